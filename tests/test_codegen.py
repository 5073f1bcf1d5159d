"""The built kernels' machine code, where the source relies on something that the
compiler cannot check (this repository's own build, disassembled; no GPU)."""
import os
import re
import struct
import subprocess

import pytest

from paper_2506_03781_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """The gfx950 code objects of a library built by hipcc (uncompressed offload bundles)."""
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(min(n, 16)):
            off, size, ln = struct.unpack_from("<QQQ", data, p)
            triple = data[p + 24:p + 24 + ln]
            if b"gfx950" in triple and size:
                yield data[at + off:at + off + size]
            p += 24 + ln
        at = data.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def w4_kernels(tmp_path_factory):
    """{name: [instruction, ...]} of the gemm_w4_kernel instantiations."""
    if not os.path.exists(build.LIB):
        build.build()
    assert os.path.exists(OBJDUMP)
    out = {}
    for co in code_objects(build.LIB):
        if b"gemm_w4_kernel" not in co:
            continue
        f = tmp_path_factory.mktemp("co") / "a.co"
        f.write_bytes(co)
        names = sorted(set(re.findall(r"_ZN2uq14gemm_w4_kernel\w+EvNS_8GemmArgsE(?!\.)", co.decode("latin1"))))
        text = subprocess.run([OBJDUMP, "-d", "--no-leading-addr", "--no-show-raw-insn",
                               "--disassemble-symbols=" + ",".join(names), str(f)],
                              capture_output=True, text=True, check=True).stdout
        for m in re.finditer(r"^(?:[0-9a-f]+ )?<(\w+)>:\n(.*?)(?=^(?:[0-9a-f]+ )?<|\Z)", text, re.S | re.M):
            out[m.group(1)] = [ln.split("//")[0].strip() for ln in m.group(2).splitlines() if ln.strip()]
    return out


def test_accumulators_are_read_after_their_products(w4_kernels):
    """A 4-pass MFMA's registers may be read by another instruction 7 wait states
    after it (another MFMA takes 4 of them).  Most products of gemm_w4_kernel are
    asm, so the compiler adds no waits for them: nothing reads an accumulator sooner,
    copies that the register allocator adds among them."""
    assert len(w4_kernels) >= 20
    for name, ins in w4_kernels.items():
        assert sum(x.startswith("v_mfma") for x in ins) == 128, name
        at, written = 0, {}
        for x in ins:
            nop = re.match(r"s_nop (\d+)", x)
            regs = [r for lo, hi in re.findall(r"\ba\[(\d+):(\d+)\]", x) for r in range(int(lo), int(hi) + 1)]
            regs += [int(r) for r in re.findall(r"\ba(\d+)\b", x)]
            if x.startswith("v_mfma"):
                at += 4
                written.update((r, at) for r in regs[:4])
                continue
            at += int(nop.group(1)) + 1 if nop else 1
            for r in regs:
                assert at - written.get(r, -99) > 7, (name, x)
                if x.startswith("v_accvgpr_write"):
                    written.pop(r, None)
