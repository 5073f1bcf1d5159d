"""The 256 x 256 tile product (K a multiple of 64) at the edges of its range:
one, two, three and five 64-deep stages, ragged rows and columns, every operand
layout.  Against an fp64 product, and bit for bit against the same product with
32 zero columns appended to K, which runs on the ping-pong kernel (the added
terms are exact zeros, the order over k is the same)."""
import numpy as np
import pytest
import torch

import oracle.uniquan as O
from paper_2506_03781_amd import uniquan as uq

pytestmark = pytest.mark.gpu
F32 = np.float32


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    uq.lib()
    torch.cuda.set_device(0)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a.astype(F32))).to("cuda").to(torch.bfloat16).contiguous()


@pytest.mark.parametrize("M,N,K", [(4104, 3848, 64), (4104, 3848, 128), (4104, 3848, 192), (4096, 4096, 320)])
@pytest.mark.parametrize("a_kslow,b_kslow", [(0, 0), (1, 1), (0, 1), (1, 0)])
def test_product_layouts_and_stages(M, N, K, a_kslow, b_kslow):
    rs = np.random.default_rng(M + N + 3 * K + 10 * a_kslow + b_kslow)
    A, B = (O.bf16_rne(rs.standard_normal((n, K)).astype(F32)) for n in (M, N))
    pad = [np.concatenate([x, np.zeros((x.shape[0], 32), F32)], axis=1) for x in (A, B)]

    def run(a, b, k):
        out = torch.full((M, N), float("nan"), device="cuda")
        uq.uniquan_gemm(M, N, k, dev(a.T if a_kslow else a), a_kslow, dev(b.T if b_kslow else b), b_kslow, out, 0.5)
        torch.cuda.synchronize()
        return out.cpu().numpy()

    got = run(A, B, K)
    assert np.array_equal(got, run(*pad, K + 32))
    ref = 0.5 * (A.astype(np.float64) @ B.astype(np.float64).T)
    mag = 0.5 * (np.abs(A) @ np.abs(B).T)
    # fp32 accumulation: at most K roundings of partial sums bounded by the sum of magnitudes
    assert np.all(np.abs(got - ref) <= (K + 1) * 2.0 ** -24 * mag + 1e-30)


@pytest.mark.parametrize("M", [4097, 4351])
def test_odd_rows(M):
    """Rows past M in the last tile are neither read nor written: guard rows stay as they are."""
    N, K = 4096, 128
    rs = np.random.default_rng(M)
    A, B = (O.bf16_rne(rs.standard_normal((n, K)).astype(F32)) for n in (M, N))
    out = torch.full((M + 8, N), 7.0, device="cuda")
    uq.uniquan_gemm_nt(M, N, K, dev(A), dev(B), out)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.all(got[M:] == 7.0)
    mag = np.abs(A) @ np.abs(B).T
    assert np.all(np.abs(got[:M] - A.astype(np.float64) @ B.astype(np.float64).T) <= (K + 1) * 2.0 ** -24 * mag)
