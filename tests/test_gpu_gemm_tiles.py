"""Products on 256 x 256 tiles: a few stages (the ping-pong kernel) and K from
which the four-wavefront kernel takes them, whole and short first stages, ragged
rows and columns, every operand layout and epilogue.  Against an fp64 product, and
bit for bit against the same product with 32 zero columns appended to K (the added
terms are exact zeros, the order over k is the same).  Then K that is no multiple
of the stages' depth, on every tile, and the loss added up beside the weight
gradient."""
import numpy as np
import pytest
import torch

import oracle.uniquan as O
import test_gpu_decoder_ops as ops
import test_gpu_fused as fused
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


# K on both sides of the line between the two kernels (512), and above it
@pytest.mark.parametrize("K", [480, 512, 544, 1088])
@pytest.mark.parametrize("a_kslow,b_kslow", [(0, 0), (1, 1), (0, 1), (1, 0)])
def test_product_layouts_deep(K, a_kslow, b_kslow):
    test_product_layouts_and_stages(4104, 3848, K, a_kslow, b_kslow)


# the other epilogues at K from which the four-wavefront kernel takes them and one step below, with full
# grids of tiles and few, short and whole first stages (the losses and the fused backward: test names of their own)
@pytest.mark.parametrize("T,H,K,L,group", [(4104, 16, 1248, 4104, 1), (4104, 16, 1312, 513, 4), (520, 4, 32, 260, 1),
                                           (520, 4, 2528, 260, 2), (520, 4, 2560, 260, 1), (520, 4, 2592, 260, 2)])
def test_heads_depths(T, H, K, L, group):
    ops.test_gemm_heads_matches_product_then_split(T, H * 2 if T > 4096 else H, K, L, group, True)


@pytest.mark.parametrize("T,I,K", [(4104, 2080, 992), (4104, 2080, 1056), (264, 352, 32), (264, 352, 2016), (264, 352, 2080)])
def test_swiglu_depths(T, I, K):
    ops.test_gemm_swiglu_matches_products_then_silu(T, I, K)


@pytest.mark.parametrize("T,I,K", [(4104, 4104, 2528), (4104, 4104, 2592), (264, 360, 32), (264, 360, 5088),
                                   (264, 360, 5152)])
@pytest.mark.parametrize("stacked", [False, True])
def test_silu_bwd_depths(T, I, K, stacked):
    ops.test_gemm_silu_bwd_matches_product_then_silu_bwd(T, I, K, stacked)


@pytest.mark.parametrize("K", [480, 544])
def test_residual_and_block_loss_depths(K):
    ops.test_gemm_nt_residual(4104, 3848, K)
    ops.test_gemm_block_loss_matches_product_then_loss(4104, 3848, K)


@pytest.mark.parametrize("C", [480, 544, 992, 1056, 1032])
def test_loss_depths(C):
    """E and the loss with a target and without, against the product itself: E is its value less the target,
    rounded to bf16."""
    T, R = 3848, 4104
    rs = np.random.default_rng(C)
    X, Wh = (dev(rs.standard_normal((n, C))) for n in (T, R))
    Yt = torch.from_numpy(rs.standard_normal((R, T)).astype(F32)).cuda() * 20.0
    P = torch.empty(R, T, device="cuda")
    uq.uniquan_gemm_nt(R, T, C, Wh, X, P)
    ws = torch.empty(uq.uniquan_recon_ws(T, R, C), device="cuda")
    for target in (Yt, None):
        Et = torch.full((R, T), float("nan"), device="cuda", dtype=torch.bfloat16)
        loss = torch.zeros(1, device="cuda")
        uq.uniquan_layer_recon(T, R, C, X, None, Wh, target, loss, Et, ws, None)
        e = P - target if target is not None else P
        torch.cuda.synchronize()
        assert torch.equal(Et, e.bfloat16())
        ref = e.double().square().sum().item()
        assert abs(loss.item() - ref) <= 1e-6 * ref


@pytest.mark.parametrize("T,g", [(6112, 128), (6176, 32)])
def test_fused_backward_depths(T, g):
    """The straight-through backward in the product's store on both sides of its line (T = 6144 tokens): 17 x 16
    tiles, ragged in both dimensions."""
    fused.sampled_rows_check(4100, 3968, T, 3, g, 38, np.array([0, 127, 128, 2049, 4095, 4096, 4099]))


@pytest.mark.parametrize("M", [4097, 4351])
@pytest.mark.parametrize("K", [128, 576])
def test_odd_rows(M, K):
    """Rows past M in the last tile are neither read nor written: guard rows stay as they are."""
    N = 4096
    rs = np.random.default_rng(M)
    A, B = (O.bf16_rne(rs.standard_normal((n, K)).astype(F32)) for n in (M, N))
    out = torch.full((M + 8, N), 7.0, device="cuda")
    uq.uniquan_gemm_nt(M, N, K, dev(A), dev(B), out)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.all(got[M:] == 7.0)
    mag = np.abs(A) @ np.abs(B).T
    assert np.all(np.abs(got[:M] - A.astype(np.float64) @ B.astype(np.float64).T) <= (K + 1) * 2.0 ** -24 * mag)


# short first stages: 128 x 128, 256 x 128 and 256 x 256 tiles, one to five
# stages, K from one chunk on (below 64 the register-staged kernel takes the
# 256-row tiles)
@pytest.mark.parametrize("M,N", [(301, 264), (4098, 2056), (4104, 3848)])
@pytest.mark.parametrize("K", [8, 24, 32, 40, 56, 72, 96, 120, 136, 264])
def test_any_k(M, N, K):
    rs = np.random.default_rng(M + K)
    A, B = (O.bf16_rne(rs.standard_normal((n, K)).astype(F32)) for n in (M, N))
    out = torch.full((M, N), float("nan"), device="cuda")
    uq.uniquan_gemm_nt(M, N, K, dev(A), dev(B), out)
    torch.cuda.synchronize()
    mag = np.abs(A) @ np.abs(B).T
    err = np.abs(out.cpu().numpy() - A.astype(np.float64) @ B.astype(np.float64).T)
    assert np.all(err <= (K + 1) * 2.0 ** -24 * mag + 1e-30)


@pytest.mark.parametrize("a_kslow,b_kslow", [(1, 1), (0, 1), (1, 0)])
@pytest.mark.parametrize("K", [32, 96, 160])
def test_kslow_half_stage(K, a_kslow, b_kslow):
    M, N = 4104, 3848
    rs = np.random.default_rng(K + 10 * a_kslow + b_kslow)
    A, B = (O.bf16_rne(rs.standard_normal((n, K)).astype(F32)) for n in (M, N))
    out = torch.full((M, N), float("nan"), device="cuda")
    uq.uniquan_gemm(M, N, K, dev(A.T if a_kslow else A), a_kslow, dev(B.T if b_kslow else B), b_kslow, out, 1.0)
    torch.cuda.synchronize()
    mag = np.abs(A) @ np.abs(B).T
    err = np.abs(out.cpu().numpy() - A.astype(np.float64) @ B.astype(np.float64).T)
    assert np.all(err <= (K + 1) * 2.0 ** -24 * mag + 1e-30)


# weight gradients on 128 x 128, 256 x 128 and 256 x 256 tiles, from the three kernels
@pytest.mark.parametrize("T,R,C", [(72, 130, 264), (8, 4096, 2056), (136, 4096, 2056), (104, 4096, 4096)])
@pytest.mark.parametrize("gdt", [torch.bfloat16, torch.float32])
def test_loss_beside_the_gradient(T, R, C, gdt):
    """The loss is the same bits whether its own launch or the gradient's extra workgroup adds it up, and the
    gradient the same as without it (its output over the partials takes the separate launch)."""
    rs = np.random.default_rng(T + C)
    X, Wh = (dev(rs.standard_normal((n, C))) for n in (T, R))
    Yt = torch.from_numpy(rs.standard_normal((R, T)).astype(F32)).cuda()
    n = uq.uniquan_recon_ws(T, R, C)
    ws = torch.empty(n, device="cuda")
    loss, loss1, loss2 = (torch.full((1,), float("nan"), device="cuda") for _ in range(3))
    Et = torch.empty(R, T, device="cuda", dtype=torch.bfloat16)
    G, G1 = (torch.full((R, C), float("nan"), device="cuda", dtype=gdt) for _ in range(2))
    Xt = X.T.contiguous()
    uq.uniquan_layer_recon(T, R, C, X, None, Wh, Yt, loss, Et, ws, None)
    uq.uniquan_layer_grad(T, R, C, Et, Xt, G)
    uq.uniquan_layer_recon(T, R, C, X, Xt, Wh, Yt, loss1, Et, ws, G1)
    torch.cuda.synchronize()
    assert loss.item() == loss1.item() and torch.equal(G, G1)
    G1.fill_(0.0)
    over = G1.reshape(-1).view(torch.float32)[:n]  # partials inside the gradient's output
    uq.uniquan_layer_recon(T, R, C, X, Xt, Wh, Yt, loss2, Et, over, G1)
    torch.cuda.synchronize()
    assert loss.item() == loss2.item() and torch.equal(G, G1)
