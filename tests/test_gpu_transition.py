"""The transition function's two device forms (one exponential per weight
while 2 cosh(2 s Delta) fits, the general one beyond) at sharpnesses on both
sides of the line between them and on it, where the groups of one launch take
both: fp32 fake weights and the factor gradients of the fp32 and the bf16
(GEMM epilogue) paths against the oracle."""
import numpy as np
import pytest

import synthgen as sg
from helpers import elem_rel_ok, f64, host, max_norm_err, to_dev_bf16, to_dev_f32
from oracle import lmst

pytestmark = pytest.mark.gpu

N, K, M = 136, 256, 192
SHARP = [0.01, 0.6, 30.0, 69.3, 75.0, 300.0]   # dz = 100 at s Delta = 34.66, Delta = 0.37 .. 0.67


@pytest.mark.parametrize("s", SHARP)
def test_soft_fp32(catq, s):
    import torch
    W = (sg.rng(41, "W").standard_normal((N, K)) * 0.02).astype(np.float32)
    W[3, :128] = 0.25                        # a constant group
    W[5, 7] = 0.0
    fac = sg.perturbed_factors(42, N * K // 128)
    ng = N * K // 128
    dm, da, dd = (to_dev_f32(f) for f in fac)
    stats = torch.zeros(ng, 2, dtype=torch.float32, device="cuda")
    Wd = to_dev_f32(W)
    wf = [torch.empty_like(Wd) for _ in range(2)]
    p = catq.lmst_params(mode=lmst.SOFT, s=s)
    catq.catq_modulate_ternarize(Wd, dm, da, dd, p, stats, 0, W_fake=wf[0])
    catq.catq_modulate_ternarize(Wd, dm, da, dd, p, stats, 1, W_fake=wf[1])
    torch.cuda.synchronize()
    assert torch.equal(wf[0], wf[1])
    ref = lmst.modulate_ternarize(W.astype(np.float64), 128, *fac, lmst.SOFT, s=s)["W_fake"]
    # f ~ e^{-2 s (Delta - |W_hat|)} in the dead zone: the exponent carries a few
    # fp32 roundings (2^-24) of 2 s Delta
    ok, worst = elem_rel_ok(host(wf[0]), ref, 4e-6 + 8 * 2.0 ** -24 * 2 * s * 0.7)
    assert ok, worst


@pytest.mark.parametrize("s", SHARP)
@pytest.mark.parametrize("mode", [lmst.SOFT, lmst.HARD])
def test_factor_gradients(catq, s, mode):
    """bf16 (fused epilogue, 192 tokens) and the separate kernel on the
    materialised G (dW_fake requested)."""
    import torch
    xb, dyb = sg.normal_bf16(43, "X", (M, K)), sg.normal_bf16(43, "Y", (M, N), std=1e-3)
    wb = sg.normal_bf16(43, "W", (N, K), std=0.02)
    fac = sg.perturbed_factors(44, N * K // 128)
    ng = N * K // 128
    dm, da, dd = (to_dev_f32(f) for f in fac)
    X, dY, W = to_dev_bf16(xb), to_dev_bf16(dyb), to_dev_bf16(wb)
    stats = torch.zeros(ng, 2, dtype=torch.float32, device="cuda")
    wf = torch.empty_like(W)
    p = catq.lmst_params(mode=mode, s=s, s_bwd=s)
    catq.catq_modulate_ternarize(W, dm, da, dd, p, stats, 0, W_fake=wf)
    ws = torch.empty(catq.catq_workspace_size(0, M, N, K), dtype=torch.uint8, device="cuda")
    ref = lmst.factor_grads(f64(dyb).T @ f64(xb), f64(wb), 128, *fac, mode, s=s, s_bwd=s)
    for dw in (None, torch.empty(N, K, dtype=torch.float32, device="cuda")):
        g = [torch.empty(ng, dtype=torch.float32, device="cuda") for _ in range(3)]
        catq.catq_fakeq_linear_bwd(dY, X, wf, M, N, K, W, stats, dm, da, dd, p, *g, ws, dW_fake=dw)
        torch.cuda.synchronize()
        for a, b in zip(g, ref):
            # f_W varies by 2 s per unit of W_hat, known to a few 2^-24; at small
            # s, f - W_hat f_W = O(s^2) is a difference of two sums of order 1
            assert max_norm_err(host(a), b) <= 2e-5 + (4 * s + 1 / s ** 2) * 2.0 ** -22


def test_constant_group_gradients(catq):
    """alpha0 = 0: all gradients of the group are zero, none is NaN, fused and
    not."""
    import torch
    X = to_dev_bf16(sg.normal_bf16(45, "X", (M, K)))
    dY = to_dev_bf16(sg.normal_bf16(45, "Y", (M, N)))
    wb = sg.normal_bf16(45, "W", (N, K), std=0.02)
    wb[9, :128] = wb[9, 0]
    W = to_dev_bf16(wb)
    ng = N * K // 128
    dm, da, dd = (to_dev_f32(f) for f in sg.perturbed_factors(46, ng))
    stats = torch.zeros(ng, 2, dtype=torch.float32, device="cuda")
    wf = torch.empty_like(W)
    p = catq.lmst_params(mode=lmst.SOFT, s=15.0)
    catq.catq_modulate_ternarize(W, dm, da, dd, p, stats, 0, W_fake=wf)
    ws = torch.empty(catq.catq_workspace_size(0, M, N, K), dtype=torch.uint8, device="cuda")
    for dw in (None, torch.empty(N, K, dtype=torch.float32, device="cuda")):
        g = [torch.empty(ng, dtype=torch.float32, device="cuda") for _ in range(3)]
        catq.catq_fakeq_linear_bwd(dY, X, wf, M, N, K, W, stats, dm, da, dd, p, *g, ws, dW_fake=dw)
        torch.cuda.synchronize()
        for t in g:
            assert torch.isfinite(t).all()
            assert t[9 * K // 128].item() == 0.0
