"""The transition function at sharpnesses from nearly linear to nearly hard: fp32
fake weights, and the factor gradients of the fp32 and the bf16 (GEMM epilogue)
paths against the oracle.  The backward has two device forms, one exponential per
weight while 2 cosh(2 s Delta) is small enough and the general one beyond; the
sharpnesses lie on both sides of the line between them and on it, where the
groups of one launch take both."""
import numpy as np
import pytest

import synthgen as sg
from helpers import elem_rel_ok, f64, host, max_norm_err, to_dev_bf16, to_dev_f32
from oracle import lmst

pytestmark = pytest.mark.gpu

N, K, M = 136, 256, 192
FUSED = (2048, 896)     # 112 tiles of 128 x 128: the factor epilogue
SHARP = [0.01, 0.6, 30.0, 41.6, 69.3, 75.0, 300.0]   # dz = 60 at s Delta = 20.8, Delta = 0.37 .. 0.67


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
@pytest.mark.parametrize("N,K", [(N, K), FUSED])
def test_factor_gradients(catq, s, mode, N, K):
    """bf16: the product with the separate kernel, or the fused epilogue, and the
    separate kernel on the materialised G (dW_fake requested)."""
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


@pytest.mark.parametrize("N,K", [(N, K), FUSED])
def test_constant_group_gradients(catq, N, K):
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


def _grads(catq, X, dY, W, fac, mode, s, s_bwd, dw):
    """The three factor gradients: fused (bf16, no dW_fake) or by the separate
    kernel (fp32, or dW_fake asked for)."""
    import torch
    (m, k), n = X.shape, W.shape[0]
    ng = n * k // 128
    f = [to_dev_f32(v) for v in fac]
    stats = torch.zeros(ng, 2, dtype=torch.float32, device="cuda")
    wf = torch.empty_like(W)
    p = catq.lmst_params(mode=mode, s=s, s_bwd=s_bwd)
    catq.catq_modulate_ternarize(W, *f, p, stats, 0, W_fake=wf)
    ws = torch.empty(catq.catq_workspace_size(0, m, n, k), dtype=torch.uint8, device="cuda")
    g = [torch.empty(ng, dtype=torch.float32, device="cuda") for _ in range(3)]
    catq.catq_fakeq_linear_bwd(dY, X, wf, m, n, k, W, stats, *f, p, *g, ws,
                               dW_fake=torch.empty(n, k, dtype=torch.float32, device="cuda") if dw else None)
    torch.cuda.synchronize()
    return [host(t) for t in g]


@pytest.mark.parametrize("path", ["f32", "bf16"])
@pytest.mark.parametrize("mode,s_bwd", [(lmst.SOFT, 30.0), (lmst.HARD, 30.0), (lmst.HARD, 0.0)])
def test_alpha_at_its_bound(catq, mode, s_bwd, path):
    """d_alpha <= 0: alpha as a divisor is the smallest normal number and W_hat
    up to 1e37, so f_W and f_Delta are 0 and f the sign: finite gradients."""
    fac = [f.copy() for f in sg.perturbed_factors(47, N * K // 128)]
    fac[1][::5] = 0.0
    fac[1][3::5] = -0.5
    # dY of 1e-3, so G below 0.1 and the straight-through sums G W_hat of 128
    # weights, |W_hat| < 0.1 / 1.2e-38, below 1e38: no overflow in fp32
    if path == "f32":
        x, dy = sg.uniform_f32(47, "X", (M, K)), sg.uniform_f32(47, "Y", (M, N)) * np.float32(1e-3)
        w = (sg.rng(47, "W").standard_normal((N, K)) * 0.02).astype(np.float32)
        X, dY, W = to_dev_f32(x), to_dev_f32(dy), to_dev_f32(w)
        x, dy, w = (t.astype(np.float64) for t in (x, dy, w))
    else:
        x, dy, w = sg.normal_bf16(47, "X", (M, K)), sg.normal_bf16(47, "Y", (M, N), std=1e-3), sg.normal_bf16(47, "W", (N, K), std=0.02)
        X, dY, W = to_dev_bf16(x), to_dev_bf16(dy), to_dev_bf16(w)
        x, dy, w = f64(x), f64(dy), f64(w)
    ref = lmst.factor_grads(dy.T @ x, w, 128, *fac, mode, s=30.0, s_bwd=s_bwd)
    got = _grads(catq, X, dY, W, fac, mode, 30.0, s_bwd, dw=True)
    low = fac[1] <= 0
    for a, b in zip(got, ref):
        for part in (low, ~low):
            assert np.isfinite(a[part]).all()
            # the bounds of test_factor_gradients at s = 30; W_hat near 1e36 (the
            # straight-through sums) adds its own rounding and that of the sums
            assert max_norm_err(a[part], b[part]) <= 2e-5 + (4 * 30 + 1 / 900) * 2.0 ** -22


@pytest.mark.parametrize("mode,s_bwd", [(lmst.SOFT, 30.0), (lmst.HARD, 30.0), (lmst.HARD, 0.0)])
def test_tiny_alpha_fused(catq, mode, s_bwd):
    """Groups of weights of 1e-31 and 1e-22 (2 s log2(e) / alpha beyond any bound
    on it that keeps constant groups finite) and groups with d_alpha <= 0, in the
    factor epilogue."""
    n, k = FUSED
    rng = sg.rng(48, "W")
    w = rng.standard_normal((n, k)) * 0.02
    for i, scale in enumerate((1e-31, 1e-22)):
        w[i::9, :256] *= scale / 0.02
    wb = sg.f32_to_bf16_bits(w.astype(np.float32))
    xb, dyb = sg.normal_bf16(48, "X", (M, k)), sg.normal_bf16(48, "Y", (M, n), std=1e-3)
    fac = [f.copy() for f in sg.perturbed_factors(48, n * k // 128)]
    low = np.zeros((n, k // 128), bool)
    low[4::9, :2] = True
    fac[1][low.reshape(-1)] = -0.25
    ref = lmst.factor_grads(f64(dyb).T @ f64(xb), f64(wb), 128, *fac, mode, s=30.0, s_bwd=s_bwd)
    got = _grads(catq, to_dev_bf16(xb), to_dev_bf16(dyb), to_dev_bf16(wb), fac, mode, 30.0, s_bwd, dw=False)
    for a, b in zip(got, ref):
        a, b = a.reshape(n, -1), b.reshape(n, -1)
        for r in range(9):
            # (the bounds of test_factor_gradients at s = 30)
            assert np.isfinite(a[r::9]).all()
            assert max_norm_err(a[r::9, :2], b[r::9, :2]) <= 2e-5 + (4 * 30 + 1 / 900) * 2.0 ** -22, r


@pytest.mark.parametrize("dy_std", [1e-3, 1e-12, 1e-18])   # G of 1e-2, 1e-11, 1e-17: the line's limit is 5e-20
@pytest.mark.parametrize("s", [15.0, 41.5, 41.7, 69.2, 100.0])  # dz 21.6, 59.9, 60.2, 99.8, 144 at Delta = 0.5
@pytest.mark.parametrize("mode", [lmst.SOFT, lmst.HARD])
@pytest.mark.parametrize("fused", [False, True])
def test_gradient_scale(catq, mode, s, dy_std, fused):
    """Small gradients keep their digits, with sharpnesses on both sides of the
    line between the two forms, and up to dz = 100, where a 2 sinh applied to the
    sum would lose them."""
    n, k = FUSED if fused else (N, K)
    xb, dyb = sg.normal_bf16(49, "X", (M, k)), sg.normal_bf16(49, "Y", (M, n), std=dy_std)
    wb = sg.normal_bf16(49, "W", (n, k), std=0.02)
    ng = n * k // 128
    fac = list(sg.perturbed_factors(49, ng))
    fac[2] = np.ones(ng, np.float32)
    ref = lmst.factor_grads(f64(dyb).T @ f64(xb), f64(wb), 128, *fac, mode, s=s, s_bwd=s)
    got = _grads(catq, to_dev_bf16(xb), to_dev_bf16(dyb), to_dev_bf16(wb), fac, mode, s, s, dw=not fused)
    for a, b in zip(got, ref):
        assert max_norm_err(a, b) <= 2e-5 + (4 * s + 1 / s ** 2) * 2.0 ** -22   # as test_factor_gradients
