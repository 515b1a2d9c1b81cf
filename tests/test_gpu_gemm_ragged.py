"""Linear layers whose extents are no tile multiples in any direction: the
direct-to-LDS products with ragged columns of a K-major operand, a ragged
contraction of a K-contiguous one, and the factor epilogue on partial tiles,
against plain float64 products and the oracle's factor gradients."""
import numpy as np
import pytest

import synthgen as sg
from helpers import f64, host, max_norm_err, to_dev_bf16, to_dev_f32
from oracle import lmst

pytestmark = pytest.mark.gpu

# bf16 outputs: one rounding, at most 2^-9 of the value, and fp32 sums of
# exact products far below that
BF16 = 2.0 ** -8


def _case(catq, M, N, K, mode=lmst.SOFT, E=1, off=None, nan_row=None):
    import torch
    xb = sg.normal_bf16(21, "X", (M, K))
    wb = sg.normal_bf16(21, "W", (E * N, K), std=0.02)
    dyb = sg.normal_bf16(21, "Y", (M, N), std=1e-3)
    if nan_row is not None:
        dyb[nan_row] = 0x7FC0
    X, W, dY = to_dev_bf16(xb), to_dev_bf16(wb), to_dev_bf16(dyb)
    ng = E * N * K // 128
    fac = sg.perturbed_factors(22, ng)
    dm, da, dd = (to_dev_f32(f) for f in fac)
    stats = torch.zeros(ng, 2, dtype=torch.float32, device="cuda")
    wf = torch.empty_like(W)
    p = catq.lmst_params(mode=mode, s=7.0, s_bwd=30.0)
    catq.catq_modulate_ternarize(W, dm, da, dd, p, stats, 0, W_fake=wf)
    ws = torch.empty(catq.catq_workspace_size(0, M, N, K, E), dtype=torch.uint8, device="cuda")
    kw = dict(n_experts=E, row_offsets=torch.tensor(off, device="cuda")) if E > 1 else {}
    # outputs inside larger buffers: nothing may be written past their ends
    Yb = torch.full((M * N + 64,), 7.0, dtype=torch.bfloat16, device="cuda")
    dXb = torch.full((M * K + 64,), 7.0, dtype=torch.bfloat16, device="cuda")
    g = [torch.full((ng + 16,), 7.0, dtype=torch.float32, device="cuda") for _ in range(3)]
    catq.catq_fakeq_linear_fwd(X, wf, Yb[:M * N].view(M, N), M, N, K, **kw)
    catq.catq_fakeq_linear_bwd(dY, X, wf, M, N, K, W, stats, dm, da, dd, p, *[t[:ng] for t in g], ws,
                               dX=dXb[:M * K].view(M, K), **kw)
    torch.cuda.synchronize()
    for t, n in [(Yb, M * N), (dXb, M * K)] + [(t, ng) for t in g]:
        assert bool((t[n:] == 7.0).all())
    off = off or [0, M]
    Wf = host(wf.float()).astype(np.float64).reshape(E, N, K)
    X64, dY64 = f64(xb), f64(dyb)
    Y, dX, G = np.zeros((M, N)), np.zeros((M, K)), np.zeros((E, N, K))
    for e in range(E):
        r = slice(off[e], off[e + 1])
        Y[r], dX[r], G[e] = X64[r] @ Wf[e].T, dY64[r] @ Wf[e], dY64[r].T @ X64[r]
    got = (host(Yb[:M * N].float()).reshape(M, N), host(dXb[:M * K].float()).reshape(M, K),
           [host(t[:ng]) for t in g])
    ref = lmst.factor_grads(G.reshape(E * N, K), f64(wb), 128, *fac, mode, s=7.0, s_bwd=30.0)
    return got, (Y, dX, ref)


@pytest.mark.parametrize("mode", [lmst.SOFT, lmst.HARD])
@pytest.mark.parametrize("M,N,K", [
    (8, 8, 128),          # one partial tile in every direction
    (130, 264, 128),      # a tile and a remainder; ragged contraction of dX (264)
    (65, 1032, 640),      # one token past a k tile; d_in = 2.5 tiles of 256
    (1000, 1048, 1152),   # 64-wide tiles over 16 k tiles, token remainder 40
    (1000, 3080, 2176),   # 128-wide tiles in four stages (forward), 34 k tiles
    (1500, 2104, 128),    # the same with two k tiles
    (1500, 64, 2176),     # and with one, in the input gradient
    (1500, 136, 2176),    # and with three, the last ragged
    (2100, 3080, 2176),   # 128-wide tiles, two per unit
    (999, 4104, 2688),    # 256-wide tiles with remainders, odd tokens
    (4100, 4104, 2688),   # the same with a partial last round
])
def test_ragged_dense(catq, M, N, K, mode):
    (y, dx, g), (Y, dX, G) = _case(catq, M, N, K, mode)
    assert max_norm_err(y, Y) <= BF16
    assert max_norm_err(dx, dX) <= BF16
    for a, b in zip(g, G):
        assert max_norm_err(a, b) <= 1e-3


@pytest.mark.parametrize("N,K", [(264, 384), (1032, 128),
                                 (1032, 1664)])   # 175 tiles of 256 x 256: the larger factor tiles
def test_ragged_experts(catq, N, K):
    off = [0, 0, 70, 71, 400, 520]   # an empty expert, one row, remainders
    (y, dx, g), (Y, dX, G) = _case(catq, 520, N, K, E=5, off=off)
    assert max_norm_err(y, Y) <= BF16
    assert max_norm_err(dx, dX) <= BF16
    for a, b in zip(g, G):
        assert max_norm_err(a, b) <= 1e-3


@pytest.mark.parametrize("N,K,rows", [(136, 256, 1), (248, 128, 1), (136, 128, 50)])
def test_narrow_experts(catq, N, K, rows):
    """Fewer than 256 columns, in the three products: 128 x 128 tiles, in four
    stages, or (26000 rows, more than one tile per unit) in two."""
    off = [rows * r for r in (0, 0, 70, 71, 400, 520)]
    (y, dx, g), (Y, dX, G) = _case(catq, off[-1], N, K, E=5, off=off)
    assert max_norm_err(y, Y) <= BF16
    assert max_norm_err(dx, dX) <= BF16
    for a, b in zip(g, G):
        assert max_norm_err(a, b) <= 1e-3


@pytest.mark.parametrize("M,N,K", [(130, 264, 256), (700, 4104, 2688)])
def test_nan_row_stays_in_its_row(catq, M, N, K):
    """dY rows are the ragged contraction operand of dX: the last chunk of row
    r - 1 must not pick up the first values of a NaN row r."""
    import torch  # noqa: F401
    (_, dx, _), _ = _case(catq, M, N, K, nan_row=67)
    bad = ~np.isfinite(dx).all(1)
    assert list(np.nonzero(bad)[0]) == [67]


@pytest.mark.parametrize("M,N,K", [
    (1, 8, 128),        # one group, most waves without work
    (33, 40, 128),      # remainders of a 32 x 32 tile, contraction of 40 and 33
    (1021, 72, 384),    # odd token contraction over eight waves
    (2100, 136, 128),   # token contraction split in two
    (2049, 1032, 256),  # 64 x 64 tiles with remainders
    (15, 24, 128),      # weight gradient on 16 x 16 tiles: less than one group
    (1025, 504, 256),   # 16 x 16 tiles, one token past sixteen waves' groups
    (1024, 520, 256),   # 32 x 32 tiles just past the 16 x 16 ones
])
def test_f32_linear(catq, M, N, K):
    """The fp32 product in its three layouts (residual in the forward) against
    float64: errors of an fp32 sum of up to 2100 terms, 2^-24 * sqrt(2100) =
    3e-6 of the largest output."""
    import torch
    x, w, dy, r = (sg.uniform_f32(31, n, s) for n, s in
                   (("X", (M, K)), ("W", (N, K)), ("Y", (M, N)), ("G", (M, N))))
    X, W, dY, R = (to_dev_f32(t) for t in (x, w, dy, r))
    ng = N * K // 128
    dm, da, dd = (to_dev_f32(f) for f in sg.perturbed_factors(32, ng))
    stats = torch.zeros(ng, 2, dtype=torch.float32, device="cuda")
    wf = torch.empty_like(W)
    p = catq.lmst_params(mode=lmst.SOFT, s=7.0)
    catq.catq_modulate_ternarize(W, dm, da, dd, p, stats, 0, W_fake=wf)
    Y, dX = torch.empty_like(R), torch.empty_like(X)
    dW = torch.empty_like(W)
    g = [torch.empty(ng, dtype=torch.float32, device="cuda") for _ in range(3)]
    ws = torch.empty(catq.catq_workspace_size(0, M, N, K), dtype=torch.uint8, device="cuda")
    catq.catq_fakeq_linear_fwd(X, wf, Y, M, N, K, residual=R)
    catq.catq_fakeq_linear_bwd(dY, X, wf, M, N, K, W, stats, dm, da, dd, p, *g, ws, dX=dX, dW_fake=dW)
    torch.cuda.synchronize()
    w64 = host(wf)
    assert max_norm_err(host(Y), host(X) @ w64.T + host(R)) <= 3e-6
    assert max_norm_err(host(dX), host(dY) @ w64) <= 3e-6
    assert max_norm_err(host(dW), host(dY).T @ host(X)) <= 3e-6
