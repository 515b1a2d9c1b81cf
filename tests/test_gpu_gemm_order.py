"""A product's element has the same bits whatever tiles the problem's size
picks: every tile kernel contracts an element over k in the same order, so the
first rows of a large product equal the product of those rows alone (64 x 64
tiles), in the three layouts of a linear layer."""
import pytest

import synthgen as sg
from helpers import to_dev_bf16, to_dev_f32

pytestmark = pytest.mark.gpu


def _products(catq, X, dY, W, y_f32):
    import torch
    (M, K), N = X.shape, W.shape[0]
    ng = N * K // 128
    fac = [to_dev_f32(f) for f in sg.perturbed_factors(72, ng)]
    stats = torch.empty(ng, 2, dtype=torch.float32, device="cuda")
    p = catq.lmst_params(s=7.0)
    catq.catq_modulate_ternarize(W, *fac, p, stats, 0, W_fake=torch.empty_like(W))
    Y = torch.empty(M, N, dtype=torch.float32 if y_f32 else torch.bfloat16, device="cuda")
    dX, G = torch.empty_like(X), torch.empty(N, K, dtype=torch.float32, device="cuda")
    g = [torch.empty(ng, dtype=torch.float32, device="cuda") for _ in range(3)]
    ws = torch.empty(catq.catq_workspace_size(0, M, N, K), dtype=torch.uint8, device="cuda")
    catq.catq_fakeq_linear_fwd(X, W, Y, M, N, K)
    catq.catq_fakeq_linear_bwd(dY, X, W, M, N, K, W, stats, *fac, p, *g, ws, dX=dX, dW_fake=G)
    torch.cuda.synchronize()
    return Y, dX, G


@pytest.mark.parametrize("y_f32", [False, True])
@pytest.mark.parametrize("M,N,K,m,n", [
    (2000, 1032, 2176, 130, 136),   # against 128 x 128 tiles; the input gradient's contraction is ragged
    (1980, 5128, 4096, 64, 264),    # against 256 x 256 tiles
])
def test_rows_of_a_larger_product(catq, M, N, K, m, n, y_f32):
    import torch
    X, dY, W = (to_dev_bf16(sg.normal_bf16(71, k, s)) for k, s in (("X", (M, K)), ("Y", (M, N)), ("W", (N, K))))
    Y, dX, G = _products(catq, X, dY, W, y_f32)
    y, dx, _ = _products(catq, X[:m], dY[:m], W, y_f32)
    assert torch.equal(y, Y[:m])
    assert torch.equal(dx, dX[:m])
    _, _, g = _products(catq, X, dY[:, :n].contiguous(), W[:n], y_f32)
    assert torch.equal(g, G[:n])


@pytest.mark.parametrize("M,N,K", [(1, 1, 8), (5, 7, 72), (70, 333, 136),   # 64 x 64 tiles
                                   (1500, 2049, 136),                       # 128 x 128 tiles in four stages
                                   (3500, 2049, 136),                       # 128 x 128 tiles
                                   (4100, 4099, 72)])                       # 256 x 256 tiles
@pytest.mark.parametrize("y,r", [("bf16", None), ("bf16", "bf16"), ("f32", "bf16"), ("f32", "f32")])
def test_odd_outputs(catq, M, N, K, y, r):
    """Any number of outputs, in a buffer of no alignment beyond its start: rows
    are stored element by element, and nothing past the last."""
    import torch
    dt = {"bf16": torch.bfloat16, "f32": torch.float32, None: None}
    X, W = (to_dev_bf16(sg.normal_bf16(73, k, s)) for k, s in (("X", (M, K)), ("W", (N, K))))
    R = None if r is None else to_dev_bf16(sg.normal_bf16(73, "Y", (M, N))).to(dt[r])
    buf = torch.full((M * N + 64,), 7.0, dtype=dt[y], device="cuda")
    catq.catq_fakeq_linear_fwd(X, W, buf[:M * N].view(M, N), M, N, K, residual=R)
    torch.cuda.synchronize()
    assert bool((buf[M * N:] == 7.0).all())
    ref = X.float() @ W.float().T + (0 if R is None else R.float())
    err = (buf[:M * N].view(M, N).float() - ref).abs().max() / ref.abs().max()
    # one rounding to the output type, and two fp32 sums of K terms
    assert err <= (2.0 ** -8 if y == "bf16" else 2e-6)
