"""LM+ST kernels at the edges of their two lane splits: one octet, or four
octets of a group per lane."""
import numpy as np
import pytest
import torch

import paper_2606_26650_amd as catq
from oracle import lmst

pytestmark = pytest.mark.gpu
DEV = "cuda"

# 2^21 weights is where lanes take four octets; groups below 32 weights never do
SHAPES = [(1, 512, 128), (7, 512, 64), (4095, 512, 128), (4096, 512, 128), (4097, 512, 128),
          (2049, 1024, 32), (2049, 1024, 64), (2049, 1024, 256), (2049, 1024, 512), (2049, 1024, 16)]


@pytest.mark.parametrize("rows,cols,g", SHAPES)
def test_modulate_and_pack(rows, cols, g):
    rng = np.random.default_rng(rows + g)
    W = torch.tensor(rng.standard_normal((rows, cols)) * 0.02, dtype=torch.bfloat16)
    W64 = W.double().numpy()
    n = rows * cols // g
    fac = [rng.uniform(-0.3, 0.3, n).astype(np.float32), rng.uniform(0.7, 1.4, n).astype(np.float32),
           rng.uniform(0.7, 1.4, n).astype(np.float32)]
    fd = [torch.tensor(f, device=DEV) for f in fac]
    Wd, wf = W.to(DEV), torch.empty((rows, cols), dtype=torch.bfloat16, device=DEV)
    stats = torch.empty((n, 2), device=DEV)
    soft, hard = (catq.lmst_params(g, m, 0.5, 15.0, 30.0) for m in (catq.SOFT, catq.HARD))
    catq.catq_modulate_ternarize(Wd, *fd, soft, stats, 0, W_fake=wf)
    ref = lmst.modulate_ternarize(W64, g, *fac, lmst.SOFT, s=15.0)
    x = W64.reshape(n, g)
    mu = x.mean(1).astype(np.float32)
    al = np.abs(x - mu.astype(np.float64)[:, None]).mean(1).astype(np.float32)
    st = stats.cpu().numpy()
    # fp64 sums rounded once: one ulp for another order of the sum
    np.testing.assert_allclose(st[:, 1], al, rtol=2.4e-7)
    np.testing.assert_allclose(st[:, 0], mu, atol=2.4e-7 * float(al.max()))
    # bf16 rounding of alpha * f: half an ulp, 2^-9, and the fp32 evaluation of f
    d = np.abs(wf.double().cpu().numpy().reshape(n, g) - ref["W_fake"].reshape(n, g))
    assert (d <= 2.0 ** -8 * np.abs(ref["W_fake"].reshape(n, g)) + 1e-5 * al[:, None]).all()
    wf2 = torch.empty_like(wf)
    catq.catq_modulate_ternarize(Wd, *fd, soft, stats, 1, W_fake=wf2)
    assert torch.equal(wf, wf2)
    # the hard branch: codes, packed words and scales agree with each other and the oracle
    codes = torch.empty((rows, cols), dtype=torch.int8, device=DEV)
    packed = torch.empty((rows, cols // 4), dtype=torch.uint8, device=DEV)
    alpha = torch.empty(n, device=DEV)
    catq.catq_modulate_ternarize(Wd, *fd, hard, stats, 1, codes=codes)
    catq.catq_ternarize_pack(Wd, *fd, hard, torch.empty_like(stats), 0, packed, alpha_out=alpha)
    rc = lmst.modulate_ternarize(W64, g, *fac, lmst.HARD)["codes"]
    np.testing.assert_array_equal(codes.cpu().numpy().reshape(rc.shape), rc)
    p = packed.cpu().numpy()
    got = np.stack([(p >> (2 * i)) & 3 for i in range(4)], -1).reshape(rows, cols).astype(np.int8) - 1
    np.testing.assert_array_equal(got, codes.cpu().numpy())
    np.testing.assert_allclose(alpha.cpu().numpy(), fac[1] * al, rtol=4e-7)


def test_more_octets_than_lanes_of_a_launch():
    """Groups of 16, one octet per lane, in a weight of 2^35 and some elements:
    more lanes than one launch may have."""
    g, cols, tail = 16, 1 << 20, 3
    rows = (1 << 15) + tail
    need = rows * cols * (2 + 1 + 0.5)          # W, codes, statistics
    if torch.cuda.mem_get_info()[0] < need * 1.1:
        pytest.skip("needs 132 GB of free device memory")
    W = torch.zeros((rows, cols), dtype=torch.bfloat16, device=DEV)
    W[0] = torch.randn(cols, device=DEV).to(torch.bfloat16)
    W[-tail:] = torch.randn((tail, cols), device=DEV).to(torch.bfloat16)
    codes = torch.full((rows, cols), 7, dtype=torch.int8, device=DEV)
    stats = torch.empty((rows * cols // g, 2), device=DEV)
    one = [torch.tensor([v], device=DEV) for v in (0.0, 1.0, 1.0)]
    p = catq.lmst_params(g, catq.HARD, strides=(0, 0, 0))
    catq.catq_modulate_ternarize(W, *one, p, stats, 0, codes=codes)
    for r in (0, rows - tail, rows - 1):
        x = W[r].double().cpu().numpy().reshape(-1, g)
        ref = lmst.modulate_ternarize(x, g, [0.0], [1.0], [1.0], lmst.HARD, strides=(0, 0, 0))["codes"]
        np.testing.assert_array_equal(codes[r].cpu().numpy().reshape(ref.shape), ref)
    assert not bool(codes[1:-tail].any())        # constant groups: all codes 0
    del W, codes, stats
    torch.cuda.empty_cache()
