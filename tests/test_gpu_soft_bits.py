"""The softened weights bit for bit: a calibration's trajectory follows the
last bit of every fake weight (a bf16 step of one weight moves the factor
gradients of a block by 1e-3), so the evaluation of f keeps its roundings.
The checksums are of the fake weights on gfx950, one octet per lane (small
arrays) and four octets of a group per lane."""
import zlib

import numpy as np
import pytest

import synthgen as sg
from helpers import to_dev_bf16, to_dev_f32
from oracle import lmst

pytestmark = pytest.mark.gpu

# rows, cols, group, sharpness, fp32 weights -> CRC-32 of W_fake
CRC = {
    (136, 256, 128, 15.0, False): 0x8958f8fc,
    (136, 256, 128, 0.6, True): 0x5659165b,
    (136, 256, 16, 75.0, True): 0x68eaf28f,
    (4104, 512, 128, 15.0, False): 0xf69a45f9,
    (4104, 512, 32, 30.0, True): 0x86749c3b,
    (4104, 512, 512, 3.0, False): 0xf340a6e7,
}


def fake(catq, rows, cols, g, s, f32):
    import torch
    if f32:
        W = to_dev_f32((sg.rng(61, "W").standard_normal((rows, cols)) * 0.02).astype(np.float32))
    else:
        W = to_dev_bf16(sg.normal_bf16(61, "W", (rows, cols), std=0.02))
    ng = rows * cols // g
    fac = [to_dev_f32(f) for f in sg.perturbed_factors(62, ng)]
    stats = torch.zeros(ng, 2, dtype=torch.float32, device="cuda")
    wf = [torch.empty_like(W) for _ in range(2)]
    p = catq.lmst_params(g, mode=lmst.SOFT, s=s)
    for i in range(2):     # statistics computed, then read back
        catq.catq_modulate_ternarize(W, *fac, p, stats, i, W_fake=wf[i])
    torch.cuda.synchronize()
    return [zlib.crc32(t.view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32).cpu().numpy().tobytes())
            for t in wf]


@pytest.mark.parametrize("case", list(CRC))
def test_fake_weight_bits(catq, case):
    assert [hex(c) for c in fake(catq, *case)] == [hex(CRC[case])] * 2
