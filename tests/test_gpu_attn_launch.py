"""Attention backward on both sides of its launch rule (dK/dV and dQ in one
launch, or two) at the edges of its 64-, 128- and 256-row tiles."""
import pytest

import synthgen as sg
from helpers import f64, host, max_norm_err, to_dev_bf16
from test_gpu_block import _oracle_attention

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,S,Hq,Hkv,d", [
    (1, 8, 1, 1, 64),       # one partial tile
    (1, 64, 4, 1, 128),     # one key tile, the group's heads split over blocks
    (2, 128, 4, 2, 64),     # exactly one block of keys, half a block of queries
    (1, 136, 5, 1, 64),     # a second key block in the first pair
    (1, 256, 4, 2, 128),    # whole query blocks
    (1, 264, 4, 2, 128),    # the second pair of key rows has one row only
    (3, 520, 2, 2, 64),     # waves of the last query block without queries
    (16, 136, 16, 16, 128),  # 768 blocks: two launches
    (32, 72, 32, 16, 64),    # 1536 or more: two launches, split heads
])
def test_backward(catq, B, S, Hq, Hkv, d):
    import torch
    cfg = sg.small_dense(batch=B, seq=S, n_q=Hq, n_kv=Hkv, head_dim=d, qk_norm=False)
    M, ld = B * S, (Hq + 2 * Hkv) * d
    qb, gb = sg.normal_bf16(3, "X", (M, ld)), sg.normal_bf16(4, "Y", (M, Hq * d), std=0.1)
    qkv, dO = to_dev_bf16(qb), to_dev_bf16(gb)
    desc = catq.attn_desc(B, S, Hq, Hkv, d, False, cfg.rope_theta)
    saved = torch.empty(catq.catq_attn_saved_bytes(desc), dtype=torch.uint8, device="cuda")
    ws = torch.empty(catq.catq_attn_bwd_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    o = torch.empty(M, Hq * d, dtype=torch.bfloat16, device="cuda")
    dq = torch.full((M * ld + 64,), 7.0, dtype=torch.bfloat16, device="cuda")
    catq.catq_aux_attention_fwd(desc, qkv, o, saved)
    catq.catq_aux_attention_bwd(desc, qkv, o, saved, dO, dq[:M * ld].view(M, ld), ws)
    torch.cuda.synchronize()
    assert bool((dq[M * ld:] == 7.0).all())
    O, ref = _oracle_attention(f64(qb), cfg, f64(gb))
    # bf16 q, k, v after rotation, P, dS and outputs: a few roundings of 2^-9
    assert max_norm_err(host(o.float()), O) <= 2e-2
    got = host(dq[:M * ld].float()).reshape(M, ld)
    for c0, c1 in ((0, Hq * d), (Hq * d, (Hq + Hkv) * d), ((Hq + Hkv) * d, ld)):
        assert max_norm_err(got[:, c0:c1], ref[:, c0:c1]) <= 2e-2
