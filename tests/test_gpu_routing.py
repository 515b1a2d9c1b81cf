"""Expert routing at the edges of its ids' segments and of its logits per lane."""
import numpy as np
import pytest
import torch

import paper_2606_26650_amd as catq

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("T,E,k", [(1, 1, 1), (3, 8, 8), (255, 4, 1), (256, 4, 2), (4097, 64, 2),
                                   (513, 65, 8), (300, 129, 16), (70, 1024, 3)])
def test_routing(T, E, k):
    g = torch.Generator().manual_seed(T + E)
    logits = torch.randn((T, E), generator=g)
    logits[:, -1] = logits[:, 0]           # ties go to the lower id
    if E > 8:
        logits[:, 3] = -10.0               # an expert without rows
    ids = torch.empty((T, k), dtype=torch.int32, device=DEV)
    wts = torch.empty((T, k), device=DEV)
    perm = torch.empty((T, k), dtype=torch.int32, device=DEV)
    offs = torch.empty(E + 1, dtype=torch.int64, device=DEV)
    ws = torch.empty(catq.catq_aux_moe_route_workspace_bytes(T, E, k), dtype=torch.uint8, device=DEV)
    catq.catq_aux_moe_route(logits.to(DEV), k, ids, wts, perm, offs, ws)
    order = np.lexsort((np.broadcast_to(np.arange(E), (T, E)), -logits.numpy()), axis=1)[:, :k]
    np.testing.assert_array_equal(ids.cpu().numpy(), order)
    sel = np.take_along_axis(logits.double().numpy(), order, 1)
    w = np.exp(sel - sel[:, :1])
    np.testing.assert_allclose(wts.cpu().numpy(), w / w.sum(1, keepdims=True), rtol=2e-6)
    flat = order.reshape(-1)
    cnt = np.bincount(flat, minlength=E)
    np.testing.assert_array_equal(offs.cpu().numpy(), np.concatenate([[0], np.cumsum(cnt)]))
    rows = np.empty(T * k, dtype=np.int64)
    rows[np.argsort(flat, kind="stable")] = np.arange(T * k)
    np.testing.assert_array_equal(perm.cpu().numpy().reshape(-1), rows)
