"""GPU: the route store where its blocks of consecutive rows meet odd tables:
routes of one row and of many, long runs of invisible routes between visible
ones, layers that end inside a block, and a buffer with rows to spare."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, i32
from paper_2608_19662_amd import recache as rc
from paper_2608_19662_amd.workloads import draw_kept, prefix

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.bfloat16, 64), (torch.float32, 128)])
@pytest.mark.parametrize("n_res,G,p,lens", [
    (1, 1, 1.0, (1, 2)), (1, 8, 1.0, (63, 66)), (700, 8, 0.01, (1, 4)), (300, 3, 0.5, (1, 200)),
    (90, 8, 1.0, (64, 65)),
    # tables around one and two steps of a wave's search
    (8, 8, 0.7, (1, 40)), (13, 5, 1.0, (1, 3)), (512, 8, 0.3, (1, 30)), (683, 6, 0.3, (1, 30)),
])
def test_store_routes_edges(dtype, d, n_res, G, p, lens):
    print("case: store edges", dtype, d, n_res, G, p, lens, flush=True)
    rng = np.random.default_rng(n_res + G)
    lengths = rng.integers(*lens, n_res).astype(np.int32)
    cu, L = prefix(lengths), 2
    cu_kept, kept = draw_kept(rng, lengths, 0.5)
    mask = (rng.random((n_res, L, G)) < p).astype(np.uint8)
    mask[0, :, 0] = mask[-1, :, -1] = 1
    T, K = int(cu[-1]), int(cu_kept[-1])
    kc = torch.randn(G, T, d, device=DEV).to(dtype)
    vc = torch.randn(G, T, d, device=DEV).to(dtype)
    off = torch.empty(L, n_res * G + 1, dtype=torch.int32, device=DEV)
    rc.route_store_offsets(torch.from_numpy(mask).to(DEV), i32(cu_kept), off, total_kept=K)
    h = off.cpu().numpy()
    assert np.array_equal(h, oracle.store_offsets(mask, cu_kept))
    for layer in range(L):
        rows = int(h[layer, -1])
        spare = min(70, G * K - rows)  # a buffer with rows to spare keeps them as they are
        ks = torch.full((rows + spare, d), 7.0, dtype=dtype, device=DEV)
        vs = torch.full_like(ks, 7.0)
        rc.store_routes(kc, vc, i32(cu), i32(cu_kept), i32(kept), off, layer, ks, vs, total_kept=K)
        at = [g * T + cu[r] + kept[j] for r in range(n_res) for g in range(G) if mask[r, layer, g]
              for j in range(cu_kept[r], cu_kept[r + 1])]
        at = torch.tensor(at, dtype=torch.long, device=DEV)
        assert torch.equal(ks[:rows], kc.view(-1, d)[at]) and torch.equal(vs[:rows], vc.view(-1, d)[at])
        assert (ks[rows:] == 7.0).all() and (vs[rows:] == 7.0).all()
