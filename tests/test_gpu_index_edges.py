"""GPU: route lists and work orders where their kernels' units meet odd sizes:
a slice of 64 (layer, group) entries per wave, 64 staged resources per step,
one pair per thread up to 1024 pairs, and a mask that is not word-aligned.
Bit-exact against the oracle and the plain Python order."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, Routes, i32, plan_reference
from paper_2608_19662_amd import recache as rc
from paper_2608_19662_amd.workloads import prefix
from test_gpu_plan import random_structure

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_req,pool,L,G,per", [
    (1, 1, 1, 1, (1, 2)), (3, 70, 8, 8, (0, 70)), (2, 130, 13, 5, (63, 66)), (5, 200, 36, 8, (0, 180)),
    (1030, 9, 1, 3, (0, 4)),
    # many requests of few entries: lanes of several requests in a wave
    (4097, 30, 1, 1, (0, 12)), (5001, 40, 5, 3, (0, 18)), (8200, 6, 2, 8, (0, 6)), (20001, 9, 1, 3, (0, 3)),
    # and where a wave takes one of them: long lists, as many waves as fit
    (4097, 70, 1, 2, (30, 70)), (4096, 9, 2, 2, (0, 4)), (9, 300, 2, 3, (7, 20)),
    # few entries and short lists, with a long one every so many requests
    (65, 90, 1, 1, (0, 7)), (64, 90, 1, 1, (1, 4, 20, 33)), (130, 300, 1, 1, (0, 3, 7, 90)),
    (50, 300, 2, 5, (0, 3, 11, 130)), (700, 90, 1, 3, (0, 2, 50, 64)), (2000, 300, 1, 1, (0, 2, 63, 300)),
    (7, 30, 36, 8, (0, 5)), (60, 90, 13, 5, (0, 3, 30, 80)),
])
def test_routes_edges(n_req, pool, L, G, per):
    print("case: route edges", n_req, pool, L, G, per, flush=True)
    rng = np.random.default_rng(n_req + L)
    kept = prefix(rng.integers(1, 50, pool))
    reqs = [rng.permutation(pool)[:rng.integers(*per[:2]) if len(per) == 2 or b % per[2] else per[3]]
            for b in range(n_req)]
    off, res = prefix([len(r) for r in reqs]), np.concatenate(reqs).astype(np.int32)
    mask = (rng.random((pool, L, G)) < 0.4).astype(np.uint8) * 3  # any non-zero byte is set
    E = n_req * L * G
    ro = torch.full((E + 1,), -1, dtype=torch.int32, device=DEV)
    rr = torch.full((max(len(res), 1) * L * G,), -1, dtype=torch.int32, device=DEV)
    rt = torch.full((E,), -1, dtype=torch.int32, device=DEV)
    rc.build_routes(i32(off), i32(res), torch.from_numpy(mask).to(DEV), i32(kept), ro, rr, rt)
    a, b, t = oracle.routes(off, res, mask, kept)
    assert np.array_equal(ro.cpu().numpy(), a)
    assert np.array_equal(rr.cpu().numpy()[:a[-1]], b)
    assert np.array_equal(rt.cpu().numpy(), t)
    # the store's row tables from an aligned mask and from one a byte off a word
    want = oracle.store_offsets(mask, kept)
    flat = torch.zeros(mask.size + 1, dtype=torch.uint8, device=DEV)
    flat[1:] = torch.from_numpy(mask.reshape(-1)).to(DEV)
    for m in (torch.from_numpy(mask).to(DEV), flat[1:].view(pool, L, G)):
        so = torch.full((L, pool * G + 1), -1, dtype=torch.int32, device=DEV)
        rc.route_store_offsets(m, i32(kept), so, total_kept=int(kept[-1]))
        assert np.array_equal(so.cpu().numpy(), want)


@pytest.mark.parametrize("n_req,Hkv", [(1, 1), (63, 1), (64, 1), (13, 5), (128, 8), (129, 8)])
def test_plan_edges(n_req, Hkv):
    print("case: plan edges", n_req, Hkv, flush=True)
    w = random_structure(151 + n_req, n_req, 4 * Hkv, Hkv, 2, 3, 5)  # many equal works
    rt = Routes(w)
    got = rt.plan().cpu().numpy()
    assert np.array_equal(got, plan_reference(w.cu_q, w.cu_ctx, rt.route_tokens.cpu().numpy(), 2, 4 * Hkv, Hkv))
