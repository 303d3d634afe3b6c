"""GPU: every form of a prefill launch (keys split over 8 or 4 waves, blocks of
4 or 8 waves) at the sizes where its tiling can go wrong, against the oracle.
The form follows from the 32-column blocks that a call's queries make
(queries x group size / 32, at least one per request, times the KV groups)
and from max_kv, so each case states the form it is there for.

Tolerances are the bf16 rules of gpu_helpers.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, Routes, check, lse_rule

from test_gpu_parity import print_case, small_attend

pytestmark = pytest.mark.gpu


def run(w, layer, max_kv):
    rt = Routes(w)
    q, ck, cv, rk, rv = w.layer_tensors(layer, DEV)
    out, lse = rt.attend(q, ck, cv, rk, rv, layer, max_kv=max_kv)
    pout, plse = rt.attend(q, ck, cv, rk, rv, layer, max_kv=max_kv, plan=rt.plan())
    torch.cuda.synchronize()
    assert torch.equal(out, pout) and torch.equal(lse, plse)
    rout, rlse = oracle.attend(q.cpu(), ck.cpu(), cv.cpu(), w.cu_q, w.cu_ctx, rk.cpu(), rv.cpu(),
                               w.cu_rows, w.req_res_off, w.req_res, w.mask, layer)
    check(out, rout, "bf16", "out")
    check(lse, rlse.T, lse_rule("bf16"), "lse")


EDGES = [1, 2, 7, 8, 9, 31, 32, 33, 65]


@pytest.mark.parametrize("form,n_req,Hq,Hkv,d,q_lens,max_kv", [
    ("split 8", 3, 20, 4, 128, [6, 7, 13], 500),          # 30, 35 and 65 columns per group
    ("split 8", 9, 6, 2, 64, EDGES, 500),
    ("split 4", 40, 32, 8, 128, EDGES, 500),              # 320 blocks
    ("split 4", 36, 24, 8, 64, EDGES, 500),
    ("split 8, blocks numbered over the columns", 41, 8, 1, 128, [1] * 20 + [128] + [1, 3, 9, 1] * 5, 500),
    ("split 8, blocks numbered over the columns", 9, 28, 4, 64, [100, 1, 1, 37, 1, 1, 1, 1, 5], 500),
    ("split 4, blocks numbered over the columns", 300, 8, 1, 128, [1] * 270 + [65] + [2] * 29, 500),
    ("split 4, blocks numbered over the columns", 256, 8, 2, 64, [33] + [1] * 255, 500),
    ("split 4, one block per request", 70, 32, 8, 128, [1, 2, 7, 8], 500),
    ("split 4, one block per request", 70, 56, 8, 64, [1, 4], 500),
    ("blocks of 4", 66, 24, 8, 128, EDGES, 500),          # groups of 3: pairs cross row blocks
    ("blocks of 4", 66, 8, 8, 64, [1, 33, 64, 65], 500),
    ("blocks of 8, one per request", 66, 56, 8, 128, [5, 31, 32], 500),
    ("blocks of 8, full grid", 5, 64, 8, 128, [240, 255, 256, 257, 33], 0),
    ("blocks of 8, full grid", 5, 56, 8, 64, [240, 255, 256, 257, 300], 0),
])
def test_prefill_form_edges(form, n_req, Hq, Hkv, d, q_lens, max_kv):
    print_case("prefill form", form, n_req, Hq, Hkv, d)
    ql = [q_lens[i % len(q_lens)] for i in range(n_req)]
    past = [0, 1, 31, 64, 200]  # causal part from nothing before the queries to several tiles
    w = small_attend(131, n_req, 6, Hq, Hkv, d, "bf16", ql, [q + past[i % 5] for i, q in enumerate(ql)],
                     L=1, max_len=120)
    run(w, 0, max_kv)
