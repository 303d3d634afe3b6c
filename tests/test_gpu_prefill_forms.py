"""GPU: every form of a prefill launch (keys split over 8 or 4 waves, blocks of
4 or 8 waves) at the sizes where its tiling can go wrong, against the oracle,
and over what each form handles for itself: route lists at and past the limit,
a route-compacted store, rows past max_q, a moving softmax reference.
The form follows from the 32-column blocks that a call's queries make
(queries x group size / 32, at least one per request, times the KV groups)
and from max_kv: form() states the rule, and every case the form it is for.

Tolerances are the bf16 rules of gpu_helpers.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, Routes, check, lse_rule

from test_gpu_parity import many_segments, print_case, run_attend_case, run_store_case, small_attend
from test_gpu_softmax import ramp

pytestmark = pytest.mark.gpu


def form(w, max_kv, max_q=None):
    """The form that the library's rules choose for the call, as it is named in the cases."""
    total_q, max_q, ratio = int(np.sum(w.q_lens)), max_q or int(np.max(w.q_lens)), w.n_q_heads // w.n_kv_heads
    n = max(-(-total_q * ratio // 32), w.n_req) * w.n_kv_heads
    if n <= 512 or max_q * ratio <= 32:
        waves = 8 if n <= 256 else 4
        per_req = -(-max_q * ratio // 32)
        numbered = per_req > 1 and w.n_req > 1 and per_req * w.n_req * w.n_kv_heads > 2048 // waves
        one = "" if n <= 512 else ", one block per request"
        return "split %d%s" % (waves, ", blocks numbered over the columns" if numbered else one)
    if n >= 2048 and (max_kv <= 0 or max_kv >= 4096):
        return "blocks of 8, full grid"
    return "blocks of 8, one per request" if max_q <= 32 and ratio > 4 else "blocks of 4"


def run(w, layer, max_kv, tensors=None):
    rt = Routes(w)
    q, ck, cv, rk, rv = tensors or w.layer_tensors(layer, DEV)
    out, lse = rt.attend(q, ck, cv, rk, rv, layer, max_kv=max_kv)
    pout, plse = rt.attend(q, ck, cv, rk, rv, layer, max_kv=max_kv, plan=rt.plan())
    torch.cuda.synchronize()
    assert torch.equal(out, pout) and torch.equal(lse, plse)
    rout, rlse = oracle.attend(q.cpu(), ck.cpu(), cv.cpu(), w.cu_q, w.cu_ctx, rk.cpu(), rv.cpu(),
                               w.cu_rows, w.req_res_off, w.req_res, w.mask, layer)
    check(out, rout, "bf16", "out")
    check(lse, rlse.T, lse_rule("bf16"), "lse")


EDGES = [1, 2, 7, 8, 9, 31, 32, 33, 65]


@pytest.mark.parametrize("name,n_req,Hq,Hkv,d,q_lens,max_kv", [
    ("split 8", 3, 20, 4, 128, [6, 7, 13], 500),          # 30, 35 and 65 columns per group
    ("split 8", 9, 6, 2, 64, EDGES, 500),
    ("blocks of 4", 40, 32, 8, 128, EDGES, 500),
    ("blocks of 4", 36, 24, 8, 64, EDGES, 500),
    ("split 4", 4, 32, 8, 128, [65, 63, 64, 65], 500),    # 264 blocks
    ("split 4", 5, 24, 8, 64, [97, 95, 96, 89, 97], 500),  # 360, some rows over two blocks
    ("split 4, blocks numbered over the columns", 18, 32, 8, 128, EDGES, 500),
    ("split 4, blocks numbered over the columns", 18, 24, 8, 64, EDGES, 500),
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
def test_prefill_form_edges(name, n_req, Hq, Hkv, d, q_lens, max_kv):
    print_case("prefill form", name, n_req, Hq, Hkv, d)
    ql = [q_lens[i % len(q_lens)] for i in range(n_req)]
    past = [0, 1, 31, 64, 200]  # causal part from nothing before the queries to several tiles
    w = small_attend(131, n_req, 6, Hq, Hkv, d, "bf16", ql, [q + past[i % 5] for i, q in enumerate(ql)],
                     L=1, max_len=120)
    assert form(w, max_kv) == name
    run(w, 0, max_kv)


# calls of each form with 8 KV heads: query heads and query rows
FORMS = [
    ("split 4", 32, [100, 64, 100]),
    ("split 4, blocks numbered over the columns", 32, [200] + [2] * 39),
    ("blocks of 4", 32, [300, 70, 200]),
    ("blocks of 8, one per request", 64, [31, 32, 30, 29, 32, 31, 32, 30, 32]),
]
FULL = ("blocks of 8, full grid", 64, [300, 240, 255, 256, 200])


def past(q_lens):
    return [q + (0, 37, 150)[i % 3] for i, q in enumerate(q_lens)]


@pytest.mark.parametrize("name,Hq,q_lens", FORMS)
def test_route_lists_at_the_limit(name, Hq, q_lens):
    """1024 tiny resources visible to every request: key tiles of many
    segments, over the per-head kept rows and over a route-compacted store."""
    print_case("prefill form, 1024 segments", name)
    w = many_segments(132, q_lens, past(q_lens), Hq=Hq)
    assert form(w, Routes(w).max_kv(0)) == name
    run_attend_case(w, 0)
    run_store_case(w, 1)


@pytest.mark.parametrize("name,Hq,q_lens", FORMS)
@pytest.mark.parametrize("d", [64, 128])
def test_store(name, Hq, q_lens, d):
    print_case("prefill form, route store", name, d)
    w = small_attend(133, len(q_lens), 6, Hq, 8, d, "bf16", q_lens, past(q_lens), L=1, max_len=300)
    assert form(w, Routes(w).max_kv(0)) == name
    run_store_case(w, 0)


@pytest.mark.parametrize("name,Hq,q_lens", FORMS + [FULL])
def test_route_list_over_the_limit(name, Hq, q_lens):
    print_case("prefill form, guard: route list over 1024", name)
    w = many_segments(134, q_lens, past(q_lens), n_res=1100, Hq=Hq)
    rt = Routes(w)
    rt.max_route_len = 1024  # understates the 1100 resources every request lists
    assert form(w, 0) == name
    out, lse = rt.attend(*w.layer_tensors(0, DEV), 0)
    torch.cuda.synchronize()
    assert torch.isnan(out.float()).all() and torch.isnan(lse).all()


@pytest.mark.parametrize("name,Hq,q_lens,max_q,done,bad", [
    # of request 0: rows [0, done) are computed, rows from `bad` on NaN (a
    # block form answers for all rows of its last row block, a split for none)
    ("split 8", 32, [100, 1, 64], 60, 60, 60),
    ("split 4", 32, [100, 64, 100], 88, 88, 88),
    ("split 4, blocks numbered over the columns", 32, [200] + [2] * 39, 150, 150, 150),
    ("blocks of 4", 32, [300, 70, 200], 192, 160, 192),
    ("blocks of 8, one per request", 64, [64] + [25] * 8, 32, 0, 32),
    ("blocks of 8, full grid", 64, [300, 240, 255, 256, 200], 256, 224, 256),
])
def test_queries_past_max_q(name, Hq, q_lens, max_q, done, bad):
    print_case("prefill form, guard: max_q", name)
    w = small_attend(135, len(q_lens), 4, Hq, 8, 128, "bf16", q_lens, past(q_lens), L=1)
    rt = Routes(w)
    rt.max_q = max_q  # understates request 0's queries
    assert form(w, 0, max_q) == name
    out, lse = rt.attend(*w.layer_tensors(0, DEV), 0)
    torch.cuda.synchronize()
    n = q_lens[0]
    assert torch.isfinite(out[:done].float()).all() and torch.isfinite(lse[:, :done]).all()
    assert torch.isnan(out[bad:n].float()).all() and torch.isnan(lse[:, bad:n]).all()
    for b, q in enumerate(q_lens):
        if q <= max_q:
            rows = slice(int(w.cu_q[b]), int(w.cu_q[b + 1]))
            assert torch.isfinite(out[rows].float()).all() and torch.isfinite(lse[:, rows]).all(), b


@pytest.mark.parametrize("name,Hq,q_lens", FORMS + [FULL])
def test_reference_moves(name, Hq, q_lens):
    """Keys that rise along their buffers, with a spike in each."""
    print_case("prefill form, softmax reference", name)
    w = small_attend(136, len(q_lens), 6, Hq, 8, 128, "bf16", q_lens, past(q_lens), L=1, max_len=400, mask_p=0.7)
    max_kv = 0 if name == FULL[0] else Routes(w).max_kv(0)
    assert form(w, max_kv) == name
    ts = w.layer_tensors(0, DEV)
    q, ck, _, rk, _ = ts
    q[:, :, 0] = 4.0
    for k, spike in ((ck, 700.0), (rk, 900.0)):
        k[:, :, 0] = ramp(k.shape[1], 0.25, k.dtype).to(DEV)[None, :]
        k[:, k.shape[1] // 2, 0] = spike
    run(w, 0, max_kv, ts)
