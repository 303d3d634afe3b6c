"""GPU: the fp32 attention kernel at the sizes where its tiling can go wrong:
columns (row, head) that do not fill a 32-column block, group sizes that do
not divide 32, key streams around a 32-key tile and around the four waves'
shares of it, more route segments than one pass of the segment table holds,
and value rows that are not finite where no query of a column may see them.

Tolerance: the fp32 rule of gpu_helpers (1e-5 absolute).  Outputs are
weighted means of N(0, 1) values; a logit is 128 products of magnitude about
1 summed in two chains of 64 (error <= 64 * 2^-24 * 12 / sqrt(128), about
4e-6 in the worst case and 3e-7 in the root mean square).
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, Routes, check, i32
from paper_2608_19662_amd import recache as rc
from paper_2608_19662_amd.workloads import EncodeWorkload

from test_gpu_parity import gpu_encode, many_segments, print_case, run_attend_case, small_attend

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,d", [(8, 8, 128), (6, 2, 64), (20, 4, 128), (24, 2, 64), (40, 1, 128)])
def test_f32_encode_edges(Hq, Hkv, d):
    print_case("f32 encode edges", Hq, Hkv, d)
    w = EncodeWorkload(seed=111, lengths=np.array([1, 31, 32, 33, 127, 128, 129, 161], np.int32),
                       n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, dtype="f32", rope_base=1e4)
    q, k, v = w.tensors("cpu")
    out, kc, vc, lse = gpu_encode(w, q.to(DEV), k.to(DEV), v.to(DEV))
    ref = oracle.encode(q, k, v, w.cu_len, w.rope_base)
    check(out, ref["out"], "f32", "out")
    check(lse, ref["lse"], "f32", "lse")


@pytest.mark.parametrize("Hq,Hkv,d,q_lens,ctx_lens", [
    (8, 8, 64, [1, 32, 33], [1, 32, 65]),
    (20, 4, 128, [6, 7, 13], [6, 39, 140]),     # 30, 35 and 65 columns per group
    (24, 2, 64, [2, 3, 1], [3, 129, 97]),       # 24, 36 and 12 columns
    (40, 1, 128, [1, 1, 1], [1, 31, 300]),      # decode, more heads than one block's columns
])
def test_f32_attend_edges(Hq, Hkv, d, q_lens, ctx_lens):
    print_case("f32 attend edges", Hq, Hkv, d, q_lens, ctx_lens)
    w = small_attend(112, 3, 5, Hq, Hkv, d, "f32", q_lens, ctx_lens, L=2)
    for layer in range(2):
        run_attend_case(w, layer)


@pytest.mark.parametrize("n_res", [1023, 1024, 1025, 2100])
def test_f32_segment_passes(n_res):
    print_case("f32 segments", n_res)
    w = many_segments(113, [9, 1], [40, 5], n_res=n_res)
    w.dtype = "f32"
    rt = Routes(w)
    rt.max_route_len = min(rt.max_route_len, 1024)
    q, ck, cv, rk, rv = w.layer_tensors(0, DEV)
    out, lse = rt.attend(q, ck, cv, rk, rv, 0)
    rout, rlse = oracle.attend(q.cpu(), ck.cpu(), cv.cpu(), w.cu_q, w.cu_ctx, rk.cpu(), rv.cpu(),
                               w.cu_rows, w.req_res_off, w.req_res, w.mask, 0)
    check(out, rout, "f32", "out")
    check(lse, rlse.T, "f32", "lse")


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_f32_unseen_values_do_not_matter(bad):
    """A value row that is not finite reaches the queries that see it, and no
    other: rows before it keep the bits they have with a finite row."""
    print_case("f32 unseen values", bad)
    w = small_attend(114, 1, 3, 8, 2, 128, "f32", [50], [90], L=1, mask_p=2.0)
    rt = Routes(w)
    q, ck, cv, rk, rv = w.layer_tensors(0, DEV)
    a, _ = rt.attend(q, ck, cv, rk, rv, 0)
    row = 63  # context row of query 23
    cv[:, row, 5] = bad
    b, _ = rt.attend(q, ck, cv, rk, rv, 0)
    torch.cuda.synchronize()
    assert torch.equal(a[:23], b[:23])
    assert not torch.isfinite(b[23:, :, 5]).any()
    other = [i for i in range(128) if i != 5]
    assert torch.equal(a[23:, :, other], b[23:, :, other])


@pytest.mark.parametrize("key", [5, 40, 90, 127])
def test_f32_unlikely_values_still_count(key):
    """A visible key whose weight underflows beside the others' keeps its say
    where its value row or its logit is not finite, whichever wave holds it:
    0 times infinity is no zero, and a NaN logit makes the row NaN."""
    print_case("f32 unlikely values", key)
    w = small_attend(115, 1, 2, 8, 2, 128, "f32", [3], [130], L=1, mask_p=0.0)
    rt = Routes(w)
    q, ck, cv, rk, rv = w.layer_tensors(0, DEV)
    q[:] = 1.0
    tile = key // 32 * 32
    ck[:, tile:tile + 32] -= 30.0  # logits of this tile about 340 below the rest
    cv[:, key, 5] = float("inf")
    a, _ = rt.attend(q, ck, cv, rk, rv, 0)
    ck[:, key, 0] = float("nan")
    b, bl = rt.attend(q, ck, cv, rk, rv, 0)
    torch.cuda.synchronize()
    # (query 0 does not see the last two of the 130 context rows)
    assert not torch.isfinite(a[:, :, 5]).any()
    assert torch.isfinite(a[:, :, [i for i in range(128) if i != 5]]).all()
    assert torch.isnan(b).all() and torch.isnan(bl).all()


def at_float(t, n):
    """A copy of t that starts n floats behind a 16-byte boundary."""
    b = torch.empty(t.numel() + 4, dtype=t.dtype, device=DEV)
    v = b[n:n + t.numel()].view(t.shape)
    assert v.data_ptr() % 16 == 4 * n
    return v.copy_(t)


@pytest.mark.parametrize("n", [1, 2, 3])
@pytest.mark.parametrize("Hq,Hkv,d", [(6, 2, 64), (20, 4, 128)])
def test_f32_tensors_at_any_float(Hq, Hkv, d, n):
    """Attention over tensors that start at any float: the bits of the same
    call on 16-byte boundaries, with all of them shifted and with one."""
    print_case("f32 alignment", Hq, Hkv, d, n)
    w = small_attend(116, 3, 5, Hq, Hkv, d, "f32", [6, 1, 33], [39, 1, 140], L=1)
    rt = Routes(w)
    ts = w.layer_tensors(0, DEV)
    assert all(t.data_ptr() % 16 == 0 for t in ts)
    want, want_lse = rt.attend(*ts, 0)
    for which in [range(5), *([i] for i in range(5))]:
        got, lse = rt.attend(*[at_float(t, n) if i in which else t for i, t in enumerate(ts)], 0)
        torch.cuda.synchronize()
        assert torch.equal(got, want) and torch.equal(lse, want_lse), which

    e = EncodeWorkload(seed=117, lengths=np.array([1, 33, 129], np.int32), n_q_heads=Hq, n_kv_heads=Hkv,
                       head_dim=d, dtype="f32", rope_base=1e4)
    q, k, v = (t.to(DEV) for t in e.tensors("cpu"))
    want, kc, vc, want_lse = gpu_encode(e, q, k, v)
    for shift in (lambda t: at_float(t, n), lambda t: t):
        got = at_float(torch.zeros_like(q), n)
        lse = torch.empty_like(want_lse)
        rc.encode_attention(shift(q), shift(kc), shift(vc), i32(e.cu_len), 129, e.rope_base, got, lse=lse)
        torch.cuda.synchronize()
        assert torch.equal(got, want) and torch.equal(lse, want_lse)
