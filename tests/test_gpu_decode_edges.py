"""GPU: decode where its addressing and its split of the key stream change:
KV planes of 4 GiB and more (addressed by pointer, smaller ones through a
buffer resource, whose offsets past 2 GiB have their top bit set), contexts of 512 MiB and more (loaded past the caches), and
ranges that end inside, at and between the resource and context rows of short
and long streams."""
import numpy as np
import pytest
import torch

from gpu_helpers import DEV, Routes, i32
from paper_2608_19662_amd import recache as rc
from test_gpu_parity import print_case, run_attend_case, small_attend

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
def test_decode_plane_of_4_gib(d):
    """The same rows at the end of a plane past 4 GiB and in a small one: the
    same bits."""
    print_case("decode 4 GiB plane", d)
    w = small_attend(141, 1, 4, 4, 1, d, "bf16", [1], [333], L=1, mask_p=2.0)
    rt = Routes(w)
    q, ck, cv, rk, rv = w.layer_tensors(0, DEV)
    mk = rt.max_kv(0)
    ws = rt.workspace(mk)
    out, lse = rt.attend(q, ck, cv, rk, rv, 0, workspace=ws, max_kv=mk)
    rows = (1 << 32) // (2 * d) + 5
    big_k = torch.empty(1, rows, d, dtype=ck.dtype, device=DEV)
    big_v = torch.empty_like(big_k)
    big_k[:, -333:], big_v[:, -333:] = ck, cv
    rt.cu_ctx = i32([rows - 333, rows])
    big, big_lse = rt.attend(q, big_k, big_v, rk, rv, 0, workspace=ws, max_kv=mk)
    torch.cuda.synchronize()
    assert torch.equal(out, big) and torch.equal(lse, big_lse)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("end", [(1 << 31) + (1 << 14), (3 << 30) + (1 << 10), (1 << 32) - (1 << 9)])
def test_decode_plane_past_2_gib(d, end):
    """The same rows across 2 GiB, past it and at the end of the largest plane
    that has 32-bit offsets, for the context and for the resources: the bits of
    a small plane."""
    print_case("decode plane past 2 GiB", d, end)
    w = small_attend(144, 1, 4, 4, 1, d, "bf16", [1], [333], L=1, mask_p=2.0)
    rt = Routes(w)
    q, ck, cv, rk, rv = w.layer_tensors(0, DEV)
    mk = rt.max_kv(0)
    ws = rt.workspace(mk)
    out, lse = rt.attend(q, ck, cv, rk, rv, 0, workspace=ws, max_kv=mk)
    rows = end // (2 * d)
    big_k = torch.empty(1, rows, d, dtype=ck.dtype, device=DEV)
    big_v = torch.empty_like(big_k)
    big_k[:, -333:], big_v[:, -333:] = ck, cv
    cu_ctx, cu_rows = rt.cu_ctx, rt.cu_rows
    rt.cu_ctx = i32([rows - 333, rows])
    big, big_lse = rt.attend(q, big_k, big_v, rk, rv, 0, workspace=ws, max_kv=mk)
    torch.cuda.synchronize()
    assert torch.equal(out, big) and torch.equal(lse, big_lse)
    n = rk.shape[1]
    big_k[:, -n:], big_v[:, -n:] = rk, rv
    rt.cu_ctx, rt.cu_rows = cu_ctx, cu_rows + (rows - n)
    big, big_lse = rt.attend(q, ck, cv, big_k, big_v, 0, workspace=ws, max_kv=mk)
    torch.cuda.synchronize()
    assert torch.equal(out, big) and torch.equal(lse, big_lse)


@pytest.mark.parametrize("Hq,Hkv,d", [(32, 8, 128), (12, 4, 64)])
@pytest.mark.parametrize("ctx", [[1, 31, 32], [33, 127, 128], [129, 4000, 9000]])
def test_decode_ranges(Hq, Hkv, d, ctx):
    print_case("decode ranges", Hq, Hkv, d, ctx)
    w = small_attend(142 + ctx[0], 3, 6, Hq, Hkv, d, "bf16", [1, 1, 1], ctx, L=2, max_len=500)
    for layer in range(2):
        run_attend_case(w, layer)


@pytest.mark.parametrize("Hq,Hkv,d", [(8, 2, 128), (6, 1, 64)])
@pytest.mark.parametrize("ctx", [[1, 5, 31], [32, 200, 1500]])
def test_decode_large_context(Hq, Hkv, d, ctx):
    """The same rows in planes and under a bound on the context that make the
    kernel load them past the caches: the same order of work, the same bits."""
    print_case("decode large context", Hq, Hkv, d, ctx)
    w = small_attend(143 + ctx[0], 3, 6, Hq, Hkv, d, "bf16", [1, 1, 1], ctx, L=1, max_len=500)
    rt = Routes(w)
    q, ck, cv, rk, rv = w.layer_tensors(0, DEV)
    mk = rt.max_kv(0)
    ws = rt.workspace(mk)
    out, lse = rt.attend(q, ck, cv, rk, rv, 0, workspace=ws, max_kv=mk)
    rows = (512 << 20) // (Hkv * d * 4) + 3
    big_k = torch.empty(Hkv, rows, d, dtype=ck.dtype, device=DEV)
    big_v = torch.empty_like(big_k)
    big_k[:, -sum(ctx):], big_v[:, -sum(ctx):] = ck, cv
    rt.cu_ctx = i32(rows - sum(ctx) + np.concatenate([[0], np.cumsum(ctx)]))
    rt.max_ctx = rows
    big, big_lse = rt.attend(q, big_k, big_v, rk, rv, 0, workspace=ws, max_kv=mk)
    torch.cuda.synchronize()
    assert torch.equal(out, big) and torch.equal(lse, big_lse)
