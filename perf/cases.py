"""Timed cases of the framework's main paths, through the Python entry points.

Every case is one attention layer's share of a serving program (one call chain
of the 36 that a pass makes), at the head layouts, resource lengths, route
densities and kept fractions of the repository's workloads and tests:

  encode   a pool of tool schemas becomes KV blocks: encode_resources, with a
           shared prefix where there is one, then prune_gather of its kept rows
  attend   conversation tokens over cached resources: attend_cached, prefill
           (several queries per request) or decode (one)
  step     one decode step of one conversation: rope_q and rope_kv of the new
           token, then attend_cached_noalloc over the caches
  store    the per-batch index work and one layer of a route-compacted store:
           build_routes, attend_plan, route_store_offsets, store_routes
  chain    a request that brings its own tools: encode_resources,
           prune_gather, attend_cached on what these wrote

Inputs are seeded N(0, 1) tensors, as the framework's workloads draw them.
"""
import math
import zlib

import numpy as np
import torch

from paper_2608_19662_amd import recache as rc
from paper_2608_19662_amd.workloads import (draw_kept, draw_lengths, draw_route_mask_exact, prefix)

DEV = "cuda"
LAYERS = 36     # layers of the served model; a case runs one of them
BASE = 1e6      # RoPE base
ENCODE = dict(kind="encode", dtype="bf16", hq=32, hkv=8, d=128, n_res=16, len_lo=200, len_hi=1500,
              prefix=0, keep=0.0, lse=False)
ATTEND = dict(kind="attend", dtype="bf16", hq=32, hkv=8, d=128, n_req=8, per_req=8, pool=64,
              len_lo=300, len_hi=1200, keep=1.0, routes=1.0, q_lo=2048, q_hi=2048, past_lo=0,
              past_hi=0, store=False, plan=True, lse=False)
PRUNED = dict(keep=0.3, routes=0.25)


def listed():
    return [
        # one new token of one conversation with eight tools: the latency of a
        # step for a single user, launches included
        dict(ATTEND, **PRUNED, name="decode_one", kind="step", n_req=1, pool=8, q_lo=1, q_hi=1,
             past_lo=3000, past_hi=3000, store=True, plan=False),
        # a moderate batch in mid-conversation, contexts of very unequal
        # length, tools shared from a common pool, smaller model (16 / 8 heads)
        dict(ATTEND, **PRUNED, name="decode_ragged", hq=16, n_req=12, per_req=12, pool=48,
             len_lo=100, q_lo=1, q_hi=1, past_lo=60, past_hi=9000, store=True, plan=False, lse=True),
        # full-rate batched decode: 64 conversations over 32 tools each
        dict(ATTEND, **PRUNED, name="decode_batch", n_req=64, per_req=32, pool=2048, len_lo=200,
             len_hi=2000, q_lo=1, q_hi=1, past_lo=4095, past_hi=4095),
        # a user's next message (a few dozen tokens) in a running conversation
        dict(ATTEND, **PRUNED, name="turn_one", n_req=1, pool=8, q_lo=75, q_hi=75, past_lo=2600,
             past_hi=2600, plan=False),
        # chunks of several prompts and messages at once, ragged in both lengths
        dict(ATTEND, **PRUNED, name="turn_batch", n_req=6, per_req=10, pool=40, len_lo=100, q_lo=17,
             q_hi=500, past_lo=0, past_hi=5000, store=True, lse=True),
        # first pass over long prompts, pruned routes and tokens
        dict(ATTEND, **PRUNED, name="prefill_pruned"),
        # the same with everything visible: the largest call
        dict(ATTEND, name="prefill_full"),
        # one tool is registered
        dict(ENCODE, name="encode_one", n_res=1, len_lo=611, len_hi=611, keep=0.3),
        # a request's tools are encoded together
        dict(ENCODE, name="encode_pool"),
        # a tool catalogue after a system prompt, 28 / 4 heads, pruned as it is built
        dict(ENCODE, name="encode_catalogue", hq=28, hkv=4, n_res=40, len_lo=30, len_hi=900,
             prefix=300, keep=0.3, lse=True),
        # the index work of a large decode batch and one layer of its store
        dict(ATTEND, **PRUNED, name="store_batch", kind="store", n_req=64, per_req=32, pool=2048,
             len_lo=200, len_hi=2000, q_lo=1, q_hi=1, past_lo=4095, past_hi=4095),
        # the fp32 path, as a precision reference for a bf16 deployment
        dict(ATTEND, name="fp32_chain", kind="chain", dtype="f32", n_req=2, per_req=3, pool=6,
             len_lo=100, len_hi=500, keep=0.3, routes=0.5, q_lo=150, q_hi=250, past_lo=0,
             past_hi=200, plan=False, lse=True),
    ]


def _span(rng, lo, hi):
    """A whole number, uniform in its logarithm over lo .. hi."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("step", "decode", "decode", "prefill", "prefill", "prefill", "encode", "encode",
                       "store", "chain"))
    hq, hkv, d = rng.choice(((32, 8, 128), (32, 8, 128), (16, 8, 128), (28, 4, 128), (64, 8, 128),
                             (8, 8, 128), (8, 2, 64), (12, 4, 64)))
    heads = dict(hq=hq, hkv=hkv, d=d, lse=rng.random() < 0.5)
    lo = _span(rng, 20, 400)
    lens = dict(len_lo=lo, len_hi=lo + _span(rng, 1, 1500))
    if kind == "encode":
        return dict(ENCODE, **heads, **lens, n_res=_span(rng, 1, 48),
                    prefix=rng.choice((0, 0, _span(rng, 1, 600))), keep=rng.choice((0.0, 0.3)))
    pruned = PRUNED if rng.random() < 0.6 else {}
    common = dict(heads, **lens, **pruned)
    if kind == "step":
        per = _span(rng, 1, 32)
        past = _span(rng, 1, 20000)
        return dict(ATTEND, **common, kind="step", n_req=1, per_req=per, pool=per, q_lo=1, q_hi=1,
                    past_lo=past, past_hi=past, store=rng.random() < 0.5, plan=False)
    if kind == "store":
        n, per = _span(rng, 1, 64), _span(rng, 1, 32)
        return dict(ATTEND, **common, kind="store", n_req=n, per_req=per,
                    pool=max(per, _span(rng, 1, 600)), q_lo=1, q_hi=1, past_lo=64, past_hi=4000)
    if kind == "chain":
        n, per = _span(rng, 1, 4), _span(rng, 1, 4)
        q = _span(rng, 1, 250)
        return dict(ATTEND, **dict(common, len_hi=lo + _span(rng, 1, 200)), kind="chain",
                    dtype=rng.choice(("f32", "f32", "bf16")), n_req=n, per_req=per,
                    pool=per + rng.randrange(4), q_lo=1 if q > 4 else q, q_hi=q, past_lo=0,
                    past_hi=_span(rng, 1, 400), plan=False)
    per = _span(rng, 1, 24)
    if kind == "decode":
        n = _span(rng, 1, 64)
        return dict(ATTEND, **common, n_req=n, per_req=per, pool=max(per, _span(rng, 1, 200)), q_lo=1,
                    q_hi=1, past_lo=_span(rng, 1, 2000), past_hi=_span(rng, 2000, 160000 // (n + 12)),
                    store=rng.random() < 0.5, plan=rng.random() < 0.5)
    n = _span(rng, 1, 10)
    # at most about half the pairs of the largest listed case
    q = min(_span(rng, 2, 2048), 16000 // n, 260000 // (hq * n) + 2)
    return dict(ATTEND, **common, n_req=n, per_req=min(per, 12), pool=min(per, 12) + rng.randrange(40),
                q_lo=max(1, q // rng.choice((1, 4, 30))), q_hi=q, past_lo=0, past_hi=_span(rng, 1, 4000),
                store=rng.random() < 0.5, plan=rng.random() < 0.5)


# ------------------------------------------------------------------ structure

def _i32(a):
    return torch.from_numpy(np.ascontiguousarray(np.asarray(a, np.int32))).to(DEV)


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _structure(case, seed):
    """Host-side lengths, kept lists, requests and route masks of a case.  The
    sizes, requests and routes belong to the case (outputs of every seed have
    one shape); which tokens are kept comes from the seed."""
    rng = np.random.default_rng(zlib.crc32(repr(sorted(case.items())).encode()))
    S = {}
    n_res = case["n_res"] if case["kind"] == "encode" else case["pool"]
    S["len"] = draw_lengths(rng, n_res, case["len_lo"], case["len_hi"])
    S["cu_len"] = prefix(S["len"])
    keep = case["keep"]
    if 0.0 < keep < 1.0:
        S["cu_kept"], S["kept"] = draw_kept(np.random.default_rng(seed), S["len"], keep)
    else:
        S["cu_kept"] = S["cu_len"]
        S["kept"] = np.concatenate([np.arange(n, dtype=np.int32) for n in S["len"]])
    if case["kind"] == "encode":
        return S
    n, per, G = case["n_req"], case["per_req"], case["hkv"]
    if n * per == n_res:
        S["req_res"] = np.arange(n_res, dtype=np.int32)
    else:
        S["req_res"] = np.concatenate([rng.permutation(n_res)[:per] for _ in range(n)]).astype(np.int32)
    S["req_off"] = prefix([per] * n)
    if case["routes"] < 1.0:
        S["mask"] = draw_route_mask_exact(rng, n_res, LAYERS, G, case["routes"])
    else:
        S["mask"] = np.ones((n_res, LAYERS, G), np.uint8)
    q = rng.integers(case["q_lo"], case["q_hi"] + 1, n)
    past = rng.integers(case["past_lo"], case["past_hi"] + 1, n)
    S["q"], S["ctx"] = q.astype(np.int32), (q + past).astype(np.int32)
    S["cu_q"], S["cu_ctx"] = prefix(S["q"]), prefix(S["ctx"])
    S["layer"] = int(rng.integers(LAYERS))
    kl = np.diff(S["cu_kept"]).astype(np.int64)
    lists = S["req_res"].reshape(n, per)
    S["vis"] = (kl[lists][:, :, None] * S["mask"][lists, S["layer"]]).sum(1)  # [n][G] visible rows
    S["rows"] = (kl[:, None] * S["mask"][:, S["layer"]]).reshape(-1)          # rows of each route
    S["n_routes"] = int(S["mask"][lists].astype(np.int64).sum())
    return S


class _Normal:
    """Seeded N(0, 1) tensors on the GPU, one after another."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed))

    def __call__(self, dtype, *shape):
        return torch.randn(*shape, generator=self.g, device=DEV, dtype=dtype)


def _encode_inputs(case, S, N):
    T, dt = int(S["cu_len"][-1]), _dtype(case)
    hq, G, d, P = case["hq"], case["hkv"], case["d"], case.get("prefix", 0)
    I = {"q": N(dt, T, hq, d), "k": N(dt, T, G, d), "v": N(dt, T, G, d)}
    if P:
        I["pk"], I["pv"] = N(dt, G, P, d), N(dt, G, P, d)
    return I


def _attend_inputs(case, S, N):
    dt = _dtype(case)
    hq, G, d = case["hq"], case["hkv"], case["d"]
    tq, tc = int(S["cu_q"][-1]), int(S["cu_ctx"][-1])
    I = {"q": N(dt, tq, hq, d), "ck": N(dt, G, tc, d), "cv": N(dt, G, tc, d)}
    if case["kind"] == "step":
        I["k_new"], I["v_new"] = N(dt, 1, G, d), N(dt, 1, G, d)
    if case["kind"] != "chain":
        shape = (int(S["rows"].sum()), d) if case["store"] else (G, int(S["cu_kept"][-1]), d)
        I["rk"], I["rv"] = N(dt, *shape), N(dt, *shape)
    return I


def _store_inputs(case, S, N):
    T, G, d = int(S["cu_len"][-1]), case["hkv"], case["d"]
    return {"kc": N(_dtype(case), G, T, d), "vc": N(_dtype(case), G, T, d)}


def _new(like, *shape, dtype=None):
    """An output buffer, filled once so that nothing in it is left undefined."""
    return torch.zeros(*shape, dtype=dtype or like.dtype, device=DEV)


# ------------------------------------------------------------------ prepare and run

def prepare(case, seed):
    S, N = _structure(case, seed), _Normal(seed)
    st = {"case": case, "cu_kept": _i32(S["cu_kept"]), "kept": _i32(S["kept"]), "cu_len": _i32(S["cu_len"])}
    kind, hq, G, d = case["kind"], case["hq"], case["hkv"], case["d"]
    T, K = int(S["cu_len"][-1]), int(S["cu_kept"][-1])
    if kind in ("encode", "chain"):
        I = _encode_inputs(case, S, N)
        st["enc"], st["max_len"] = I, int(S["len"].max())
        st["enc_out"] = torch.zeros_like(I["q"])
        st["kc"], st["vc"] = _new(I["q"], G, T, d), _new(I["q"], G, T, d)
        st["enc_lse"] = _new(I["q"], hq, T, dtype=torch.float32) if case["lse"] else None
        if case.get("prefix"):
            st["pos_base"] = torch.full((len(S["len"]),), case["prefix"], dtype=torch.int32, device=DEV)
        if case["keep"]:
            st["kk"], st["vk"] = _new(I["q"], G, K, d), _new(I["q"], G, K, d)
        if kind == "encode":
            return st
    E, n, L = case["n_req"] * LAYERS * G, case["n_req"], LAYERS
    st["routes"] = (_i32(S["req_off"]), _i32(S["req_res"]), torch.from_numpy(S["mask"]).to(DEV),
                    st["cu_kept"])
    st["route_out"] = (_new(None, E + 1, dtype=torch.int32),
                       _new(None, len(S["req_res"]) * L * G, dtype=torch.int32),
                       _new(None, E, dtype=torch.int32))
    rc.build_routes(*st["routes"], *st["route_out"])
    st["cu_q"], st["cu_ctx"], st["layer"] = _i32(S["cu_q"]), _i32(S["cu_ctx"]), S["layer"]
    st["plan"] = None
    if case["plan"] or kind == "store":
        st["plan"] = _new(None, L, n * G, dtype=torch.int32)
        rc.attend_plan(st["cu_q"], st["cu_ctx"], st["route_out"][2], L, hq, G, st["plan"])
    st["res_off"] = None
    if case["store"] or kind == "store":
        st["store_off"] = _new(None, L, case["pool"] * G + 1, dtype=torch.int32)
        rc.route_store_offsets(st["routes"][2], st["cu_kept"], st["store_off"], total_kept=K)
        st["res_off"] = st["store_off"][st["layer"]]
    st["total_kept"] = K
    if kind == "store":
        st.update(_store_inputs(case, S, N))
        rows = int(S["rows"].sum())
        st["ks"], st["vs"] = _new(st["kc"], rows, d), _new(st["kc"], rows, d)
        return st
    I = _attend_inputs(case, S, N)
    st.update(I)
    if kind == "chain":
        st["rk"], st["rv"] = (st["kk"], st["vk"]) if case["keep"] < 1.0 else (st["kc"], st["vc"])
    st["out"] = torch.zeros_like(I["q"])
    st["lse"] = _new(None, hq, I["q"].shape[0], dtype=torch.float32) if case["lse"] else None
    st["max_q"], st["max_ctx"] = int(S["q"].max()), int(S["ctx"].max())
    st["max_kv"] = int((S["vis"].max(1) + S["ctx"]).max())
    nb = rc.attend_workspace_bytes(n, st["max_q"], st["max_ctx"], st["max_kv"], hq, G, d)
    st["ws"] = torch.empty(nb // 4, dtype=torch.float32, device=DEV) if nb and kind != "step" else None
    if kind == "step":
        st["pos"] = torch.full((1,), T + int(S["ctx"][0]) - 1, dtype=torch.int32, device=DEV)
        st["q_rot"] = torch.empty_like(I["q"])
    return st


def _run_encode(st):
    I, case = st["enc"], st["case"]
    rc.encode_resources(I["q"], I["k"], I["v"], st["cu_len"], st["max_len"], BASE, st["enc_out"], st["kc"],
                        st["vc"], lse=st["enc_lse"], pos_base=st.get("pos_base"), prefix_k=I.get("pk"),
                        prefix_v=I.get("pv"))
    got = [st["enc_out"], st["kc"], st["vc"], st["enc_lse"]]
    if 0.0 < case["keep"] < 1.0:
        rc.prune_gather(st["kc"], st["vc"], st["cu_len"], st["cu_kept"], st["kept"], st["kk"], st["vk"])
        got += [st["kk"], st["vk"]]
    return got


def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "encode":
        return _run_encode(st)
    if kind == "store":
        rc.build_routes(*st["routes"], *st["route_out"])
        rc.attend_plan(st["cu_q"], st["cu_ctx"], st["route_out"][2], LAYERS, case["hq"], case["hkv"], st["plan"])
        rc.route_store_offsets(st["routes"][2], st["cu_kept"], st["store_off"], total_kept=st["total_kept"])
        rc.store_routes(st["kc"], st["vc"], st["cu_len"], st["cu_kept"], st["kept"], st["store_off"],
                        st["layer"], st["ks"], st["vs"], total_kept=st["total_kept"])
        return [*st["route_out"], st["plan"], st["store_off"], st["ks"], st["vs"]]
    got = _run_encode(st) if kind == "chain" else []
    q = st["q"]
    args = (st["ck"], st["cv"], st["cu_q"], st["cu_ctx"], st["max_q"], st["max_ctx"], st["rk"], st["rv"],
            st["cu_kept"], *st["route_out"], st["layer"], LAYERS, st["out"])
    more = dict(max_route_len=case["per_req"], lse=st["lse"], max_kv=st["max_kv"], res_off=st["res_off"],
                plan=st["plan"])
    if kind == "step":
        # the copy stands for the projection that writes a fresh query each step
        q = st["q_rot"].copy_(q)
        rc.rope_q(q, st["pos"], BASE)
        rc.rope_kv(st["k_new"], st["v_new"], st["pos"], BASE, st["ck"], st["cv"], row0=st["max_ctx"] - 1)
        rc.attend_cached_noalloc(q, *args, **more)
        return [st["out"], st["lse"], st["ck"][:, -1], st["cv"][:, -1]]
    rc.attend_cached(q, *args, workspace=st["ws"], **more)
    return got + [st["out"], st["lse"]]


# ------------------------------------------------------------------ work and tolerance

def work(case):
    S, G, d = _structure(case, 1), case["hkv"], case["d"]
    row = d * (4 if case["dtype"] == "f32" else 2)
    b = f = 0.0
    T, K = float(S["cu_len"][-1]), float(S["cu_kept"][-1])
    if case["kind"] in ("encode", "chain"):
        n = S["len"].astype(np.float64)
        P = case.get("prefix", 0)
        f += 4.0 * d * case["hq"] * float((n * (n + 1) / 2 + n * P).sum())
        b += row * (2 * T * case["hq"] + 4 * T * G + 2 * P * G)
        if 0.0 < case["keep"] < 1.0:
            b += row * 4 * K * G
    if case["kind"] == "encode":
        return {"bytes": b, "flops": f}
    rows = float(S["rows"].sum())
    if case["kind"] == "store":
        E = case["n_req"] * LAYERS * G
        index = S["mask"].size + 4.0 * (3 * E + S["n_routes"] + LAYERS * case["pool"] * G)
        return {"bytes": index + row * 4 * rows, "flops": 0.0}
    q, ctx = S["q"].astype(np.float64)[:, None], S["ctx"].astype(np.float64)[:, None]
    pairs = q * S["vis"] + q * (q + 1) / 2 + q * (ctx - q)     # per query head of a group
    f += 4.0 * d * (case["hq"] // G) * float(pairs.sum())
    b += row * 2 * (float(S["vis"].sum()) + float(ctx.sum()) * G) + row * 2 * float(q.sum()) * case["hq"]
    return {"bytes": b, "flops": f}


def tolerance(case):
    # bf16: rounding of rotated rows, of the weights and of the outputs, about
    # 3e-3 in all; fp32: sums of a few thousand terms in another order
    if case["kind"] == "store":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.2}


# ------------------------------------------------------------------ in 64 bits

def _rope64(x, pos):
    """x[T][H][d] rotated at pos[T] (pairs i, i + d/2)."""
    x, half = x.double(), x.shape[2] // 2
    a = pos.double()[:, None] * BASE ** (-torch.arange(half, device=DEV, dtype=torch.float64) / half)
    c, s = a.cos()[:, None], a.sin()[:, None]
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], 2)


def _softmax64(q, k, v, off):
    """out, lse of q[n][R][d] over k, v[m][d], query i seeing keys <= off + i."""
    n, R, d = q.shape
    out, lse = torch.empty_like(q), torch.empty(n, R, dtype=torch.float64, device=DEV)
    for a in range(0, n, 512):
        z = min(n, a + 512)
        s = (q[a:z].reshape(-1, d) @ k.t()).reshape(z - a, R, -1) / math.sqrt(d)
        if off + a + 1 < k.shape[0]:
            last = off + torch.arange(a, z, device=DEV)
            s.masked_fill_(torch.arange(k.shape[0], device=DEV)[None, None] > last[:, None, None], -math.inf)
        lse[a:z] = torch.logsumexp(s, 2)
        out[a:z] = ((s - lse[a:z, :, None]).exp().reshape(-1, k.shape[0]) @ v).reshape(z - a, R, d)
    return out, lse


def _exact_encode(case, S, I):
    G, R, P = case["hkv"], case["hq"] // case["hkv"], case.get("prefix", 0)
    pos = P + torch.cat([torch.arange(int(n), device=DEV) for n in S["len"]])
    q, kc = _rope64(I["q"], pos), _rope64(I["k"], pos).permute(1, 0, 2).contiguous()
    vc = I["v"].double().permute(1, 0, 2).contiguous()
    out = torch.empty_like(q)
    lse = torch.empty(case["hq"], q.shape[0], dtype=torch.float64, device=DEV)
    for r in range(len(S["len"])):
        a, z = int(S["cu_len"][r]), int(S["cu_len"][r + 1])
        for g in range(G):
            k, v = kc[g, a:z], vc[g, a:z]
            if P:
                k, v = torch.cat([I["pk"][g].double(), k]), torch.cat([I["pv"][g].double(), v])
            h = slice(g * R, (g + 1) * R)
            out[a:z, h], l = _softmax64(q[a:z, h], k, v, P)
            lse[h, a:z] = l.t()
    return out, kc, vc, lse


def exact(case, seed):
    if case["kind"] == "store":
        return None  # copies and whole numbers
    S, N = _structure(case, seed), _Normal(seed)
    got, G, R = [], case["hkv"], case["hq"] // case["hkv"]
    start, kept = torch.from_numpy(S["cu_len"]).to(DEV), torch.from_numpy(S["kept"]).to(DEV)
    owner = torch.repeat_interleave(torch.arange(len(S["len"]), device=DEV),
                                    torch.from_numpy(np.diff(S["cu_kept"])).to(DEV).long())
    if case["kind"] in ("encode", "chain"):
        I = _encode_inputs(case, S, N)
        out, kc, vc, lse = _exact_encode(case, S, I)
        got = [out, kc, vc, lse if case["lse"] else None]
        at = (start[owner] + kept).long()
        kk, vk = kc[:, at], vc[:, at]
        if 0.0 < case["keep"] < 1.0:
            got += [kk, vk]
        if case["kind"] == "encode":
            return got
    I = _attend_inputs(case, S, N)
    q, ck, cv = I["q"].double(), I["ck"], I["cv"]
    if case["kind"] == "step":
        pos = torch.full((1,), int(S["cu_len"][-1]) + int(S["ctx"][0]) - 1, device=DEV)
        q = _rope64(I["q"], pos)
        ck, cv = ck.double(), cv.double()
        ck[:, -1], cv[:, -1] = _rope64(I["k_new"], pos)[0], I["v_new"][0].double()
    out = torch.empty_like(q)
    lse = torch.empty(case["hq"], q.shape[0], dtype=torch.float64, device=DEV)
    off = np.concatenate([[0], np.cumsum(S["rows"])])
    for b in range(case["n_req"]):
        a, z = int(S["cu_q"][b]), int(S["cu_q"][b + 1])
        c0, c1 = int(S["cu_ctx"][b]), int(S["cu_ctx"][b + 1])
        mine = S["req_res"][S["req_off"][b]:S["req_off"][b + 1]]
        for g in range(G):
            ks, vs = [], []
            for r in mine[S["mask"][mine, S["layer"], g] != 0]:
                if case["kind"] == "chain":
                    rk, rv, x = kk[g], vk[g], int(S["cu_kept"][r])
                elif case["store"]:
                    rk, rv, x = I["rk"], I["rv"], int(off[r * G + g])
                else:
                    rk, rv, x = I["rk"][g], I["rv"][g], int(S["cu_kept"][r])
                n = int(S["cu_kept"][r + 1] - S["cu_kept"][r])
                ks.append(rk[x:x + n])
                vs.append(rv[x:x + n])
            vis = sum(len(t) for t in ks)
            k = torch.cat([t.double() for t in ks] + [ck[g, c0:c1].double()])
            v = torch.cat([t.double() for t in vs] + [cv[g, c0:c1].double()])
            h = slice(g * R, (g + 1) * R)
            out[a:z, h], l = _softmax64(q[a:z, h], k, v, vis + (c1 - c0) - (z - a))
            lse[h, a:z] = l.t()
    got += [out, lse if case["lse"] else None]
    if case["kind"] == "step":
        got += [ck[:, -1], cv[:, -1]]
    return got
