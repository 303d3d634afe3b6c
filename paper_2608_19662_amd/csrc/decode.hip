// Split-KV decode: one new conversation token per request attends the kept
// rows of the resources routed to its (layer, KV group) and the whole
// conversation context (final ReCache mask, Fig. 2, with Tq = 1), followed
// by a log-sum-exp merge of the splits.
//
// Memory-bound: every visible K/V row is read from HBM once per (request,
// layer, group), whatever the number of query heads in the group.  The
// products run on the matrix cores with the group's query heads as the N
// dimension of 16x16x32 bf16 MFMAs:
//     S^T = K Q^T      (A = 16 keys x 32 dims of K, straight from HBM into VGPRs)
//     O^T += V^T P^T   (A = V^T read from LDS with transpose reads, B = P^T
//                       packed from the S^T accumulators without shuffles)
// which leaves the VALU a few dozen instructions per 32 keys (the softmax),
// so the kernel streams at the memory system's pace.
//
// One block handles one contiguous range of the (request, group) key stream.
// Its four waves take 32-key tiles of the range in turn and run independent
// pipelines (own registers, own LDS buffers, no barriers in the loop): K and
// V of tile t + 1 are in flight while tile t is computed.  The four partial
// softmax states are merged in LDS at the end, and a second kernel merges the
// splits.  64 requests over 32 resources (30% of tokens, 25% of routes) plus
// 4,096 context rows, 32 / 8 heads, head_dim 128: 283 us a layer, 6.4 TB/s; a
// large elementwise copy reaches 6.2 (325 us while the compiler's waits
// drained the prefetch, see load_tile; 306 with the context through the
// caches).
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"

namespace rc {

namespace {

constexpr int kThreads = 256;
constexpr int kTk = 32;  // keys per wave tile
constexpr int kMaxSeg = 1024;
// Third dword of a gfx9 buffer resource for raw (unformatted) loads.
constexpr int kBufferFlags = 0x00020000;

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) void lds_void;
// (addresses held as integers: a plain pointer made from one is a flat access)
typedef __attribute__((address_space(1))) u32x4 global_u32x4;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

template <int C>
struct Tag {
    static constexpr int value = C;
};

template <int HD>
struct DT {
    static constexpr int CPR = HD / 8;        // 16-byte chunks per row
    static constexpr int ROWB = HD * 2;       // bytes per row
    static constexpr int TILEB = kTk * ROWB;  // bytes of one V tile
    static constexpr int NKS = HD / 32;       // k-steps of S^T over head_dim
    static constexpr int NDB = HD / 16;       // 16-dim blocks of O^T
    static constexpr int RPI = 64 / CPR;      // rows per 1 KB wave copy
    static constexpr int NJ = kTk / RPI;      // copies per V tile
    static constexpr int NLOAD = 2 * NKS + NJ;  // vector memory operations per tile
    // s_waitcnt immediate for vmcnt(NLOAD) (the loads of the newer tile may
    // still be in flight), other counters unconstrained
    static constexpr int WAIT_PREV = (NLOAD & 15) | ((NLOAD >> 4) << 14) | 0x0F70;
};

struct DecSmem {
    int seg_start[kMaxSeg + 1];
    int seg_row[kMaxSeg];
    int scan[8];  // of the segment-length scan
    float ml[4][16][2];  // per wave and head: max, sum (for the merge)
};

// Chunk swizzle of a V tile row: the 16 rows x 32 bytes that one transpose
// read touches spread over all 64 banks exactly twice.
template <int CPR>
__device__ __forceinline__ int v_mask(int row) {
    return CPR == 16 ? 2 * (row & 7) : 2 * ((row >> 1) & 3);
}

__device__ __forceinline__ float xor16_max(float x) { return fmaxf(x, __shfl_xor(x, 16)); }
__device__ __forceinline__ float xor16_sum(float x) { return x + __shfl_xor(x, 16); }

// A wave-uniform 64-bit value, pinned to scalar registers.
__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

// BIG: a plane of 4 GiB or more, which a buffer resource cannot address.  NT:
// context rows are loaded with the non-temporal hint (no request reads
// another's); resource rows never are, since requests share them.
template <int HD, bool BIG, bool NT>
__global__ __launch_bounds__(kThreads, 2) void decode_kernel(const DecodeArgs a) {
    using T = DT<HD>;
    __shared__ DecSmem sm;
    // Per wave two V tile buffers, in two arrays: the compiler then sees that
    // the copies in flight into one do not touch the tile being read, and
    // does not wait for them.  After the loop the first takes the wave's O,
    // fp32 [16 heads][HD].
    __shared__ __attribute__((aligned(16))) char v_all0[4][T::TILEB], v_all1[4][T::TILEB];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: a scalar
    const int l16 = lane & 15, grp = lane >> 4;  // MFMA column and row group of this lane

    int bid = blockIdx.x;
    const int split = bid % a.n_splits;
    bid /= a.n_splits;
    int g = bid % a.n_kv_heads;
    int b = bid / a.n_kv_heads;
    if (a.plan) {
        // with a work order the streams run longest first, so that the grid
        // does not end on a tail of long ones
        const int n_pairs = a.n_req * a.n_kv_heads;
        int p = a.plan[(size_t)a.layer * n_pairs + bid];
        p = min(max(p, 0), n_pairs - 1);  // in bounds whatever the plan holds
        b = p / a.n_kv_heads;
        g = p % a.n_kv_heads;
    }
    const int R = a.ratio;

    // ---- Q^T (B operand), loaded first since it depends on nothing else
    // (but the pair):
    // lane holds head l16 of the group (zero beyond R), dims ks*32 + grp*8 + [0, 8).
    const int qrow = min(a.cu_q[b], (int)a.lse_rows - 1);
    bf16x8_t qf[T::NKS];
#pragma unroll
    for (int ks = 0; ks < T::NKS; ++ks) {
        u32x4 w = {0u, 0u, 0u, 0u};
        if (l16 < R)
            w = *reinterpret_cast<const u32x4*>(a.q + ((size_t)qrow * a.n_q_heads + g * R + l16) * HD +
                                                ks * 32 + grp * 8);
        qf[ks] = __builtin_bit_cast(bf16x8_t, w);
    }

    // ---- visible segments of this (request, layer, group): kept rows of the
    // routed resources, request order.
    const size_t e = ((size_t)b * a.n_layers + a.layer) * a.n_kv_heads + g;
    const int r0 = a.route_off[e];
    const int n_seg = a.route_off[e + 1] - r0;
    if (n_seg > kMaxSeg || a.cu_q[b + 1] - a.cu_q[b] != 1) {
        // A route list longer than the segment table, or a request that does
        // not have exactly one query: this split's partial becomes NaN with
        // an infinite max, which the merge turns into NaN outputs for the
        // group (a caller's size error shows instead of dropped keys).
        for (int idx = tid; idx < R * HD; idx += kThreads) {
            const size_t slot = ((size_t)b * a.n_q_heads + g * R + idx / HD) * a.n_splits + split;
            a.ws_o[slot * HD + idx % HD] = __builtin_nanf("");
            if (idx % HD == 0) {
                a.ws_ml[slot * 2 + 0] = INFINITY;
                a.ws_ml[slot * 2 + 1] = __builtin_nanf("");
            }
        }
        return;
    }
    const int s_vis = segment_table<4, false>(a.route_res + r0, n_seg, a.cu_kept, a.res_off, a.n_kv_heads, g, 0,
                                              sm.seg_start, sm.seg_row, sm.scan);
    const int c0 = a.cu_ctx[b];
    const int tc = a.cu_ctx[b + 1] - c0;
    const int n_keys = s_vis + tc;
    // This split's key range [s0, s1): its resource rows [g0, g1) of the
    // stream, 32 keys per tile, then its context rows [x0, x1), so that every
    // tile has its rows in one buffer.
    int chunk = (n_keys + a.n_splits - 1) / a.n_splits;
    chunk = (chunk + kTk - 1) / kTk * kTk;
    const int s0 = min(split * chunk, n_keys);
    const int s1 = min(s0 + chunk, n_keys);
    const int g0 = min(s0, s_vis), g1 = min(s1, s_vis);
    const int x0 = max(s0, s_vis) - s_vis, x1 = max(s1, s_vis) - s_vis;
    const int n_segt = (g1 - g0 + kTk - 1) / kTk;
    const int n_tiles = n_segt + (x1 - x0 + kTk - 1) / kTk;

    // Last rows of the two buffers, pinned to scalar registers: selected from
    // the argument block they become a load and a wait per lookup.
    const int r_last = __builtin_amdgcn_readfirstlane((int)a.r_rows - 1);
    const int c_last = __builtin_amdgcn_readfirstlane((int)a.c_rows - 1);
    // this lane's segment walk (key l32 of each tile), forward only
    int ls_i = 0, ls_hi = n_seg > 0 ? sm.seg_start[1] : 0, ls_dl = n_seg > 0 ? sm.seg_row[0] : 0;
    // first stream position (resource rows) or context row of tile t, and its
    // range's end
    auto tile_begin = [&](int t) { return t < n_segt ? g0 + t * kTk : x0 + (t - n_segt) * kTk; };
    auto tile_end = [&](int t) { return t < n_segt ? g1 : x1; };

    // ---- loads of one tile.  K: lane holds key kb*16 + l16 of the tile,
    // dims ks*32 + grp*8 + [0, 8), in registers.  V: copy j of the wave moves
    // rows j*RPI + i / CPR of the tile; lane i lands at byte 16 i, i.e.
    // physical chunk i % CPR, which holds logical chunk (i % CPR) ^ v_mask(row).
    // Lane k looks up the row of key k (clamped into its buffer) and the loads
    // fetch row offsets from there: one straight line of 16 loads, whatever
    // the tile straddles, so that the compiler's waits count them exactly (a
    // branch per kind of tile made it wait for all loads in flight).
    char* const v_st0 = v_all0[wave];
    char* const v_st1 = v_all1[wave];
    uint32_t v_lane[2];  // byte offset of this lane's chunk within its row, copies 2i and 2i + 1
#pragma unroll
    for (int j = 0; j < 2; ++j)
        v_lane[j] = (uint32_t)(((lane % T::CPR) ^ v_mask<T::CPR>(j * T::RPI + lane / T::CPR)) << 4);
    u32x4 kreg[2][2][T::NKS];  // [buffer][key block][k-step]
    auto load_tile = [&](auto buf_tag, auto aux_tag, int i) {
        constexpr int buf = decltype(buf_tag)::value, AUX = decltype(aux_tag)::value;
        const int t = wave + 4 * i;
        const bool seg = t < n_segt;
        const int p = min(tile_begin(t) + (lane & 31), tile_end(t) - 1);  // past the range: its last key
        int row;
        if (seg) {
            while (p >= ls_hi && ls_i + 1 < n_seg) {
                ++ls_i;
                ls_hi = sm.seg_start[ls_i + 1];
                ls_dl = sm.seg_row[ls_i] - sm.seg_start[ls_i];
            }
            row = min(ls_dl + p, r_last);
        } else {
            row = min(c0 + p, c_last);
        }
        row = max(row, 0);
        const uint32_t off = BIG ? (uint32_t)row : (uint32_t)row * T::ROWB;  // (a plane may reach 4 GiB)
        const uint64_t kp = uniform64((uint64_t)((seg ? a.rk : a.ck) + (size_t)g * (seg ? a.r_gstride : a.c_rows) * HD));
        const uint64_t vp = uniform64((uint64_t)((seg ? a.rv : a.cv) + (size_t)g * (seg ? a.r_gstride : a.c_rows) * HD));
        char* dst = buf ? v_st1 : v_st0;
        if constexpr (BIG) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                const uint64_t r = (uint64_t)(uint32_t)__builtin_amdgcn_ds_bpermute(l16 * 4 + kb * 64, (int)off);
                const uint64_t src = kp + r * T::ROWB + grp * 16;
#pragma unroll
                for (int ks = 0; ks < T::NKS; ++ks) kreg[buf][kb][ks] = ((const global_u32x4*)src)[ks * 4];
            }
#pragma unroll
            for (int j = 0; j < T::NJ; ++j) {
                const uint64_t r =
                    (uint64_t)(uint32_t)__builtin_amdgcn_ds_bpermute(lane / T::CPR * 4 + j * T::RPI * 4, (int)off);
                const uint64_t src = vp + r * T::ROWB + v_lane[j & 1];
                __builtin_amdgcn_global_load_lds((const uint16_t*)src, (lds_void*)(dst + j * 1024), 16, 0, 0);
            }
        } else {
            const int bytes = __builtin_amdgcn_readfirstlane((int)((seg ? a.r_rows : a.c_rows) * T::ROWB));
            const __amdgpu_buffer_rsrc_t kr =
                __builtin_amdgcn_make_buffer_rsrc((void*)kp, (short)0, bytes, kBufferFlags);
            const __amdgpu_buffer_rsrc_t vr =
                __builtin_amdgcn_make_buffer_rsrc((void*)vp, (short)0, bytes, kBufferFlags);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                const uint32_t o = (uint32_t)__builtin_amdgcn_ds_bpermute(l16 * 4 + kb * 64, (int)off) + grp * 16;
#pragma unroll
                for (int ks = 0; ks < T::NKS; ++ks)
                    kreg[buf][kb][ks] = __builtin_amdgcn_raw_buffer_load_b128(kr, (int)(o + ks * 64), 0, AUX);
            }
#pragma unroll
            for (int j = 0; j < T::NJ; ++j) {
                const uint32_t o =
                    (uint32_t)__builtin_amdgcn_ds_bpermute(lane / T::CPR * 4 + j * T::RPI * 4, (int)off) + v_lane[j & 1];
                __builtin_amdgcn_raw_ptr_buffer_load_lds(vr, (lds_void*)(dst + j * 1024), 16, (int)o, 0, 0, AUX);
            }
        }
    };

    // ---- transpose-read offsets: lane (grp, i) of a 16-lane group points at
    // row w*16 + grp*4 + i/4, dims db*16 + 4*(i % 4), so that it receives dim
    // db*16 + i of rows w*16 + grp*4 + [0, 4): keys grp*4 + [0, 4) (w = 0) and
    // 16 + grp*4 + [0, 4) (w = 1), the keys whose weights this lane holds in
    // the S^T accumulators of the two 16-key blocks.
    auto tr_off = [&](int db, int w) -> uint32_t {
        const int row = w * 16 + grp * 4 + (l16 >> 2);
        const int col = db * 16 + 4 * (l16 & 3);
        return (uint32_t)(row * T::ROWB + (((col >> 3) ^ v_mask<T::CPR>(row)) << 4) + (col & 7) * 2);
    };

    const float sl2 = a.scale_log2;
    const bf16x2 ones2 = __builtin_bit_cast(bf16x2, 0x3F803F80u);  // (1.0, 1.0) in bf16
    float m = -INFINITY;  // running max (log2 units) for head l16
    float lsum = 0.f;     // this lane's part of the row sum
    f32x4 oacc[T::NDB];   // O^T: dims db*16 + grp*4 + [0, 4) of head l16
#pragma unroll
    for (int db = 0; db < T::NDB; ++db) oacc[db] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto compute = [&](auto buf_tag, int i) {
        constexpr int buf = decltype(buf_tag)::value;
        const int t = wave + 4 * i;
        const int n_in = tile_end(t) - tile_begin(t);  // keys of the tile in its range (32 or more: all)
        f32x4 sacc[2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            sacc[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < T::NKS; ++ks)
                sacc[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    __builtin_bit_cast(bf16x8_t, kreg[buf][kb][ks]), qf[ks], sacc[kb], 0, 0, 0);
        }
        // keys past the range's end (its last tile only)
        if (n_in < kTk) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (kb * 16 + grp * 4 + r >= n_in) sacc[kb][r] = -INFINITY;
        }
        float mt = fmaxf(fmaxf(fmaxf(sacc[0][0], sacc[0][1]), fmaxf(sacc[0][2], sacc[0][3])),
                         fmaxf(fmaxf(sacc[1][0], sacc[1][1]), fmaxf(sacc[1][2], sacc[1][3])));
        mt = pair_max(xor16_max(mt)) * sl2;  // over the tile's 32 keys, log2 units
        // lazy rescale: m moves only when a logit exceeds it by more than 8
        // (weights stay <= 2^8); O and the row sum share m, so this is exact
        if (__builtin_amdgcn_ballot_w64(mt > m + 8.f)) {
            const float m_new = fmaxf(m, mt);
            const float alpha = __builtin_amdgcn_exp2f(m - m_new);  // 0 when m == -inf
            lsum *= alpha;
#pragma unroll
            for (int db = 0; db < T::NDB; ++db) oacc[db] *= alpha;
            m = m_new;
        }
        uint32_t w[4];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 4; r += 2) {
                const float p0 = __builtin_amdgcn_exp2f(fmaf(sacc[kb][r], sl2, -m));
                const float p1 = __builtin_amdgcn_exp2f(fmaf(sacc[kb][r + 1], sl2, -m));
                const uint32_t pk = pack_bf16x2(p0, p1);
                w[kb * 2 + r / 2] = pk;
                // row sum of the weights as rounded for the P V product
                lsum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pk), ones2, lsum, false);
            }
        const bf16x8_t pf = __builtin_bit_cast(bf16x8_t, u32x4{w[0], w[1], w[2], w[3]});
        const char* st = buf ? v_st1 : v_st0;
#pragma unroll
        for (int db = 0; db < T::NDB; ++db) {
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(st + tr_off(db, 0)));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(st + tr_off(db, 1)));
            const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
            const bf16x8_t av = __builtin_bit_cast(bf16x8_t, u32x4{l2[0], l2[1], h2[0], h2[1]});
            oacc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, pf, oacc[db], 0, 0, 0);
        }
    };

    // This wave's tiles are wave, wave + 4, ... of the range; the loads of
    // the next one are in flight while one is computed.  Only this wave
    // reads its V buffers, so waiting for its own copies is enough.  (Each
    // exit has its own copy of the computation, so that inside the loop the
    // compiler's waits count the newer tile's loads as these do; a macro, since
    // the K registers of a lambda around these two went to scratch.)
#define RC_TILES(AUX, FIRST, LAST)                            \
    if (const int i0 = FIRST, i1 = LAST; i0 < i1) {           \
        load_tile(Tag<0>{}, Tag<AUX>{}, i0);                  \
        for (int i = i0;; i += 2) {                           \
            if (i + 1 >= i1) {                                \
                __builtin_amdgcn_s_waitcnt(0x0F70);           \
                compute(Tag<0>{}, i);                         \
                break;                                        \
            }                                                 \
            load_tile(Tag<1>{}, Tag<AUX>{}, i + 1);           \
            __builtin_amdgcn_s_waitcnt(T::WAIT_PREV);         \
            compute(Tag<0>{}, i);                             \
            if (i + 2 >= i1) {                                \
                __builtin_amdgcn_s_waitcnt(0x0F70);           \
                compute(Tag<1>{}, i + 1);                     \
                break;                                        \
            }                                                 \
            load_tile(Tag<0>{}, Tag<AUX>{}, i + 2);           \
            __builtin_amdgcn_s_waitcnt(T::WAIT_PREV);         \
            compute(Tag<1>{}, i + 1);                         \
        }                                                     \
    }
    auto tiles_of = [&](int n) { return n > wave ? (n - wave + 3) / 4 : 0; };
    if constexpr (NT) {
        // the resource tiles, then the context tiles with their own loads
        RC_TILES(0, 0, tiles_of(n_segt))
        RC_TILES(2, tiles_of(n_segt), tiles_of(n_tiles))
    } else {
        RC_TILES(0, 0, tiles_of(n_tiles))
    }
#undef RC_TILES

    // ---- merge: the four row groups of a head hold disjoint dims of O^T and
    // parts of its row sum; then the four waves, through LDS.
    lsum = pair_sum(xor16_sum(lsum));
    static_assert(16 * HD * 4 == T::TILEB, "a wave's O fills a V buffer");
    // (16-byte chunks swizzled by head; only this wave touched its buffers, so
    // no barrier before the writes)
#pragma unroll
    for (int db = 0; db < T::NDB; ++db)
        *reinterpret_cast<f32x4*>(v_st0 + (l16 * (HD / 4) + ((db * 4 + grp) ^ l16)) * 16) = oacc[db];
    if (grp == 0) {
        sm.ml[wave][l16][0] = m;
        sm.ml[wave][l16][1] = lsum;
    }
    __syncthreads();
    for (int idx = tid; idx < R * HD; idx += kThreads) {
        const int h = idx / HD, d = idx % HD;
        float mx = -INFINITY;
#pragma unroll
        for (int w = 0; w < 4; ++w) mx = fmaxf(mx, sm.ml[w][h][0]);
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float mw = sm.ml[w][h][0];
            const float sc = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw - mx);
            const char* o = v_all0[w] + (h * (HD / 4) + ((d >> 2) ^ h)) * 16 + (d & 3) * 4;
            num += sc * *reinterpret_cast<const float*>(o);
            den += sc * sm.ml[w][h][1];
        }
        const size_t slot = ((size_t)b * a.n_q_heads + g * R + h) * a.n_splits + split;
        a.ws_o[slot * HD + d] = num;
        if (d == 0) {
            a.ws_ml[slot * 2 + 0] = mx;
            a.ws_ml[slot * 2 + 1] = den;
        }
    }
}

// out[b][h] = sum_s w_s O_s / sum_s w_s l_s with w_s = exp2(m_s - max m);
// splits that saw no key carry m_s = -inf and weigh nothing.  One wave per
// (request, head), lane s holding split s's (max, sum) and weight: one round
// trip for those, beside the partials' own (each lane HD / 64 dims of every
// split, four or eight splits in flight), whatever the number of splits.
template <int HD>
__global__ __launch_bounds__(kThreads) void combine_kernel(const DecodeArgs a) {
    constexpr int V = HD / 64;  // dims per lane
    typedef float vec __attribute__((ext_vector_type(V)));
    const int lane = threadIdx.x & 63;
    const int bh = blockIdx.x * (kThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (bh >= a.n_req * a.n_q_heads) return;
    const int b = bh / a.n_q_heads, h = bh % a.n_q_heads;
    const int row = a.cu_q[b];
    const size_t slot0 = (size_t)bh * a.n_splits;
    const float2 ml = lane < a.n_splits ? reinterpret_cast<const float2*>(a.ws_ml)[slot0 + lane]
                                        : make_float2(-INFINITY, 0.f);
    const float* o = a.ws_o + slot0 * HD + lane * V;
    float mx, den;
    vec num = {};
    auto merge = [&](auto in_flight) {
        constexpr int C = decltype(in_flight)::value;
        vec x[C];
        auto load = [&](int s0) {
#pragma unroll
            for (int c = 0; c < C; ++c)  // (past the last split: the last one again, not used)
                x[c] = *reinterpret_cast<const vec*>(o + (size_t)min(s0 + c, a.n_splits - 1) * HD);
        };
        load(0);
        // over the lanes that may hold splits (C = 4: lanes 0 .. 3)
        constexpr int TOP = C == 4 ? 2 : 32;
        mx = ml.x;
        for (int f = TOP; f >= 1; f >>= 1) mx = fmaxf(mx, __shfl_xor(mx, f));
        mx = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(mx)));
        const float w = ml.x == -INFINITY ? 0.f : exp2f(ml.x - mx);
        den = w * ml.y;
        for (int f = TOP; f >= 1; f >>= 1) den += __shfl_xor(den, f);
        den = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(den)));
        for (int s0 = 0;;) {
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float wc = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w), min(s0 + c, 63)));
                if (s0 + c < a.n_splits) num += wc * x[c];
            }
            s0 += C;
            if (s0 >= a.n_splits) break;
            load(s0);
        }
    };
    if (a.n_splits <= 4)
        merge(Tag<4>{});
    else
        merge(Tag<8>{});
    if (row < 0 || row >= a.lse_rows) return;
    uint16_t* out = a.out + ((size_t)row * a.n_q_heads + h) * HD + lane * V;
    if constexpr (V == 2)
        *reinterpret_cast<uint32_t*>(out) = pack_bf16x2(num[0] / den, num[1] / den);
    else
        *out = f32_to_bf16_bits(num[0] / den);
    if (a.lse && lane == 0) a.lse[(size_t)h * a.lse_rows + row] = (mx + log2f(den)) * 0.69314718055994531f;
}

template <int HD>
hipError_t launch_dec(const DecodeArgs& a, hipStream_t s) {
    const long blocks = (long)a.n_req * a.n_kv_heads * a.n_splits;
    const bool big = (unsigned long)std::max(a.r_rows, a.c_rows) * HD * 2 >= (1UL << 32);
    // Context rows past the caches where a layer of them (at most n_req *
    // max_ctx rows) is twice the 256 MB last-level cache or more: they evict
    // what would be found there, of the resources too.  64 requests, 4,096
    // context rows (1 GB): 283 us a layer instead of 306.  Twelve layers in
    // turn, 4,096 rows per request over 32 / 256 resources, us a layer with the
    // hint (without): 512 MiB 102 / 114 (107 / 117), 1 GiB 187 / 205 (199 /
    // 220).  Below, little speaks for either while the layers take turns: 400
    // MiB 88 / 96 (90 / 98), but 98 (95) with contexts of unequal length; 256
    // MiB 62 / 69 (61 / 67); 128 MiB 37 / 42 (37 / 41).  Where the next call
    // reads the same layer, the part that stays cached counts: 256 MiB 60 / 64
    // (52 / 60).
    const bool nt = (unsigned long)std::min(a.c_rows, a.max_ctx_rows) * a.n_kv_heads * HD * 4 >= (512UL << 20);
    if (big)
        hipLaunchKernelGGL((decode_kernel<HD, true, false>), dim3((unsigned)blocks), dim3(kThreads), 0, s, a);
    else if (nt)
        hipLaunchKernelGGL((decode_kernel<HD, false, true>), dim3((unsigned)blocks), dim3(kThreads), 0, s, a);
    else
        hipLaunchKernelGGL((decode_kernel<HD, false, false>), dim3((unsigned)blocks), dim3(kThreads), 0, s, a);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    const unsigned waves = (unsigned)(a.n_req * a.n_q_heads), per = kThreads / 64;
    hipLaunchKernelGGL((combine_kernel<HD>), dim3((waves + per - 1) / per), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace

namespace {

// Blocks that a grid is filled to at 512 keys or more each, and where that
// leaves CUs idle at 128 keys (one tile per wave) or more: three rounds of two
// blocks per CU, and one.
constexpr long kManyBlocks = 1536, kFewBlocks = 512;

long split_limit(long units, int max_kv, long blocks, int keys) {
    return std::min({(blocks + units - 1) / units, ((long)max_kv + keys - 1) / keys, 64L});
}

}  // namespace

// About three rounds of two blocks per CU, at least 512 keys per block; and
// where that leaves CUs idle, finer: up to 512 blocks of at least 128 keys
// (one request over 3,400 keys, 32 / 8 heads: 27 splits instead of 7, the
// kernel 7.2 us instead of 10.5, the merge of the splits 4.7 and 3.9).
int decode_splits(int n_req, int n_kv_heads, int max_kv) {
    const long units = (long)n_req * n_kv_heads;
    const long s = split_limit(units, max_kv, kManyBlocks, 512);
    const long few = std::min(kFewBlocks / units, split_limit(units, max_kv, kFewBlocks, 128));
    return (int)std::max({s, few, 1L});
}

// Splits fall as requests are added, so requests times splits is largest at
// the last request count of some split count: the walk goes from n_req to
// smaller batches, to the largest one that can have another split each time.
long decode_max_parts(int n_req, int n_kv_heads, int max_kv) {
    const long g = n_kv_heads, by512 = ((long)max_kv + 511) / 512, by128 = ((long)max_kv + 127) / 128;
    const int top = decode_splits(1, n_kv_heads, max_kv);
    long n = n_req, most = 0;
    for (;;) {
        const long c = decode_splits((int)n, n_kv_heads, max_kv);
        most = std::max(most, n * c);
        if (c >= top) return most;
        n = std::min(n - 1, std::max(c < by512 ? (kManyBlocks - 1) / c : 0, c < by128 ? kFewBlocks / (c + 1) : 0) / g);
    }
}

size_t decode_workspace_bytes(long parts, int n_q_heads, int head_dim) {
    return (size_t)parts * n_q_heads * (head_dim + 2) * sizeof(float);
}

hipError_t launch_decode(const DecodeArgs& a, hipStream_t s) {
    if ((long)a.n_req * a.n_kv_heads * a.n_splits > 0x7fffffffL) return hipErrorInvalidValue;
    if (a.ratio < 1 || a.ratio > 16) return hipErrorInvalidValue;
    return a.head_dim == 128 ? launch_dec<128>(a, s) : launch_dec<64>(a, s);
}

}  // namespace rc
