// fp32 attention (encode, conversation prefill and decode) on the fp32 matrix
// instructions of gfx950.  Every product and sum stays in fp32: it runs the
// method at fp32 input precision, with no bf16 rounding anywhere.
//
// Visibility follows the same definitions as the bf16 kernels: encode rows
// see the shared prefix and their own resource causally (ReCache Sec. 3,
// "Resource-Wise Attention"); conversation rows see the kept rows of their routed resources
// in request order and then the context causally, bottom-right aligned
// (Fig. 2, final mask).
//
// Work decomposition.  The query rows of a unit and KV group are flattened to
// columns j = row * ratio + head, and a block owns 32 of them: few queries
// still fill the matrix tile when they have several heads, and a causal block
// of 32 columns spans only 32 / ratio rows.  Its four waves take the 32-key
// tiles of the key stream in turn, each with its own softmax state, merged in
// LDS at the end: fp32 calls are small (short streams, few columns), so the
// keys are split to have enough waves, and always four ways, so that a
// resource's results do not depend on what is packed beside it.  Per tile
//     S^T = K Q^T      (32x32x2 fp32 MFMA; A = K straight from memory in
//                       VGPRs, B = Q^T in VGPRs)
//     O^T += V^T P^T   (A = V rows from LDS, B = P^T as it stands in the S^T
//                       accumulators)
// so that a lane owns one column, and half of its keys and dims.  The order
// of the MFMA's inner index is free: half h of the lanes holds dims 8 j + 4 h
// + [0, 4) of Q and K (one 16-byte load each), and the keys that the S^T
// accumulators leave in half h of P.
//
// Bound: one tile after another in a wave, its V's round trip in each, with
// two blocks per CU to cover it (a wave tile is 128 MFMAs of 64 cycles at
// head_dim 128; its 32 KB of K and V ask the L2 for 16 B/clk per CU).  The K
// loads of the next tile are issued behind this tile's S products.  The V
// copies of a tile are issued before its S products, but flat copies into LDS
// make the compiler wait for all of them in front of all but the first of
// these products; and in the attend form at head_dim 128 16 VGPRs spill, whose
// reloads wait for the K loads too.
// Measured at 32 / 8 heads, head_dim 128: six resources of 100 to 500 tokens
// encode in 140 us (one wave per row and head, a shuffle reduction per key:
// 965 us), two requests of 150 to 250 queries over them attend in 73 us (669).
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace rc {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = 4;
constexpr int kCols = 32;     // columns (row, head) per block
constexpr int kKeys = 32;     // keys per wave tile
constexpr int kMaxSeg = 1024; // route segments per pass over the segment table

typedef __attribute__((address_space(3))) void lds_void;
typedef float f32x4_dword __attribute__((ext_vector_type(4), aligned(4)));

template <int HD>
struct F32Smem {
    int seg_start[kMaxSeg + 1];
    int seg_row[kMaxSeg];
    int scan[2 * kWaves];
    float ml[kWaves][kCols][2];
    // per wave: the V tile [32 keys][HD]; before the loop the cos / sin table,
    // after it the wave's O [32 columns][HD]
    alignas(16) float v[kWaves][kKeys * HD];
};

// DWORD: a tensor that is not on 16 bytes (a view that starts at any float).
// Its rows are read and written as four floats each way, and V copied into LDS
// dword by dword.
template <int HD, bool ENCODE, bool DWORD>
__global__ __launch_bounds__(kThreads, 2) void attn_f32_kernel(const AttnF32Args a) {
    constexpr int NJ = HD / 8;    // 8-dim steps of S^T (four MFMAs each)
    constexpr int NDB = HD / 32;  // 32-dim blocks of O^T
    constexpr int LPR = HD / 4;   // lanes per row of a V copy (16 bytes each)
    constexpr int NVC = kKeys * HD / 256;  // 1 KB copies per V tile
    using vec = std::conditional_t<DWORD, f32x4_dword, f32x4>;  // four floats in memory
    __shared__ F32Smem<HD> sm;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int R = a.ratio;

    // block -> (unit, column block [longest first], group)
    int bid = blockIdx.x;
    const int g = bid % a.n_kv_heads;
    bid /= a.n_kv_heads;
    const int cb = a.n_cb - 1 - bid % a.n_cb;
    const int unit = bid / a.n_cb;

    int q_row0, q_len, c0, tc;
    if constexpr (ENCODE) {
        q_row0 = a.cu_len[unit];
        q_len = a.cu_len[unit + 1] - q_row0;
        c0 = q_row0;
        tc = q_len;
    } else {
        q_row0 = a.cu_q[unit];
        q_len = a.cu_q[unit + 1] - q_row0;
        c0 = a.cu_ctx[unit];
        tc = a.cu_ctx[unit + 1] - c0;
    }
    if (cb == a.n_cb - 1 && q_len > a.max_rows) {
        // rows past the grid's max_rows: NaN, so that a caller's size error
        // shows in the outputs instead of leaving them unwritten
        for (int r = a.max_rows; r < q_len && (long)q_row0 + r < a.lse_rows; ++r)
            for (int i = tid; i < R * HD; i += kThreads) {
                const int h = g * R + i / HD;
                a.out[((size_t)(q_row0 + r) * a.n_q_heads + h) * HD + i % HD] = __builtin_nanf("");
                if (i % HD == 0 && a.lse) a.lse[(size_t)h * a.lse_rows + q_row0 + r] = __builtin_nanf("");
            }
    }
    const int rows = min(q_len, a.max_rows);
    const int j0 = cb * kCols, n_cols = rows * R;  // (rows <= lse_rows: n_cols indexes LSE)
    if (j0 >= n_cols) return;
    const int used = min(kCols, n_cols - j0);   // columns of this block
    const int my_j = j0 + min(l32, used - 1);   // spare lanes repeat the last column
    const int my_row = my_j / R, my_head = my_j % R;
    const int first_row = j0 / R, last_row = (j0 + used - 1) / R;
    const long max_q = a.lse_rows - 1;  // rows outside [0, lse_rows) of q / out are never touched

    // ---- Q^T (B operand): dims 8 j + 4 half + [0, 4) of this lane's column
    f32x4 qf[NJ];
    {
        const long row = max(0L, min((long)q_row0 + my_row, max_q));
        const float* qp = a.q + ((size_t)row * a.n_q_heads + g * R + my_head) * HD + half * 4;
#pragma unroll
        for (int j = 0; j < NJ; ++j) qf[j] = *reinterpret_cast<const vec*>(qp + j * 8);
    }
    if constexpr (ENCODE) {
        // RoPE at the resource-local position: cos / sin of the block's rows
        // once per (row, frequency) into LDS; the pairs (f, f + HD / 2) are
        // (j, j + NJ / 2) in this lane
        constexpr int HALF = HD / 2;
        float2* tab = reinterpret_cast<float2*>(&sm.v[0][0]);
        const int pos0 = a.pos_base ? a.pos_base[unit] : 0;
        const int n = (last_row - first_row + 1) * HALF;
        for (int i = tid; i < n; i += kThreads) {
            float s, c;
            sincos_rev(rope_revolutions(pos0 + first_row + i / HALF, a.rope.rev[i % HALF]), &s, &c);
            tab[i] = make_float2(c, s);
        }
        __syncthreads();
        const float2* t = tab + (my_row - first_row) * HALF + half * 4;
#pragma unroll
        for (int j = 0; j < NJ / 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float2 k = t[j * 8 + e];
                const float x1 = qf[j][e], x2 = qf[j + NJ / 2][e];
                // the rounding of the key rotation, written out
                qf[j][e] = fmaf(x1, k.x, -(x2 * k.y));
                qf[j + NJ / 2][e] = fmaf(x2, k.x, x1 * k.y);
            }
        __syncthreads();  // the table's place takes V tiles next
    }
    const float sc = a.scale * 1.44269504088896340736f;

    float m = -INFINITY, l = 0.f;  // this wave's reference max and this lane's part of the sum
    f32x16 oacc[NDB];              // O^T: dims db*32 + 8 (r / 4) + 4 half + r % 4 of the column
#pragma unroll
    for (int db = 0; db < NDB; ++db) oacc[db] = f32x16{};

    // ---- the key stream: route segments (at most kMaxSeg per pass), the
    // last pass followed by the causal rows
    int n_seg, r0 = 0;
    if constexpr (ENCODE) {
        n_seg = a.p_len > 0 ? 1 : 0;
    } else {
        const size_t e = ((size_t)unit * a.n_layers + a.layer) * a.n_kv_heads + g;
        r0 = a.route_off[e];
        n_seg = a.route_off[e + 1] - r0;
    }
    const int off = tc - q_len;  // the row's last visible causal row is off + row
    const int c_max = (int)min((long)a.c_rows - 1 - c0, (long)tc - 1);
    const int my_last = min(off + my_row, c_max), block_last = min(off + last_row, c_max);
    const int block_first = min(off + first_row, c_max);
    float* vbuf = sm.v[wave];

    for (int seg0 = 0;; seg0 += kMaxSeg) {
        const bool last_pass = seg0 + kMaxSeg >= n_seg;
        const int ns = max(0, min(kMaxSeg, n_seg - seg0));
        int s_vis;
        if constexpr (ENCODE) {
            s_vis = a.p_len;
            if (tid == 0) sm.seg_start[0] = 0, sm.seg_start[1] = s_vis, sm.seg_row[0] = 0;
            __syncthreads();
        } else {
            if (seg0 > 0) __syncthreads();  // every wave is done with the previous pass's table
            s_vis = segment_table<kWaves, true>(a.route_res + r0 + seg0, ns, a.cu_kept, a.res_off, a.n_kv_heads, g,
                                                a.k_rows, sm.seg_start, sm.seg_row, sm.scan);
        }
        const int n_keys = s_vis + (last_pass ? max(0, block_last + 1) : 0);
        const int n_tiles = (n_keys + kKeys - 1) / kKeys;
        // stream positions up to these are visible to the column / to all columns
        const int vis_hi = last_pass ? s_vis + my_last : s_vis - 1;
        const int all_hi = last_pass ? s_vis + block_first : s_vis - 1;

        // Row of this lane's key l32 of a tile: the segment plane's row, or
        // ~row of the causal plane.  Keys past the stream repeat its last
        // one.  A lane's segment index only moves forward.
        int sidx = 0;
        auto row_code = [&](int t) -> int {
            const int p = min(t * kKeys + l32, n_keys - 1);
            if (p >= s_vis) return ~max(0, min(c0 + (p - s_vis), (int)a.c_rows - 1));
            while (sidx + 1 < ns && p >= sm.seg_start[sidx + 1]) ++sidx;
            return max(0, min(sm.seg_row[sidx] + (p - sm.seg_start[sidx]), (int)a.k_rows - 1));
        };
        const float* seg_k = a.k + (size_t)g * a.k_gstride * HD;
        const float* seg_v = a.v + (size_t)g * a.k_gstride * HD;
        const float* ctx_k = a.ck + (size_t)g * a.c_rows * HD;
        const float* ctx_v = a.cv + (size_t)g * a.c_rows * HD;

        f32x4 kf[NJ];  // K tile (A operand): key l32, dims 8 j + 4 half + [0, 4)
        int code = 0;
        auto load_k = [&](int t) {
            code = row_code(t);
            const float* kp = (code < 0 ? ctx_k + (size_t)(~code) * HD : seg_k + (size_t)code * HD) + half * 4;
#pragma unroll
            for (int j = 0; j < NJ; ++j) kf[j] = *reinterpret_cast<const vec*>(kp + j * 8);
        };
        auto copy_v = [&]() {  // of the tile whose row codes are in `code`
            if constexpr (DWORD) {
#pragma unroll 4
                for (int c = 0; c < kKeys * HD / 64; ++c) {  // 64 floats of one row
                    const int rc_ = __builtin_amdgcn_readlane(code, c * 64 / HD);
                    const float* vp = rc_ < 0 ? ctx_v + (size_t)(~rc_) * HD : seg_v + (size_t)rc_ * HD;
                    __builtin_amdgcn_global_load_lds(vp + c * 64 % HD + lane, (lds_void*)(vbuf + c * 64), 4, 0, 0);
                }
                return;
            }
#pragma unroll
            for (int c = 0; c < NVC; ++c) {
                // lane k holds key k's code (the byte address folds into the instruction)
                const int rc_ = __builtin_amdgcn_ds_bpermute(lane / LPR * 4 + c * (256 / LPR), code);
                const float* vp = rc_ < 0 ? ctx_v + (size_t)(~rc_) * HD : seg_v + (size_t)rc_ * HD;
                __builtin_amdgcn_global_load_lds(vp + (lane % LPR) * 4, (lds_void*)(vbuf + c * 256), 16, 0, 0);
            }
        };

        if (wave < n_tiles) load_k(wave);
        for (int t = wave; t < n_tiles; t += kWaves) {
            copy_v();
            // two chains, added at the end: half the rounding of one long chain
            f32x16 s0 = {}, s1 = {};
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (j & 1)
                        s1 = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j][e], qf[j][e], s1, 0, 0, 0);
                    else
                        s0 = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j][e], qf[j][e], s0, 0, 0, 0);
                }
            s0 += s1;
            __builtin_amdgcn_sched_barrier(0);  // the K loads wait for the registers of this tile's
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the V tile is in LDS
            asm volatile("" ::: "memory");
            if (t + kWaves < n_tiles) load_k(t + kWaves);
            const bool masked = t * kKeys + kKeys - 1 > all_hi;
            const int rem = vis_hi - t * kKeys - half * 4;  // key offsets above it are masked
#pragma unroll
            for (int r = 0; r < 16; ++r) s0[r] *= sc;
            if (masked) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if ((r >> 2) * 8 + (r & 3) > rem) s0[r] = -INFINITY;
            }
            float mt = s0[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) mt = fmaxf(mt, s0[r]);
            mt = pair_max(mt);
            if (__builtin_amdgcn_ballot_w64(mt > m)) {
                const float mn = fmaxf(m, mt);
                const float alpha = m == mn ? 1.f : exp2f(m - mn);  // 0 when m == -inf
                l *= alpha;
#pragma unroll
                for (int db = 0; db < NDB; ++db) oacc[db] *= alpha;
                m = mn;
            }
            const float mr = m == -INFINITY ? 0.f : m;  // a column that has seen no key yet
            float ts = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                s0[r] = exp2f(s0[r] - mr);
                ts += s0[r];
            }
            l += ts;
            const float* vr = vbuf + half * 4 * HD + l32;
            // A masked key weighs 0, but 0 times an infinity or NaN of its
            // value row is no zero: in a masked tile that holds one, the
            // product takes 0 in its place, and the columns that see the key
            // add it afterwards.
            uint32_t top = 0;  // largest magnitude in the tile
            if (masked) {
#pragma unroll 1
                for (int i = 0; i < NVC; ++i) {
                    const u32x4 w = *reinterpret_cast<const u32x4*>(vbuf + i * 256 + lane * 4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) top = max(top, w[e] & 0x7fffffffu);
                }
            }
            const bool unclean = __builtin_amdgcn_ballot_w64(top >= 0x7f800000u) != 0;
            const uint32_t keep = unclean ? 0x7f7fffffu : 0x7fffffffu;  // magnitudes that enter the product
#pragma unroll
            for (int r = 0; r < 16; ++r)
#pragma unroll
                for (int db = 0; db < NDB; ++db) {
                    const float v = vr[((r >> 2) * 8 + (r & 3)) * HD + db * 32];
                    oacc[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                        (__float_as_uint(v) & 0x7fffffffu) <= keep ? v : 0.f, s0[r], oacc[db], 0, 0, 0);
                }
            if (__builtin_expect(unclean, 0)) {
                const int rem0 = min(vis_hi, n_keys - 1) - t * kKeys;
#pragma unroll 1
                for (int key = 0; key <= rem0 && key < kKeys; ++key)
#pragma unroll
                    for (int db = 0; db < NDB; ++db)
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const float v = vbuf[key * HD + db * 32 + (r >> 2) * 8 + half * 4 + (r & 3)];
                            oacc[db][r] += __builtin_isfinite(v) ? 0.f : v;
                        }
            }
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the V tile is read before the next copy
            asm volatile("" ::: "memory");
        }
        if (last_pass) break;
    }

    // ---- merge of the four waves: O rows in LDS (16-byte chunks swizzled by
    // column), the two halves of a column's sum first
    l = pair_sum(l);
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const int c = db * 8 + r4 * 2 + half;
            *reinterpret_cast<f32x4*>(vbuf + l32 * HD + ((c ^ (l32 % LPR)) << 2)) =
                f32x4{oacc[db][r4 * 4], oacc[db][r4 * 4 + 1], oacc[db][r4 * 4 + 2], oacc[db][r4 * 4 + 3]};
        }
    if (half == 0) {
        sm.ml[wave][l32][0] = m;
        sm.ml[wave][l32][1] = l;
    }
    __syncthreads();
    for (int i = tid; i < used * LPR; i += kThreads) {
        const int col = i / LPR, c = i % LPR;
        const int j = j0 + col;
        const long row = (long)q_row0 + j / R;
        const int head = g * R + j % R;
        if (row < 0 || row > max_q) continue;
        float mx = -INFINITY;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) mx = fmaxf(mx, sm.ml[w][col][0]);
        f32x4 num = {0.f, 0.f, 0.f, 0.f};
        float den = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            // A wave that saw no visible key carries no weight (its O and sum
            // are 0; its NaN sum, from a NaN logit, counts).  One whose weight
            // underflows still passes on an infinity or NaN.
            const float mw = sm.ml[w][col][0], lw = sm.ml[w][col][1];
            const float f = mw == -INFINITY ? (lw == 0.f ? 0.f : lw) : exp2f(mw - mx);
            const f32x4 o = *reinterpret_cast<const f32x4*>(&sm.v[w][col * HD + ((c ^ (col % LPR)) << 2)]);
#pragma unroll
            for (int e = 0; e < 4; ++e) num[e] += f * o[e];
            den += f * lw;
        }
        const float inv = 1.0f / den;
#pragma unroll
        for (int e = 0; e < 4; ++e) num[e] *= inv;
        *reinterpret_cast<vec*>(a.out + ((size_t)row * a.n_q_heads + head) * HD + c * 4) = num;
        if (a.lse && c == 0)
            a.lse[(size_t)head * a.lse_rows + row] = (mx + log2f(den)) * 0.69314718055994531f;
    }
}

}  // namespace

hipError_t launch_attn_f32(const AttnF32Args& a, bool encode, hipStream_t stream) {
    AttnF32Args b = a;
    b.max_rows = (int)std::min((long)a.max_rows, a.lse_rows);  // no unit has more rows
    b.n_cb = (int)(((long)b.max_rows * a.ratio + kCols - 1) / kCols);
    const long blocks = (long)b.n_cb * a.n_units * a.n_kv_heads;
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
    const uintptr_t at = (uintptr_t)a.q | (uintptr_t)a.out | (uintptr_t)a.k | (uintptr_t)a.v | (uintptr_t)a.ck |
                         (uintptr_t)a.cv;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kThreads), 0, stream, b);
        return hipGetLastError();
    };
    if (a.head_dim == 128) {
        if (at & 15) return encode ? go(attn_f32_kernel<128, true, true>) : go(attn_f32_kernel<128, false, true>);
        return encode ? go(attn_f32_kernel<128, true, false>) : go(attn_f32_kernel<128, false, false>);
    }
    if (at & 15) return encode ? go(attn_f32_kernel<64, true, true>) : go(attn_f32_kernel<64, false, true>);
    return encode ? go(attn_f32_kernel<64, true, false>) : go(attn_f32_kernel<64, false, false>);
}

}  // namespace rc
