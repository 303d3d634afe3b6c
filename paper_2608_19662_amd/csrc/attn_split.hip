// bf16 conversation prefill for small grids: few requests or few queries,
// where blocks that own whole key streams leave most of the GPU idle.
// Visibility, key stream and softmax are those of the prefill kernel
// (attn_mfma.hip); what differs is the decomposition.
//
// The query rows of a request and KV group are flattened to columns
// j = row * ratio + head; a block owns 32 of them, and its W waves take the
// 32-key tiles of the stream in turn, each with its own softmax state and
// pipeline (no barriers in the loop), merged in LDS at the end.  A stream of
// n keys then costs a block n / (32 W) tiles instead of n / 64, and a group's
// blocks number rows * ratio / 32 instead of rows * ratio / 256.  What it
// gives up is sharing: every wave reads its own K and V (16 KB per tile of
// 16 MFMAs), so a full grid would run at the L2's 64 B/clk per CU, about half
// of the matrix rate.  The launcher's rule weighs the two.
//
// Per tile (32 keys):
//     S^T = K Q^T      (32x32x16 bf16 MFMA; A = K rows from LDS, B = Q^T in VGPRs)
//     O^T += V^T P^T   (A = V^T by LDS transpose reads, B = P^T from the S^T
//                       accumulators)
// K and V go straight into LDS.  (K fragments loaded into VGPRs touch 32 rows
// with 32 bytes each per load: 46 us against 32 at 64 queries, 4,000 keys.)
#include <algorithm>

#include "attn_tile.hpp"
#include "common.hpp"
#include "kernels.hpp"

namespace rc {

namespace {

constexpr int kCols = 32;  // columns (row, head) per block
constexpr int kKeys = 32;  // keys per wave tile

template <int W>
struct SplitSmem {
    int seg_start[kMaxSeg + 1];
    int seg_row[kMaxSeg];
    int scan[2 * W];
    float ml[W][kCols][2];
};

// Reads a K tile's fragments from LDS and waits for them.
template <int N>
__device__ __forceinline__ void read_k(const uint32_t* addr, u32x4* f) {
    static_assert(N == 4 || N == 8, "head_dim 64 or 128");
    if constexpr (N == 8)
        asm volatile(
            "ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %11\n\t"
            "ds_read_b128 %4, %12\n\tds_read_b128 %5, %13\n\tds_read_b128 %6, %14\n\tds_read_b128 %7, %15\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[4]), "=&v"(f[5]), "=&v"(f[6]), "=&v"(f[7])
            : "v"(addr[0]), "v"(addr[1]), "v"(addr[2]), "v"(addr[3]), "v"(addr[4]), "v"(addr[5]), "v"(addr[6]),
              "v"(addr[7])
            : "memory");
    else
        asm volatile(
            "ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3])
            : "v"(addr[0]), "v"(addr[1]), "v"(addr[2]), "v"(addr[3])
            : "memory");
}

// Whether a launch numbers its blocks over the column blocks that there are
// rather than n_qt for every request (and leaves a work order aside).  In a
// batch of few long and many short requests most blocks of the full grid are
// empty, and the others fall on few XCDs and CUs wherever n_qt has a factor in
// common with their number: 63 requests of one query and one of 128 over 100
// keys, 8 / 1 heads, 83 us against 14; 511 and one 431 against 31.  A full grid
// of one block per free CU slot (two 4-wave blocks or one of 8 per CU) has no
// such problem and saves the search (0.5 us: four requests of 9 to 300 queries,
// 8 / 2 heads, 28.4 us against 29.0).
bool compact_grid(const AttnArgs& a, int waves) {
    return a.n_qt > 1 && a.n_units > 1 && (long)a.n_qt * a.n_units * a.n_kv_heads > 2048 / waves;
}

// The idx-th column block in order of the requests, each one's last columns
// first: (request, column block), or request -1 past the last.  Each wave
// searches for itself, four requests per lane and step.
__device__ __forceinline__ int2 nth_col_block(const AttnArgs& a, int idx, int lane) {
    for (int u0 = 0; u0 < a.n_units; u0 += 256) {
        const int u = u0 + lane * 4;
        int c[5], n[4], sum = 0;
#pragma unroll
        for (int i = 0; i < 5; ++i) c[i] = a.cu_q[min(u + i, a.n_units)];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            n[i] = (max(0, min(c[i + 1] - c[i], a.max_rows)) * a.ratio + kCols - 1) / kCols;
            sum += n[i];
        }
        int incl = sum;
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o);
            if (lane >= o) incl += y;
        }
        int at = idx - (incl - sum);  // of the lane's column blocks
        const uint64_t hit = __builtin_amdgcn_ballot_w64(at >= 0 && at < sum);
        if (hit) {
            int2 r = make_int2(0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (at >= 0 && at < n[i]) r = make_int2(u + i, n[i] - 1 - at);
                at -= n[i];
            }
            const int l = __builtin_ctzll(hit);
            return make_int2(__builtin_amdgcn_readlane(r.x, l), __builtin_amdgcn_readlane(r.y, l));
        }
        idx -= __builtin_amdgcn_readlane(incl, 63);
    }
    return make_int2(-1, 0);
}

template <int HD, int W, bool COMPACT>
__global__ __launch_bounds__(W * 64, 2) void attn_split_kernel(const AttnArgs a) {
    constexpr int kThreads = W * 64;
    constexpr int CPR = HD / 8;        // 16-byte chunks per row
    constexpr int ROWB = HD * 2;       // bytes per row
    constexpr int NT = HD / 16;        // MFMA k-steps over head_dim
    constexpr int NDB = HD / 32;       // 32-wide blocks of head_dim
    constexpr int RPI = 64 / CPR;      // rows per 1 KB wave copy
    constexpr int NJ = kKeys / RPI;    // copies per V tile
    constexpr int NP = CPR == 16 ? 4 : 1;  // copy j's swizzle repeats with this period
    constexpr int TILEB = kKeys * ROWB;
    __shared__ SplitSmem<W> sm;
    // Per wave one K and one V tile (two arrays: the compiler then sees that
    // copies in flight into one do not touch the other); after the loop the
    // lower and upper dims of the wave's O, fp32 [32 columns][HD / 2] each.
    __shared__ __attribute__((aligned(16))) char k_st[W][TILEB], v_st[W][TILEB];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int R = a.ratio;

    // block -> (unit, column block [longest first], group), as in the prefill
    // kernel: the blocks of one (request, group) run side by side on one XCD
    int bid = blockIdx.x;
    int g = bid % a.n_kv_heads;
    bid /= a.n_kv_heads;
    int cb, unit;
    if constexpr (COMPACT) {
        const int2 at = nth_col_block(a, bid, lane);
        unit = at.x, cb = at.y;
        if (unit < 0) return;  // the grid is a bound on the blocks there are
        g = (g + unit) % a.n_kv_heads;
    } else {
        cb = a.n_qt - 1 - bid % a.n_qt;
        unit = bid / a.n_qt;
        if (a.plan) {
            const int n_pairs = a.n_units * a.n_kv_heads;
            int p = a.plan[(size_t)a.layer * n_pairs + unit * a.n_kv_heads + g];
            p = min(max(p, 0), n_pairs - 1);  // in bounds whatever the plan holds
            unit = p / a.n_kv_heads;
            g = p % a.n_kv_heads;
        } else {
            g = (g + unit) % a.n_kv_heads;
        }
    }
    const int q_row0 = a.cu_q[unit], q_len = a.cu_q[unit + 1] - q_row0;
    const int c0 = a.cu_ctx[unit], tc = a.cu_ctx[unit + 1] - c0;
    // the grid covers max_rows rows; the last block answers for any beyond
    if (cb == a.n_qt - 1 && q_len > a.max_rows)
        poison_rows<HD>(a, g * R, R, q_row0, a.max_rows, q_len, tid, kThreads);
    const int j0 = cb * kCols, n_cols = min(q_len, a.max_rows) * R;
    if (j0 >= n_cols) return;
    const int used = min(kCols, n_cols - j0);
    const int my_j = j0 + min(l32, used - 1);  // spare lanes repeat the last column
    const int my_row = my_j / R, my_head = g * R + my_j % R;
    const int first_row = j0 / R, last_row = (j0 + used - 1) / R;

    // ---- Q^T (B operand): dims t*16 + half*8 + [0, 8) of this lane's column
    bf16x8 qf[NT];
    {
        const long row = max(0L, min((long)q_row0 + my_row, a.lse_rows - 1));
        const uint16_t* qp = a.q + ((size_t)row * a.n_q_heads + my_head) * HD + half * 8;
#pragma unroll
        for (int t = 0; t < NT; ++t)
            qf[t] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(qp + t * 16));
    }

    // ---- visible segments of this (request, layer, group)
    const size_t e = ((size_t)unit * a.n_layers + a.layer) * a.n_kv_heads + g;
    const int r0 = a.route_off[e];
    const int n_seg = a.route_off[e + 1] - r0;
    if (n_seg > kMaxSeg) {
        for (int j = j0 + wave; j < j0 + used; j += W)
            poison_rows<HD>(a, g * R + j % R, 1, q_row0, j / R, j / R + 1, lane, 64);
        return;
    }
    const int s_vis = segment_table<W, false>(a.route_res + r0, n_seg, a.cu_kept, a.res_off, a.n_kv_heads, g, 0,
                                              sm.seg_start, sm.seg_row, sm.scan);
    // Tiles: the segment rows' 32 at a time, then the causal rows', so that
    // every tile has its rows in one plane.
    const int off = tc - q_len;                          // a column sees causal rows <= off + row
    const int n_ctx = max(0, min(off + last_row + 1, tc));  // causal rows the block sees
    const int n_segt = (s_vis + kKeys - 1) / kKeys;
    const int n_tiles = n_segt + (n_ctx + kKeys - 1) / kKeys;

    // ---- HBM -> LDS copies.  Two planes (segment rows, causal rows), each a
    // buffer resource for K and one for V: a load past a plane's end returns
    // zeros.  A tile of consecutive rows takes their offset in a scalar
    // register plus per-lane constants; any other tile looks its keys up, key
    // l32 per lane, and its copies fetch the row offsets from those lanes.
    // Copy j moves rows j*RPI + [0, RPI); lane i lands at byte 16 i of them,
    // chunk i % CPR, which holds logical chunk (i % CPR) ^ mask(row).
    // The resource is formed at each copy from values pinned to scalar
    // registers: one in vector registers would cost every copy a loop.
    auto plane = [&](bool is_v, bool causal) {
        const uint16_t* p = causal ? (is_v ? a.cv : a.ck) : (is_v ? a.v : a.k);
        const uint64_t u = (uint64_t)(p + (size_t)g * (causal ? a.c_rows : a.k_gstride) * HD);
        const uint64_t base = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(u >> 32)) << 32) |
                              (uint32_t)__builtin_amdgcn_readfirstlane((int)u);
        const int bytes = __builtin_amdgcn_readfirstlane((int)((causal ? a.c_rows : a.k_rows) * ROWB));
        return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, bytes, kBufferFlags);
    };
    const int v_row = lane / CPR;  // row of this lane in a copy
    u32x4 lane_off;                // its byte offset in copy j % NP, from the copy's first row
#pragma unroll
    for (int j = 0; j < 4; ++j)
        lane_off[j] = (uint32_t)(v_row * ROWB + (((lane % CPR) ^ chunk_mask<CPR>(j % NP * RPI + v_row)) << 4));
    bool causal = true;   // the plane of the tile being copied
    bool t_fast = false;  // its rows are consecutive:
    uint32_t t_off = 0;   // the first one's byte offset
    uint32_t key_off = 0; // else this lane's key l32: its row's byte offset
    int u_i = 0, u_hi = 0, u_dl = 0;   // wave-uniform segment walk
    int sidx = 0, s_hi = 0, s_dl = 0;  // this lane's segment walk
    if (n_seg > 0) {
        u_hi = __builtin_amdgcn_readfirstlane(sm.seg_start[1]);
        u_dl = __builtin_amdgcn_readfirstlane(sm.seg_row[0]);
        s_hi = u_hi;
        s_dl = u_dl;
    }
    auto set_tile = [&](int t) {
        long row;
        if (t < n_segt) {
            const int p0 = t * kKeys;
            while (p0 >= u_hi && u_i + 1 < n_seg) {
                ++u_i;
                u_hi = __builtin_amdgcn_readfirstlane(sm.seg_start[u_i + 1]);
                u_dl = __builtin_amdgcn_readfirstlane(sm.seg_row[u_i]) -
                       __builtin_amdgcn_readfirstlane(sm.seg_start[u_i]);
            }
            causal = false;
            row = (long)u_dl + p0;
            t_fast = p0 + kKeys <= u_hi && row >= 0 && row + kKeys <= a.k_rows;
            if (!t_fast) {
                const int p = min(p0 + l32, s_vis - 1);  // keys past the end repeat the last one
                while (p >= s_hi && sidx + 1 < n_seg) {
                    ++sidx;
                    s_hi = sm.seg_start[sidx + 1];
                    s_dl = sm.seg_row[sidx] - sm.seg_start[sidx];
                }
                key_off = (uint32_t)(s_dl + p) * ROWB;
            }
        } else {
            const int p0 = (t - n_segt) * kKeys;
            causal = true;
            row = (long)c0 + p0;
            t_fast = p0 + kKeys <= n_ctx && row >= 0 && row + kKeys <= a.c_rows;
            key_off = (uint32_t)(c0 + min(p0 + l32, n_ctx - 1)) * ROWB;
        }
        t_off = (uint32_t)row * ROWB;
    };
    auto copy = [&](bool is_v, char* dst) {
        const __amdgpu_buffer_rsrc_t r = plane(is_v, causal);
        const uint32_t off0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)t_off);
        if (__builtin_amdgcn_readfirstlane((int)t_fast)) {
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)(dst + j * 1024), 16, (int)lane_off[j % NP],
                                                         (int)(off0 + j * RPI * ROWB), 0, 0);
        } else {
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const uint32_t vo = (uint32_t)__builtin_amdgcn_ds_bpermute(v_row * 4 + j * RPI * 4, (int)key_off) +
                                    (lane_off[j % NP] - (uint32_t)(v_row * ROWB));
                __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)(dst + j * 1024), 16, (int)vo, 0, 0, 0);
            }
        }
    };

    // V^T transpose-read offset (see attn_mfma.hip): rows s*16 + w*8 + half*4
    // + [0, 4), the keys that P^T holds in slots w*4 + [0, 4) of step s
    uint32_t v_rd0;
    {
        const int G = lane >> 4, i = lane & 15;
        const int row = (G >> 1) * 4 + (i >> 2);
        const int col = (G & 1) * 16 + (i & 3) * 4;
        v_rd0 = swz<HD>(row, col >> 3) + (col & 7) * 2;
    }
    auto v_rd = [&](int db, int w) -> uint32_t {
        return v_rd0 ^ (uint32_t)(db << 6) ^ (uint32_t)(w * (8 * ROWB + (CPR == 16 ? 32 : 0)));
    };

    const float sl2 = a.scale_log2;
    const bf16x2 ones2 = __builtin_bit_cast(bf16x2, 0x3F803F80u);  // (1.0, 1.0) in bf16
    float m = kNoKey, lsum = 0.f;
    f32x16 oacc[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db) oacc[db] = f32x16{};

    // This wave's tiles are wave, wave + W, ...; only it touches its buffers,
    // so waiting for its own copies is enough.  K(t + W) is copied behind the
    // reads of K(t), V(t + W) behind those of V(t): one of the two is in
    // flight at any time, and the block's other waves fill the waits.
    constexpr int WAIT_OLD = NJ | 0x0F70;  // vmcnt(NJ): all but the newest tile copy
    static_assert(NJ < 16, "vmcnt(NJ) fits the low counter bits");
    char* kb = k_st[wave];
    char* vb = v_st[wave];
    // K as the A operand: key l32, chunk 2t + half (t moves chunk bits 1..3)
    uint32_t k_addr[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) k_addr[i] = (uint32_t)(uintptr_t)(lds_void*)kb + (swz<HD>(l32, half) ^ (i << 5));
    if (wave < n_tiles) {
        set_tile(wave);
        copy(false, kb);
        // (the first wait counts on this order, which two arrays alone leave open)
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        copy(true, vb);
    }
    // (the loop ends from its middle, so that on its back edge a V copy always
    // follows the K copy: the compiler's own waits then count as these do)
    for (int t = wave; wave < n_tiles; t += W) {
        const bool more = t + W < n_tiles;
        __builtin_amdgcn_s_waitcnt(WAIT_OLD);  // K(t)
        // (The compiler would wait here for the V copies in flight as well.)
        u32x4 kf[NT];
        read_k<NT>(k_addr, kf);
        f32x16 sc = {};
#pragma unroll
        for (int i = 0; i < NT; ++i)
            sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[i]), qf[i], sc, 0, 0, 0);
        if (more) {
            set_tile(t + W);
            copy(false, kb);
        }
        // key offsets that every column of the block sees, and this lane's
        const int p0 = (t < n_segt ? t : t - n_segt) * kKeys;
        if (kKeys - 1 > (t < n_segt ? s_vis - 1 : off + first_row) - p0) {
            const int rem = (t < n_segt ? s_vis - 1 : off + my_row) - p0 - half * 4;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if ((r >> 2) * 8 + (r & 3) > rem) sc[r] = -INFINITY;
        }
        bf16x8 pf[2];
        float tsum;
        auto weights = [&]() {
            const float msl = m * sl2;
            tsum = 0.f;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                uint32_t w[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float p0 = __builtin_amdgcn_exp2f(fmaf(sc[8 * s + 2 * i], sl2, -msl));
                    const float p1 = __builtin_amdgcn_exp2f(fmaf(sc[8 * s + 2 * i + 1], sl2, -msl));
                    w[i] = pack_bf16x2(p0, p1);
                    tsum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w[i]), ones2, tsum, false);
                }
                pf[s] = __builtin_bit_cast(bf16x8, u32x4{w[0], w[1], w[2], w[3]});
            }
        };
        // Weights against the reference max m, set by the wave's first tile
        // and moved (O and the row sum rescaled) only when a lane's sum of
        // them shows that one could pass 2^16.  A column that its wave's first
        // tile does not show a key sees none of the later ones either.
        auto row_max = [&]() {
            float mt = sc[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) mt = fmaxf(mt, sc[r]);
            return pair_max(mt);
        };
        if (t == wave) {
            m = row_max();
            if (m == -INFINITY) m = kNoKey;
        }
        weights();
        if (__builtin_amdgcn_ballot_w64(!(tsum <= kWeightCap)) != 0) {
            const float m_new = fmaxf(m, row_max());
            const float alpha = __builtin_amdgcn_exp2f((m - m_new) * sl2);
            lsum *= alpha;
#pragma unroll
            for (int db = 0; db < NDB; ++db) oacc[db] *= alpha;
            m = m_new;
            weights();
        }
        lsum += tsum;
        if (more)
            __builtin_amdgcn_s_waitcnt(WAIT_OLD);  // V(t)
        else
            __builtin_amdgcn_s_waitcnt(0x0F70);
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (lds_s16x4*)(vb + v_rd(db, 0) + s * 16 * ROWB));
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (lds_s16x4*)(vb + v_rd(db, 1) + s * 16 * ROWB));
                const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
                const bf16x8 av = __builtin_bit_cast(bf16x8, u32x4{l2[0], l2[1], h2[0], h2[1]});
                oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, pf[s], oacc[db], 0, 0, 0);
            }
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): V(t) is read
        if (!more) break;
        copy(true, vb);
    }

    // ---- merge of the waves: O rows in LDS (16-byte chunks swizzled by
    // column), then eight dims of one column per thread
    lsum = pair_sum(lsum);
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const int c = db % (NDB / 2) * 8 + r4 * 2 + half;  // 16-byte chunk of the half row
            *reinterpret_cast<f32x4*>((db < NDB / 2 ? kb : vb) + l32 * ROWB + ((c ^ (l32 % CPR)) << 4)) =
                f32x4{oacc[db][r4 * 4], oacc[db][r4 * 4 + 1], oacc[db][r4 * 4 + 2], oacc[db][r4 * 4 + 3]};
        }
    if (half == 0) {
        sm.ml[wave][l32][0] = m == kNoKey ? -INFINITY : m;
        sm.ml[wave][l32][1] = lsum;
    }
    __syncthreads();
    for (int i = tid; i < used * CPR; i += kThreads) {
        const int col = i / CPR, c = i % CPR;
        const int j = j0 + col, row = j / R, head = g * R + j % R;
        float mx = -INFINITY;
#pragma unroll
        for (int w = 0; w < W; ++w) mx = fmaxf(mx, sm.ml[w][col][0]);
        float num[8] = {}, den = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const float mw = sm.ml[w][col][0];
            const float f = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((mw - mx) * sl2);
            den += f * sm.ml[w][col][1];
            const char* o = (c < CPR / 2 ? k_st[w] : v_st[w]) + col * ROWB;
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2) {
                const f32x4 x =
                    *reinterpret_cast<const f32x4*>(o + (((c % (CPR / 2) * 2 + h2) ^ (col % CPR)) << 4));
#pragma unroll
                for (int k = 0; k < 4; ++k) num[h2 * 4 + k] += f * x[k];
            }
        }
        const float inv = 1.0f / den;
        const u32x4 o = {pack_bf16x2(num[0] * inv, num[1] * inv), pack_bf16x2(num[2] * inv, num[3] * inv),
                         pack_bf16x2(num[4] * inv, num[5] * inv), pack_bf16x2(num[6] * inv, num[7] * inv)};
        if ((long)q_row0 + row < 0 || (long)q_row0 + row >= a.lse_rows) continue;
        *reinterpret_cast<u32x4*>(a.out + ((size_t)(q_row0 + row) * a.n_q_heads + head) * HD + c * 8) = o;
        if (a.lse && c == 0)
            a.lse[(size_t)head * a.lse_rows + q_row0 + row] = mx * sl2 * 0.69314718055994531f + logf(den);
    }
}

template <int HD, int W>
hipError_t launch(const AttnArgs& b, bool compact, unsigned blocks, hipStream_t stream) {
    if (compact)
        hipLaunchKernelGGL((attn_split_kernel<HD, W, true>), dim3(blocks), dim3(W * 64), 0, stream, b);
    else
        hipLaunchKernelGGL((attn_split_kernel<HD, W, false>), dim3(blocks), dim3(W * 64), 0, stream, b);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_split(const AttnArgs& a, int head_dim, int waves, hipStream_t stream) {
    AttnArgs b = a;
    b.max_rows = (int)std::min((long)a.max_rows, a.lse_rows);  // no unit has more rows
    b.n_qt = (int)(((long)b.max_rows * a.ratio + kCols - 1) / kCols);
    // compact: no more column blocks than the full ones and one begun by every request
    const bool compact = compact_grid(b, waves);
    const long full = (long)b.n_qt * b.n_units;
    const long blocks =
        (compact ? std::min(full, (a.lse_rows * a.ratio + (kCols - 1L) * b.n_units) / kCols) : full) * b.n_kv_heads;
    if (blocks <= 0) return hipSuccess;
    if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
    const unsigned n = (unsigned)blocks;
    if (head_dim == 128)
        return waves == 8 ? launch<128, 8>(b, compact, n, stream) : launch<128, 4>(b, compact, n, stream);
    return waves == 8 ? launch<64, 8>(b, compact, n, stream) : launch<64, 4>(b, compact, n, stream);
}

}  // namespace rc
