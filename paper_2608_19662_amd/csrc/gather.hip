// Index work of the method, all integer and exact:
//   - kept-row gather (ReCache Sec. 3, "Semantic Pruning"): the retained
//     subsequence of every resource, copied bit for bit into a compacted,
//     head-major buffer;
//   - route lists (Sec. 3, "Structural Pruning"): for every (request, layer,
//     KV group), the request's resources whose route is in Omega, in request
//     order, as a CSR with a per-entry kept-token total;
//   - a route-compacted store (both pruning stages): per layer, only the
//     visible (resource, group) routes hold rows, resource-major, each with
//     the kept rows of its resource.
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"

namespace rc {

namespace {

// Blocks per (resource r, KV head g): n_parts of them share the kept rows of
// r for head g (contiguous, equal shares), which go to rows g * total_kept +
// cu_kept[r] + j of the compacted caches.  Each thread moves U 16-byte
// chunks per step, all loads issued before the stores; source rows are
// clamped into the caches.
__global__ __launch_bounds__(256) void prune_gather_kernel(
    int chunks_per_row, int n_kv_heads, int n_parts, const int32_t* __restrict__ cu_len,
    const int32_t* __restrict__ cu_kept, const int32_t* __restrict__ kept_idx, long total_T,
    long total_kept, const u32x4* __restrict__ kc, const u32x4* __restrict__ vc,
    u32x4* __restrict__ ko, u32x4* __restrict__ vo) {
    constexpr int U = 8;
    const int part = blockIdx.x % n_parts, rg = blockIdx.x / n_parts;
    const int r = rg / n_kv_heads, g = rg % n_kv_heads;
    const long r0 = cu_kept[r];
    const long r1 = min((long)cu_kept[r + 1], total_kept);
    if (r0 < 0 || r1 <= r0) return;
    // this block's share of the resource's kept rows
    const long k0 = r0 + (r1 - r0) * part / n_parts;
    const long k1 = r0 + (r1 - r0) * (part + 1) / n_parts;
    if (k1 <= k0) return;
    const long beg = cu_len[r];
    const int sh = __builtin_ctz(chunks_per_row);  // a power of two
    const long n = (k1 - k0) * chunks_per_row;
    const size_t src_base = (size_t)g * total_T;
    const size_t dst_base = ((size_t)g * total_kept + k0) * chunks_per_row;
    for (long c0 = threadIdx.x; c0 < n; c0 += 256 * U) {
        u32x4 kx[U], vx[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long c = min(c0 + u * 256, n - 1);
            const long j = c >> sh;
            const int e = (int)(c & (chunks_per_row - 1));
            long src = beg + kept_idx[k0 + j];
            src = src < 0 ? 0 : (src >= total_T ? total_T - 1 : src);
            const size_t si = (src_base + src) * chunks_per_row + e;
            kx[u] = kc[si];
            vx[u] = vc[si];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long c = c0 + u * 256;
            if (c < n) {
                ko[dst_base + c] = kx[u];
                vo[dst_base + c] = vx[u];
            }
        }
    }
}

// The resources of a request, kRouteStage at a time, one per lane: id (-1 where
// the request lists none that exists) and kept length.  This costs two round
// trips whatever the list, and the mask bytes are then independent loads.
constexpr int kRouteStage = 64;

__device__ __forceinline__ int2 stage_resource(int j, int j1, int n_res, const int32_t* req_res,
                                               const int32_t* cu_kept) {
    int r = j < j1 ? req_res[j] : -1;
    if (r < 0 || r >= n_res) return make_int2(-1, 0);
    return make_int2(r, cu_kept[r + 1] - cu_kept[r]);
}

// Slices of the entries, one per wave: 64 entries of a request, fewer in its
// last slice, or with FLAT any 64 consecutive entries.  Index in route_off of
// the last entry of slice sl.
struct Slices {
    int n;        // slices in all
    int per_req;  // of each request
    int LG, E;    // entries of a request, and in all
};

template <bool FLAT>
__device__ __forceinline__ size_t slice_last(const Slices& z, uint32_t sl) {
    if (FLAT) return min((long)sl * 64 + 64, (long)z.E);
    return (size_t)(sl / (uint32_t)z.per_req) * z.LG + min((int)(sl % (uint32_t)z.per_req) * 64 + 64, z.LG);
}

// Resources k0 .. k0 + 15 of a staged list for the entries of the lanes that
// are `in`: mask bytes first, then the counts or, with FILL, the ids.
template <bool FILL>
__device__ __forceinline__ void walk_step(const int2 mine, const int k0, const bool in, const uint8_t* m, const int LG,
                                          int& cnt, int& tok, int& w, int32_t* __restrict__ route_res) {
    constexpr int U = 16;
    uint8_t v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        // lanes of k0 + u < 64 hold ids, or -1 past the list
        const int r = __builtin_amdgcn_readlane(mine.x, k0 + u);
        v[u] = m[(size_t)max(r, 0) * LG];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int r = __builtin_amdgcn_readlane(mine.x, k0 + u);
        if (r >= 0 && in && v[u]) {
            if constexpr (FILL) {
                route_res[w++] = r;
            } else {
                ++cnt;
                tok += __builtin_amdgcn_readlane(mine.y, k0 + u);
            }
        }
    }
}

// Entry e = (b * L + l) * G + g, one wave per slice of 64 entries of a request.
// First pass: count the visible resources and their kept rows; route_off[e + 1]
// gets the counts' inclusive scan within the slice.  route_scan_kernel makes
// the slices' last entries final.  Second pass (FILL): the other entries, from
// the last one of the slice before, and the resource ids in request order.
// Bound by latency: 18,432 entries of 32 resources each in 4.8 and 4.9 us (a
// thread per entry that walked the list itself, on 72 CUs: 13.7 and 11.5).
// FLAT: lanes of several requests, each of which walks its own list.
template <bool FILL, bool FLAT>
__global__ __launch_bounds__(64) void route_walk_kernel(
    const Slices z, int n_res, const int32_t* __restrict__ req_res_off,
    const int32_t* __restrict__ req_res, const uint8_t* __restrict__ mask,
    const int32_t* __restrict__ cu_kept, int32_t* __restrict__ route_off,
    int32_t* __restrict__ route_tokens, int32_t* __restrict__ route_res) {
    const int LG = z.LG, lane = threadIdx.x;
    const uint32_t sl = blockIdx.x;
    int b, lg;  // request and (layer, group) of this lane
    bool in, last;  // whether its entry exists, and ends its slice
    if constexpr (FLAT) {
        const uint32_t e = sl * 64 + lane;
        b = (int)(min(e, (uint32_t)z.E - 1) / (uint32_t)LG);
        lg = (int)(e - (uint32_t)b * LG);
        in = e < (uint32_t)z.E;
        last = lane == 63 || e == (uint32_t)z.E - 1;
    } else {
        b = (int)(sl / (uint32_t)z.per_req);
        lg = (int)(sl % (uint32_t)z.per_req) * 64 + lane;
        in = lg < LG;
        last = lane == 63 || lg == LG - 1;
    }
    const uint8_t* m = mask + (in ? lg : 0);
    const int j0 = req_res_off[b], j1 = req_res_off[b + 1];
    const size_t e = (size_t)b * LG + lg;
    int cnt = 0, tok = 0, w = 0, incl = 0;
    if constexpr (FILL) {
        const int base = sl > 0 ? route_off[slice_last<FLAT>(z, sl - 1)] : 0;
        // (a slice's last entry holds its final value already)
        incl = in ? (last ? route_off[e + 1] : base + route_off[e + 1]) : 0;
        const int before = __shfl_up(incl, 1);
        w = lane == 0 ? base : before;
    }
    if constexpr (FLAT) {
        // (one or two long lists among short ones by the wave, 0.08 us per
        // resource each, instead of 0.2 by one lane each side by side)
        const bool is_long = in && j1 - j0 > 32;
        const int b_before = __shfl_up(b, 1);
        const bool by_wave = __popcll(__builtin_amdgcn_ballot_w64(is_long && (lane == 0 || b != b_before))) <= 2;
        for (uint64_t left = by_wave ? __builtin_amdgcn_ballot_w64(is_long) : 0; left;) {
            const int l = __builtin_ctzll(left);
            const bool its = in && b == __builtin_amdgcn_readlane(b, l);
            const int end = __builtin_amdgcn_readlane(j1, l);
            for (int js = __builtin_amdgcn_readlane(j0, l); js < end; js += kRouteStage) {
                const int2 mine = stage_resource(js + lane, end, n_res, req_res, cu_kept);
                for (int k0 = 0; k0 < min(kRouteStage, end - js); k0 += 16)
                    walk_step<FILL>(mine, k0, its, m, LG, cnt, tok, w, route_res);
            }
            left &= ~__builtin_amdgcn_ballot_w64(its);
        }
        const int end = in && !(is_long && by_wave) ? j1 : j0;
#pragma unroll 4
        for (int j = j0; j < end; ++j) {
            const int r = req_res[j];
            if (r < 0 || r >= n_res || !m[(size_t)r * LG]) continue;
            if constexpr (FILL) {
                route_res[w++] = r;
            } else {
                ++cnt;
                tok += cu_kept[r + 1] - cu_kept[r];
            }
        }
    }
    for (int js = j0; !FLAT && js < j1; js += kRouteStage) {
        const int2 mine = stage_resource(js + lane, j1, n_res, req_res, cu_kept);
        const int n = min(kRouteStage, j1 - js);
        for (int k0 = 0; k0 < n; k0 += 16) walk_step<FILL>(mine, k0, in, m, LG, cnt, tok, w, route_res);
    }
    if constexpr (FILL) {
        if (in && !last) route_off[e + 1] = incl;
        if (sl == 0 && lane == 0) route_off[0] = 0;
    } else {
        int s = cnt;
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(s, o);
            if (lane >= o) s += y;
        }
        if (in) {
            route_off[e + 1] = s;
            route_tokens[e] = tok;
        }
    }
}

// The slices' totals (their last entries of route_off) become the entries'
// final values: an inclusive scan over the slices by one block.  (Over all
// entries, 18,432 of them: 11.3 us; over their 320 slices 4.6.)
template <bool FLAT>
__global__ __launch_bounds__(1024) void route_scan_kernel(const Slices z, int32_t* __restrict__ route_off) {
    __shared__ int wave_tot[2][16];  // alternate buffers: one barrier per chunk suffices
    int carry = 0, k = 0;
    for (long base = 0; base < z.n; base += 1024, k ^= 1) {
        const long sl = base + threadIdx.x;
        const size_t at = slice_last<FLAT>(z, (uint32_t)min(sl, z.n - 1L));
        const int v = sl < z.n ? route_off[at] : 0;
        int total;
        const int before = carry + block_exclusive_scan<16>(v, wave_tot[k], &total);
        if (sl < z.n) route_off[at] = before + v;
        carry += total;
    }
}

// One block per layer: exclusive scan over routes i = r * G + g of
// mask[r][l][g] * kept_r, written to the layer's row of the table, plus the
// layer's total.  The routes go through in chunks of 4096 consecutive ones,
// four per thread, four chunks' loads in flight together, with a block-wide
// scan of the thread sums per chunk and the chunk totals carried on.  QUAD: G
// and the mask's address are multiples of 4, so that a thread's four routes
// are one resource's and their mask one word (36 layers of 16,384 routes: 8.2
// us; byte by byte, chunk after chunk: 15.4).
template <bool QUAD>
__global__ __launch_bounds__(1024) void store_offsets_kernel(
    int n_res, int L, int G, const uint8_t* __restrict__ mask,
    const int32_t* __restrict__ cu_kept, int32_t* __restrict__ store_off) {
    constexpr int V = 4, NC = 4;
    __shared__ int wave_tot[2][16];  // alternate buffers: one barrier per chunk suffices
    const int l = blockIdx.x, tid = threadIdx.x;
    const long n = (long)n_res * G;
    int32_t* off = store_off + (size_t)l * (n + 1);
    int carry = 0;
    for (long base = 0; base < n; base += 1024L * V * NC) {
        int v[NC][V], k0[NC][V], k1[NC][V], m[NC][V];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
#pragma unroll
            for (int j = 0; j < V; ++j) k0[c][j] = k1[c][j] = m[c][j] = 0;
            const long i = base + (c * 1024L + tid) * V;
            if (i < n) {  // (else neither divided nor loaded: a small table is bound by this)
                int r = (int)i / G, g = (int)i - r * G;
                if constexpr (QUAD) {
                    k0[c][0] = cu_kept[r];
                    k1[c][0] = cu_kept[r + 1];
                    m[c][0] = *reinterpret_cast<const int*>(mask + ((size_t)r * L + l) * G + g);
                    continue;
                }
#pragma unroll
                for (int j = 0; j < V; ++j) {
                    // (routes past the last read the last resource's entries)
                    k0[c][j] = cu_kept[r];
                    k1[c][j] = cu_kept[r + 1];
                    m[c][j] = mask[((size_t)r * L + l) * G + g];
                    if (++g == G) g = 0, r = min(r + 1, n_res - 1);
                }
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int j = 0; j < V; ++j) {
                if constexpr (QUAD)
                    v[c][j] = ((uint32_t)m[c][0] >> (8 * j)) & 0xffu ? k1[c][0] - k0[c][0] : 0;
                else
                    v[c][j] = m[c][j] && base + (c * 1024L + tid) * V + j < n ? k1[c][j] - k0[c][j] : 0;
            }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const long i0 = base + (c * 1024L + tid) * V;
            if (base + c * 1024L * V >= n) break;
            int total;
            int run = carry + block_exclusive_scan<16>(v[c][0] + v[c][1] + v[c][2] + v[c][3], wave_tot[c & 1], &total);
#pragma unroll
            for (int j = 0; j < V; ++j) {
                if (i0 + j < n) off[i0 + j] = run;
                run += v[c][j];
            }
            carry += total;
        }
    }
    if (tid == 0) off[n] = carry;
}

// Last index i in [lo, hi] with off[i] <= row (off non-decreasing, off[lo] <=
// row), by the 64 lanes of a wave together: two or three round trips for a
// table that a binary search crosses in fourteen.
__device__ __forceinline__ int wave_find_route(const int32_t* off, int lo, int hi, long row) {
    const int lane = threadIdx.x & 63;
    int n = hi - lo + 1;
    while (n > 1) {
        const int step = (n + 63) / 64;
        const bool le = lane * step < n && off[lo + lane * step] <= row;
        const int c = max(1, (int)__popcll(__builtin_amdgcn_ballot_w64(le)));
        const int skip = (c - 1) * step;
        n = min(step, n - skip);
        lo += skip;
    }
    return lo;
}

// One block per 256 U / chunks_per_row consecutive rows of the layer's store,
// whatever routes they belong to, so that every block moves the same bytes.
// One thread per row finds its source row: the wave looks up the route of its
// first row, the 64 routes after it are at hand in the lanes, and only a row
// past those searches the table.
// Rows past the routes' total (or past the store) are not written.  NT: loads
// and stores that leave no trace in the caches, for a layer larger than these
// hold.  A thread's chunks go one after another (load, wait, store: the bounds
// test keeps the compiler from loading ahead), with 2,048 threads per CU to
// cover it.  Bound by HBM: one layer of 2,048 resources (1.3 M rows of 256 bytes,
// K and V, out of 9.2 GB) in 242 us, 5.7 TB/s.  Without NT 268, with 8 chunks
// per thread instead of 4 252 (both with each thread looking its rows up);
// with a block per route in steps of eight chunks per thread 286.
template <int U, bool NT>
__global__ __launch_bounds__(256) void store_routes_kernel(
    int chunks_per_row, int G, int n_routes, const int32_t* __restrict__ off,
    const int32_t* __restrict__ cu_len, const int32_t* __restrict__ cu_kept,
    const int32_t* __restrict__ kept_idx, long total_T, long total_kept, long store_rows,
    const u32x4* __restrict__ kc, const u32x4* __restrict__ vc, u32x4* __restrict__ ko,
    u32x4* __restrict__ vo) {
    __shared__ long src_row[32 * U];  // (8 chunks per row or more)
    const int sh = __builtin_ctz(chunks_per_row);  // a power of two
    const long first = (long)blockIdx.x * (256 * U >> sh);
    const long end = min(first + (256 * U >> sh), min(store_rows, (long)off[n_routes]));
    if (end <= first) return;
    const int n_rows = (int)(end - first);
    if ((int)(threadIdx.x & ~63u) < n_rows) {
        const long row = min(first + (long)threadIdx.x, end - 1);
        const int i0 = wave_find_route(off, 0, n_routes - 1, first + (threadIdx.x & ~63u));
        const int lane = threadIdx.x & 63;
        const int next = off[min(i0 + 1 + lane, n_routes)];  // where the routes after i0 start
        int lo = 0;  // routes after i0 that start at or before the row (all lanes take every step)
#pragma unroll
        for (int step = 32; step >= 1; step >>= 1)
            if (__shfl(next, lo + step - 1) <= row) lo += step;
        if (__shfl(next, lo) <= row) ++lo;
        int i = min(i0 + lo, n_routes - 1);
        if (lo == 64) {
            int to = n_routes - 1;
            while (i < to) {
                const int mid = (i + to + 1) >> 1;
                if (off[mid] <= row) i = mid; else to = mid - 1;
            }
        }
        const int r = i / G, g = i % G;
        const long kj = max(0L, min((long)cu_kept[r] + (row - off[i]), total_kept - 1));
        const long src = max(0L, min((long)cu_len[r] + kept_idx[kj], total_T - 1));
        if ((int)threadIdx.x < n_rows) src_row[threadIdx.x] = g * total_T + src;
    }
    __syncthreads();
    const int n = n_rows << sh;  // chunks
    u32x4 kx[U], vx[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int c = min((int)threadIdx.x + u * 256, n - 1);
        const size_t si = (size_t)src_row[c >> sh] * chunks_per_row + (c & (chunks_per_row - 1));
        kx[u] = NT ? __builtin_nontemporal_load(kc + si) : kc[si];
        vx[u] = NT ? __builtin_nontemporal_load(vc + si) : vc[si];
    }
    const size_t dst = (size_t)first << sh;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int c = (int)threadIdx.x + u * 256;
        if (c >= n) break;
        if constexpr (NT) {
            __builtin_nontemporal_store(kx[u], ko + dst + c);
            __builtin_nontemporal_store(vx[u], vo + dst + c);
        } else {
            ko[dst + c] = kx[u];
            vo[dst + c] = vx[u];
        }
    }
}

}  // namespace

hipError_t launch_store_offsets(int n_res, int n_layers, int n_kv_heads, const uint8_t* mask,
                                const int32_t* cu_kept, int32_t* store_off, hipStream_t s) {
    const bool quad = n_kv_heads % 4 == 0 && ((uintptr_t)mask & 3) == 0;
    if (quad)
        hipLaunchKernelGGL(store_offsets_kernel<true>, dim3(n_layers), dim3(1024), 0, s, n_res, n_layers,
                           n_kv_heads, mask, cu_kept, store_off);
    else
        hipLaunchKernelGGL(store_offsets_kernel<false>, dim3(n_layers), dim3(1024), 0, s, n_res, n_layers,
                           n_kv_heads, mask, cu_kept, store_off);
    return hipGetLastError();
}

hipError_t launch_store_routes(int elem_bytes, int layer, int n_res, const int32_t* cu_len,
                               const int32_t* cu_kept, const int32_t* kept_idx, long total_T,
                               long total_kept, int n_kv_heads, int head_dim,
                               const int32_t* store_off, long store_rows, const void* k_cache,
                               const void* v_cache, void* k_store, void* v_store, hipStream_t s) {
    if (store_rows == 0) return hipSuccess;
    const int cpr = head_dim * elem_bytes / 16;
    const long n_routes = (long)n_res * n_kv_heads;
    if (n_routes > 0x7fffffffL) return hipErrorInvalidValue;
    constexpr int U = 4;
    const long rows = 256 * U / cpr;  // per block
    const long blocks = (store_rows + rows - 1) / rows;
    if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
    // Past the caches where K and V, read and written, take more than the 256
    // MB of the last-level cache.  The store alone is faster so at every size
    // (24 / 91 / 185 / 473 MiB of stored rows: 12.4 / 39 / 75 / 174 us instead
    // of 13.6 / 42 / 81 / 188), and with it a program that fills all layers
    // before it attends.  Where the layer's attention follows at once, a
    // cached store is found by it: both together, for 91 / 185 / 275 / 473 MiB,
    // 87 / 126 / 165 / 245 us through the caches, 92 / 131 / 167 / 236 past them.
    const bool nt = 4 * store_rows * cpr * 16 > (256L << 20);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, s, cpr, n_kv_heads, (int)n_routes,
                           store_off + (size_t)layer * (n_routes + 1), cu_len, cu_kept, kept_idx, total_T,
                           total_kept, store_rows, static_cast<const u32x4*>(k_cache),
                           static_cast<const u32x4*>(v_cache), static_cast<u32x4*>(k_store),
                           static_cast<u32x4*>(v_store));
    };
    if (nt)
        go(store_routes_kernel<U, true>);
    else
        go(store_routes_kernel<U, false>);
    return hipGetLastError();
}

hipError_t launch_prune_gather(int elem_bytes, int n_res, const int32_t* cu_len,
                               const int32_t* cu_kept, const int32_t* kept_idx, long total_T,
                               long total_kept, int n_kv_heads, int head_dim, const void* k_cache,
                               const void* v_cache, void* k_kept, void* v_kept, hipStream_t s) {
    const int cpr = head_dim * elem_bytes / 16;
    const long rg = (long)n_res * n_kv_heads;
    if (rg == 0) return hipSuccess;
    // about 2048 blocks (eight per CU) whatever the resource count
    const int parts = (int)std::min(16L, std::max(1L, (2048 + rg - 1) / rg));
    const long blocks = rg * parts;
    if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(prune_gather_kernel, dim3((unsigned)blocks), dim3(256), 0, s, cpr, n_kv_heads, parts,
                       cu_len, cu_kept, kept_idx, total_T, total_kept,
                       static_cast<const u32x4*>(k_cache), static_cast<const u32x4*>(v_cache),
                       static_cast<u32x4*>(k_kept), static_cast<u32x4*>(v_kept));
    return hipGetLastError();
}

hipError_t launch_build_routes(int n_req, const int32_t* req_res_off, const int32_t* req_res,
                               int total_req_res, int n_res, int n_layers, int n_kv_heads, const uint8_t* mask,
                               const int32_t* cu_kept, int32_t* route_off, int32_t* route_res,
                               int32_t* route_tokens, hipStream_t s) {
    Slices z{};
    z.LG = n_layers * n_kv_heads;
    z.E = n_req * z.LG;
    z.per_req = (z.LG + 63) / 64;
    const long n = (long)n_req * z.per_req;
    // With few entries per request a wave for each leaves most lanes idle and
    // costs 1.7 us per thousand requests, and some 1 us more to start with than
    // lanes that walk lists themselves; these cost 0.4 us per resource.  One
    // entry each, 20,000 requests: lists of 2 in 12.6 us instead of 44, of 30 in
    // 22 instead of 56; 4,000 of 2: 7.4 instead of 12.4; 64 of 1 / 6 / 8: 5.9 /
    // 8.2 / 9.2 instead of 7.3 / 8.7 / 8.7; 4,097 of 64: 39 instead of 26.
    // With more entries the line lies at 4: 288 entries, 8 requests of 1 / 2 / 4 /
    // 5 resources 6.7 / 7.3 / 8.3 / 8.9 instead of 8.6, 8.6, 8.6 and 8.8.
    const bool flat = (long)total_req_res <= (z.LG <= 16 ? std::max(6L, n / 256) : 4L) * n_req;
    z.n = flat ? (z.E + 63L) / 64 : n;
    auto go = [&](auto count, auto scan, auto fill) {
        hipLaunchKernelGGL(count, dim3((unsigned)z.n), dim3(64), 0, s, z, n_res, req_res_off, req_res, mask, cu_kept,
                           route_off, route_tokens, route_res);
        hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
        hipLaunchKernelGGL(scan, dim3(1), dim3(1024), 0, s, z, route_off);
        err = hipGetLastError();
        if (err != hipSuccess) return err;
        hipLaunchKernelGGL(fill, dim3((unsigned)z.n), dim3(64), 0, s, z, n_res, req_res_off, req_res, mask, cu_kept,
                           route_off, route_tokens, route_res);
        return hipGetLastError();
    };
    return flat ? go(route_walk_kernel<false, true>, route_scan_kernel<true>, route_walk_kernel<true, true>)
                : go(route_walk_kernel<false, false>, route_scan_kernel<false>, route_walk_kernel<true, false>);
}

}  // namespace rc
