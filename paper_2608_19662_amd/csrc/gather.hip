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

// Entry e = (b * L + l) * G + g: count the visible resources and their kept rows.
__global__ __launch_bounds__(256) void route_count_kernel(
    int n_req, int L, int G, int n_res, const int32_t* __restrict__ req_res_off,
    const int32_t* __restrict__ req_res, const uint8_t* __restrict__ mask,
    const int32_t* __restrict__ cu_kept, int32_t* __restrict__ route_off,
    int32_t* __restrict__ route_tokens) {
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (long)n_req * L * G) return;
    const int g = (int)(e % G);
    const int l = (int)((e / G) % L);
    const int b = (int)(e / ((long)G * L));
    int cnt = 0, tok = 0;
#pragma unroll 4
    for (int j = req_res_off[b]; j < req_res_off[b + 1]; ++j) {
        const int r = req_res[j];
        if (r < 0 || r >= n_res) continue;
        if (mask[((size_t)r * L + l) * G + g]) {
            ++cnt;
            tok += cu_kept[r + 1] - cu_kept[r];
        }
    }
    route_off[e + 1] = cnt;
    route_tokens[e] = tok;
}

// In-place inclusive scan of route_off[1..E] by one block; route_off[0] = 0.
// The entries go through in chunks of 4096 consecutive ones, four per thread
// (coalesced loads and stores), with a block-wide scan of the thread sums per
// chunk and the chunk totals carried on.
__global__ __launch_bounds__(1024) void route_scan_kernel(long E, int32_t* __restrict__ route_off) {
    constexpr int V = 4;
    __shared__ int wave_tot[2][16];  // alternate buffers: one barrier per chunk suffices
    const int tid = threadIdx.x;
    int carry = 0, k = 0;
    for (long base = 1; base <= E; base += 1024L * V, k ^= 1) {
        const long i0 = base + (long)tid * V;
        int v[V], s = 0;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            v[j] = i0 + j <= E ? route_off[i0 + j] : 0;
            s += v[j];
        }
        int total;
        int run = carry + block_exclusive_scan<16>(s, wave_tot[k], &total);
#pragma unroll
        for (int j = 0; j < V; ++j) {
            run += v[j];
            if (i0 + j <= E) route_off[i0 + j] = run;
        }
        carry += total;
    }
    if (tid == 0) route_off[0] = 0;
}

__global__ __launch_bounds__(256) void route_fill_kernel(
    int n_req, int L, int G, int n_res, const int32_t* __restrict__ req_res_off,
    const int32_t* __restrict__ req_res, const uint8_t* __restrict__ mask,
    const int32_t* __restrict__ route_off, int32_t* __restrict__ route_res) {
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (long)n_req * L * G) return;
    const int g = (int)(e % G);
    const int l = (int)((e / G) % L);
    const int b = (int)(e / ((long)G * L));
    int w = route_off[e];
#pragma unroll 4
    for (int j = req_res_off[b]; j < req_res_off[b + 1]; ++j) {
        const int r = req_res[j];
        if (r < 0 || r >= n_res) continue;
        if (mask[((size_t)r * L + l) * G + g]) route_res[w++] = r;
    }
}

// One block per layer: exclusive scan over routes i = r * G + g of
// mask[r][l][g] * kept_r, written to the layer's row of the table, plus the
// layer's total.  The routes go through in chunks of 4096 consecutive ones,
// four per thread, with a block-wide scan of the thread sums per chunk and
// the chunk totals carried on.
__global__ __launch_bounds__(1024) void store_offsets_kernel(
    int n_res, int L, int G, const uint8_t* __restrict__ mask,
    const int32_t* __restrict__ cu_kept, int32_t* __restrict__ store_off) {
    constexpr int V = 4;
    __shared__ int wave_tot[2][16];  // alternate buffers: one barrier per chunk suffices
    const int l = blockIdx.x, tid = threadIdx.x;
    const long n = (long)n_res * G;
    int32_t* off = store_off + (size_t)l * (n + 1);
    auto rows = [&](long i) {
        const int r = (int)(i / G), g = (int)(i % G);
        return mask[((size_t)r * L + l) * G + g] ? cu_kept[r + 1] - cu_kept[r] : 0;
    };
    int carry = 0, k = 0;
    for (long base = 0; base < n; base += 1024L * V, k ^= 1) {
        const long i0 = base + (long)tid * V;
        int v[V], s = 0;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            v[j] = i0 + j < n ? rows(i0 + j) : 0;
            s += v[j];
        }
        int total;
        int run = carry + block_exclusive_scan<16>(s, wave_tot[k], &total);
#pragma unroll
        for (int j = 0; j < V; ++j) {
            if (i0 + j < n) off[i0 + j] = run;
            run += v[j];
        }
        carry += total;
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
// whatever routes they belong to, so that every block moves the same bytes in
// one step, all loads in flight at once.  One thread per row finds its source
// row: the wave looks up the route of its first row, the 64 routes after it
// are at hand in the lanes, and only a row past those searches the table.
// Rows past the routes' total (or past the store) are not written.  NT: loads
// and stores that leave no trace in the caches, for a layer larger than these
// hold.  Bound by HBM: one layer of 2,048 resources (1.3 M rows of 256 bytes,
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
    hipLaunchKernelGGL(store_offsets_kernel, dim3(n_layers), dim3(1024), 0, s, n_res, n_layers,
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
    // K and V read and written: above the last-level cache's 256 MB nothing
    // of it would be found there by the next reader; a smaller store is left
    // in reach of the attention that follows
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
                               int n_res, int n_layers, int n_kv_heads, const uint8_t* mask,
                               const int32_t* cu_kept, int32_t* route_off, int32_t* route_res,
                               int32_t* route_tokens, hipStream_t s) {
    const long E = (long)n_req * n_layers * n_kv_heads;
    const unsigned blocks = (unsigned)((E + 255) / 256);
    hipLaunchKernelGGL(route_count_kernel, dim3(blocks), dim3(256), 0, s, n_req, n_layers,
                       n_kv_heads, n_res, req_res_off, req_res, mask, cu_kept, route_off,
                       route_tokens);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(route_scan_kernel, dim3(1), dim3(1024), 0, s, E, route_off);
    err = hipGetLastError();
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(route_fill_kernel, dim3(blocks), dim3(256), 0, s, n_req, n_layers,
                       n_kv_heads, n_res, req_res_off, req_res, mask, route_off, route_res);
    return hipGetLastError();
}

}  // namespace rc
