// Helpers shared by the bf16 MFMA attention kernels of encode and prefill:
// LDS tile swizzle, buffer resources, NaN rows for calls whose sizes
// understate their inputs.
#pragma once

#include "common.hpp"
#include "kernels.hpp"

namespace rc {

namespace {

// A lane's sum of a tile's weights above this moves the reference max.
constexpr float kWeightCap = 65536.0f;  // 2^16
constexpr int kMaxSeg = 1024;
// Stands for "no visible key" as a reference max where a wave may hold columns
// that see none of its keys: finite, so that masked logits still weigh
// exp2(-inf) = 0 against it.
constexpr float kNoKey = -1e30f;
// Third dword of a gfx9 buffer resource for raw (unformatted) loads.
constexpr int kBufferFlags = 0x00020000;

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// XOR mask of a row's chunk index: for 256-byte rows the two 2-bit halves of
// row % 16 are swapped, which keeps the 16 rows of an A-operand read on 16
// distinct chunks and puts the four rows of one transpose-read lane group on
// four distinct 4-chunk groups (both bank-conflict free, as measured with the
// LDS conflict counter).
template <int CPR>
__device__ __forceinline__ int chunk_mask(int row) {
    return CPR == 16 ? (((row & 3) << 2) | ((row >> 2) & 3)) : (row % CPR);
}

template <int HD>
__device__ __forceinline__ uint32_t swz(int row, int chunk) {
    constexpr int CPR = HD / 8;
    return (uint32_t)(row * HD * 2 + ((chunk ^ chunk_mask<CPR>(row)) << 4));
}

// Rows a block is responsible for but cannot compute (its route list is
// longer than the segment table, or they lie past the query rows the grid
// was sized for): NaN in out and lse, so that a caller's size error shows in
// the outputs instead of leaving rows unwritten or dropping resources.
// Rows [r_begin, r_end) of the unit whose rows start at q_row0, heads
// [head0, head0 + n_heads), by n threads of which this is number i0.
template <int HD>
__device__ __forceinline__ void poison_rows(const AttnArgs& a, int head0, int n_heads, int q_row0,
                                            int r_begin, int r_end, int i0, int n_threads) {
    constexpr int CPR = HD / 8;
    const u32x4 nan8 = {0x7FC07FC0u, 0x7FC07FC0u, 0x7FC07FC0u, 0x7FC07FC0u};  // bf16 NaNs
    const long n = (long)max(r_end - r_begin, 0) * n_heads * CPR;
    for (long i = i0; i < n; i += n_threads) {
        const int c = (int)(i % CPR);
        const long rest = i / CPR;
        const int h = head0 + (int)(rest % n_heads);
        const long row = (long)q_row0 + r_begin + rest / n_heads;
        if (row < 0 || row >= a.lse_rows) continue;
        *reinterpret_cast<u32x4*>(a.out + ((size_t)row * a.n_q_heads + h) * HD + c * 8) = nan8;
        if (c == 0 && a.lse) a.lse[(size_t)h * a.lse_rows + row] = __builtin_nanf("");
    }
}

}  // namespace

}  // namespace rc
