// Shared by the kernels for small products (small.hip, small_complex.hip): one launch splits both operands and multiplies.
#pragma once

#include "mfma_common.h"
#include "split_common.h"

namespace ozimmu {
namespace {

constexpr int kSmallThreads = 512;
constexpr int kSmallTile = 32;       // rows and columns of C per workgroup
constexpr int kSmallStep = 64;       // positions of k per MFMA
constexpr int kSmallGroups = kSmallThreads / kSmallTile;   // threads that share a vector of an operand

// byte of a fragment that holds (row, position): lane l of the operand takes row l % 16, positions 16 (l / 16) .. + 15
__device__ __forceinline__ int small_offset(int row, int pos) { return ((pos >> 4) * 16 + row) * 16 + (pos & 15); }

inline int64_t small_tiles(int64_t m, int64_t n) { return ((m + kSmallTile - 1) / kSmallTile) * ((n + kSmallTile - 1) / kSmallTile); }

// The bits that the thread's elements of a word lose with s and with s - 1 slices, added to lost[0] and lost[1] (Section 4.4).
__device__ __forceinline__ void small_count(unsigned (&lost)[2], const unsigned long long (&word)[4], int E, int s) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        uint32_t z, L;
        loss_position(word[u], E, z, L);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int edge = OZIMMU_SLICE_BITS * (s - i), below = (int)(z + L) - edge, above = (int)z - edge;
            lost[i] += (unsigned)((below > 0 ? below : 0) - (above > 0 ? above : 0));
        }
    }
}
// Which workgroup counts a tile of rows, and which a tile of columns: one each, and not the same one where that can be had.
__device__ __forceinline__ bool small_counts_rows(int tm, int tn, const SmallArgs& g) {
    return tn == tm % ((g.n + kSmallTile - 1) / kSmallTile);
}
__device__ __forceinline__ bool small_counts_columns(int tm, int tn, const SmallArgs& g) {
    const int last = (g.m + kSmallTile - 1) / kSmallTile - 1, next = (tn + 1) % ((g.n + kSmallTile - 1) / kSmallTile);
    return tm == (next < last ? next : last);
}
// The counts of a workgroup's vectors of one operand (N per thread) to N words of `out`; lds: N zeroed words. A tile counts at most
// 32 x 256 elements of fewer than 166 bits. Every thread calls this.
template <int N>
__device__ __forceinline__ void small_put_counts(const unsigned (&lost)[N], unsigned* lds, unsigned* out) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
        unsigned c = lost[i];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off, 64);
        if ((threadIdx.x & 63) == 0 && c) atomicAdd(&lds[i], c);
    }
    __syncthreads();
    if (threadIdx.x < N) out[threadIdx.x] = lds[threadIdx.x];
}

}  // namespace
}  // namespace ozimmu
