// Shared by the kernels for small products (small.hip, small_complex.hip): one launch splits both operands and multiplies.
#pragma once

#include "mfma_common.h"
#include "split_common.h"

namespace ozimmu {
namespace {

constexpr int kSmallThreads = 512;
constexpr int kSmallTile = kSmallTileRows;   // rows and columns of C per workgroup
constexpr int kSmallStep = 64;       // positions of k per MFMA
constexpr int kSmallGroups = kSmallThreads / kSmallTile;   // threads that share a vector of an operand

// byte of a fragment that holds (row, position): lane l of the operand takes row l % 16, positions 16 (l / 16) .. + 15
__device__ __forceinline__ int small_offset(int row, int pos) { return ((pos >> 4) * 16 + row) * 16 + (pos & 15); }

inline int64_t small_tiles(int64_t m, int64_t n) { return ((m + kSmallTile - 1) / kSmallTile) * ((n + kSmallTile - 1) / kSmallTile); }

// What a thread holds of a workgroup's tile of each operand, PL planes of each (2: interleaved complex): words group, group + kSmallGroups, ... (of
// four consecutive positions) of vector vec (neighbouring threads take what is contiguous in memory).
template <int KS, int PL>
struct SmallElements {
    static constexpr int W = KS * (kSmallStep / 4) / kSmallGroups;
    unsigned long long v[2][PL][W][4];
    int vec[2], group[2];
};

// Both operands: exponents to ex, slices to lds as operand fragments, [operand][plane][slice][step][fragment of 16 rows], which may be read when it
// returns. KS steps of 64 positions cover k.
template <int S, int KS, int PL>
__device__ __forceinline__ void small_split(SmallElements<KS, PL>& el, const SmallArgs& g, int tm, int tn, unsigned char* lds,
                                            unsigned long long (&maxima)[2][PL][kSmallGroups][kSmallTile], int (&ex)[2][PL][kSmallTile]) {
    constexpr bool WIDE = S > 9;
    constexpr int GROUPS = kSmallGroups, W = SmallElements<KS, PL>::W;
    constexpr int STEP = 2 * kFragBytes, SLICE = KS * STEP, PLANE = S * SLICE, OPERAND = PL * PLANE;
    const int tid = threadIdx.x;
    auto& v = el.v;
    auto& vec = el.vec;
    auto& group = el.group;
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        const SmallOperand& x = g.x[o];
        vec[o] = x.by_cols ? tid & (kSmallTile - 1) : tid / GROUPS;
        group[o] = x.by_cols ? tid / kSmallTile : tid & (GROUPS - 1);
        const int at = (o ? tn : tm) * kSmallTile + vec[o];
        const int64_t first = x.by_cols ? at : (int64_t)at * x.ld, stride = x.by_cols ? x.ld : 1;
        const unsigned long long* src = reinterpret_cast<const unsigned long long*>(x.X) + PL * first;
        const bool live = at < (o ? g.n : g.m);
#pragma unroll
        for (int i = 0; i < W; ++i)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int l = 4 * (group[o] + GROUPS * i) + u;
                const bool in = live && l < g.k;
#pragma unroll
                for (int pl = 0; pl < PL; ++pl) v[o][pl][i][u] = in ? src[PL * l * stride + pl] : 0ull;
            }
    }
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int pl = 0; pl < PL; ++pl) {
            unsigned long long mx = 0;
#pragma unroll
            for (int i = 0; i < W; ++i)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const unsigned long long a = v[o][pl][i][u] & kAbsMask;
                    mx = a > mx ? a : mx;
                }
            maxima[o][pl][group[o]][vec[o]] = mx;
        }
    __syncthreads();
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int pl = 0; pl < PL; ++pl) {
            unsigned long long mx = 0;
#pragma unroll
            for (int i = 0; i < GROUPS; ++i) {
                const unsigned long long a = maxima[o][pl][i][vec[o]];
                mx = a > mx ? a : mx;
            }
            const int E = exponent_of_max(mx);
            if (group[o] == 0) ex[o][pl][vec[o]] = E;
#pragma unroll
            for (int i = 0; i < W; ++i) {
                const int word = group[o] + GROUPS * i;
                unsigned char* dst = lds + o * OPERAND + pl * PLANE + (word >> 4) * STEP + (vec[o] >> 4) * kFragBytes + small_offset(vec[o] & 15, (word & 15) * 4);
                Fixed x[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) x[u] = to_fixed<WIDE>(v[o][pl][i][u], E);
                const SignMask sm = sign_mask(v[o][pl][i][0], v[o][pl][i][1], v[o][pl][i][2], v[o][pl][i][3]);
                static_for<1, S + 1>([&](auto pc) __attribute__((always_inline)) {
                    constexpr int p = decltype(pc)::value;
                    *reinterpret_cast<uint32_t*>(dst + (p - 1) * SLICE) = packed_slice<WIDE>(x, sm, p);
                });
            }
        }
    __syncthreads();
}

// The 16 x 16 patch of a wavefront: one plane of each operand from its fragments (a, b: of its sixteen rows and columns), all diagonals, and their
// FP64 sum without the exponents. DD: double-double.
template <int S, int KS, bool DD>
__device__ __forceinline__ void small_patch(const unsigned char* a_frag, const unsigned char* b_frag, double (&sum)[4], double (&lo)[4]) {
    constexpr int STEP = 2 * kFragBytes, SLICE = KS * STEP;
    const int lane = threadIdx.x & 63;
    v4i acc[S];
#pragma unroll
    for (int e = 0; e < S; ++e) acc[e] = v4i{0, 0, 0, 0};
#pragma unroll
    for (int step = 0; step < KS; ++step) {
        v4i a[S], b[S];
#pragma unroll
        for (int p = 0; p < S; ++p) {
            a[p] = *reinterpret_cast<const v4i*>(a_frag + p * SLICE + step * STEP + 16 * lane);
            b[p] = *reinterpret_cast<const v4i*>(b_frag + p * SLICE + step * STEP + 16 * lane);
        }
#pragma unroll
        for (int q = 0; q < S; ++q)
#pragma unroll
            for (int p = S - 1 - q; p >= 0; --p) acc[p + q] = mfma16(a[p], b[q], acc[p + q]);
    }
    // least significant first (a product with a power of two is exact, so the fused operation rounds like the sum)
#pragma unroll
    for (int u = 0; u < 4; ++u) sum[u] = lo[u] = 0.0;
#pragma unroll
    for (int e = S - 1; e >= 0; --e) {
        const double sc = __longlong_as_double((long long)(1023 - OZIMMU_SLICE_BITS * (e + 2)) << 52);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if constexpr (DD) dd_add(sum[u], lo[u], (double)acc[e][u] * sc);
            else sum[u] = fma((double)acc[e][u], sc, sum[u]);
        }
    }
}

// Which workgroup counts a tile of rows (o = 0), and which a tile of columns: one each, and not the same one where that can be had.
__device__ __forceinline__ bool small_counts(int o, int tm, int tn, const SmallArgs& g) {
    const int tiles_n = (g.n + kSmallTile - 1) / kSmallTile;
    if (o == 0) return tn == tm % tiles_n;
    const int last = (g.m + kSmallTile - 1) / kSmallTile - 1, next = (tn + 1) % tiles_n;
    return tm == (next < last ? next : last);
}
// The bits that the elements of this workgroup's vectors lose with S and with S - 1 slices (Section 4.4), the check of S as the automatic slice count,
// to g.counts where the workgroup has them to count. lost: [operand][plane][2] zeroed words. A tile counts at most 32 x 256 elements of fewer than 166 bits.
// Every thread calls it (the wavefronts that do not multiply count while the others do).
template <int S, int KS, int PL>
__device__ __forceinline__ void small_count(const SmallElements<KS, PL>& el, const SmallArgs& g, int tm, int tn, const int (&ex)[2][PL][kSmallTile],
                                            unsigned (&lost)[2][PL][2]) {
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        if (!small_counts(o, tm, tn, g)) continue;
        unsigned c[PL][2] = {};
#pragma unroll
        for (int pl = 0; pl < PL; ++pl) {
            const int E = ex[o][pl][el.vec[o]];
#pragma unroll
            for (int i = 0; i < SmallElements<KS, PL>::W; ++i)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    uint32_t z, L;
                    loss_position(el.v[o][pl][i][u], E, z, L);
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const int edge = OZIMMU_SLICE_BITS * (S - j), below = (int)(z + L) - edge, above = (int)z - edge;
                        c[pl][j] += (unsigned)((below > 0 ? below : 0) - (above > 0 ? above : 0));
                    }
                }
        }
#pragma unroll
        for (int pl = 0; pl < PL; ++pl)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                unsigned x = c[pl][j];
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
                if ((threadIdx.x & 63) == 0 && x) atomicAdd(&lost[o][pl][j], x);
            }
        __syncthreads();
        unsigned* out = g.counts + 2 * PL * (o ? (g.m + kSmallTile - 1) / kSmallTile + tn : tm);
        if (threadIdx.x < 2 * PL) out[threadIdx.x] = (&lost[o][0][0])[threadIdx.x];
    }
}

}  // namespace
}  // namespace ozimmu
