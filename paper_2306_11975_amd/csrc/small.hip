// Small real products in one launch: split, slice products and FP64 sum (the whole algorithm of Section 3.1).
//
// A product of a few tiles with a short inner dimension is two launches on the general path, each of 5 to 6 us of which its work is
// the smaller part. Here a workgroup takes a 32 x 32 tile of C: it splits the tile's rows of A and columns of B for itself, all of
// k at once, straight into LDS as operand fragments of v_mfma_i32_16x16x64_i8 (16 rows x 64 positions), and four of its eight wavefronts
// multiply a 16 x 16 patch each, all diagonals resident. What bounds it is latency (a launch, a trip to memory, three barriers), and
// the splitting that the tiles of a row or column repeat: so few tiles and a short k only (small_product_applies). Per call, two launches
// -> one (about 9 us is what the host takes for one): 64^3 at five slices 12.0 -> 9.0 us, at thirteen 22.2 -> 9.0; 512 x 512 x 128 at eight 15.1 -> 9.3.
#include "small_common.h"

namespace ozimmu {
namespace {

// KS steps of 64 positions cover k. DD: double-double sum into C and C_lo.
template <int S, int KS, bool DD>
__global__ __launch_bounds__(kSmallThreads) void small_product_kernel(const SmallArgs g) {
    constexpr bool WIDE = S > 9;
    constexpr int GROUPS = kSmallGroups;
    constexpr int W = KS * (kSmallStep / 4) / GROUPS;                // words of four consecutive positions to a thread
    constexpr int STEP = 2 * kFragBytes, SLICE = KS * STEP, OPERAND = S * SLICE;   // [operand][slice][step][fragment of 16 rows]
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ unsigned long long maxima[2][GROUPS][kSmallTile];
    __shared__ int ex[2][kSmallTile];
    __shared__ unsigned count_lds[2][2];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles_n = (g.n + kSmallTile - 1) / kSmallTile;
    const int tm = (int)blockIdx.x / tiles_n, tn = (int)blockIdx.x % tiles_n;

    // ---- both operands: vector `vec` of the tile, words group, group + GROUPS, ... (neighbouring threads take what is contiguous in memory)
    unsigned long long v[2][W][4];
    int vec[2], group[2];
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        const SmallOperand& x = g.x[o];
        vec[o] = x.by_cols ? tid & (kSmallTile - 1) : tid / GROUPS;
        group[o] = x.by_cols ? tid / kSmallTile : tid & (GROUPS - 1);
        const int at = (o ? tn : tm) * kSmallTile + vec[o];
        const int64_t first = x.by_cols ? at : (int64_t)at * x.ld, stride = x.by_cols ? x.ld : 1;
        const unsigned long long* src = reinterpret_cast<const unsigned long long*>(x.X) + first;
        const bool live = at < (o ? g.n : g.m);
#pragma unroll
        for (int i = 0; i < W; ++i)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int l = 4 * (group[o] + GROUPS * i) + u;
                v[o][i][u] = live && l < g.k ? src[l * stride] : 0ull;
            }
    }
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        unsigned long long mx = 0;
#pragma unroll
        for (int i = 0; i < W; ++i)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const unsigned long long a = v[o][i][u] & kAbsMask;
                mx = a > mx ? a : mx;
            }
        maxima[o][group[o]][vec[o]] = mx;
    }
    if (tid < 4) count_lds[tid >> 1][tid & 1] = 0u;
    __syncthreads();
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        unsigned long long mx = 0;
#pragma unroll
        for (int i = 0; i < GROUPS; ++i) {
            const unsigned long long a = maxima[o][i][vec[o]];
            mx = a > mx ? a : mx;
        }
        const int E = exponent_of_max(mx);
        if (group[o] == 0) ex[o][vec[o]] = E;
#pragma unroll
        for (int i = 0; i < W; ++i) {
            const int word = group[o] + GROUPS * i;
            unsigned char* dst = lds + o * OPERAND + (word >> 4) * STEP + (vec[o] >> 4) * kFragBytes + small_offset(vec[o] & 15, (word & 15) * 4);
            Fixed x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = to_fixed<WIDE>(v[o][i][u], E);
            const SignMask sm = sign_mask(v[o][i][0], v[o][i][1], v[o][i][2], v[o][i][3]);
            static_for<1, S + 1>([&](auto pc) __attribute__((always_inline)) {
                constexpr int p = decltype(pc)::value;
                *reinterpret_cast<uint32_t*>(dst + (p - 1) * SLICE) = packed_slice<WIDE>(x, sm, p);
            });
        }
    }
    __syncthreads();

    // ---- a 16 x 16 patch to a wavefront
    if (wave < 4) {
        const int pi = wave >> 1, pj = wave & 1;
        const int row0 = tm * kSmallTile + 16 * pi + 4 * (lane >> 4), col = tn * kSmallTile + 16 * pj + (lane & 15);
        double old_c[4] = {0.0, 0.0, 0.0, 0.0};
        if (g.c_mode != 0 && g.beta != 0.0) {   // requested ahead of the products
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (row0 + u < g.m && col < g.n) old_c[u] = g.C[(int64_t)(row0 + u) * g.ldc + col];
        }
        v4i acc[S];
#pragma unroll
        for (int e = 0; e < S; ++e) acc[e] = v4i{0, 0, 0, 0};
#pragma unroll
        for (int step = 0; step < KS; ++step) {
            v4i a[S], b[S];
#pragma unroll
            for (int p = 0; p < S; ++p) {
                a[p] = *reinterpret_cast<const v4i*>(lds + p * SLICE + step * STEP + pi * kFragBytes + 16 * lane);
                b[p] = *reinterpret_cast<const v4i*>(lds + OPERAND + p * SLICE + step * STEP + pj * kFragBytes + 16 * lane);
            }
#pragma unroll
            for (int q = 0; q < S; ++q)
#pragma unroll
                for (int p = S - 1 - q; p >= 0; --p) acc[p + q] = mfma16(a[p], b[q], acc[p + q]);
        }
        // the diagonals, least significant first (a product with a power of two is exact, so the fused operation rounds like the sum), ...
        double sum[4] = {0.0, 0.0, 0.0, 0.0}, lo[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = S - 1; e >= 0; --e) {
            const double sc = __longlong_as_double((long long)(1023 - OZIMMU_SLICE_BITS * (e + 2)) << 52);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if constexpr (DD) dd_add(sum[u], lo[u], (double)acc[e][u] * sc);
                else sum[u] = fma((double)acc[e][u], sc, sum[u]);
            }
        }
        // ... scaled, combined and stored
        const int eb = ex[1][16 * pj + (lane & 15)];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = ex[0][16 * pi + 4 * (lane >> 4) + u] + eb;
            double val = ldexp(sum[u], e);
            if (DD && row0 + u < g.m && col < g.n) g.C_lo[(int64_t)(row0 + u) * g.ldc + col] = ldexp(lo[u], e);
            if (g.c_mode != 0) {   // RN(alpha G), then RN(RN(alpha G) + RN(beta C)); C is not read if beta == 0
                val = g.alpha * val;
                if (g.beta != 0.0) val = val + g.beta * old_c[u];
            }
            if (row0 + u < g.m && col < g.n) g.C[(int64_t)(row0 + u) * g.ldc + col] = val;
        }
    }

    // ---- the check of S as the automatic slice count (the other wavefronts count while those four multiply)
    if (!g.counts) return;
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        if (!(o ? small_counts_columns(tm, tn, g) : small_counts_rows(tm, tn, g))) continue;
        unsigned lost[2] = {0u, 0u};
        const int E = ex[o][vec[o]];
#pragma unroll
        for (int i = 0; i < W; ++i) small_count(lost, v[o][i], E, S);
        small_put_counts(lost, count_lds[o], g.counts + 2 * (o ? (g.m + kSmallTile - 1) / kSmallTile + tn : tm));
    }
}

template <int S, int KS, bool DD>
hipError_t launch_small_one(const SmallArgs& g, hipStream_t st) {
    constexpr int lds = 2 * S * KS * 2 * kFragBytes;
    hipError_t e = allow_dynamic_lds<&small_product_kernel<S, KS, DD>>(lds);
    if (e != hipSuccess) return e;
    small_product_kernel<S, KS, DD><<<dim3((unsigned)small_tiles(g.m, g.n)), dim3(kSmallThreads), lds, st>>>(g);
    return hipGetLastError();
}
template <int S, bool DD>
hipError_t launch_small(const SmallArgs& g, hipStream_t st) {
    if (g.k <= kSmallStep) return launch_small_one<S, 1, DD>(g, st);
    if constexpr (S <= kBand) {
        if (g.k > 2 * kSmallStep) return launch_small_one<S, 4, DD>(g, st);
    }
    return launch_small_one<S, 2, DD>(g, st);
}

}  // namespace

// All of k has to fit the LDS (128 KiB: two steps, four up to eight slices). What the tiles repeat makes the rest: a compute unit's time goes with its
// tiles times steps, and four of those are where two launches are as fast (1024 x 1024 x 64 at three, eight and sixteen slices 11.5, 14.8 and 23.0 us, here 9.9, 13.1 and
// 22.7; 2048 x 1024 x 64 at eight 17.8, here 22.1; 512 x 1024 x 128 at eight 15.3, here 10.9; 512 x 512 x 200 at eight 18.1, here 11.6, 512 x 1024 x 256 at five 14.8, here 19.4).
bool small_product_applies(int64_t m, int64_t n, int64_t k, int s) {
    if (s < 1 || s > OZIMMU_MAX_SLICES || m < 1 || n < 1 || k < 1 || k > (s <= kBand ? 4 : 2) * kSmallStep) return false;
    const int64_t steps = k <= kSmallStep ? 1 : k <= 2 * kSmallStep ? 2 : 4;
    return small_tiles(m, n) * steps <= 4 * kComputeUnits;
}

hipError_t launch_small_product(const SmallArgs& g, int s, hipStream_t st) {
    if (!small_product_applies(g.m, g.n, g.k, s)) return hipErrorInvalidValue;
    switch (s) {
#define OZ_CASE(S_) case S_: return g.C_lo ? launch_small<S_, true>(g, st) : launch_small<S_, false>(g, st);
        OZ_CASE(1) OZ_CASE(2) OZ_CASE(3) OZ_CASE(4) OZ_CASE(5) OZ_CASE(6) OZ_CASE(7) OZ_CASE(8)
        OZ_CASE(9) OZ_CASE(10) OZ_CASE(11) OZ_CASE(12) OZ_CASE(13) OZ_CASE(14) OZ_CASE(15) OZ_CASE(16)
#undef OZ_CASE
    }
    return hipErrorInvalidValue;
}

}  // namespace ozimmu
