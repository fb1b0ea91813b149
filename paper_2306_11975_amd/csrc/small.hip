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

// KS steps of 64 positions cover k. DD: double-double sum into C and C_lo. COUNT: counts to g.counts.
template <int S, int KS, bool DD, bool COUNT>
__global__ __launch_bounds__(kSmallThreads) void small_product_kernel(const SmallArgs g) {
    constexpr int OPERAND = S * KS * 2 * kFragBytes;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ unsigned long long maxima[2][1][kSmallGroups][kSmallTile];
    __shared__ int ex[2][1][kSmallTile];
    __shared__ unsigned lost[2][1][2];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles_n = (g.n + kSmallTile - 1) / kSmallTile;
    const int tm = (int)blockIdx.x / tiles_n, tn = (int)blockIdx.x % tiles_n;
    if (COUNT && tid < 4) lost[tid >> 1][0][tid & 1] = 0u;
    SmallElements<KS, 1> el;
    small_split<S, KS, 1>(el, g, tm, tn, lds, maxima, ex);

    if (wave < 4) {   // a 16 x 16 patch to a wavefront
        const int pi = wave >> 1, pj = wave & 1;
        const int row0 = tm * kSmallTile + 16 * pi + 4 * (lane >> 4), col = tn * kSmallTile + 16 * pj + (lane & 15);
        double old_c[4] = {0.0, 0.0, 0.0, 0.0};
        if (g.c_mode != 0 && g.beta != 0.0) {   // requested ahead of the products
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (row0 + u < g.m && col < g.n) old_c[u] = g.C[(int64_t)(row0 + u) * g.ldc + col];
        }
        double sum[4], lo[4];
        small_patch<S, KS, DD>(lds + pi * kFragBytes, lds + OPERAND + pj * kFragBytes, sum, lo);
        const int eb = ex[1][0][16 * pj + (lane & 15)];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = ex[0][0][16 * pi + 4 * (lane >> 4) + u] + eb;
            double val = ldexp(sum[u], e);
            if (DD && row0 + u < g.m && col < g.n) g.C_lo[(int64_t)(row0 + u) * g.ldc + col] = ldexp(lo[u], e);
            if (g.c_mode != 0) {   // RN(alpha G), then RN(RN(alpha G) + RN(beta C)); C is not read if beta == 0
                val = g.alpha * val;
                if (g.beta != 0.0) val = val + g.beta * old_c[u];
            }
            if (row0 + u < g.m && col < g.n) g.C[(int64_t)(row0 + u) * g.ldc + col] = val;
        }
    }
    if constexpr (COUNT) small_count<S, KS, 1>(el, g, tm, tn, ex, lost);
}

template <int S, int KS, bool DD, bool COUNT>
hipError_t launch_small_kernel(const SmallArgs& g, hipStream_t st) {
    constexpr int lds = 2 * S * KS * 2 * kFragBytes;
    hipError_t e = allow_dynamic_lds<&small_product_kernel<S, KS, DD, COUNT>>(lds);
    if (e != hipSuccess) return e;
    small_product_kernel<S, KS, DD, COUNT><<<dim3((unsigned)small_tiles(g.m, g.n)), dim3(kSmallThreads), lds, st>>>(g);
    return hipGetLastError();
}
template <int S, int KS>
hipError_t launch_small_one(const SmallArgs& g, hipStream_t st) {
    if (g.counts) return g.C_lo ? hipErrorInvalidValue : launch_small_kernel<S, KS, false, true>(g, st);
    return g.C_lo ? launch_small_kernel<S, KS, true, false>(g, st) : launch_small_kernel<S, KS, false, false>(g, st);
}
template <int S>
hipError_t launch_small(const SmallArgs& g, hipStream_t st) {
    if (g.k <= kSmallStep) return launch_small_one<S, 1>(g, st);
    if constexpr (S <= kBand) {
        if (g.k > 2 * kSmallStep) return launch_small_one<S, 4>(g, st);
    }
    return launch_small_one<S, 2>(g, st);
}

}  // namespace

// All of k has to fit the LDS (128 KiB: two steps, four up to eight slices). What the tiles repeat makes the rest: a compute unit's time goes with its
// tiles times steps, and four of those are where two launches are as fast (1024 x 1024 x 64 at three, eight and sixteen slices 12.0, 15.1 and 24.3 us, here 9.9, 12.9 and
// 22.4; 2048 x 1024 x 64 at eight 17.8, here 22.1; 512 x 1024 x 128 at eight 15.5, here 10.9, at thirteen 29.6, here 20.5; 512 x 512 x 200 at eight 18.1, here 11.6,
// 512 x 1024 x 256 at five 14.8, here 19.4). The two launches take less where
//  - both operands are read along k (rows: the BLAS-style call of A transposed and B not): at one step three, but for ten to thirteen slices (1024 x 1024 x 64 in a graph at one, six, nine
//    and sixteen 9.0, 12.3, 14.7 and 21.0 us, here 10.5, 13.0, 15.4 and 23.2; at thirteen 22.5, here 19.7);
//  - the product kernel saves half a step of one (k up to 32 with more than nine slices): three for rows along k (1024 x 1024 x 30 at twelve 16.1, here 18.3), and from fourteen slices
//    on one less of either (at fourteen 17.7, here 18.4, 768 x 1024 x 30 17.4, here 14.8; rows along k 768 x 1024 x 30 14.8, here 15.6, 512 x 1024 x 30 14.6, here 11.4).
bool small_product_applies(int64_t m, int64_t n, int64_t k, int s, bool both_by_rows) {
    if (s < 1 || s > OZIMMU_MAX_SLICES || m < 1 || n < 1 || k < 1 || k > (s <= kBand ? 4 : 2) * kSmallStep) return false;
    const int64_t steps = k <= kSmallStep ? 1 : k <= 2 * kSmallStep ? 2 : 4;
    const bool half_step = k <= kSlab && s > 9;
    int64_t per_unit = kSmallTilesPerUnit;
    if (both_by_rows && steps == 1 && (s <= 9 || s >= 14 || half_step)) per_unit -= 1;
    if (half_step && s >= 14) per_unit -= 1;
    return small_tiles(m, n) * steps <= per_unit * kComputeUnits;
}

hipError_t launch_small_product(const SmallArgs& g, int s, hipStream_t st) {
    if (!small_product_applies(g.m, g.n, g.k, s, !g.x[0].by_cols && !g.x[1].by_cols)) return hipErrorInvalidValue;
    switch (s) {
#define OZ_CASE(S_) case S_: return launch_small<S_>(g, st);
        OZ_CASE(1) OZ_CASE(2) OZ_CASE(3) OZ_CASE(4) OZ_CASE(5) OZ_CASE(6) OZ_CASE(7) OZ_CASE(8)
        OZ_CASE(9) OZ_CASE(10) OZ_CASE(11) OZ_CASE(12) OZ_CASE(13) OZ_CASE(14) OZ_CASE(15) OZ_CASE(16)
#undef OZ_CASE
    }
    return hipErrorInvalidValue;
}

}  // namespace ozimmu
