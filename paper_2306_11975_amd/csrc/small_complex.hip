// Small complex products in one launch: as small.hip, with both planes of every element and four real products to a patch. A gate on a
// small register, above all: what such a call takes is launches (gate split, product and the counters' sums were three). Per call: 1024 x 64 x 64 with the
// slice count checked on the way 36.8 -> 28.6 us (most of it the wait for the device), without 12.3 -> 9.8; 256 x 256 x 64 at eight slices 54.8 -> 9.7.
#include "small_common.h"

namespace ozimmu {
namespace {

// KS steps of 64 positions cover k. A workgroup takes 32 x 32 complex elements, four of its wavefronts 16 x 16 each.
template <int S, int KS>
__global__ __launch_bounds__(kSmallThreads) void small_complex_kernel(const SmallArgs g) {
    constexpr bool WIDE = S > 9;
    constexpr int GROUPS = kSmallGroups, W = KS * (kSmallStep / 4) / GROUPS;       // words of four positions to a thread
    constexpr int STEP = 2 * kFragBytes, SLICE = KS * STEP, PLANE = S * SLICE, OPERAND = 2 * PLANE;   // [operand][plane][slice][step][16 rows]
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ unsigned long long maxima[2][2][GROUPS][kSmallTile];
    __shared__ int ex[2][2][kSmallTile];
    __shared__ unsigned count_lds[2][4];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles_n = (g.n + kSmallTile - 1) / kSmallTile;
    const int tm = (int)blockIdx.x / tiles_n, tn = (int)blockIdx.x % tiles_n;

    // ---- both operands, as in small.hip: element l of a vector is (re, im)
    unsigned long long v[2][2][W][4];   // [operand][plane]
    int vec[2], group[2];
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        const SmallOperand& x = g.x[o];
        vec[o] = x.by_cols ? tid & (kSmallTile - 1) : tid / GROUPS;
        group[o] = x.by_cols ? tid / kSmallTile : tid & (GROUPS - 1);
        const int at = (o ? tn : tm) * kSmallTile + vec[o];
        const int64_t first = x.by_cols ? at : (int64_t)at * x.ld, stride = x.by_cols ? x.ld : 1;
        const unsigned long long* src = reinterpret_cast<const unsigned long long*>(x.X) + 2 * first;
        const bool live = at < (o ? g.n : g.m);
#pragma unroll
        for (int i = 0; i < W; ++i)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int l = 4 * (group[o] + GROUPS * i) + u;
                const bool in = live && l < g.k;
#pragma unroll
                for (int pl = 0; pl < 2; ++pl) v[o][pl][i][u] = in ? src[2 * l * stride + pl] : 0ull;
            }
    }
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int pl = 0; pl < 2; ++pl) {
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
    if (tid < 8) count_lds[tid >> 2][tid & 3] = 0u;
    __syncthreads();
#pragma unroll
    for (int o = 0; o < 2; ++o) {
#pragma unroll
        for (int pl = 0; pl < 2; ++pl) {
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
    }
    __syncthreads();

    // ---- 16 x 16 complex elements to a wavefront: G(Ar,Br), G(Ai,Bi), G(Ar,Bi), G(Ai,Br) in turn
    if (wave < 4) {
        const int pi = wave >> 1, pj = wave & 1;
        const int row0 = tm * kSmallTile + 16 * pi + 4 * (lane >> 4), col = tn * kSmallTile + 16 * pj + (lane & 15);
        double re[4], im[4];
        static_for<0, 4>([&](auto ic) __attribute__((always_inline)) {
            constexpr int product = decltype(ic)::value, pa = product & 1, pb = product == 1 || product == 2 ? 1 : 0;
            v4i acc[S];
#pragma unroll
            for (int e = 0; e < S; ++e) acc[e] = v4i{0, 0, 0, 0};
#pragma unroll
            for (int step = 0; step < KS; ++step) {
                v4i a[S], b[S];
#pragma unroll
                for (int p = 0; p < S; ++p) {
                    a[p] = *reinterpret_cast<const v4i*>(lds + pa * PLANE + p * SLICE + step * STEP + pi * kFragBytes + 16 * lane);
                    b[p] = *reinterpret_cast<const v4i*>(lds + OPERAND + pb * PLANE + p * SLICE + step * STEP + pj * kFragBytes + 16 * lane);
                }
#pragma unroll
                for (int q = 0; q < S; ++q)
#pragma unroll
                    for (int p = S - 1 - q; p >= 0; --p) acc[p + q] = mfma16(a[p], b[q], acc[p + q]);
            }
            double sum[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int e = S - 1; e >= 0; --e) {
                const double sc = __longlong_as_double((long long)(1023 - OZIMMU_SLICE_BITS * (e + 2)) << 52);
#pragma unroll
                for (int u = 0; u < 4; ++u) sum[u] = fma((double)acc[e][u], sc, sum[u]);
            }
            const int eb = ex[1][pb][16 * pj + (lane & 15)];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const double val = ldexp(sum[u], ex[0][pa][16 * pi + 4 * (lane >> 4) + u] + eb);
                if constexpr (product == 0) re[u] = val;
                else if constexpr (product == 1) re[u] = re[u] - val;
                else if constexpr (product == 2) im[u] = val;
                else im[u] = im[u] + val;
            }
        });
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (row0 + u < g.m && col < g.n) {
                double* c = g.C + 2 * ((int64_t)(row0 + u) * g.ldc + col);
                c[0] = re[u];
                c[1] = im[u];
            }
    }

    // ---- the check of S as the automatic slice count (the other wavefronts count while those four multiply)
    if (!g.counts) return;
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        if (!(o ? small_counts_columns(tm, tn, g) : small_counts_rows(tm, tn, g))) continue;
        unsigned lost[4];
#pragma unroll
        for (int pl = 0; pl < 2; ++pl) {
            unsigned of_plane[2] = {0u, 0u};
            const int E = ex[o][pl][vec[o]];
#pragma unroll
            for (int i = 0; i < W; ++i) small_count(of_plane, v[o][pl][i], E, S);
            lost[2 * pl] = of_plane[0];
            lost[2 * pl + 1] = of_plane[1];
        }
        small_put_counts(lost, count_lds[o], g.counts + 4 * (o ? (g.m + kSmallTile - 1) / kSmallTile + tn : tm));
    }
}

template <int S, int KS>
hipError_t launch_small_complex_one(const SmallArgs& g, hipStream_t st) {
    constexpr int lds = 4 * S * KS * 2 * kFragBytes;
    hipError_t e = allow_dynamic_lds<&small_complex_kernel<S, KS>>(lds);
    if (e != hipSuccess) return e;
    small_complex_kernel<S, KS><<<dim3((unsigned)small_tiles(g.m, g.n)), dim3(kSmallThreads), lds, st>>>(g);
    return hipGetLastError();
}
template <int S>
hipError_t launch_small_complex_for(const SmallArgs& g, hipStream_t st) {
    if constexpr (S <= kBand) {
        if (g.k > kSmallStep) return launch_small_complex_one<S, 2>(g, st);
    }
    return launch_small_complex_one<S, 1>(g, st);
}

}  // namespace

// All of k has to fit the LDS (128 KiB: one step, two up to eight slices), and a tile a compute unit: a second round takes longer than the other kernels'
// two launches (complex 4096 x 64 x 64 at eight slices, 256 tiles, 12.4 us there, here 10.2; 8192 x 64 x 64 13.6, here 18.9; 2048 x 128 x 128 21.7, here 14.8).
bool small_complex_applies(int64_t m, int64_t n, int64_t k, int s) {
    if (s < 1 || s > OZIMMU_MAX_SLICES || m < 1 || n < 1 || k < 1 || k > (s <= kBand ? 2 : 1) * kSmallStep) return false;
    return small_tiles(m, n) <= kComputeUnits;
}

hipError_t launch_small_complex(const SmallArgs& g, int s, hipStream_t st) {
    if (!small_complex_applies(g.m, g.n, g.k, s)) return hipErrorInvalidValue;
    switch (s) {
#define OZ_CASE(S_) case S_: return launch_small_complex_for<S_>(g, st);
        OZ_CASE(1) OZ_CASE(2) OZ_CASE(3) OZ_CASE(4) OZ_CASE(5) OZ_CASE(6) OZ_CASE(7) OZ_CASE(8)
        OZ_CASE(9) OZ_CASE(10) OZ_CASE(11) OZ_CASE(12) OZ_CASE(13) OZ_CASE(14) OZ_CASE(15) OZ_CASE(16)
#undef OZ_CASE
    }
    return hipErrorInvalidValue;
}

}  // namespace ozimmu
