// Small complex products in one launch: as small.hip, with both planes of every element and four real products to a patch. A gate on a
// small register, above all: what such a call takes is launches (gate split, product and the counters' sums were three). Per call: 1024 x 64 x 64 with the
// slice count checked on the way 36.8 -> 28.6 us (most of it the wait for the device), without 12.3 -> 9.8; 256 x 256 x 64 at eight slices 54.8 -> 9.7; 2048 x 128 x 128 at eight 21.7 -> 15.5.
#include "small_common.h"

namespace ozimmu {
namespace {

// KS steps of 64 positions cover k. A workgroup takes 32 x 32 complex elements, four of its wavefronts 16 x 16 each. COUNT: counts to g.counts.
template <int S, int KS, bool COUNT>
__global__ __launch_bounds__(kSmallThreads) void small_complex_kernel(const SmallArgs g) {
    constexpr int PLANE = S * KS * 2 * kFragBytes, OPERAND = 2 * PLANE;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ unsigned long long maxima[2][2][kSmallGroups][kSmallTile];
    __shared__ int ex[2][2][kSmallTile];
    __shared__ unsigned lost[2][2][2];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles_n = (g.n + kSmallTile - 1) / kSmallTile;
    const int tm = (int)blockIdx.x / tiles_n, tn = (int)blockIdx.x % tiles_n;
    if (COUNT && tid < 8) lost[tid >> 2][(tid >> 1) & 1][tid & 1] = 0u;
    SmallElements<KS, 2> el;
    small_split<S, KS, 2>(el, g, tm, tn, lds, maxima, ex);

    if (wave < 4) {   // 16 x 16 complex elements to a wavefront: G(Ar,Br), G(Ai,Bi), G(Ar,Bi), G(Ai,Br) in turn
        const int pi = wave >> 1, pj = wave & 1;
        const int row0 = tm * kSmallTile + 16 * pi + 4 * (lane >> 4), col = tn * kSmallTile + 16 * pj + (lane & 15);
        double re[4], im[4];
        static_for<0, 4>([&](auto ic) __attribute__((always_inline)) {
            constexpr int product = decltype(ic)::value, pa = product & 1, pb = product == 1 || product == 2 ? 1 : 0;
            double sum[4], lo[4];
            small_patch<S, KS, false>(lds + pa * PLANE + pi * kFragBytes, lds + OPERAND + pb * PLANE + pj * kFragBytes, sum, lo);
            // The sums are formed here: put off to the stores behind the other products (the compiler's choice where nothing else needs them), they
            // would keep every product's diagonals, more than the registers hold: 156 spilled at sixteen slices, 1024 x 64 x 64 28.0 us per call, now 15.4 (with two launches 21.3).
            // Where they do fit, the compiler's choice is the faster one (300 x 200 x 40 at five slices 8.45 us, formed here 8.71; 338 x 183 x 95 at six 12.4, 12.8).
            if constexpr (KS == 1 ? S >= 6 : S >= (COUNT ? 5 : 7)) {
#pragma unroll
                for (int u = 0; u < 4; ++u) asm volatile("" : "+v"(sum[u])::"memory");
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
    if constexpr (COUNT) small_count<S, KS, 2>(el, g, tm, tn, ex, lost);
}

template <int S, int KS, bool COUNT>
hipError_t launch_small_complex_kernel(const SmallArgs& g, hipStream_t st) {
    constexpr int lds = 4 * S * KS * 2 * kFragBytes;
    hipError_t e = allow_dynamic_lds<&small_complex_kernel<S, KS, COUNT>>(lds);
    if (e != hipSuccess) return e;
    small_complex_kernel<S, KS, COUNT><<<dim3((unsigned)small_tiles(g.m, g.n)), dim3(kSmallThreads), lds, st>>>(g);
    return hipGetLastError();
}
template <int S, int KS>
hipError_t launch_small_complex_one(const SmallArgs& g, hipStream_t st) {
    return g.counts ? launch_small_complex_kernel<S, KS, true>(g, st) : launch_small_complex_kernel<S, KS, false>(g, st);
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
// two launches (complex 4096 x 64 x 64 at eight slices, 256 tiles, 12.4 us there, here 10.2; 8192 x 64 x 64 13.6, here 18.9).
bool small_complex_applies(int64_t m, int64_t n, int64_t k, int s) {
    if (s < 1 || s > OZIMMU_MAX_SLICES || m < 1 || n < 1 || k < 1 || k > (s <= kBand ? 2 : 1) * kSmallStep) return false;
    static_assert(kComputeUnits <= kSmallMaxTiles, "the room for the counters");
    return small_tiles(m, n) <= kComputeUnits;
}

// A gate of up to sixteen columns leaves half of a tile and more empty, and its MFMAs are what many slices take: there the gate kernel's two launches are
// as fast at eleven slices and ahead beyond (per call, 8192 x 2 x 2 at eleven, thirteen and sixteen 11.5, 12.2, 13.5 us, here 11.3, 12.8, 14.9; 2000 x 16 x 16
// at sixteen 13.6, here 14.7; 20 columns 14.6, here 14.7; counting, where that kernel takes a third launch, this one stays ahead).
bool small_complex_ahead(const double* Z, const double* B, const double* Cz, int64_t m, int64_t n, int64_t k, int s) {
    return small_complex_applies(m, n, k, s) && !(n <= 16 && s > 11 && gate_product_applies(Z, B, Cz, n, k, s));
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
