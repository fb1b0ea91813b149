// The gate's split, the counters' sums and the dispatch of the kernel in gate_kernel.h (a gate on a state vector, Section 4.4); more than eight
// slices are compiled in a translation unit of their own (gate_many.hip), so that they build in parallel.
#include "gate_kernel.h"

namespace ozimmu {

hipError_t launch_gate_many(const GateArgs& g, int cls, int s, hipStream_t st);

namespace {

// bits an element at (z, L) loses with s slices
__device__ __forceinline__ unsigned lost_bits(uint32_t z, uint32_t L, int s) {
    const int edge = OZIMMU_SLICE_BITS * s, below = (int)(z + L) - edge, above = (int)z - edge;
    return (unsigned)((below > 0 ? below : 0) - (above > 0 ? above : 0));
}

// ---------------------------------------------------------------------------- the gate -> T1, T2, exponents
// One workgroup per fragment f (8 columns of B). Thread (c, w) = (tid % 8, tid / 8) owns column 8 f + c and the four
// positions 4 w .. 4 w + 3 of k. T: tensor t at t * s * nfr * ks KiB, slice q at q * nfr * ks KiB, fragment (f, step)
// at (f ks + step) KiB. E: [t][f][16] exponents of the fragments' rows.
template <bool WIDE>   // more than nine slices: the fraction takes both words of the fixed-point value
__global__ __launch_bounds__(512) void gate_split_kernel(const double* __restrict__ B, int64_t ldb, int k, int n, int s,
                                                         int ks, int nfr, int8_t* __restrict__ T, int32_t* __restrict__ E,
                                                         unsigned* __restrict__ scan) {
    const int tid = threadIdx.x, r8 = tid & 7, w = tid >> 3, f = blockIdx.x, c = f * 8 + r8;
    const ulonglong2* src = reinterpret_cast<const ulonglong2*>(B);
    ulonglong2 v[4];
    unsigned long long mx_re = 0, mx_im = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int l = 4 * w + u;
        v[u] = ulonglong2{0ull, 0ull};
        if (l < k && c < n) v[u] = src[(int64_t)l * ldb + c];
        const unsigned long long a = v[u].x & kAbsMask, b = v[u].y & kAbsMask;
        mx_re = a > mx_re ? a : mx_re;
        mx_im = b > mx_im ? b : mx_im;
    }
    __shared__ unsigned long long colmax[64][8][2];
    __shared__ unsigned lost_lds[4];
    if (scan && tid < 4) lost_lds[tid] = 0u;
    const int words = blockDim.x >> 3;   // 32 (k <= 128) or 64
    colmax[w][r8][0] = mx_re;
    colmax[w][r8][1] = mx_im;
    __syncthreads();
    for (int i = 0; i < words; ++i) {
        mx_re = colmax[i][r8][0] > mx_re ? colmax[i][r8][0] : mx_re;
        mx_im = colmax[i][r8][1] > mx_im ? colmax[i][r8][1] : mx_im;
    }
    const int e_re = exponent_of_max(mx_re), e_im = exponent_of_max(mx_im);
    if (w == 0) {
        E[f * 16 + r8] = e_re;
        E[f * 16 + 8 + r8] = e_im;
        E[nfr * 16 + f * 16 + r8] = e_im;
        E[nfr * 16 + f * 16 + 8 + r8] = e_re;
    }
    if (scan) {
        // the bits the fragment's columns lose with s and with s - 1 slices (Section 4.4): [re s, re s - 1, im s, im s - 1][nfr]
        unsigned lost[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            uint32_t z, L;
            loss_position(v[u].x, e_re, z, L);
            lost[0] += lost_bits(z, L, s);
            lost[1] += lost_bits(z, L, s - 1);
            loss_position(v[u].y, e_im, z, L);
            lost[2] += lost_bits(z, L, s);
            lost[3] += lost_bits(z, L, s - 1);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) lost[i] += __shfl_xor(lost[i], off, 64);
            if ((tid & 63) == 0 && lost[i]) atomicAdd(&lost_lds[i], lost[i]);
        }
        __syncthreads();
        if (tid < 4) scan[tid * nfr + f] = lost_lds[tid];
    }
    if (4 * w >= kGateStep * ks) return;
    const int64_t slice = (int64_t)nfr * ks * kFragBytes, tensor = (int64_t)s * slice;
    Fixed xr[4], xi[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        xr[u] = to_fixed<WIDE>(v[u].x, e_re);
        xi[u] = to_fixed<WIDE>(v[u].y, e_im);
    }
    const SignMask sr = sign_mask(v[0].x, v[1].x, v[2].x, v[3].x);
    const SignMask si = sign_mask(v[0].y, v[1].y, v[2].y, v[3].y);
    const int l0 = 4 * w, step = l0 / kGateStep, ll = l0 % kGateStep;
    const int64_t lo = (int64_t)(f * ks + step) * kFragBytes + frag_offset(r8, ll);       // first plane of the fragment
    const int64_t hi = (int64_t)(f * ks + step) * kFragBytes + frag_offset(8 + r8, ll);   // second plane
#pragma unroll
    for (int p = 1; p <= (WIDE ? OZIMMU_MAX_SLICES : 9); ++p) {
        if (p <= s) {
            const uint32_t pr = packed_slice<WIDE>(xr, sr, p), pi = packed_slice<WIDE>(xi, si, p);
            int8_t* d = T + (p - 1) * slice;
            *reinterpret_cast<uint32_t*>(d + lo) = pr;
            *reinterpret_cast<uint32_t*>(d + hi) = pi;
            *reinterpret_cast<uint32_t*>(d + tensor + lo) = pi;
            *reinterpret_cast<uint32_t*>(d + tensor + hi) = pr;
        }
    }
}

// The counters of all tiles ([counter][tile]) and of the gate's fragments (behind them, [4][nfr]) -> the bits the two
// planes of Z (planes 0, 1) and of B (planes 2, 3) lose with s and with s - 1 slices: out[plane * 16 + s - 1] and
// out[plane * 16 + s - 2], the layout of the slice-count sums. `out` may be mapped host memory. One workgroup.
// U: tiles to a thread at a time.
template <int U>
__global__ __launch_bounds__(1024) void gate_scan_reduce_kernel(const unsigned* __restrict__ partials, int64_t tiles, int nfr,
                                                                int s, unsigned long long* __restrict__ out) {
    __shared__ unsigned long long sums[2 * kScanCounters + 4];
    if (threadIdx.x < 2 * kScanCounters + 4) sums[threadIdx.x] = 0ull;
    __syncthreads();
    // ten U loads in flight per thread (the words come from beyond the L2, written by other XCDs); a tile index past
    // the end reads the last tile and adds nothing
    unsigned long long mine[2 * kScanCounters] = {};
    for (int64_t base = threadIdx.x; base < tiles; base += 1024 * U) {
        unsigned v[U][2 * kScanCounters];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t t = base + 1024 * u, tc = t < tiles ? t : tiles - 1;
#pragma unroll
            for (int i = 0; i < 2 * kScanCounters; ++i) v[u][i] = partials[i * tiles + tc];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = base + 1024 * u < tiles;
#pragma unroll
            for (int i = 0; i < 2 * kScanCounters; ++i) mine[i] += in ? v[u][i] : 0u;
        }
    }
#pragma unroll
    for (int i = 0; i < 2 * kScanCounters; ++i) {
        const unsigned long long v = wave_sum(mine[i]);
        if ((threadIdx.x & 63) == 0 && v) atomicAdd(&sums[i], v);
    }
    const unsigned* of_gate = partials + 2 * kScanCounters * tiles;
    if ((int)threadIdx.x < 4 * nfr) atomicAdd(&sums[2 * kScanCounters + threadIdx.x / nfr], (unsigned long long)of_gate[threadIdx.x]);
    __syncthreads();
    if (threadIdx.x < 2) {
        const unsigned long long* c = sums + threadIdx.x * kScanCounters;
        out[threadIdx.x * OZIMMU_MAX_SLICES + s - 1] = (c[0] - c[1] + c[4]) >> 1;
        if (s > 1) out[threadIdx.x * OZIMMU_MAX_SLICES + s - 2] = (c[2] - c[3] + c[4]) >> 1;
    } else if (threadIdx.x < 4) {
        const unsigned long long* c = sums + 2 * kScanCounters + 2 * (threadIdx.x - 2);
        out[threadIdx.x * OZIMMU_MAX_SLICES + s - 1] = c[0];
        if (s > 1) out[threadIdx.x * OZIMMU_MAX_SLICES + s - 2] = c[1];
    }
}

inline int gate_class(int64_t k, int64_t n) { return k > 128 || n > 128 ? 2 : k > 64 || n > 64 ? 1 : 0; }
inline int64_t gate_limit(int s) { return s <= kBand ? kGateMaxFew : kGateMax; }

}  // namespace

bool gate_product_applies(const double* Z, const double* B, const double* Cz, int64_t n, int64_t k, int s) {
    return s >= 1 && s <= OZIMMU_MAX_SLICES && n >= 1 && n <= gate_limit(s) && k >= 1 && k <= gate_limit(s) &&
           reinterpret_cast<uintptr_t>(Z) % 16 == 0 && reinterpret_cast<uintptr_t>(B) % 16 == 0 && reinterpret_cast<uintptr_t>(Cz) % 16 == 0;
}

size_t gate_scratch_bytes(int64_t n, int64_t k, int s) {
    if (s < 1 || s > OZIMMU_MAX_SLICES || n < 1 || n > gate_limit(s) || k < 1 || k > gate_limit(s)) return 0;
    const size_t nfr = (size_t)8 << gate_class(k, n), ks = (size_t)1 << gate_class(k, n);
    return 2 * nfr * 16 * sizeof(int32_t) + (size_t)2 * s * nfr * ks * kFragBytes;
}

size_t gate_scan_bytes(int64_t m) {
    return ((size_t)((m + kGateRows - 1) / kGateRows) * 2 * kScanCounters + 4 * (8 << 2)) * sizeof(unsigned);
}

hipError_t launch_gate_product(const double* Z, int64_t ldz, int64_t m, int64_t k, int64_t n, const double* B, int64_t ldb,
                               int s, void* scratch, double* Cz, int64_t ldcz, hipStream_t st, unsigned* scan_partials,
                               unsigned long long* scan_sums) {
    if (m <= 0) return hipSuccess;
    if (!gate_product_applies(Z, B, Cz, n, k, s)) return hipErrorInvalidValue;
    const int cls = gate_class(k, n), ks = 1 << cls, nfr = 8 << cls;
    int32_t* E = static_cast<int32_t*>(scratch);
    int8_t* T = reinterpret_cast<int8_t*>(E + 2 * nfr * 16);
    const unsigned split_threads = cls == 2 ? 512 : 256;   // a thread per word of four positions and column of the fragment
    const int64_t tiles = (m + kGateRows - 1) / kGateRows;
    unsigned* scan_gate = scan_partials ? scan_partials + 2 * kScanCounters * tiles : nullptr;
    if (s > 9) gate_split_kernel<true><<<dim3(nfr), dim3(split_threads), 0, st>>>(B, ldb, (int)k, (int)n, s, ks, nfr, T, E, scan_gate);
    else gate_split_kernel<false><<<dim3(nfr), dim3(split_threads), 0, st>>>(B, ldb, (int)k, (int)n, s, ks, nfr, T, E, scan_gate);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    GateArgs g{};
    g.Z = Z;
    g.ldz = ldz;
    g.m = m;
    g.k = (int)k;
    g.n = (int)n;
    g.T = T;
    g.E = E;
    g.Cz = Cz;
    g.ldcz = ldcz;
    g.scan = scan_partials;
    e = hipErrorInvalidValue;
    switch (s) {
#define OZ_CASE(S_) case S_: e = cls == 2 ? launch_gate<S_, 2>(g, st) : cls == 1 ? launch_gate<S_, 1>(g, st) : launch_gate<S_, 0>(g, st); break;
        OZ_CASE(1) OZ_CASE(2) OZ_CASE(3) OZ_CASE(4) OZ_CASE(5) OZ_CASE(6) OZ_CASE(7) OZ_CASE(8)
#undef OZ_CASE
        default: e = launch_gate_many(g, cls, s, st);
    }
    if (e == hipSuccess && scan_partials) {
        // (with few tiles the loads past the end would be most of them)
        if (tiles <= 2048) gate_scan_reduce_kernel<2><<<dim3(1), dim3(1024), 0, st>>>(scan_partials, tiles, nfr, s, scan_sums);
        else gate_scan_reduce_kernel<8><<<dim3(1), dim3(1024), 0, st>>>(scan_partials, tiles, nfr, s, scan_sums);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace ozimmu
