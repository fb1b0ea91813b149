// A gate on a state vector (Section 4.4): the complex product of a tall operand Z (m x k, the reshaped state,
// interleaved re/im) with a small one (B: k x n, the gate), k and n at most 128 (256 with up to eight slices), in ONE kernel
// that reads Z once and writes the result once.
//
// With so short an inner dimension the product is bound by the memory traffic of the state and by the vector
// work around the matrix cores (cutting the state into slices, folding the diagonals in FP64), and splitting the
// state in a kernel of its own doubles that traffic (slices written, slices read back). Here a workgroup of four
// wavefronts (eight when k or n exceeds 64, sixteen beyond 128) takes 32 rows of Z: it finds the exponents of their
// real and imaginary parts and cuts both planes into
// slices (SplitInt, Section 3.1; the same bit operations as the splitter kernels) straight into LDS, as operand
// fragments of v_mfma_i32_16x16x64_i8 (16 rows x 64 positions of k).
//
// The gate is split beforehand (gate_split_kernel) into two slice tensors whose 16-row fragments interleave its
// planes: fragment f of T1 holds columns 8 f .. 8 f + 7 of Br in rows 0..7 and the same columns of Bi in rows
// 8..15, T2 the other way round. A wavefront owns 16 rows and 8 complex columns at a time: Ar times a T1 fragment
// gives G(Ar,Br) in lanes 0..7 (of every 16) and G(Ar,Bi) in lanes 8..15, Ai times the T2 fragment gives G(Ai,Bi)
// and G(Ai,Br) in the same lanes, so that one rounded FP64 operation per lane forms re = G(Ar,Br) - G(Ai,Bi) or
// im = G(Ar,Bi) + G(Ai,Br); lanes 8 apart exchange half of their values and every lane stores whole (re, im) pairs.
// All anti-diagonals of a product are resident in registers (four per diagonal), every product is folded in FP64
// in the fixed order, least significant first, and scaled by 2^(EA_i + EB_j) (the summing-up step of the algorithm,
// Section 3.1).
//
// Why the small MFMA shape: a wavefront issues vector instructions at half the rate its SIMD can take them, and
// with the 32 x 32 shape the eight resident diagonals of a patch cost 128 registers, which leaves room for two
// wavefronts per SIMD only: whenever one of them waited for memory or for the matrix core, the vector pipeline ran
// at half speed. With 16 x 16 patches (32 registers for the diagonals) four wavefronts fit a SIMD; beyond eight
// slices (up to 64 registers for the diagonals and as many again for the fragments) two.
// Register allocation is left to the compiler: without accumulation-register operands in inline assembly the MFMA
// results land in ordinary vector registers, where the FP64 fold reads them directly, and a product's first MFMA
// per diagonal takes the constant 0 as its addend instead of cleared registers.
#pragma once

#include "mfma_common.h"
#include "split_common.h"

namespace ozimmu {
namespace {

constexpr int kGateMax = 128;    // largest k and n with more than eight slices
constexpr int kGateMaxFew = 256; // largest k and n with up to eight slices
constexpr int kGateRows = 32;    // rows of Z per workgroup: two fragments of 16
constexpr int kGateStep = 64;    // positions of k per MFMA

// A fragment: 16 rows x 64 positions, 1 KiB. Lane l of the MFMA operand holds row l % 16, positions 16 (l / 16) .. + 15
// (both operands alike, which is all a sum over k needs); its 16 bytes sit at byte 16 l.
__device__ __forceinline__ int frag_offset(int row, int pos) { return ((pos >> 4) * 16 + row) * 16 + (pos & 15); }

// |x| 2^(-E) < 1 to its upper 56 binary places as two words of 28: the scaled number's integer part, then that of the scaled
// rest (conversion and fraction are exact, truncation is what SplitInt wants, subnormals and zeros need no cases of their own). With
// integer instructions the same takes two 64-bit shifts and the handling of the exponent field; and FP64 instructions
// overlap better with the MFMAs of the other wavefronts (6 qubits of 24 201.0 -> 198.8 us, 5 qubits 213 -> 206).
struct Words28 {
    unsigned w[2];
};
__device__ __forceinline__ Words28 to_words28(unsigned long long bits, int E) {
    const double y = ldexp(__longlong_as_double((long long)(bits & kAbsMask)), 28 - E);
    Words28 f;
    f.w[0] = (unsigned)y;
    f.w[1] = (unsigned)ldexp(__builtin_amdgcn_fract(y), 28);
    return f;
}
// 28 bits to the low seven bits of four bytes, most significant first in the top byte; bit 7 of a byte is left over.
__device__ __forceinline__ unsigned spread28(unsigned x) {
    const unsigned y = (x & 0x3fffu) | ((x << 2) & ~0x3fffu);
    return (y & 0x007f007fu) | ((y << 1) & ~0x007f007fu);
}
// Slices 4 g + 1 .. 4 g + 4 of four elements, a slice to a word (element u in byte u), the bytes still to be cut to seven bits.
__device__ __forceinline__ void slices_of_four(const Words28 (&x)[4], int g, unsigned (&out)[4]) {
    unsigned e[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) e[u] = spread28(x[u].w[g]);
    // 4 x 4 bytes transposed: pairs of elements, then pairs of pairs
    const unsigned a_hi = __builtin_amdgcn_perm(e[1], e[0], 0x07030602u), a_lo = __builtin_amdgcn_perm(e[1], e[0], 0x05010400u);
    const unsigned b_hi = __builtin_amdgcn_perm(e[3], e[2], 0x07030602u), b_lo = __builtin_amdgcn_perm(e[3], e[2], 0x05010400u);
    out[0] = __builtin_amdgcn_perm(b_hi, a_hi, 0x07060302u);   // the top bytes: the first of the four slices
    out[1] = __builtin_amdgcn_perm(b_hi, a_hi, 0x05040100u);
    out[2] = __builtin_amdgcn_perm(b_lo, a_lo, 0x07060302u);
    out[3] = __builtin_amdgcn_perm(b_lo, a_lo, 0x05040100u);
}

// scan_count4 with the edges of a compile-time slice count (no counters for S - 1 = 0 slices)
template <int S>
__device__ __forceinline__ void scan_count4(ScanCount& a, const unsigned long long (&b)[4], int E) {
    scan_count4(a, b, E, 0x01010101u * (uint32_t)(OZIMMU_SLICE_BITS * S), 0x01010101u * (uint32_t)(OZIMMU_SLICE_BITS * (S > 1 ? S - 1 : 1)));
}

// ---------------------------------------------------------------------------- the product
// S slices; CLS, the size class of k and n: 0 up to 64 (one step of 64 positions, eight fragments of B, four wavefronts),
// 1 up to 128 (two steps, sixteen fragments), 2 up to 256 (four steps, 32 fragments, sixteen wavefronts; up to eight slices).
// SCAN: the kernel also counts, for the two planes of Z, what the slice-count choice needs to know about S and S - 1
// slices (Section 4.4; five counters per plane and tile, added up by gate_scan_reduce_kernel), so that a caller who
// guessed S can have the guess checked without another pass over Z.
// WAVES: wavefronts of the workgroup: 8 for CLS 1, 16 for CLS 2, 4 for CLS 0 (a gate of at most 32 x 32 has work for no
// more per tile; up to 64 x 64 a lane takes two words of its row and a wavefront four patches): four such workgroups
// then share a compute unit up to eight slices, and the latency of a tile's loads and its barrier hide behind three
// other tiles instead of one.
constexpr int gate_waves(int cls, int few) { return cls == 2 ? 16 : few == 3 ? 2 : few ? 4 : 8; }
// The narrowest gates (k <= 16, n <= 8: up to three qubits) have work for two wavefronts, and a quarter of a fragment's
// positions: their slices take a quarter of the LDS (the operand's other lanes read the same 16 positions again, and meet
// the zeros of the gate's fragments), so that eight such workgroups share a compute unit. A tile of so few bytes is all
// latency, and twice as many in flight take two thirds of the time (2 qubits of 24: 552 -> 360 us).
// FEW: 1 = four wavefronts, k <= 32; 2 = four wavefronts, two words to a lane; 3 = two wavefronts, k <= 16, n <= 8
// BOTH: a wavefront takes both row fragments of the tile, one after the other, with the gate's fragments it has loaded, instead of sharing the
// columns with a wavefront on the other sixteen rows: half the fragments on their way from the L2, which were the largest part of the time beside the MFMAs
// (6 qubits of 24 at eight slices 206 -> 189 us, at five 153 -> 137, at eleven 305 -> 296, 5 qubits 202 -> 192). Where that leaves a wavefront
// no more walks than before (launch_gate), and with one step only: with more, both fragments' sums would have to be resident, and four wavefronts
// to a SIMD have no registers for them.
template <int S, int CLS, bool SCAN, int FEW, bool BOTH>
__global__ __launch_bounds__(64 * gate_waves(CLS, FEW)) __attribute__((amdgpu_waves_per_eu(S <= kBand ? 4 : 2, S <= kBand ? 4 : 2)))
void gate_kernel(const GateArgs g) {
    static_assert(!FEW || CLS == 0, "four wavefronts: the smallest class only");
    static_assert(!BOTH || CLS == 0, "both row fragments: one step");
    constexpr bool WIDE = S > 9;   // the slices beyond the ninth come from the lower word of the fixed-point fraction
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr int KS = 1 << CLS, NFR = 8 << CLS, WAVES = gate_waves(CLS, FEW), NT = 64 * WAVES;
    constexpr int FRAG = FEW == 3 ? kFragBytes / 4 : kFragBytes;
    constexpr int SLICE = KS * 2 * FRAG;   // one slice of one plane of the tile's rows: [step][row fragment]
    constexpr int PLANE = S * SLICE;
    // behind the two planes: exponents of the tile's rows, [plane][32], then those of the gate's fragments, [tensor][NFR][16]
    int* ex = reinterpret_cast<int*>(lds + 2 * PLANE);
    int* ex_gate = ex + 2 * kGateRows;
    unsigned* scan_lds = reinterpret_cast<unsigned*>(ex_gate + 2 * NFR * 16);   // SCAN: [wavefront][plane][5] counters
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t row_tile = (int64_t)blockIdx.x * kGateRows;

    // ---- this wavefront's patches: rows 16 rf .. + 15 of the tile, complex columns 8 f .. 8 f + 7 for f = cg, cg + CGS, ...
    constexpr int CGS = BOTH ? WAVES : WAVES / 2, RF = BOTH ? 2 : 1;   // wavefronts side by side over the fragments of B; row fragments of each
    const int rf0 = BOTH ? 0 : wave & 1, cg = BOTH ? wave : wave >> 1;
    const unsigned char* a_rd = lds + rf0 * FRAG + 16 * (FEW == 3 ? lane & 15 : lane);
    constexpr int BSLICE = NFR * KS * kFragBytes, TENSOR = S * BSLICE;
    auto read_a = [&](int rf, int plane, int p, int step) __attribute__((always_inline)) -> v4i {   // rf: from rf0 on
        return *reinterpret_cast<const v4i*>(a_rd + rf * FRAG + plane * PLANE + p * SLICE + step * 2 * FRAG);
    };
    // fragments of the gate: a wave-uniform byte offset (tensor, fragment) plus the lane's 16 bytes, unsigned, so that the
    // loads take the tensor's address as their scalar base and a 32-bit register as offset
    const unsigned b_lane = 16u * (unsigned)lane;
    auto b_base = [&](int t, int f) __attribute__((always_inline)) -> unsigned {
        return (unsigned)__builtin_amdgcn_readfirstlane(t * TENSOR + f * KS * kFragBytes);
    };
    auto load_b = [&](unsigned base, int q, int step) __attribute__((always_inline)) -> v4i {
        return *reinterpret_cast<const v4i*>(g.T + (base + (unsigned)(q * BSLICE + step * kFragBytes) + b_lane));
    };
    // the gate's fragments of the first walk are requested before anything else: they are on their way while Z is split
    v4i b[S];
    {
        const unsigned first = b_base(0, cg);
        static_for<0, S>([&](auto pc) __attribute__((always_inline)) { b[decltype(pc)::value] = load_b(first, decltype(pc)::value, 0); });
    }

    // ---- the rows of Z -> exponents and slices in LDS. LPR lanes work on a row (16, or 32 with sixteen wavefronts); a
    // lane owns W words of four consecutive complex elements of it (words cl, LPR + cl, ...). A narrow gate (k <= 32,
    // k <= 16) has its rows' live words in 8 or 4 lanes: then half or a quarter of the wavefronts split all 32 rows and
    // the others skip this part. The positions of a step beyond those words are never written: the gate's fragments
    // hold zeros there (gate_split_kernel), and an integer times zero is zero whatever the LDS holds.
    for (int i = tid; i < 2 * NFR * 16; i += NT) ex_gate[i] = g.E[i];
    constexpr int LPR = FEW == 1 || FEW == 3 ? 16 : NT / kGateRows, W = KS * 16 / LPR;   // (FEW 1, 3: k <= 32, 16, never 16 lanes to a row)
    const int lshift = FEW == 3 ? 2 : FEW == 2 ? 3 : CLS == 0 ? (g.k <= 16 ? 2 : g.k <= 32 ? 3 : 4) : (LPR == 32 ? 5 : 4);   // log2 of the lanes per row
    if (tid < (kGateRows << lshift)) {   // whole wavefronts
        const int lrow = tid >> lshift, cl = tid & ((1 << lshift) - 1);
        const int64_t row = row_tile + lrow;
        const bool live = row < g.m;
        const ulonglong2* src = reinterpret_cast<const ulonglong2*>(g.Z) + (live ? row : 0) * g.ldz;
        ulonglong2 v[W][4];
#pragma unroll
        for (int j = 0; j < W; ++j)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int l = (cl + LPR * j) * 4 + u;
                v[j][u] = ulonglong2{0ull, 0ull};
                if (live && l < g.k) v[j][u] = src[l];
            }
        // Exponents of the row's two planes. The high words of the |x| bit patterns decide unless the row's maximum is
        // zero or subnormal: maxima of those over the row's 16 lanes with rotations inside the row, one instruction each.
        unsigned hw_re = 0, hw_im = 0;
#pragma unroll
        for (int j = 0; j < W; ++j)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const unsigned a = (unsigned)(v[j][u].x >> 32) & 0x7fffffffu, b2 = (unsigned)(v[j][u].y >> 32) & 0x7fffffffu;
                hw_re = a > hw_re ? a : hw_re;
                hw_im = b2 > hw_im ? b2 : hw_im;
            }
        if (CLS != 0 || lshift == 4) {
            hw_re = row_max_step<1>(row_max_step<2>(row_max_step<4>(row_max_step<8>(hw_re))));
            hw_im = row_max_step<1>(row_max_step<2>(row_max_step<4>(row_max_step<8>(hw_im))));
            if constexpr (LPR == 32) {   // the row's other sixteen lanes
                const unsigned o = __shfl_xor(hw_re, 16, 64), q = __shfl_xor(hw_im, 16, 64);
                hw_re = o > hw_re ? o : hw_re;
                hw_im = q > hw_im ? q : hw_im;
            }
        } else {   // rows of 4 or 8 lanes
            for (int off = 1 << (lshift - 1); off >= 1; off >>= 1) {
                const unsigned o = __shfl_xor(hw_re, off, 64), q = __shfl_xor(hw_im, off, 64);
                hw_re = o > hw_re ? o : hw_re;
                hw_im = q > hw_im ? q : hw_im;
            }
        }
        int e_re = (int)(hw_re >> 20) - 1022, e_im = (int)(hw_im >> 20) - 1022;   // as exponent_of_max for a normal maximum
        const bool normal = __all(hw_re >= 0x00100000u && hw_im >= 0x00100000u);
        if (!normal) {
            // some row of this wavefront has a zero or subnormal maximum (rows past the end of Z among them): full 64-bit maxima
            unsigned long long mx_re = 0, mx_im = 0;
#pragma unroll
            for (int j = 0; j < W; ++j)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const unsigned long long a = v[j][u].x & kAbsMask, b2 = v[j][u].y & kAbsMask;
                    mx_re = a > mx_re ? a : mx_re;
                    mx_im = b2 > mx_im ? b2 : mx_im;
                }
            for (int off = 1 << (lshift - 1); off >= 1; off >>= 1) {
                const unsigned long long o = __shfl_xor(mx_re, off, 64), q = __shfl_xor(mx_im, off, 64);
                mx_re = o > mx_re ? o : mx_re;
                mx_im = q > mx_im ? q : mx_im;
            }
            e_re = exponent_of_max(mx_re);
            e_im = exponent_of_max(mx_im);
        }
        if (cl == 0) {
            ex[lrow] = e_re;
            ex[kGateRows + lrow] = e_im;
        }
        ScanCount cnt_re = {}, cnt_im = {};
        auto emit = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < W; ++j) {
                const SignMask sr = sign_mask(v[j][0].x, v[j][1].x, v[j][2].x, v[j][3].x);
                const SignMask si = sign_mask(v[j][0].y, v[j][1].y, v[j][2].y, v[j][3].y);
                if constexpr (SCAN) {
                    const unsigned long long re4[4] = {v[j][0].x, v[j][1].x, v[j][2].x, v[j][3].x};
                    const unsigned long long im4[4] = {v[j][0].y, v[j][1].y, v[j][2].y, v[j][3].y};
                    scan_count4<S>(cnt_re, re4, e_re);
                    scan_count4<S>(cnt_im, im4, e_im);
                }
                const int word = cl + LPR * j;   // sixteen words to a step
                unsigned char* dst = lds + ((word >> 4) * 2 + (lrow >> 4)) * FRAG + frag_offset(lrow & 15, (word & 15) * 4);
                if constexpr (S <= kBand) {
#pragma unroll
                    for (int plane = 0; plane < 2; ++plane) {
                        Words28 x[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) x[u] = plane ? to_words28(v[j][u].y, e_im) : to_words28(v[j][u].x, e_re);
#pragma unroll
                        for (int g4 = 0; g4 < 2; ++g4) {
                            if (4 * g4 >= S) continue;
                            unsigned c[4];
                            slices_of_four(x, g4, c);
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                if (4 * g4 + q < S)
                                    *reinterpret_cast<uint32_t*>(dst + plane * PLANE + (4 * g4 + q) * SLICE) =
                                        apply_sign(c[q] & 0x7f7f7f7fu, plane ? si : sr);
                        }
                        __builtin_amdgcn_sched_barrier(0);   // one plane's temporaries at a time
                    }
                } else {
                    Fixed xr[4], xi[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        xr[u] = to_fixed<WIDE>(v[j][u].x, e_re);
                        xi[u] = to_fixed<WIDE>(v[j][u].y, e_im);
                    }
                    static_for<1, S + 1>([&](auto pc) __attribute__((always_inline)) {
                        constexpr int p = decltype(pc)::value;
                        *reinterpret_cast<uint32_t*>(dst + (p - 1) * SLICE) = packed_slice<WIDE>(xr, sr, p);
                        *reinterpret_cast<uint32_t*>(dst + PLANE + (p - 1) * SLICE) = packed_slice<WIDE>(xi, si, p);
                    });
                }
                __builtin_amdgcn_sched_barrier(0);   // one word's temporaries at a time
            }
        };
        emit();
        if constexpr (SCAN) {
            // sums over the wavefront (rotations inside the rows of 16 lanes, then the four rows through scalar registers),
            // one LDS word per wavefront and counter: no atomics, which a tile of few elements would feel
            unsigned c[2 * kScanCounters] = {cnt_re.sv_g, cnt_re.sz_g, cnt_re.sv_h, cnt_re.sz_h, cnt_re.bits,
                                             cnt_im.sv_g, cnt_im.sz_g, cnt_im.sv_h, cnt_im.sz_h, cnt_im.bits};
            unsigned mine = 0;
#pragma unroll
            for (int i = 0; i < 2 * kScanCounters; ++i) {
                const unsigned r = row_sum_step<1>(row_sum_step<2>(row_sum_step<4>(row_sum_step<8>(c[i]))));
                const unsigned total = (unsigned)__builtin_amdgcn_readlane((int)r, 0) + (unsigned)__builtin_amdgcn_readlane((int)r, 16) +
                                       (unsigned)__builtin_amdgcn_readlane((int)r, 32) + (unsigned)__builtin_amdgcn_readlane((int)r, 48);
                mine = lane == i ? total : mine;
            }
            if (lane < 2 * kScanCounters) scan_lds[wave * (2 * kScanCounters) + lane] = mine;
        }
    } else if constexpr (SCAN) {
        if (lane < 2 * kScanCounters) scan_lds[wave * (2 * kScanCounters) + lane] = 0u;
    }
    __syncthreads();
    if constexpr (SCAN) {
        if (tid < 2 * kScanCounters) {
            unsigned total = 0;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) total += scan_lds[w * (2 * kScanCounters) + tid];
            g.scan[(int64_t)tid * gridDim.x + blockIdx.x] = total;   // [counter][tile]
        }
    }

    // ---- the products
    // accumulator layout of the 16x16 MFMA: lane holds column (lane % 16); register u holds row 4 (lane / 16) + u
    const int lrow_first = rf0 * 16 + 4 * (lane >> 4), c8 = lane & 7;
    const bool is_im = (lane & 8) != 0;
    // patches of this wavefront that hold a column of C at all (wave-uniform)
    const int np = g.n > 8 * cg ? (g.n - 8 * cg - 1) / (8 * CGS) + 1 : 0;
    if (np == 0) return;

    v4i acc[S];
    v4i a[S];
    double part[RF][4];
    // iteration it: patch it / 2, pass it % 2 (0: Ar with T1, 1: Ai with T2)
    for (int it = 0; it < 2 * np; ++it) {
        const int pass = it & 1, f = cg + CGS * (it >> 1);
        const int nit = it + 1 < 2 * np ? it + 1 : 0;   // (after the last one the first one's fragments again, unused)
        const unsigned b_this = b_base(pass, f), b_next = b_base(nit & 1, cg + CGS * (nit >> 1));
        static_for<0, RF>([&](auto rc) __attribute__((always_inline)) {
            constexpr int rf = decltype(rc)::value;
            static_for<0, S>([&](auto pc) __attribute__((always_inline)) { a[decltype(pc)::value] = read_a(rf, pass, decltype(pc)::value, 0); });
            __builtin_amdgcn_sched_barrier(0);
            // Group q of a step = the MFMAs of B fragment q with the A fragments S - 1 - q .. 0, each into the sum of
            // its anti-diagonal p + q: b[q] and a[S - 1 - q] have their last use of the step there and are fetched again,
            // in place, for the next step. Across the end of a walk only the B fragments are (they come from memory); the
            // A fragments are read from LDS after the fold, which needs their registers.
            static_for<0, KS>([&](auto sc) __attribute__((always_inline)) {
                constexpr int step = decltype(sc)::value;
                constexpr bool last_step = step == KS - 1;
                static_for<0, S>([&](auto qc) __attribute__((always_inline)) {
                    constexpr int q = decltype(qc)::value, pmax = S - 1 - q;
                    static_for<0, pmax + 1>([&](auto ic) __attribute__((always_inline)) {
                        constexpr int p = pmax - decltype(ic)::value;
                        if constexpr (step == 0 && q == 0) acc[p] = mfma16(a[p], b[0], v4i{0, 0, 0, 0});
                        else acc[p + q] = mfma16(a[p], b[q], acc[p + q]);
                    });
                    if constexpr (last_step) {
                        if constexpr (rf == RF - 1) b[q] = load_b(b_next, q, 0);
                    } else {
                        b[q] = load_b(b_this, q, step + 1);
                        a[pmax] = read_a(rf, pass, pmax, step + 1);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
            // G = the diagonals, least significant first: acc = RN(acc + S_e 2^(-7 (e + 2))) (the product of an integer
            // below 2^31 and a power of two is exact, so the fused operation rounds like the sum it stands for) ...
            // (the first term as a plain product: RN(0 + t) = t, and t is exact)
            // The four least significant diagonals, two at a time as one integer 2^7 S_(e-1) + S_e: diagonal e sums e + 1 slice
            // products of at most 64 KS positions and 127^2 each, so while ((S - 1) 2^7 + S) 64 KS 127^2 < 2^31 that integer
            // fits 32 bits; and the partial sums of those four terms are integers of less than 2^53 units of 2^(-7 (S + 1)),
            // so no rounding happens among them and any grouping gives the value the one-by-one sequence gives.
            constexpr bool MERGE = S >= 4 && ((long long)(S - 1) * 128 + S) * (64 * KS) * (127 * 127) < (1ll << 31);
            constexpr int E_FIRST = MERGE ? S - 5 : S - 2;   // the diagonals from here down are added one by one
            auto scale_of = [](int e) __attribute__((always_inline)) {
                return __longlong_as_double((long long)(1023 - OZIMMU_SLICE_BITS * (e + 2)) << 52);
            };
            double sum[4];
    #pragma unroll
            for (int u = 0; u < 4; ++u) {
                if constexpr (MERGE) {
                    const int low = acc[S - 2][u] * (1 << OZIMMU_SLICE_BITS) + acc[S - 1][u];
                    const int next = acc[S - 4][u] * (1 << OZIMMU_SLICE_BITS) + acc[S - 3][u];
                    sum[u] = fma((double)next, scale_of(S - 3), (double)low * scale_of(S - 1));
                } else {
                    sum[u] = (double)acc[S - 1][u] * scale_of(S - 1);
                }
            }
    #pragma unroll
            for (int e = E_FIRST; e >= 0; --e) {
                const double sc = scale_of(e);
    #pragma unroll
                for (int u = 0; u < 4; ++u) sum[u] = fma((double)acc[e][u], sc, sum[u]);
            }
            // ... times 2^(EA_i + EB_j)
            const int lrow0 = lrow_first + 16 * rf;
            const v4i ea = *reinterpret_cast<const v4i*>(ex + pass * kGateRows + lrow0);   // four consecutive rows
            const int eb = ex_gate[pass * (NFR * 16) + f * 16 + (lane & 15)];
    #pragma unroll
            for (int u = 0; u < 4; ++u) sum[u] = ldexp(sum[u], ea[u] + eb);
            if (pass == 0) {
    #pragma unroll
                for (int u = 0; u < 4; ++u) part[rf][u] = sum[u];
            } else {
                // lanes 0..7 of every 16: re = G(Ar,Br) - G(Ai,Bi); lanes 8..15: im = G(Ar,Bi) + G(Ai,Br)
                // (the subtraction as the addition of the negated term: one flipped sign bit, no selection)
                const long long flip = is_im ? 0ll : (long long)(1ull << 63);
                double other[4];
    #pragma unroll
                for (int u = 0; u < 4; ++u) {
                    sum[u] = part[rf][u] + __longlong_as_double(__double_as_longlong(sum[u]) ^ flip);
                    // the other part of the same element, from the lane 8 further (rotation of the row of 16 lanes by 8)
                    const unsigned long long x = (unsigned long long)__double_as_longlong(sum[u]);
                    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)x, 0x128, 0xf, 0xf, false);
                    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(x >> 32), 0x128, 0xf, 0xf, false);
                    other[u] = __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
                }
                // the lane with the real parts stores rows 0 and 1 of its four, the one with the imaginary parts rows 2 and 3
                const int col = f * 8 + c8;
                const int64_t row0 = row_tile + lrow0 + (is_im ? 2 : 0);
                double* c = g.Cz + 2 * (row0 * g.ldcz + col);
    #pragma unroll
                for (int u = 0; u < 2; ++u) {
                    double2 z;
                    z.x = is_im ? other[u + 2] : sum[u];
                    z.y = is_im ? sum[u + 2] : other[u];
                    if (row0 + u < g.m && col < g.n) *reinterpret_cast<double2*>(c + 2 * (int64_t)u * g.ldcz) = z;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    }
}

template <int S, int CLS, bool SCAN, int FEW, bool BOTH>
hipError_t launch_gate_one(const GateArgs& g, hipStream_t st) {
    constexpr int lds = 2 * S * (1 << CLS) * 2 * (FEW == 3 ? kFragBytes / 4 : kFragBytes) + (2 * kGateRows + 2 * (8 << CLS) * 16 + 16 * 2 * kScanCounters) * (int)sizeof(int);
    static_assert(lds <= 160 * 1024 && (S > kBand || CLS == 2 || 2 * lds <= 160 * 1024) && (!FEW || S > kBand || (FEW == 3 ? 8 : 4) * lds <= 160 * 1024),
                  "the LDS of a compute unit: two workgroups of eight wavefronts (four of four) up to eight slices, else one workgroup");
    hipError_t e = allow_dynamic_lds<&gate_kernel<S, CLS, SCAN, FEW, BOTH>>(lds);
    if (e != hipSuccess) return e;
    const unsigned grid = (unsigned)((g.m + kGateRows - 1) / kGateRows);
    gate_kernel<S, CLS, SCAN, FEW, BOTH><<<dim3(grid), dim3(64 * gate_waves(CLS, FEW)), lds, st>>>(g);
    return hipGetLastError();
}
template <int S, int CLS, bool SCAN, int FEW>
hipError_t launch_gate(const GateArgs& g, hipStream_t st) {
    if constexpr (CLS == 0 && FEW == 0 && (SCAN || S <= 11)) {   // (more than 32 columns: fewer, with so few rows, are small_complex.hip's, but for small_complex_ahead's)
        return launch_gate_one<S, CLS, SCAN, FEW, true>(g, st);
    } else {
        if constexpr (CLS == 0 && FEW != 3) {
            constexpr int waves = gate_waves(CLS, FEW);
            const int fragments = (g.n + 7) / 8, walks = (fragments + waves / 2 - 1) / (waves / 2), walks_both = 2 * ((fragments + waves - 1) / waves);
            if (walks_both <= walks) return launch_gate_one<S, CLS, SCAN, FEW, true>(g, st);
        }
        return launch_gate_one<S, CLS, SCAN, FEW, false>(g, st);
    }
}
template <int S, int CLS>
hipError_t launch_gate(const GateArgs& g, hipStream_t st) {
    if constexpr (CLS == 0) {
        // no more tiles than compute units: eight wavefronts share a tile, whose time is what the call takes; with more tiles
        // four wavefronts each, four tiles to a compute unit, are faster (8192 x 64 x 64 at eight slices 14.7 us per call with four
        // wavefronts, 13.3 with eight; 4200 x 64 x 64 at sixteen 24.0, 21.9)
        if (g.m <= (int64_t)kGateRows * kComputeUnits) return g.scan ? launch_gate<S, 0, true, 0>(g, st) : launch_gate<S, 0, false, 0>(g, st);
        if (g.k <= 16 && g.n <= 8) return g.scan ? launch_gate<S, 0, true, 3>(g, st) : launch_gate<S, 0, false, 3>(g, st);
        if (g.k <= 32 && g.n <= 32) return g.scan ? launch_gate<S, 0, true, 1>(g, st) : launch_gate<S, 0, false, 1>(g, st);
        return g.scan ? launch_gate<S, 0, true, 2>(g, st) : launch_gate<S, 0, false, 2>(g, st);
    } else {
        return g.scan ? launch_gate<S, CLS, true, 0>(g, st) : launch_gate<S, CLS, false, 0>(g, st);
    }
}

}  // namespace
}  // namespace ozimmu
