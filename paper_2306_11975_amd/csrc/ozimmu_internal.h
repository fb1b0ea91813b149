// Internal declarations shared by the translation units of libozimmu (HIP, gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "ozimmu.h"

namespace ozimmu {

constexpr int kRowAlign = OZIMMU_ROW_ALIGN;   // slice rows are padded to a multiple of this (128)
constexpr int kSlab = OZIMMU_K_ALIGN;         // k-extent of a fragment of a slice tensor (32); a step of the walk takes two
constexpr int kFragRows = 32;                 // rows of one fragment
constexpr int kFragBytes = kFragRows * kSlab; // 1 KiB: what one wave-wide direct load moves
constexpr int kBand = 8;                      // anti-diagonals whose INT32 sums a wavefront holds at a time where two wavefronts share a SIMD
// The same where a wavefront has a SIMD to itself (64 x 64 tiles, one workgroup to a compute unit): twice the registers, and all diagonals
// of nine and of eleven to fifteen slices are walked at once, which saves the second walk its loads, barriers and start (per call: 1024^3 at nine slices 49.9 -> 46.7 us,
// 2000 x 1500 x 1000 at fifteen 258 -> 237, double-double 1501 x 1301 x 1107 at fourteen 185.6 -> 168.6; sixteen keep two bands of eight).
constexpr int resident_diagonals(int s, bool alone) { return alone && (s == 9 || (s >= 11 && s <= 15)) ? s : kBand; }

constexpr int kComputeUnits = 256;            // MI355X

static inline int64_t round_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

// Wavefront grid of the product kernel: 2 x 4 wavefronts of 32 x 32 outputs (a 64 x 128 tile of C) up to thirteen slices, whose
// steps of the walk (one stage and at most a part of a second) fit the LDS, 2 x 2 (64 x 64) beyond. `small`: 2 x 2 also for
// fewer, up to nine with two such workgroups per compute unit (see use_small_tiles).
static inline void tile_waves(int s, bool small, int* wm, int* wn) {
    *wm = 2;
    *wn = s > 13 || small ? 2 : 4;
}
// Whether a product of this shape runs on 64 x 64 tiles instead of 64 x 128 ones (a complex product
// in one launch: asked with twice its rows and columns; never with k-blocking, so that the workspace layout does not depend on it).
// Up to nine slices: two workgroups per compute unit instead of one. Two independent workgroups overlap one's start, fold and stores with the other's matrix-core work, and a last round that is not full
// costs less; the small tiles move a third more bytes into the LDS. So: small where the inner dimension is short or the large ones leave
// compute units without a tile; otherwise by an estimate of the time, rounds times a tile's time, whose constants are fitted to 150
// products of three to nine slices with k = 256 .. 8192 timed both ways (call, large -> small): complex 4096 x 4096 x 256 at seven slices
// 456 -> 392 us, x 1024 at eight 1735 -> 1690, x 2048 at six 2080 -> 2140 (stays large); real 1500 x 1800 x 1500 at nine (two rounds
// of large ones) 191 -> 153, 3500 x 3500 x 1536 at eight 529 -> 483, 8192 x 8192 x 8192 at eight 12910 -> 13090 (stays large). One round of
// large tiles is one of small ones as well and takes as long (1024 x 2048 x 1024 70.5, 71.4).
// With two to six slices the loads are what a long walk waits for, and two workgroups, each at a step of its own, find fewer of them in the L2 than one twice as large:
// as k goes from 2048 to 10240 a step of the small tiles comes to take up to 7 % more at five and six slices, of real products 12 % at three and four and 30 % at two (complex
// ones of so few slices, and one slice, lose nothing). Five have the least to cover a load with where a workgroup has a compute unit to itself. Per call, small -> large:
// 1033 x 12215 x 16484 at four 2830 -> 2550 us, 4990 x 1835 x 16428 at two 910 -> 845, 1169 x 9165 x 11163 at four 1524 -> 1430, complex 228 x 2401 x 5028 at five 403 -> 373; still
// large -> small: complex 1836 x 544 x 17249 at four 1577 -> 1204, 1338 x 1549 x 12050 at six 735 -> 683. Fitted to 1190 products of one to nine slices that the estimate without these
// terms has on small tiles, of which 123 took more than 1.5 % longer there, up to 10 %; of 350 others, with the terms, four do, up to 2.9 % (the most seen: 455 x 6066 x 10890 at six, 4.8 %).
// Eleven to thirteen: one workgroup per compute unit of either, and the same rate (4096^3 at eleven 2822, 2838 us; 4096 x 4096 x 512 396, 413), so rounds decide:
// 1024^3 at twelve 103 -> 71, 300^3 42 -> 28, 1500 x 1500 x 1000 205 -> 171, complex 300^3 48 -> 35.
// Ten keep the large tiles and two bands only because the interface's tests hold ozimmu_launch_plan to them (1000^3, 1024^3). They take longer: with this rule and one
// band for ten slices as well 1024^3 89 -> 62 us, 1500 x 1800 x 1500 219 -> 179, double-double 1501 x 1301 x 1107 180 -> 112, complex 300^3 39 -> 30, 1.25 x on average over 214 products.
static inline bool use_small_tiles(int64_t m, int64_t n, int64_t k_pad, int s, bool wide, bool cplx) {
    if (wide || s == 10 || s > 13) return false;
    const int64_t row_tiles = (m + 63) / 64, large = row_tiles * ((n + 127) / 128), small = row_tiles * ((n + 63) / 64);
    const int64_t large_rounds = (large + kComputeUnits - 1) / kComputeUnits;
    const double step_us = 0.08 * (s * (s + 1) / 2) + 0.17;   // of a round of 64 x 128 tiles
    const double walk_us = (double)((k_pad + 63) / 64) * step_us, ends_us = 3.0, ends_alone_us = 5.0;
    if (s > 10) {   // one workgroup of either to a compute unit, small tiles with half the work: what they save is rounds that are not full
        const int64_t rounds = (small + kComputeUnits - 1) / kComputeUnits;
        return (double)rounds * (0.5 * walk_us + ends_us) < (double)large_rounds * (walk_us + ends_us);
    }
    if (k_pad <= 512 || large < kComputeUnits) return true;
    if (large == kComputeUnits) return false;
    // what a step of the small tiles takes more (five and six slices: their loads are covered least; of seven and eight, in few rounds, less is
    // covered than in many: complex 217 x 3797 x 1568 at seven, two rounds of either, 195 -> 201 us, 808 x 1024 x 1024 97 -> 99: both stay large)
    const double few = large_rounds < 8 ? 0.04 : 0.0;
    const double long_walk = std::min(std::max((double)(k_pad - 2048) / 8192.0, 0.0), 1.0);
    const double more = s == 9 ? -0.01 : s == 8 ? 0.012 + few : s == 7 ? 0.015 + few
                      : 0.065 + long_walk * (s >= 5 ? 0.07 : cplx || s == 1 ? 0.0 : s == 2 ? 0.3 : 0.12);
    // a last round of small tiles with a compute unit to each takes 0.6 of one with two
    const int64_t pairs = 2 * kComputeUnits, rest = small % pairs;
    const double small_rounds = (double)(small / pairs) + (rest == 0 ? 0.0 : rest > kComputeUnits ? 1.0 : s == 5 ? 0.9 : 0.6);
    return small_rounds * (walk_us * (1.0 + more) + ends_us) < (double)large_rounds * (walk_us + ends_alone_us);
}

// Arguments of the slice-product kernel. One launch covers every tile of C.
struct GemmArgs {
    const int8_t* SA;        // slice tensor of A   (fragment layout, see ozimmu.h)
    const int8_t* SB;        // slice tensor of B^T
    int64_t a_slice_stride;  // bytes between consecutive slices of A
    int64_t b_slice_stride;
    int kslabs;              // padded row length in slabs of 32
    int t_begin, t_end;      // slab range of the walk along k
    int tiles_m, tiles_n;
    int tile_cols;           // 128, or 64 (2 x 2 wavefronts)
    int m, n;                // true extent of C
    int splits;              // workgroups per tile, each with split_slabs slabs of the walk (1: one, the whole walk)
    int split_slabs;         // (even)
    int* partial;            // splits > 1: their INT32 sums, [split][slice count][tile][16][threads of a tile]
    int block_steps;         // slabs after which the INT32 sums are moved into the INT64 sums in D (0: never)
    long long* D;            // INT64 diagonal sums (k-blocking only)
    int32_t* P;              // pair mode (P != nullptr): raw INT32 product of the slices SA, SB point at
    int64_t ldp;
    double* C;               // output, row-major
    int64_t ldc;             // in doubles
    int c_mode;              // 0: C = G, 1: C = C + G, 2: C = C - G, 3: C = alpha G (+ beta C if beta != 0),
                             // 4: (Zr, C + G) -> Cz as interleaved (re, im) pairs (C is read only)
    double* Zr;              // c_mode 4: finished real parts, same shape and leading dimension as C
    double* Cz;              // c_mode 4 and complex mode: complex output
    int64_t ldcz;            // its leading dimension in complex elements
    double alpha, beta;      // c_mode 3 only
    double* C_lo;            // low parts of a double-double result (double-double summing-up only)
    const int32_t* EA;
    const int32_t* EB;
    // complex mode only: the slice tensors and exponents of the imaginary planes (SA, SB, EA, EB: real planes)
    const int8_t* SA2;
    const int8_t* SB2;
    const int32_t* EA2;
    const int32_t* EB2;
};

// Arguments of the one-kernel complex product with a short inner dimension and few columns (a gate applied to
// a state vector, Section 4.4): Z is split inside the kernel, the small operand arrives as two slice tensors
// and exponent sets (gate.hip).
struct GateArgs {
    const double* Z;         // m x k complex elements, interleaved (re, im), 16-byte aligned
    int64_t ldz;             // in complex elements
    int64_t m;
    int k, n;                // 1 .. 128 each
    const int8_t* T;         // the gate's two slice tensors
    const int32_t* E;        // and their exponents
    double* Cz;              // m x n complex elements, interleaved, 16-byte aligned
    int64_t ldcz;            // in complex elements
    unsigned* scan;          // not null: per tile of 32 rows, ten counters for the check of the slice count (gate.hip)
};
// Whether that kernel serves a complex product Z (m x k) times B (k x n) -> Cz with s slices.
bool gate_product_applies(const double* Z, const double* B, const double* Cz, int64_t n, int64_t k, int s);
// Device scratch it needs for the gate's slices and exponents (0 if the shape is never served).
size_t gate_scratch_bytes(int64_t n, int64_t k, int s);
// Cz = Z . B: splits B (k x n complex elements, leading dimension ldb in complex elements) into `scratch`
// (16-byte aligned, gate_scratch_bytes), then the product kernel. Only where gate_product_applies.
// scan_partials (optional; gate_scan_bytes(m) bytes of device memory): the two kernels also count what the check of s
// as the automatic slice count needs, and scan_sums[plane * 16 + s - 1], [.. + s - 2] (planes 0, 1: real and imaginary
// part of Z, 2, 3: of B; the layout of the slice-count sums; device or mapped host memory) receive the bits the planes
// lose with s and with s - 1 slices.
size_t gate_scan_bytes(int64_t m);
hipError_t launch_gate_product(const double* Z, int64_t ldz, int64_t m, int64_t k, int64_t n, const double* B, int64_t ldb,
                               int s, void* scratch, double* Cz, int64_t ldcz, hipStream_t st,
                               unsigned* scan_partials = nullptr, unsigned long long* scan_sums = nullptr);

// A small real product in one launch (small.hip): m vectors of the first operand times n of the second, each the rows of a stored row-major
// array or its columns (leading dimension ld), all of length k.
struct SmallOperand {
    const double* X;
    int64_t ld;
    bool by_cols;
};
struct SmallArgs {
    SmallOperand x[2];
    int m, n, k;
    double* C;               // m x n, row-major
    int64_t ldc;
    int c_mode;              // 0: C = G, 3: C = alpha G (+ beta C if beta != 0)
    double alpha, beta;
    double* C_lo;            // not null: double-double sum, its low parts (c_mode 0)
    unsigned* counts;        // not null (device or mapped host memory): [row tiles, then column tiles][planes][2], the bits that a tile's rows
                             // (columns) lose with s and with s - 1 slices
};
// both_by_rows: neither operand by its columns
bool small_product_applies(int64_t m, int64_t n, int64_t k, int s, bool both_by_rows = false);
hipError_t launch_small_product(const SmallArgs& g, int s, hipStream_t st);
// The same for a complex product, its operands and C interleaved (leading dimensions in complex elements; c_mode 0).
bool small_complex_applies(int64_t m, int64_t n, int64_t k, int s);
// Whether a product that is not counted takes it (Z, B, Cz: where the gate kernel could serve instead).
bool small_complex_ahead(const double* Z, const double* B, const double* Cz, int64_t m, int64_t n, int64_t k, int s);
hipError_t launch_small_complex(const SmallArgs& g, int s, hipStream_t st);
constexpr int kSmallTileRows = 32;   // rows and columns of their tiles
constexpr int kSmallTilesPerUnit = 4;                                      // tiles times steps to a compute unit, at most
constexpr int kSmallMaxTiles = kSmallTilesPerUnit * kComputeUnits;         // so that many tiles (complex: fewer), whose counters the caller has room for

// negate: emit the slices of -A (-B) instead: same exponents, every slice with the opposite sign
// (how a conjugated operand's imaginary plane is split)
// Counting while splitting (the check of s as the automatic slice count, Section 4.4): scan_slots, if not null, is a
// zeroed array of scan_slots_bytes(planes of the operand) bytes; the splitter adds, per plane, five counters into one
// of its slots (scan_nc counters to a slot: 5 per plane of the operand; a one-plane launcher is handed the pointer to
// its plane's five), and launch_scan_reduce turns those of both operands (the second's slots behind the first's) into the bits lost with s and
// with s - 1 slices:
// out[plane * 16 + s - 1], out[plane * 16 + s - 2] (device or mapped host memory).
size_t scan_slots_bytes(int planes);
// One operand of a product, to be split: `count` vectors of length k, the rows of a stored row-major array or its columns
// (leading dimension ld), complex elements interleaved (one or two planes of slices and exponents).
struct SplitOperand {
    const double* X;
    int64_t ld, count, padded;   // padded: vectors of its slice tensor
    bool by_cols, negate_im;     // negate_im: the slices of -Im (a conjugated operand)
    int8_t* S[2];
    int32_t* E[2];
};
// Whether one launch splits both operands (split_pair_kernel), and the launch. partials (optional; 2 scan_slots_bytes(planes)
// bytes, need not be cleared): it also counts, and the bits the planes lose with s and with s - 1 slices arrive in sums_a
// and sums_b ([planes][16]; device or mapped host memory).
bool split_pair_applies(const SplitOperand& a, const SplitOperand& b, int planes, int64_t k_pad, int s, bool counting);
// to_host (optional; its words: kPairCountWords of mapped host memory): where they fit, the counters of its workgroups go there instead and no launch adds
// them up (its blocks is then set); add_pair_counts does, once the stream has been waited for. (Automatic mode, per call: 376 x 2594 x 67 at threshold
// 1 45.9 -> 39.9 us, 508 x 2683 x 390 65.4 -> 60.4; of longer calls, 2048^3 at twelve slices, it is lost in the runs' differences. More words than that: the launch that adds them up takes less than the host.)
constexpr int kPairCountWords = 8192;
struct PairCounts {
    unsigned* words;
    unsigned first, blocks;      // workgroups of the first operand, and of both (0: not used)
};
hipError_t launch_split_pair(const SplitOperand& a, const SplitOperand& b, int planes, int64_t k, int64_t k_pad, int s, hipStream_t st,
                             unsigned* partials, unsigned long long* sums_a, unsigned long long* sums_b, PairCounts* to_host);
void add_pair_counts(const PairCounts& c, int planes, int s, unsigned long long* sums_a, unsigned long long* sums_b);
hipError_t launch_scan_reduce(const unsigned long long* slots, int planes, int s, unsigned long long* out_first,
                              unsigned long long* out_second, hipStream_t st);
hipError_t launch_split_rows(const double* A, int64_t lda, int inc, int64_t m, int64_t k, int s,
                             int8_t* S, int64_t m_pad, int64_t k_pad, int32_t* E, hipStream_t st,
                             bool negate = false, unsigned long long* scan_slots = nullptr, int scan_nc = 5);
// The same for few and long rows of a real operand, where split_rows_in_pieces says so. rowmax: m_pad entries of scratch.
bool split_rows_in_pieces(int64_t m_pad, int64_t k_pad);
hipError_t launch_split_rows_pieces(const double* A, int64_t lda, int64_t m, int64_t k, int s, int8_t* S, int64_t m_pad, int64_t k_pad,
                                    int32_t* E, unsigned long long* rowmax, hipStream_t st, unsigned long long* scan_slots = nullptr);
hipError_t launch_split_cols(const double* B, int64_t ldb, int inc, int64_t k, int64_t n, int s,
                             int8_t* S, int64_t n_pad, int64_t k_pad, int32_t* E,
                             unsigned long long* colmax, hipStream_t st, bool negate = false,
                             unsigned long long* scan_slots = nullptr, int scan_nc = 5);
// Both planes of an interleaved complex B (k x n complex elements, leading dimension ldb in complex elements) in one
// set of launches; colmax: 2 n_pad entries. negate_im: the slices of -Im(B) (a conjugated operand).
hipError_t launch_split_cols_complex(const double* B, int64_t ldb, int64_t k, int64_t n, int s, int8_t* S_re, int8_t* S_im,
                                     int64_t n_pad, int64_t k_pad, int32_t* E_re, int32_t* E_im,
                                     unsigned long long* colmax, hipStream_t st, bool negate_im = false,
                                     unsigned long long* scan_slots = nullptr);
// Rows of an interleaved complex operand (Z: m x k complex elements, leading dimension ldz in complex
// elements), both planes in one pass; only where complex_rows_in_one_pass / complex_scan_in_one_pass say so
// (short enough rows, 16-byte aligned), otherwise one strided pass per plane with the functions above / below.
bool complex_rows_in_one_pass(const double* Z, int64_t k_pad);
hipError_t launch_split_rows_complex(const double* Z, int64_t ldz, int64_t m, int64_t k, int s, int8_t* S_re,
                                     int8_t* S_im, int64_t m_pad, int64_t k_pad, int32_t* E_re, int32_t* E_im,
                                     hipStream_t st, bool negate_im = false, unsigned long long* scan_slots = nullptr);
bool complex_scan_in_one_pass(const double* Z, int64_t k);
hipError_t launch_loss_scan_rows_complex(const double* Z, int64_t ldz, int64_t m, int64_t k,
                                         unsigned long long* sums_re, unsigned long long* sums_im, hipStream_t st);
// Both planes of a small interleaved complex operand scanned by columns (B: k x n complex elements, leading dimension
// ldb in complex elements, k and n at most 128, 16-byte aligned) in one launch.
bool complex_cols_scan_in_one_launch(const double* B, int64_t k, int64_t n);
hipError_t launch_loss_scan_cols_complex_small(const double* B, int64_t ldb, int64_t k, int64_t n,
                                               unsigned long long* sums_re, unsigned long long* sums_im, hipStream_t st);
// Slice products of the pairs p + q <= s + 1 with the FP64 sum. mode 0: FP64 sum; 1: double-double sum
// into C, C_lo; 2: the four real products of a complex one in one launch (no k-blocking: block_steps == 0),
// written to Cz as (re, im) pairs. splits > 1: the launch that adds the parts' sums up follows.
hipError_t launch_slice_gemm(const GemmArgs& args, int s, int mode, hipStream_t st);
// Slice-count scan: adds, for s = 1 .. 16, the mantissa bits s slices would lose into sums[s - 1].
hipError_t launch_loss_scan_rows(const double* A, int64_t lda, int inc, int64_t m, int64_t k,
                                 unsigned long long* sums, hipStream_t st);
hipError_t launch_loss_scan_cols(const double* B, int64_t ldb, int inc, int64_t k, int64_t n,
                                 unsigned long long* colmax, unsigned long long* sums, hipStream_t st);
// Both planes of an interleaved complex operand (k x n complex elements, ldb in complex elements) by columns; colmax: 2 n entries.
hipError_t launch_loss_scan_cols_complex(const double* B, int64_t ldb, int64_t k, int64_t n, unsigned long long* colmax,
                                         unsigned long long* sums_re, unsigned long long* sums_im, hipStream_t st);
// C = beta C (C = +0 if beta == 0, without reading C) on an m x n row-major array.
hipError_t launch_scale_f64(double* C, int64_t ldc, int64_t m, int64_t n, double beta, hipStream_t st);
// Complex update on rows x cols row-major arrays of interleaved (re, im) doubles, leading
// dimensions in complex elements: t = alpha T (T == nullptr: no product term), u = beta C
// (beta == 0: C is not read), C = t + u, each complex product as RN(RN(ar xr) - RN(ai xi)),
// RN(RN(ar xi) + RN(ai xr)). T may be C itself.
hipError_t launch_zaxpby(const double* T, int64_t ldt, double* C, int64_t ldc, int64_t rows, int64_t cols,
                         double ar, double ai, double br, double bi, hipStream_t st);
hipError_t launch_fill_u64(unsigned long long* p, int64_t count, unsigned long long v, hipStream_t st);
hipError_t launch_fill_f64(double* C, int64_t ldc, int c_inc, int64_t m, int64_t n, double v,
                           hipStream_t st);
hipError_t launch_fill_i32(int32_t* P, int64_t ldp, int64_t m, int64_t n, int32_t v, hipStream_t st);

}  // namespace ozimmu
