// Slice products on the CDNA4 INT8 matrix cores with the FP64 sum fused in
// (the pair loop of the IMMU algorithm with its product and summing-up steps, Section 3.1).
//
// Loop nest: "all diagonals resident". A wavefront owns a 32 x 32 patch of C, four 16 x 16 results of
// v_mfma_i32_16x16x64_i8, and keeps the exact INT32 sums of up to eight anti-diagonals d = p + q of that patch in its
// accumulation registers (16 registers per diagonal) for the whole walk along k. A workgroup of 2 x 4 wavefronts owns a
// 64 x 128 tile. One step covers 64 positions of k (two slabs of 32): the 32-row fragments of ALL slices of
// the tile's rows of A and of B^T (12 s KiB) are brought into LDS once, each wavefront reads its
// fragments (ds_read_b128) and issues the MFMAs of all pairs
// p + q <= s + 1, every one into the accumulator of its own diagonal. Integer addition is exact, so
// all pairs of a diagonal share one INT32 sum; nothing but the slices is read and nothing but C is
// written: no product and no diagonal sum ever exists in memory. At the end the diagonals are added
// in the fixed order (least significant first) in FP64, scaled by 2^(EA_i + EB_j), and stored.
//
// More than eight slices: the diagonals are walked in two bands, the upper eight first, then the
// remaining s - 8 (which are exactly the diagonals of the s - 8 slice problem); the FP64 sum of the
// first band waits in registers. Where a wavefront has a SIMD and its registers to itself one band holds all diagonals of 9 and
// of 11 to 15 slices (resident_diagonals). Long k (more than 2^17 products per INT32 sum, cf. Section 2.4 on
// splitting long k): every block_steps slabs the INT32 sums are added into INT64 sums in the
// workspace (k-blocking) and the FP64 sum is formed from those.
//
// Complex product (kModeComplex, Section 4.4): the same walk on tiles whose rows are the same complex rows twice, from the
// real and from the imaginary plane of A, and whose columns are complex columns twice. A wavefront's patch pairs 16 rows
// of Ar and the same 16 of Ai with 16 columns of Br and the same 16 of Bi, so that its four 16 x 16 results are the
// four real products of the same 16 x 16 complex elements, in the same lanes and registers: one fold, one rounded FP64
// operation per part, and C is written once as (re, im) pairs without anything having waited in memory.
//
// An odd number of slabs: the last step would be half empty. With nine slices and more a kernel of its own (HEAD) takes the last
// slab ahead of the steps instead, with two pairs of a diagonal to an MFMA (see band_walk); below, where the other workgroup of the
// compute unit fills the gap (and at nine where there is none: a call is then mostly launches), the last step runs with zeros
// for A's second slab.
//
// Why the small MFMA shape: what bounds this kernel at large k is the clock that the power management grants, and with
// signed 7-bit operands a register-only loop of 16x16x64 sustains about a fifth more operations than one of 32x32x32.
//
// Data path of a step: global -> LDS with wave-wide direct loads (global_load_lds_dwordx4, no
// staging registers; a fragment is 1 KiB contiguous in memory and in LDS);
// LDS -> registers with ds_read_b128 (fragment rows are 32 bytes with the two 16-byte halves
// swapped in rows 8..15 and 24..31, so that any 16 consecutive lanes cover all 64 banks).
#pragma once

#include "ozimmu_internal.h"

#include "mfma_common.h"

namespace ozimmu {
namespace {

constexpr int kLdsLimit = 160 * 1024;
constexpr int kLdsReserve = 2048;             // of a compute unit: exponents behind the stages
constexpr int kStepBytes = 2 * kFragBytes;    // two slabs: what a step advances along the fragments of a row group

// One band of a walk: the pairs (p, q), 0-based, with E0 <= p + q <= SB - 1 of an SB-slice problem, and how a step of it
// is run.
//
// Group q of a step = the MFMAs of B slice q with the A slices p = pmax(q) .. pmin(q), highest first. Registers hold the
// ND slices of A that a group can need (slice p in slot p % ND) and three or four slices of B (all of them up to five):
// after group q, A slice SB - 1 - q has had its last use and its slot takes the next slice that belongs there (of this
// step while there is one, else of the next step), and so does the slot of B slice q. These SB "reads" r = 0 .. SB - 1
// (one slice of A, one of B, behind group r) are all LDS reads of a step; in LDS a read's two slices share a slot, filled
// by direct loads from the step (t or t + 1) the read is for.
//
// One phase (Y == 0), where two or three whole stages fit the LDS: one barrier per step, X, behind group 0. Behind X
// of step t the reads take version t of the slots and version t + NB2 - 1 is requested into the buffer read in step t - 1.
// Two phases: the slots of the reads r < Y (phase 1) are read between X and the second barrier, Y, behind group Y, the
// others between Y and the next X. Phase 2 has one buffer, requested anew behind X (version t). Phase 1 has one, requested
// anew behind Y (version t + 1), or two, and then the same request needs not wait for Y and follows phase 2's. So a
// buffer is filled again as soon as every wavefront has read it, and its loads have the time up to the other barrier to
// land; one stage and at most a part of a second are enough, which is what lets a step be 64 positions long at up to
// 13 slices.
// KB: diagonals that a wavefront's registers hold.
template <int SB, int KB, int WM, int WN, bool SOLO>
struct Band {
    static constexpr int ND = SB < KB ? SB : KB;          // resident diagonals
    static constexpr int E0 = SB - ND;                    // lowest one (e = p + q, 0-based; d = e + 2)
    static constexpr int NW = WM * WN;
    static constexpr int SLOT = (WM + WN) * kStepBytes;   // LDS of one slice of A and one of B
    // 2 x 2 wavefronts with up to nine slices: two workgroups share a compute unit (and its LDS), unless there are not
    // more workgroups than compute units (SOLO): the whole LDS then holds the loads further ahead, which is what a
    // workgroup with nothing beside it to hide their latency needs
    static constexpr bool PAIRED = NW == 4 && SB <= 9 && !SOLO;
    static constexpr int CAP = PAIRED ? (kLdsLimit - kLdsReserve) / 2 : kLdsLimit - kLdsReserve;

    // register slots of B: blocks of three and four slices, so that a slot's next slice is three or four groups away
    static constexpr int FOURS = SB <= 5 ? 0 : SB % 3;
    static constexpr int NBUF = SB <= 5 ? SB : FOURS ? 4 : 3;
    static constexpr int b_slot(int q) {
        if (SB <= 5) return q;
        const int threes = SB - 4 * FOURS;
        return q < threes ? q % 3 : (q - threes) % 4;
    }
    // the slice of B that follows slice r in its slot (<= r: it belongs to the next step)
    static constexpr int b_next(int r) {
        for (int d = 1; d < SB; ++d)
            if (b_slot((r + d) % SB) == b_slot(r)) return (r + d) % SB;
        return r;
    }
    static constexpr int b_first(int slot) {
        for (int q = 0; q < SB; ++q)
            if (b_slot(q) == slot) return q;
        return 0;
    }
    static constexpr bool b_ahead(int r) { return b_next(r) <= r; }   // the read is for the next step
    static constexpr int a_next(int r) { return r < E0 ? E0 - 1 - r : E0 + (SB - 1 - r - E0 + 2 * ND) % ND; }
    static constexpr bool a_ahead(int r) { return r >= E0; }

    static constexpr int pmax(int q) { return SB - 1 - q; }
    static constexpr int pmin(int q) { return E0 - q > 0 ? E0 - q : 0; }
    static constexpr int pairs(int q) { return pmax(q) - pmin(q) + 1; }
    static constexpr int pairs_to(int q) { int n = 0; for (int i = 0; i <= q; ++i) n += pairs(i); return n; }   // groups 0 .. q

    // direct loads per wavefront for `slots` slots: wavefront w brings slab w % 2, row group (w / 2) % WM of A and w / 2 of B
    static constexpr int GA = NW / (2 * WM);              // wavefronts that share a row group of A (and slab)
    static constexpr int loads_a(int slots) { return (slots + GA - 1) / GA; }
    static constexpr int loads(int slots) { return loads_a(slots) + slots; }
    static_assert(NW == 2 * WN && GA >= 1, "one row group of B per pair of wavefronts");

    // Loads are requested one at a time behind pairs of the step, counted from its start: phase 2's (one phase: all) one per
    // pair from X on, phase 1's from BEGIN1 on, every STRIDE1 pairs (or PER1 to a pair). Spread, because a wavefront stalls
    // while a direct load is issued, and eight wavefronts that issue theirs at once queue behind each other.
    struct Plan { int y, nb1, nb2; };
    static constexpr int total_pairs() { return pairs_to(SB - 1); }
    static constexpr int begin1(Plan p) { return p.nb1 == 2 ? pairs_to(0) + loads(SB - p.y) : pairs_to(p.y); }
    static constexpr int stride1(Plan p) {
        const int room = (total_pairs() - begin1(p)) / loads(p.y);
        return room > 3 ? 3 : room < 1 ? 1 : room;
    }
    static constexpr int per1(Plan p) {
        const int room = total_pairs() - begin1(p);
        return room <= 0 ? loads(p.y) : (loads(p.y) + room - 1) / room;
    }
    static constexpr Plan plan() {
        constexpr int stage = SB * SLOT;
        if (2 * stage <= CAP) return {0, 1, CAP / stage > 3 ? 3 : CAP / stage};
        Plan best{1, 1, 1};
        int best_score = -1000;
        for (int y = 1; y < SB - 1; ++y)
            for (int nb1 = 1; nb1 <= 2; ++nb1) {
                const Plan p{y, nb1, 1};
                if ((y * nb1 + SB - y) * SLOT > CAP) continue;
                // pairs of MFMA work between the last request of a phase and its first read: fourteen are enough
                // (1800 cycles of the matrix cores); beyond that fewer loads count
                const int last2 = pairs_to(0) + loads(SB - y) - 1, last1 = begin1(p) + (loads(y) - 1) / per1(p) * stride1(p);
                if (last2 >= pairs_to(y)) continue;
                const int lead2 = pairs_to(y) - last2, lead1 = total_pairs() + pairs_to(0) - last1;
                const int lead = lead1 < lead2 ? lead1 : lead2;
                const int score = (lead < 14 ? lead : 14) * 8 + (lead < 32 ? lead : 32) - 16 * (loads(y) + loads(SB - y) - loads(SB));
                if (score > best_score) { best_score = score; best = p; }
            }
        return best;
    }
    static constexpr Plan P = plan();
    static constexpr int Y = P.y, NB1 = P.nb1, NB2 = P.nb2;
    static constexpr bool TWO = Y > 0;
    static constexpr int SIZE1 = Y * SLOT, SIZE2 = (SB - Y) * SLOT, BASE2 = SIZE1 * NB1;
    static constexpr int LDS = BASE2 + SIZE2 * NB2;
    static constexpr int N1 = TWO ? loads(Y) : 0, N2 = loads(SB - Y);
    static_assert(LDS <= CAP, "the stages must fit the LDS");
    static_assert(N1 + NB2 * N2 < 63, "vmcnt is a 6-bit counter");
    static constexpr int BEGIN1 = TWO ? begin1(P) : 0, STRIDE1 = TWO ? stride1(P) : 1, PER1 = TWO ? per1(P) : 1;
    // where phase 2's loads go: one to a pair, or more where a step has too few pairs
    static constexpr int room2() { return (TWO ? pairs_to(Y) : total_pairs()) - pairs_to(0); }
    static constexpr int PER2 = room2() > 0 ? (N2 + room2() - 1) / room2() : N2;
    // first and one-past-last load of phase f requested behind pair `at` (0-based, counted from the start of the step)
    static constexpr int load_begin(int f, int at) {
        const int d = f ? at - pairs_to(0) : at - BEGIN1, n = f ? N2 : N1, per = f ? PER2 : PER1, stride = f ? 1 : STRIDE1;
        if (d < 0 || d % stride != 0) return n;
        const int i = d / stride * per;
        return i < n ? i : n;
    }
    static constexpr int load_end(int f, int at) {
        const int i = load_begin(f, at) + (f ? PER2 : PER1), n = f ? N2 : N1;
        return i < n ? i : n;
    }
    // of phase 1's loads, those that are requested ahead of Y
    static constexpr int early1() {
        int n = 0;
        for (int at = 0; at < pairs_to(Y); ++at)
            if (load_begin(0, at) < N1) n = load_end(0, at);
        return n;
    }
    // loads that may still be in flight when a phase's slots are about to be read
    static constexpr int WAIT_X = TWO ? 0 : (NB2 - 2) * N2;
    static constexpr int WAIT_Y = TWO ? early1() : 0;
    static_assert(!TWO || NB1 == 2 || BEGIN1 >= pairs_to(Y), "a single buffer is refilled behind Y");
};

template <int S, int WM, int WN, bool SOLO>
struct Shape {
    static constexpr int KB = resident_diagonals(S, WM * WN == 4 && (S > 9 || SOLO));
    static constexpr int LDS1 = Band<S, KB, WM, WN, SOLO>::LDS;
    static constexpr int LDS2 = S > KB ? Band<(S > KB ? S - KB : 1), KB, WM, WN, SOLO>::LDS : 0;
    static constexpr int LDS = LDS1 > LDS2 ? LDS1 : LDS2;
};

// What a wavefront needs to know about its place in the walk.
struct Walk {
    unsigned char* lds;      // dynamic LDS segment
    unsigned lds_base;       // its LDS address
    int lane, wave, wm, wn;
    int tm, tn;
    int t_begin, t_end;      // slabs of this workgroup's walk
    int tid;
};

// A fragment of zeros: what A's second slab is read from when the walk ends with half a step, and what stands before its
// slice 0 in the head of a walk.
__device__ __align__(16) const int8_t zero_fragment[kFragBytes] = {};

__device__ __forceinline__ const int8_t* uniform_ptr(const int8_t* p) {
    const unsigned long long v = (unsigned long long)p;
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(v >> 32));
    return (const int8_t*)(((unsigned long long)hi << 32) | lo);
}

template <int N>
__device__ __forceinline__ void wait_loads() {
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
__device__ __forceinline__ void workgroup_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Offset of a lane's 16 bytes in the two slabs of a row group's step: an operand of the 16x16x64 MFMA takes row lane % 16
// (of the fragment's first 16; the other 16 are 512 bytes on) and 16 positions, chosen by lane / 16: the slab by its low
// bit, the half of the slab by its high one. (Both operands alike, which is all a sum over k needs. This assignment puts
// the lanes on the LDS banks exactly as a whole 32-row fragment read by the 32-row shape would, which has no conflicts;
// with slab and half exchanged every read takes twice as long.)
__device__ __forceinline__ unsigned operand_offset(int lane) {
    return (unsigned)(((lane >> 4) & 1) * kFragBytes + (lane & 15) * 32 + ((((lane >> 5) ^ (lane >> 3)) & 1) << 4));
}

// The walk of one band over the slabs [w.t_begin, w.t_end): acc[e - E0] receives the pairs of diagonal e;
// while_filling() is called once when the first loads are on their way, and clears acc; after_step(slabs done) is called
// after every step (k-blocking hooks in there). HEAD: the number of slabs is odd, and acc need not be cleared. All LDS traffic of the walk is complete when it returns.
template <int SB, int KB, int WM, int WN, bool SOLO, bool CPLX, bool HEAD, class WhileFilling, class AfterStep>
__device__ __forceinline__ void band_walk(v4i (&acc)[KB][4], const GemmArgs& g, const Walk& w, WhileFilling&& while_filling,
                                          AfterStep&& after_step) {
    using B = Band<SB, KB, WM, WN, SOLO>;
    constexpr int ND = B::ND, E0 = B::E0, Y = B::Y;
    static_assert(!CPLX || WM == 2, "one row group of a complex tile is real, one imaginary");
    const int slabs = w.t_end - w.t_begin;
    // the last slab of an odd number is taken ahead of the steps (HEAD; the number is odd), or shares the last step with zeros
    constexpr int head = HEAD ? 1 : 0;
    const int steps = HEAD ? slabs >> 1 : (slabs + 1) >> 1;
    const int last_off = (slabs - head - 1) * kFragBytes;

    // ---- the request side
    // This wavefront's share of a slot: slab `half` of one row group of A (of every GA-th slot) and of one of B.
    const int half = w.wave & 1, pairw = w.wave >> 1;
    const int ga = pairw / WM;                    // which of the GA wavefronts that share A's row group
    const bool zero_tail = !HEAD && (slabs & 1) && half;   // the last step has no second slab: A's is read as zeros, B's as the slab before
    constexpr int NA1 = B::TWO ? B::loads_a(Y) : 0, NA2 = B::loads_a(SB - Y);
    const int8_t* pa[NA1 + NA2];                  // phase 1's loads of A, then phase 2's
    const int8_t* pb[SB];                         // by read
    // A's j-th load of a phase of ns slots serves slot min(GA j + ga, ns - 1) (the last one again where there is none: the
    // same bytes to the same place, so that every wavefront has the same number of loads in flight)
    auto read_of_a = [&](int f, int j) __attribute__((always_inline)) -> int {
        const int x = B::GA * j + ga, ns = f ? SB - Y : Y;
        return (f ? Y : 0) + (x < ns ? x : ns - 1);
    };
    // complex: the row groups of a tile's A are its rows' real and imaginary parts, and the first half of B's row groups
    // is its columns' real parts
    auto first_a = [&](int r) __attribute__((always_inline)) -> const int8_t* {
        const int group = pairw % WM;
        const int8_t* base = CPLX && group ? g.SA2 : g.SA;
        return uniform_ptr(base + (int64_t)B::a_next(r) * g.a_slice_stride +
                           ((int64_t)(CPLX ? w.tm : w.tm * WM + group) * g.kslabs + w.t_begin) * kFragBytes);
    };
    auto first_b = [&](int q) __attribute__((always_inline)) -> const int8_t* {
        const int group = CPLX ? w.tn * (WN / 2) + pairw % (WN / 2) : w.tn * WN + pairw;
        const int8_t* base = CPLX && pairw >= WN / 2 ? g.SB2 : g.SB;
        return uniform_ptr(base + (int64_t)q * g.b_slice_stride + ((int64_t)group * g.kslabs + w.t_begin) * kFragBytes);
    };
    // Where each phase's next request stands: [phase][0] for the slices read for the version's own step, [1] for those read
    // for the step after it. Past the last step requests go on, so that the number of loads in flight stays what the waits
    // count on, but all lanes of them ask for the same 16 bytes (of the last step; into slots nobody reads any more).
    int kst[2][2];
    unsigned koff[2][2];   // its offset along the slabs
    unsigned lanes[2][2];  // mask of the lane's own offset
    auto place = [&](auto fc, auto dc, int k) __attribute__((always_inline)) {
        constexpr int F = decltype(fc)::value, d = decltype(dc)::value;
        constexpr int NA = F ? NA2 : NA1, A0 = F ? NA1 : 0;
        kst[F][d] = k;
        const int o = k * kStepBytes + half * kFragBytes;
        const unsigned off = (unsigned)(o < last_off ? o : last_off);
        koff[F][d] = off;
        lanes[F][d] = ~0u;
        if (zero_tail && k == steps - 1) {
#pragma unroll
            for (int j = 0; j < NA; ++j)
                if (B::a_ahead(read_of_a(F, j)) == (d == 1)) pa[A0 + j] = uniform_ptr(zero_fragment - (int64_t)off);
        }
    };
    auto advance_one = [&](auto fc, auto dc) __attribute__((always_inline)) {
        constexpr int F = decltype(fc)::value, d = decltype(dc)::value;
        if (kst[F][d] + 1 < steps) place(fc, dc, kst[F][d] + 1);
        else lanes[F][d] = 0u;
    };
    constexpr std::integral_constant<int, 0> PH1{}, OWN{};
    constexpr std::integral_constant<int, 1> PH2{}, AHEAD{};
    auto advance = [&](auto fc) __attribute__((always_inline)) {
        advance_one(fc, OWN);
        advance_one(fc, AHEAD);
    };
    auto start = [&](auto fc) __attribute__((always_inline)) {
        constexpr int F = decltype(fc)::value, R0 = F ? Y : 0, NS = F ? SB - Y : Y, NA = F ? NA2 : NA1, A0 = F ? NA1 : 0;
#pragma unroll
        for (int j = 0; j < NA; ++j) pa[A0 + j] = first_a(read_of_a(F, j));
        static_for<R0, R0 + NS>([&](auto rc) __attribute__((always_inline)) { pb[decltype(rc)::value] = first_b(B::b_next(decltype(rc)::value)); });
        place(fc, OWN, 0);
        place(fc, AHEAD, 0);
        advance_one(fc, AHEAD);
    };
    const unsigned lane16 = (unsigned)w.lane * 16u;
    const unsigned dst_a = w.lds_base + (unsigned)(ga * B::SLOT + (pairw % WM) * kStepBytes + half * kFragBytes);
    const unsigned dst_b = w.lds_base + (unsigned)((WM + pairw) * kStepBytes + half * kFragBytes);
    // the i-th load of phase F into the buffer at buf: with(source, lane offset, LDS address, constant part of it)
    auto request = [&](auto fc, auto ic, unsigned buf, auto&& with) __attribute__((always_inline)) {
        constexpr int F = decltype(fc)::value, i = decltype(ic)::value;
        constexpr int R0 = F ? Y : 0, NS = F ? SB - Y : Y, NA = F ? NA2 : NA1;
        if constexpr (i < NA) {
            constexpr int r0 = R0 + B::GA * i, r1 = r0 + B::GA - 1;
            constexpr bool dup = r1 >= R0 + NS;   // the last load may serve an earlier slot
            unsigned off, own, d = dst_a + buf;
            if constexpr (dup || B::a_ahead(r0) == B::a_ahead(r1)) { off = koff[F][B::a_ahead(r0)]; own = lanes[F][B::a_ahead(r0)]; }
            else { off = ga ? koff[F][B::a_ahead(r1)] : koff[F][B::a_ahead(r0)]; own = ga ? lanes[F][B::a_ahead(r1)] : lanes[F][B::a_ahead(r0)]; }
            if constexpr (dup) d -= (unsigned)((B::GA * i + ga - (read_of_a(F, i) - R0)) * B::SLOT);
            with(pa[(F ? NA1 : 0) + i], (lane16 & own) | off, d, std::integral_constant<unsigned, (unsigned)(i * B::GA * B::SLOT)>{});
        } else {
            constexpr int r = R0 + i - NA;
            with(pb[r], (lane16 & lanes[F][B::b_ahead(r)]) | koff[F][B::b_ahead(r)], dst_b + buf, std::integral_constant<unsigned, (unsigned)((i - NA) * B::SLOT)>{});
        }
    };
    auto issue_all = [&](auto fc, unsigned buf) __attribute__((always_inline)) {
        constexpr int F = decltype(fc)::value;
        static_for<0, (F ? B::N2 : B::N1)>([&](auto ic) __attribute__((always_inline)) {
            request(fc, ic, buf, [&](const int8_t* src, unsigned voff, unsigned dst, auto imm) __attribute__((always_inline)) {
                dma_load16<decltype(imm)::value>(src, voff, dst);
            });
        });
        advance(fc);
    };

    // ---- the read side
    v4i a[ND][2], b[B::NBUF][2];
    const unsigned op_off = operand_offset(w.lane);
    const unsigned rd_a = op_off + (unsigned)(CPLX ? w.wm * 512 : w.wm * kStepBytes);
    const unsigned rd_b = op_off + (unsigned)(CPLX ? (WM + (w.wn >> 1)) * kStepBytes + (w.wn & 1) * 512 : (WM + w.wn) * kStepBytes);
    // from a patch's first 16 rows (columns) to its second
    constexpr unsigned IA = CPLX ? kStepBytes : 512, JB = CPLX ? (WN / 2) * kStepBytes : 512;
    // Operands straight from memory, for step 0 (nothing in LDS is older than what the steps read there) and for the head.
    struct Sources { const int8_t* a[2]; const int8_t* b[2]; };   // of the patch's two halves, at slab t, slice 0
    auto sources = [&](int t) __attribute__((always_inline)) -> Sources {
        const int64_t ga = CPLX ? w.tm : w.tm * WM + w.wm, gb = CPLX ? w.tn * (WN / 2) + (w.wn >> 1) : w.tn * WN + w.wn;
        const int64_t oa = (ga * g.kslabs + t) * kFragBytes + (CPLX ? w.wm * 512 : 0);
        const int64_t ob = (gb * g.kslabs + t) * kFragBytes + (CPLX ? (w.wn & 1) * 512 : 0);
        return {{g.SA + oa, CPLX ? g.SA2 + oa : g.SA + oa + 512}, {g.SB + ob, CPLX ? g.SB2 + ob : g.SB + ob + 512}};
    };
    auto load = [&](const int8_t* p) __attribute__((always_inline)) -> v4i { return *reinterpret_cast<const v4i*>(p); };
    auto load_a = [&](auto pc, const Sources& from, unsigned off) __attribute__((always_inline)) {
        constexpr int p = decltype(pc)::value;
#pragma unroll
        for (int i = 0; i < 2; ++i) a[p % ND][i] = load(from.a[i] + p * g.a_slice_stride + off);
    };
    auto load_b = [&](auto sc, const Sources& from, unsigned off) __attribute__((always_inline)) {   // by register slot
        constexpr int slot = decltype(sc)::value, q = B::b_first(slot);
#pragma unroll
        for (int j = 0; j < 2; ++j) b[slot][j] = load(from.b[j] + q * g.b_slice_stride + off);
    };
    auto load_first = [&]() __attribute__((always_inline)) {
        // (a walk of one slab: the second half of every lane's positions does not exist; A's are zeros, B's whatever slab 0 holds)
        const int lane = lane_here();
        const bool half_step = !HEAD && slabs == 1;
        const unsigned off = operand_offset(half_step ? lane & ~16 : lane);
        const Sources from = sources(w.t_begin);
        static_for<0, ND>([&](auto xc) __attribute__((always_inline)) {   // in the order of their first use
            if constexpr (decltype(xc)::value < B::NBUF) load_b(xc, from, off);
            load_a(std::integral_constant<int, SB - 1 - decltype(xc)::value>{}, from, off);
        });
        if (half_step) {
            static_for<0, ND>([&](auto xc) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < 2; ++i) a[decltype(xc)::value][i] = lane & 16 ? v4i{0, 0, 0, 0} : a[decltype(xc)::value][i];
            });
        }
    };

    // The head: one slab, with two pairs of a diagonal to an MFMA. The lanes that hold the second slab of a step hold the
    // neighbouring slices instead, p - 1 of A beside p (zeros beside slice 0) and q + 1 of B beside q, so that the groups of the
    // even q make up all pairs, in about half the MFMAs of a step. Its operands come straight from memory into the registers of
    // the steps' operands, and those of step 0 follow as registers fall free: beside the first loads of the walk, which it would
    // wait for anyway, the head costs little more than its MFMAs.
    // (One address at a time: a lane's own part of it is 64 bits wide, and there are no registers for several.)
    int64_t lane_a, lane_b;   // its own part: where its 16 bytes lie, and the neighbouring slice
    auto head_a = [&](auto pc, const Sources& from) __attribute__((always_inline)) {
        constexpr int p = decltype(pc)::value;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if constexpr (p > 0) {
                a[p % ND][i] = load(from.a[i] + p * g.a_slice_stride + lane_a);
            } else {
                const int lane = lane_here();
                // (as an offset, so that the load stays one from global memory)
                const int64_t to_zeros = (int64_t)zero_fragment - (int64_t)from.a[i];
                a[0][i] = load(from.a[i] + ((lane & 16 ? to_zeros : 0) + operand_offset(lane & ~16)));
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto head_b = [&](auto hc, const Sources& from) __attribute__((always_inline)) {   // slice q = 2 h
        constexpr int h = decltype(hc)::value, q = 2 * h;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int8_t* const slice = from.b[j] + q * g.b_slice_stride;
            // (beside the last slice, which meets slice 0 of A only, stands the same one again)
            b[h % B::NBUF][j] = q + 1 < SB ? load(slice + lane_b) : load(slice + operand_offset(lane_here() & ~16));
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    constexpr int HEAD_GROUPS = (SB + 1) / 2;
    auto head_first = [&]() __attribute__((always_inline)) {
        const int lane = lane_here();
        const Sources from = sources(w.t_end - 1);
        lane_a = (int64_t)operand_offset(lane & ~16) - (lane & 16 ? g.a_slice_stride : 0);
        lane_b = (int64_t)operand_offset(lane & ~16) + (lane & 16 ? g.b_slice_stride : 0);
        static_for<0, ND>([&](auto xc) __attribute__((always_inline)) {
            constexpr int x = decltype(xc)::value;
            if constexpr (x < B::NBUF && x < HEAD_GROUPS) head_b(xc, from);
            head_a(std::integral_constant<int, SB - 1 - x>{}, from);
        });
    };
    auto head_step = [&]() __attribute__((always_inline)) {
        // (a walk without steps: the same slab once more, for nothing)
        const Sources from = sources(w.t_end - 1), next = sources(w.t_begin);
        const unsigned off = operand_offset(steps ? lane_here() : lane_here() & ~16);
        valu_results_ready();
        static_for<0, HEAD_GROUPS>([&](auto hc) __attribute__((always_inline)) {
            constexpr int h = decltype(hc)::value, q = 2 * h;
            static_for<0, B::pairs(q)>([&](auto ic) __attribute__((always_inline)) {
                constexpr int p = B::pmax(q) - decltype(ic)::value;
                const v4i(&x)[2] = a[p % ND], (&y)[2] = b[h % B::NBUF];
                v4i(&c)[4] = acc[p + q - E0];
                if constexpr (h == 0) {   // every diagonal's first product: nothing to clear
                    mfma16_new(x[0], y[0], c[0]);
                    mfma16_new(x[0], y[1], c[1]);
                    mfma16_new(x[1], y[1], c[3]);
                    mfma16_new(x[1], y[0], c[2]);
                } else {
                    mfma16_acc(x[0], y[0], c[0]);
                    mfma16_acc(x[0], y[1], c[1]);
                    mfma16_acc(x[1], y[1], c[3]);
                    mfma16_acc(x[1], y[0], c[2]);
                }
            });
            __builtin_amdgcn_sched_barrier(0);
            // behind this group two slices of A and one of B have had their last use
            static_for<q, (q + 2 < SB ? q + 2 : SB)>([&](auto rc) __attribute__((always_inline)) {
                constexpr int r = decltype(rc)::value;
                if constexpr (B::a_ahead(r)) load_a(std::integral_constant<int, B::a_next(r)>{}, next, off);
                else head_a(std::integral_constant<int, B::a_next(r)>{}, from);
            });
            if constexpr (h + B::NBUF < HEAD_GROUPS) head_b(std::integral_constant<int, h + B::NBUF>{}, from);
            else load_b(std::integral_constant<int, h % B::NBUF>{}, next, off);
            __builtin_amdgcn_sched_barrier(0);
        });
        // register slots of B that the head had no use for
        static_for<(HEAD_GROUPS < B::NBUF ? HEAD_GROUPS : B::NBUF), B::NBUF>([&](auto sc) __attribute__((always_inline)) { load_b(sc, next, off); });
        last_mfma_issued();
    };

    // read positions (lane offsets into the buffers phase 1 and 2 are read from) and request buffers
    unsigned cur1 = 0, cur2 = B::BASE2, req1 = (B::NB1 - 1) * B::SIZE1, req2 = B::BASE2 + (B::NB2 - 1) * B::SIZE2;
    unsigned ra1 = rd_a, rb1 = rd_b, ra2 = rd_a + B::BASE2, rb2 = rd_b + B::BASE2;
    if constexpr (B::NB2 == 1) asm("" : "+v"(ra2), "+v"(rb2));   // (registers of their own: the reads' offsets then fit the instruction)
    auto step = [&]() __attribute__((always_inline)) {
        valu_results_ready();
        static_for<0, SB>([&](auto qc) __attribute__((always_inline)) {
            constexpr int q = decltype(qc)::value;
            static_for<0, B::pairs(q)>([&](auto ic) __attribute__((always_inline)) {
                constexpr int p = B::pmax(q) - decltype(ic)::value;
                constexpr int at = (q ? B::pairs_to(q - 1) : 0) + decltype(ic)::value;   // pairs ahead of this one
                const v4i(&x)[2] = a[p % ND], (&y)[2] = b[B::b_slot(q)];
                v4i(&c)[4] = acc[p + q - E0];
                constexpr int i1 = B::load_begin(0, at), n1 = B::load_end(0, at) - i1, i2 = B::load_begin(1, at), n2 = B::load_end(1, at) - i2;
                if constexpr (SB > 1 && n1 + n2 > 0) {
                    constexpr bool second = n2 > 0;
                    __builtin_amdgcn_sched_barrier(0);
                    // one load behind the pair's first MFMA; more than one only where a step has few pairs
                    auto with_mfma = [&](const int8_t* src, unsigned voff, unsigned dst, auto imm) __attribute__((always_inline)) {
                        mfma16_acc_and_load<decltype(imm)::value>(x[0], y[0], c[0], src, voff, dst);
                    };
                    auto alone = [&](const int8_t* src, unsigned voff, unsigned dst, auto imm) __attribute__((always_inline)) {
                        dma_load16<decltype(imm)::value>(src, voff, dst);
                    };
                    if constexpr (second) request(PH2, std::integral_constant<int, i2>{}, req2, with_mfma);
                    else request(PH1, std::integral_constant<int, i1>{}, req1, with_mfma);
                    static_for<1, n2>([&](auto lc) __attribute__((always_inline)) { request(PH2, std::integral_constant<int, i2 + decltype(lc)::value>{}, req2, alone); });
                    static_for<(second ? 0 : 1), n1>([&](auto lc) __attribute__((always_inline)) { request(PH1, std::integral_constant<int, i1 + decltype(lc)::value>{}, req1, alone); });
                    __builtin_amdgcn_sched_barrier(0);
                } else {
                    mfma16_acc(x[0], y[0], c[0]);
                }
                mfma16_acc(x[0], y[1], c[1]);
                mfma16_acc(x[1], y[1], c[3]);
                mfma16_acc(x[1], y[0], c[2]);
            });
            if constexpr (q == 0) {
                // every wavefront has read what the last step read behind its last barrier, and what is read from here
                // on has landed everywhere
                __builtin_amdgcn_sched_barrier(0);
                wait_loads<B::WAIT_X>();
                workgroup_barrier();
                if constexpr (SB == 1) issue_all(PH2, req2);
            }
            if constexpr (B::TWO && q == Y) {
                __builtin_amdgcn_sched_barrier(0);
                advance(PH2);
                wait_loads<B::WAIT_Y>();
                workgroup_barrier();
            }
            {
                constexpr unsigned slot = (unsigned)((q < Y ? q : q - Y) * B::SLOT);
                constexpr int pn = B::a_next(q) % ND, bn = B::b_slot(q);
#pragma unroll
                for (int j = 0; j < 2; ++j) b[bn][j] = *reinterpret_cast<const v4i*>(w.lds + (q < Y ? rb1 : rb2) + (slot + j * JB));
#pragma unroll
                for (int i = 0; i < 2; ++i) a[pn][i] = *reinterpret_cast<const v4i*>(w.lds + (q < Y ? ra1 : ra2) + (slot + i * IA));
                __builtin_amdgcn_sched_barrier(0);   // keep the reads where their registers fall free
            }
        });
        last_mfma_issued();
        if constexpr (!B::TWO && SB > 1) advance(PH2);
        if constexpr (B::TWO) advance(PH1);
        if constexpr (B::NB1 == 2) {
            req1 = cur1;
            cur1 = B::SIZE1 - cur1;
            ra1 += cur1 - req1;
            rb1 += cur1 - req1;
        }
        if constexpr (B::NB2 > 1) {
            req2 = cur2;
            cur2 = cur2 + B::SIZE2 < (unsigned)B::LDS ? cur2 + B::SIZE2 : (unsigned)B::BASE2;
            ra2 += cur2 - req2;
            rb2 += cur2 - req2;
        }
    };
    if constexpr (HEAD) head_first();
    else load_first();
    __builtin_amdgcn_sched_barrier(0);
    if (!HEAD || steps) {
        if constexpr (B::TWO) start(PH1);
        start(PH2);
        if constexpr (B::TWO) issue_all(PH1, 0u);
        static_for<0, B::NB2 - 1>([&](auto vc) __attribute__((always_inline)) { issue_all(PH2, (unsigned)(B::BASE2 + decltype(vc)::value * B::SIZE2)); });
    }
    __builtin_amdgcn_sched_barrier(0);
    while_filling();
    if constexpr (HEAD) head_step();
    // Nothing that shares the counter of the LDS reads may be in flight when the step loop is entered (a scalar load of
    // a kernel argument, say): scalar loads complete out of order, and with one possibly in flight on entry every wait
    // for a fragment inside the loop becomes a wait for all of them.
    // The same goes for step 0's operands from memory: left to the first use, the wait for them stands in the loop, where it waits
    // for the direct loads of every step.
    __builtin_amdgcn_s_waitcnt(HEAD ? 0x0070 : 0xC07F);   // lgkmcnt(0) (and vmcnt(0))
    for (int t = 0; t < steps; ++t) {
        step();
        after_step(t + 1 < steps ? 2 * (t + 1) : slabs);
    }
    // requests of the repeated last step may still be in flight: they must land before the
    // LDS is used for anything else or handed to another workgroup
    __builtin_amdgcn_sched_barrier(0);
    wait_loads<0>();
    workgroup_barrier();
}

template <int SB, int KB>
__device__ __forceinline__ void fold_band_dd(double (&h)[16], double (&l)[16], const v4i (&acc)[KB][4]) {
    constexpr int ND = SB < KB ? SB : KB, E0 = SB - ND;
    mfma_results_ready();
#pragma unroll
    for (int e = SB - 1; e >= E0; --e) {
        const double sc = __longlong_as_double((long long)(1023 - OZIMMU_SLICE_BITS * (e + 2)) << 52);
#pragma unroll
        for (int u = 0; u < 16; ++u) dd_add(h[u], l[u], (double)acc_read(acc[e - E0][u >> 2][u & 3]) * sc);
    }
}

// Whether a combine mode reads the old contents of C.
__device__ __forceinline__ bool c_mode_reads(const GemmArgs& g, int c_mode) {
    return c_mode == 1 || c_mode == 2 || c_mode == 4 || (c_mode == 3 && g.beta != 0.0);
}

// One element of the result: `old_c` combined with val by combine mode c_mode (0: val alone). Mode 4 is not among them.
__device__ __forceinline__ double combined(const GemmArgs& g, double old_c, double val) {
    if (g.c_mode == 1) return old_c + val;
    if (g.c_mode == 2) return old_c - val;
    // BLAS update: RN(alpha G), then RN(RN(alpha G) + RN(beta C)); C is not read if beta == 0
    const double v = g.alpha * val;
    return g.beta != 0.0 ? v + g.beta * old_c : v;
}

// kModeComplex: a complex product in one launch (planes SA/SA2, SB/SB2; result interleaved in Cz).
constexpr int kModeReal = 0, kModeDD = 1, kModeComplex = 2;

// Element u of a thread's sixteen: patch (i, j) = (u / 8, u / 4 % 2), register u % 4 of it. Accumulator layout of the
// 16x16 MFMA: lane holds column lane % 16; register r holds row 4 (lane / 16) + r.
constexpr int elem_row(int u) { return 16 * (u >> 3) + (u & 3); }
constexpr int elem_col(int u) { return 16 * ((u >> 2) & 1); }

template <int S, int WM, int WN, int MODE, bool SOLO, bool HEAD>
__global__ __launch_bounds__(64 * WM * WN)
__attribute__((amdgpu_waves_per_eu((WM * WN == 4 && S <= 9 && !SOLO) ? 2 : WM * WN / 4, (WM * WN == 4 && S <= 9 && !SOLO) ? 2 : WM * WN / 4)))
void product_kernel(const GemmArgs g) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr int T = 64 * WM * WN;
    constexpr int KB = Shape<S, WM, WN, SOLO>::KB;
    constexpr int S2 = S > KB ? S - KB : 1;         // slice count of the second band (unused if there is one)
    constexpr bool CPLX = MODE == kModeComplex;
    constexpr int NEX = CPLX ? 2 : 1;                     // exponent sets staged (one per plane)
    constexpr int TR = (CPLX ? 16 : 32) * WM, TC = (CPLX ? 16 : 32) * WN;   // tile of C (complex: in complex elements)

    Walk w;
    w.tid = threadIdx.x;
    w.lane = w.tid & 63;
    w.wave = __builtin_amdgcn_readfirstlane(w.tid >> 6);   // wave-uniform, kept in a scalar register
    w.wm = w.wave / WN;
    w.wn = w.wave % WN;
    if (WM * WN == 8 && w.wave >= 4) __builtin_amdgcn_s_setprio(2);   // (the two wavefronts of a SIMD drift apart: 0.5 %)
    const int tiles = g.tiles_m * g.tiles_n;
    const int split = g.splits > 1 ? (int)blockIdx.x / tiles : 0;
    tile_of_block((int)blockIdx.x - split * tiles, g.tiles_m, g.tiles_n, w.tm, w.tn);
    w.t_begin = g.t_begin + split * g.split_slabs;
    w.t_end = g.splits > 1 && w.t_begin + g.split_slabs < g.t_end ? w.t_begin + g.split_slabs : g.t_end;
    w.lds = lds;
    w.lds_base = (unsigned)(unsigned long)(__attribute__((address_space(3))) unsigned char*)lds;

    const int tile_id = w.tm * g.tiles_n + w.tn;
    const int64_t num_tiles = tiles;
    const bool wide = !CPLX && !HEAD && g.block_steps > 0;   // complex calls with k-blocking take four real launches

    // The exponents of the tile's rows and columns wait in LDS behind the pipeline stages (rows at
    // ex, columns at ex + TR): the epilogue must not stall on a round trip to memory. The first
    // barrier of the walk publishes them.
    int* ex = reinterpret_cast<int*>(lds + Shape<S, WM, WN, SOLO>::LDS);   // complex: the imaginary planes' set follows at TR + TC
    // They are requested here and written there while the walk's first loads are on their way.
    static_assert(NEX * (TR + TC) <= T, "an exponent to a thread");
    int my_exponent = 0;
    if (!g.P && w.tid < NEX * (TR + TC)) {
        const int plane = w.tid / (TR + TC), i = w.tid % (TR + TC);
        const bool is_a = i < TR;
        const int pos = is_a ? w.tm * TR + i : w.tn * TC + (i - TR);
        const int32_t* E = is_a ? (plane ? g.EA2 : g.EA) : (plane ? g.EB2 : g.EB);
        if (pos < (is_a ? g.m : g.n)) my_exponent = E[pos];
    }

    v4i acc[KB][4];
    auto zero_acc = [&](int nd) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < nd; ++i)
#pragma unroll
            for (int u = 0; u < 16; ++u) acc[i][u >> 2][u & 3] = acc_zero();
    };
    // k-blocking: INT32 sums of the band with lowest diagonal e0 -> INT64 sums in the workspace.
    // Thread t of the workgroup owns element t of every 16 x (diagonal, tile) run: coalesced, and
    // nobody else ever touches it.
    auto flush = [&](int e0, int nd, bool first) __attribute__((always_inline)) {
        // one running pointer (made opaque so that it is formed here, not ahead of the k-walk)
        long long* q = g.D + (((int64_t)e0 * num_tiles + tile_id) * 16) * T + (w.wave * 64 + lane_here());
        const int64_t diag_stride = num_tiles * 16 * T - 16 * T;
        mfma_results_ready();
#pragma unroll
        for (int i = 0; i < KB; ++i) {
            if (i < nd) {
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    const long long v = (long long)acc_read(acc[i][u >> 2][u & 3]);
                    // later blocks add with an atomic that returns nothing: no round trip per element
                    if (first) *q = v;
                    else __hip_atomic_fetch_add(q, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    q += T;
                    __builtin_amdgcn_sched_barrier(0);   // keep register pressure flat
                }
                q += diag_stride;
            }
        }
        // no store of this block may still be in flight when the walk goes back to counting its
        // direct loads (stores and loads share the counter)
        wait_loads<0>();
    };

    // The coordinates are formed where the epilogue needs them, from the lane number read there: kept
    // across the walk they would be spilled, and a reload of a spilled register waits for every memory
    // operation in flight, the direct loads of the next steps included.
    struct Where { int lrow0, lcol, row0, col; };
    auto where = [&]() __attribute__((always_inline)) -> Where {
        const int lane = lane_here();
        Where p;
        p.lrow0 = w.wm * (CPLX ? 16 : 32) + 4 * (lane >> 4);
        p.lcol = w.wn * (CPLX ? 16 : 32) + (lane & 15);
        p.row0 = w.tm * TR + p.lrow0;
        p.col = w.tn * TC + p.lcol;
        return p;
    };

    double sum[16], lo[MODE == kModeDD ? 16 : 1];
    auto clear_sum = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 16; ++u) sum[u] = 0.0;
        if constexpr (MODE == kModeDD) {
#pragma unroll
            for (int u = 0; u < 16; ++u) lo[u] = 0.0;
        }
    };

    // whether the whole tile lies inside C (then the epilogue tests nothing per element); formed where it is used
    auto tile_inside = [&]() __attribute__((always_inline)) -> bool {
        const int z = opaque_scalar_zero();
        return (w.tm + 1 + z) * TR <= g.m && (w.tn + 1 + z) * TC <= g.n;
    };
    // The elements that the combine mode reads are requested before the diagonals are folded, so
    // that they arrive while the fold runs (dependent round trips to memory otherwise); those of
    // Zr (complex interleave of the four-launch form only) in one batch after it, when the fold's registers are free again.
    double old_c[MODE == kModeReal ? 16 : 1], old_zr[MODE == kModeReal ? 16 : 1];
    auto fetch_old = [&](double (&dst)[16], const double* src, bool wanted) __attribute__((always_inline)) {
        if (!wanted) return;   // (then nothing reads them)
        const Where at = where();
        const double* c = src + (int64_t)at.row0 * g.ldc + at.col;
        if (tile_inside()) {
#pragma unroll
            for (int u = 0; u < 16; ++u) dst[u] = c[(int64_t)elem_row(u) * g.ldc + elem_col(u)];
            return;
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const bool in = at.row0 + elem_row(u) < g.m && at.col + elem_col(u) < g.n;
            dst[u] = in ? c[(int64_t)elem_row(u) * g.ldc + elem_col(u)] : 0.0;
        }
    };
    // The sum is complete (in `sum`, or in the INT64 sums of the workspace): scale it,
    // combine it, store what is final.
    auto finish_product = [&]() __attribute__((always_inline)) {
        // Everything this step addresses is formed here, from values made opaque, and not ahead of the
        // walk, where it would occupy registers the matrix-core loop needs.
        const Where at = where();
        const int oz = (int)opaque_zero();
        const int row0 = at.row0, col = at.col, lrow0 = at.lrow0, lcol = at.lcol;
        if (g.P) {   // pair mode (S == 1): the raw INT32 sums
            mfma_results_ready();
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int row = row0 + elem_row(u), c = col + elem_col(u);
                if (row < g.m && c < g.n) g.P[(int64_t)row * g.ldp + c] = acc_read(acc[0][u >> 2][u & 3]);
            }
            return;
        }
        if (wide) {   // the FP64 sum from the INT64 sums, same order
            const long long* q = g.D + ((int64_t)tile_id * 16) * T + (w.wave * 64 + lane_here()) + oz;
            for (int e = S - 1; e >= 0; --e) {
                const double sc = __longlong_as_double((long long)(1023 - OZIMMU_SLICE_BITS * (e + 2)) << 52);
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    // read at the L2, where the atomic adds of the blocks were applied
                    const long long s_e = __hip_atomic_load(q + ((int64_t)e * num_tiles * 16 + u) * T, __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT);
                    const double term = (double)s_e * sc;   // exact: |S_e| < 2^53
                    if constexpr (MODE == kModeDD) dd_add(sum[u], lo[u], term);
                    else sum[u] = sum[u] + term;
                }
            }
        }
        if constexpr (CPLX) {
            // patch (i, j): plane i of A with plane j of B
            const int* const exb = ex + TR + lcol;
            const int eb[2] = {exb[0], exb[TR + TC]};
            const v4i ea[2] = {*reinterpret_cast<const v4i*>(ex + lrow0), *reinterpret_cast<const v4i*>(ex + TR + TC + lrow0)};   // four consecutive rows
            double* z = g.Cz + 2 * ((int64_t)row0 * g.ldcz + col);
            const bool inside = tile_inside();
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                double2 v;
                v.x = ldexp(sum[r], ea[0][r] + eb[0]) - ldexp(sum[12 + r], ea[1][r] + eb[1]);
                v.y = ldexp(sum[4 + r], ea[0][r] + eb[1]) + ldexp(sum[8 + r], ea[1][r] + eb[0]);
                if (inside || (row0 + r < g.m && col < g.n)) *reinterpret_cast<double2*>(z + 2 * (int64_t)r * g.ldcz) = v;
            }
        } else {
            const int* exb = ex + TR + lcol;
            const int eb[2] = {exb[0], exb[16]};
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const v4i ea = *reinterpret_cast<const v4i*>(ex + lrow0 + 16 * i);   // four consecutive rows
#pragma unroll
                for (int u = 8 * i; u < 8 * i + 8; ++u) {
                    const int e = ea[u & 3] + eb[(u >> 2) & 1];
                    sum[u] = ldexp(sum[u], e);
                    if constexpr (MODE == kModeDD) lo[u] = ldexp(lo[u], e);
                }
            }
            // one decision per tile on the combine mode and on whether all of it lies inside C
            const bool inside = tile_inside();
            auto each = [&](auto&& store) __attribute__((always_inline)) {   // store(element, its offset)
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    const int row = row0 + elem_row(u), c = col + elem_col(u);
                    if (inside || (row < g.m && c < g.n)) store(u, (int64_t)elem_row(u));
                }
            };
            double* c0 = g.C + (int64_t)row0 * g.ldc + col;
            if constexpr (MODE == kModeDD) {
                double* l0 = g.C_lo + (int64_t)row0 * g.ldc + col;
                each([&](int u, int64_t dr) __attribute__((always_inline)) {
                    c0[dr * g.ldc + elem_col(u)] = sum[u];
                    l0[dr * g.ldc + elem_col(u)] = lo[u];
                });
            } else {
                if (g.c_mode == 4) {   // last of the four real products of a complex one: (re, im) = (Zr, C + val) -> interleaved Cz
                    fetch_old(old_zr, g.Zr, true);
                    double* z0 = g.Cz + 2 * ((int64_t)row0 * g.ldcz + col);
                    each([&](int u, int64_t dr) __attribute__((always_inline)) {
                        double2 z;
                        z.x = old_zr[u];
                        z.y = old_c[u] + sum[u];
                        *reinterpret_cast<double2*>(z0 + 2 * (dr * g.ldcz + elem_col(u))) = z;
                    });
                    return;
                }
                // (as `combined`, with one decision for all sixteen)
                if (g.c_mode == 1) {
#pragma unroll
                    for (int u = 0; u < 16; ++u) sum[u] = old_c[u] + sum[u];
                } else if (g.c_mode == 2) {
#pragma unroll
                    for (int u = 0; u < 16; ++u) sum[u] = old_c[u] - sum[u];
                } else if (g.c_mode == 3) {
                    if (g.alpha != 1.0) {
#pragma unroll
                        for (int u = 0; u < 16; ++u) sum[u] = g.alpha * sum[u];
                    }
                    if (g.beta != 0.0) {
#pragma unroll
                        for (int u = 0; u < 16; ++u) sum[u] = sum[u] + g.beta * old_c[u];
                    }
                }
                if (inside) {
#pragma unroll
                    for (int u = 0; u < 16; ++u) c0[(int64_t)elem_row(u) * g.ldc + elem_col(u)] = sum[u];
                } else {
                    each([&](int u, int64_t dr) __attribute__((always_inline)) { c0[dr * g.ldc + elem_col(u)] = sum[u]; });
                }
            }
        }
    };

    bool first_block;
    int until_flush;
    // the band's sums into the FP64 sum
    auto fold = [&](auto sb_tag) __attribute__((always_inline)) {
        if (!wide && !g.P) {
            if constexpr (MODE == kModeDD) fold_band_dd<decltype(sb_tag)::value, KB>(sum, lo, acc);
            else fold_band<decltype(sb_tag)::value, KB>(sum, acc);
        }
    };
    auto walk = [&](auto sb_tag, auto&& while_filling) __attribute__((always_inline)) {
        constexpr int SB = decltype(sb_tag)::value;
        using B = Band<SB, KB, WM, WN, SOLO>;
        first_block = true;
        until_flush = g.block_steps;
        band_walk<SB, KB, WM, WN, SOLO, CPLX, HEAD>(acc, g, w, while_filling, [&](int done) __attribute__((always_inline)) {
            // a step adds two slabs: the block is full when it has no room for two more
            if (wide && ((until_flush -= 2) < 2 || done == w.t_end - w.t_begin)) {
                flush(B::E0, B::ND, first_block);
                first_block = false;
                until_flush = g.block_steps;
                zero_acc(B::ND);
            }
        });
        // nothing of the epilogue is to be scheduled up into the last step, where the fragment
        // registers are still in use and there is no room for its values
        __builtin_amdgcn_sched_barrier(0);
    };
    // One of several workgroups on a tile, each with a part of k: the INT32 sums go to the workspace as they are, where
    // fold_kernel adds them up. Thread t owns element t of every run, [split][diagonal][tile][u].
    auto put_partial = [&](auto sb_tag) __attribute__((always_inline)) {
        using B = Band<decltype(sb_tag)::value, KB, WM, WN, SOLO>;
        mfma_results_ready();
        int* q = g.partial + ((((int64_t)split * S + B::E0) * num_tiles + tile_id) * 16) * T + (w.wave * 64 + lane_here());
#pragma unroll
        for (int e = 0; e < B::ND; ++e) {
#pragma unroll
            for (int u = 0; u < 16; ++u) q[u * T] = acc_read(acc[e][u >> 2][u & 3]);
            q += num_tiles * 16 * T;
        }
    };
    walk(std::integral_constant<int, S>{}, [&]() __attribute__((always_inline)) {
        if (w.tid < NEX * (TR + TC)) ex[w.tid] = my_exponent;
        if constexpr (!HEAD) zero_acc(S < KB ? S : KB);
    });
    clear_sum();
    // a band's sums into the FP64 sum, or to where all parts' sums meet
    auto take = [&](auto sb_tag) __attribute__((always_inline)) {
        if (MODE != kModeDD && g.splits > 1) put_partial(sb_tag);
        else fold(sb_tag);
    };
    if constexpr (S > KB) {
        // the first band is taken while the second one's first loads are on their way (before them where the sum takes
        // two registers per part: there is no room for both)
        if constexpr (MODE == kModeDD) take(std::integral_constant<int, S>{});
        walk(std::integral_constant<int, S2>{}, [&]() __attribute__((always_inline)) {
            if constexpr (MODE != kModeDD) take(std::integral_constant<int, S>{});
            if constexpr (!HEAD) zero_acc(S2 < KB ? S2 : KB);
        });
    }
    if (MODE != kModeDD && g.splits > 1) {
        put_partial(std::integral_constant<int, (S > KB ? S2 : S)>{});
        return;
    }
    if constexpr (MODE == kModeReal) fetch_old(old_c, g.C, !g.P && c_mode_reads(g, g.c_mode));
    fold(std::integral_constant<int, (S > KB ? S2 : S)>{});
    finish_product();
}

template <int S, int WM, int WN, int MODE, bool SOLO = false, bool HEAD = false>
hipError_t launch_one(const GemmArgs& g, hipStream_t st) {
    constexpr int lds = Shape<S, WM, WN, SOLO>::LDS + 32 * (WM + WN) * (int)sizeof(int);
    static_assert(lds <= kLdsLimit, "stages and exponents must fit the LDS");
    hipError_t e = allow_dynamic_lds<&product_kernel<S, WM, WN, MODE, SOLO, HEAD>>(lds);
    if (e != hipSuccess) return e;
    product_kernel<S, WM, WN, MODE, SOLO, HEAD><<<dim3((unsigned)(g.tiles_m * g.tiles_n * g.splits)), dim3(64 * WM * WN), lds, st>>>(g);
    return hipGetLastError();
}

// The sums of a product whose tiles were walked by several workgroups each, and everything behind them: one element of C
// (complex: one of the four real products of one) per thread of the first four wavefronts. A workgroup takes 64 of a
// tile's threads and one of their four registers per patch. What takes time here is the way to memory and back (the parts
// come from other XCDs), so sixteen wavefronts share it: wavefront w takes the parts w / 4, w / 4 + 4, ... of patch w % 4,
// four parts at a time in flight, and the four groups meet in LDS.
template <int S, int MODE>
__global__ __launch_bounds__(1024) void fold_kernel(const GemmArgs g, int wn_waves) {
    constexpr bool CPLX = MODE == kModeComplex;
    __shared__ unsigned long long lds_sums[S][256];
    const int T = 128 * wn_waves;                                  // threads of a tile (2 x wn_waves wavefronts)
    const int64_t tiles = (int64_t)g.tiles_m * g.tiles_n;
    const int tile = blockIdx.x, tm = tile / g.tiles_n, tn = tile % g.tiles_n;
    const int r = blockIdx.y & 3, wave = blockIdx.y >> 2;          // register of the patch, wavefront of the tile
    const int tid = threadIdx.x & 255, group = threadIdx.x >> 8;
    const int lane = tid & 63, patch = tid >> 6, i = patch >> 1, j = patch & 1;
    const int u = patch * 4 + r;
    const int* q = g.partial + ((int64_t)tile * 16 + u) * T + wave * 64 + lane;
    const int64_t diag = tiles * 16 * T, split = diag * S;
    long long d[S];
#pragma unroll
    for (int e = 0; e < S; ++e) d[e] = 0;
    constexpr int V = S > 8 ? 2 : 4;
    for (int sp = group; sp < g.splits; sp += 4 * V) {   // V S loads in flight (past the last part the last one again, for nothing)
        int x[V][S];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int part = sp + 4 * v < g.splits ? sp + 4 * v : g.splits - 1;
#pragma unroll
            for (int e = 0; e < S; ++e) x[v][e] = q[part * split + e * diag];
        }
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const bool live = sp + 4 * v < g.splits;
#pragma unroll
            for (int e = 0; e < S; ++e) d[e] += live ? x[v][e] : 0;
        }
    }
    if (group == 0) {
#pragma unroll
        for (int e = 0; e < S; ++e) lds_sums[e][tid] = (unsigned long long)d[e];
    }
    __syncthreads();
    if (group != 0) {
#pragma unroll
        for (int e = 0; e < S; ++e) atomicAdd(&lds_sums[e][tid], (unsigned long long)d[e]);
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < S; ++e) d[e] = (long long)lds_sums[e][tid];
    const int wm = wave / wn_waves, wn = wave % wn_waves;
    const int TR = CPLX ? 32 : 64, TC = (CPLX ? 16 : 32) * wn_waves;
    const int row = tm * TR + wm * (TR / 2) + (CPLX ? 0 : 16 * i) + 4 * (lane >> 4) + r;
    const int col = tn * TC + wn * (CPLX ? 16 : 32) + (CPLX ? 0 : 16 * j) + (lane & 15);
    const bool in = group == 0 && row < g.m && col < g.n;
    int ex = 0;
    if (in) ex = (CPLX && i ? g.EA2 : g.EA)[row] + (CPLX && j ? g.EB2 : g.EB)[col];
    double h = 0.0, l = 0.0;
#pragma unroll
    for (int e = S - 1; e >= 0; --e) {
        // exact: |S_e| < 2^53 and a power of two
        const double term = (double)d[e] * __longlong_as_double((long long)(1023 - OZIMMU_SLICE_BITS * (e + 2)) << 52);
        if constexpr (MODE == kModeDD) dd_add(h, l, term);
        else h = h + term;
    }
    h = ldexp(h, ex);
    if constexpr (CPLX) {
        __shared__ double part[4][64];
        if (group == 0) part[patch][lane] = h;
        __syncthreads();
        if (patch < 2 && in) {   // re = G(Ar,Br) - G(Ai,Bi), im = G(Ar,Bi) + G(Ai,Br)
            const double v = patch == 0 ? part[0][lane] - part[3][lane] : part[1][lane] + part[2][lane];
            g.Cz[2 * ((int64_t)row * g.ldcz + col) + patch] = v;
        }
    } else if (in) {
        double* c = g.C + (int64_t)row * g.ldc + col;
        if constexpr (MODE == kModeDD) {
            *c = h;
            g.C_lo[(int64_t)row * g.ldc + col] = ldexp(l, ex);
        } else if (g.c_mode == 4) {
            double2 z;
            z.x = g.Zr[(int64_t)row * g.ldc + col];
            z.y = *c + h;
            *reinterpret_cast<double2*>(g.Cz + 2 * ((int64_t)row * g.ldcz + col)) = z;
        } else {
            *c = g.c_mode == 0 ? h : combined(g, c_mode_reads(g, g.c_mode) ? *c : 0.0, h);
        }
    }
}

template <int MODE>
hipError_t launch_fold(const GemmArgs& g, int s, hipStream_t st) {
    const int wn_waves = g.tile_cols / 32;
    const dim3 grid((unsigned)(g.tiles_m * g.tiles_n), (unsigned)(4 * 2 * wn_waves));
    switch (s) {
#define OZ_CASE(S_) case S_: fold_kernel<S_, MODE><<<grid, dim3(1024), 0, st>>>(g, wn_waves); return hipGetLastError();
        OZ_CASE(1) OZ_CASE(2) OZ_CASE(3) OZ_CASE(4) OZ_CASE(5) OZ_CASE(6) OZ_CASE(7) OZ_CASE(8)
        OZ_CASE(9) OZ_CASE(10) OZ_CASE(11) OZ_CASE(12) OZ_CASE(13) OZ_CASE(14) OZ_CASE(15) OZ_CASE(16)
#undef OZ_CASE
    }
    return hipErrorInvalidValue;
}

template <int MODE>
hipError_t launch_for(const GemmArgs& g, int s, hipStream_t st) {
    // An odd number of slabs, all of them walked by one workgroup: whatever their number, the half step saved counts (per call,
    // half-empty last step against head: 4044 x 1069 x 72 at nine slices 43 -> 39 us, 4966 x 2346 x 28 at fifteen 163 -> 113, 8192 x 2351 x 82 at eleven 192 -> 168,
    // 5372 x 5100 x 3744 at fourteen 7450 -> 7360). A shared walk has an odd slab in its last part only.
    const bool head = g.block_steps == 0 && g.splits == 1 && ((g.t_end - g.t_begin) & 1);
    if (g.tile_cols == 64 && s <= 9) {   // 64 x 64 tiles, two workgroups per compute unit: not for the double-double sum
        if constexpr (MODE == kModeReal || MODE == kModeComplex) {
            const bool solo = (int64_t)g.tiles_m * g.tiles_n * g.splits <= kComputeUnits;
            switch (s) {
#define OZ_CASE(S_) case S_: return solo ? launch_one<S_, 2, 2, MODE, true>(g, st) : launch_one<S_, 2, 2, MODE>(g, st);
                OZ_CASE(1) OZ_CASE(2) OZ_CASE(3) OZ_CASE(4) OZ_CASE(5) OZ_CASE(6) OZ_CASE(7) OZ_CASE(8)
#undef OZ_CASE
                case 9:
                    return solo ? launch_one<9, 2, 2, MODE, true>(g, st) : head ? launch_one<9, 2, 2, MODE, false, true>(g, st) : launch_one<9, 2, 2, MODE>(g, st);
            }
        }
        return hipErrorInvalidValue;
    }
    switch (s) {
#define OZ_CASE(S_, WN_) case S_: return launch_one<S_, 2, WN_, MODE>(g, st);
        OZ_CASE(1, 4) OZ_CASE(2, 4) OZ_CASE(3, 4) OZ_CASE(4, 4) OZ_CASE(5, 4) OZ_CASE(6, 4) OZ_CASE(7, 4) OZ_CASE(8, 4) OZ_CASE(9, 4)
#undef OZ_CASE
#define OZ_CASE(S_, WN_) case S_: return head ? launch_one<S_, 2, WN_, MODE, false, true>(g, st) : launch_one<S_, 2, WN_, MODE>(g, st);
#define OZ_BOTH(S_) case S_: if (g.tile_cols == 64) return head ? launch_one<S_, 2, 2, MODE, false, true>(g, st) : launch_one<S_, 2, 2, MODE>(g, st); \
                             return head ? launch_one<S_, 2, 4, MODE, false, true>(g, st) : launch_one<S_, 2, 4, MODE>(g, st);
        OZ_CASE(10, 4) OZ_BOTH(11) OZ_BOTH(12) OZ_BOTH(13) OZ_CASE(14, 2) OZ_CASE(15, 2) OZ_CASE(16, 2)
#undef OZ_BOTH
#undef OZ_CASE
    }
    return hipErrorInvalidValue;
}

}  // namespace

// One translation unit per mode instantiates these for its sixteen slice counts.
template <int MODE>
hipError_t launch_product_mode(const GemmArgs& g, int s, hipStream_t st) {
    return launch_for<MODE>(g, s, st);
}
template <int MODE>
hipError_t launch_fold_mode(const GemmArgs& g, int s, hipStream_t st) {
    return launch_fold<MODE>(g, s, st);
}

}  // namespace ozimmu
