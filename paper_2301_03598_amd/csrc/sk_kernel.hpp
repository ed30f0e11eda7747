// Stream-K GEMM kernels for gfx950 (CDNA4): MFMA mainloop, partial-tile
// fixup and the data-parallel / Stream-K / hybrid work walk.
//
// Work decomposition (paper section 4, Algorithm 5): the MAC-loop iterations
// of the Stream-K region (tiles in m->n->k order, k innermost) are split into
// g contiguous ranges whose lengths differ by at most one; each workgroup
// walks its range tile by tile.  A segment that does not start at its tile's
// first iteration stores its accumulators to its own workspace slot and
// raises its flag; the segment that does start there (the owner) adds the
// later contributors' slots in ascending workgroup order, so the summation
// order is fixed and runs are bitwise repeatable, then applies alpha/beta and
// writes the tile.  Tiles outside the Stream-K region are produced whole, in
// data-parallel waves (section 5.2 hybrids; Algorithm 2 when g = tiles).
//
// MAC loop (Algorithm 3): each k-tile of BLK_K is staged from global memory
// into LDS with 16-byte LDS-DMA loads and consumed by MFMA instructions from
// LDS; the loads of later k-tiles overlap the MFMAs of the running one.  LDS
// rows are 128 bytes of one A row (or B column) along k, the 16-byte chunks of
// a row XOR-swizzled by the row index so the MFMA operand reads are free of
// bank conflicts.  An operand that is contiguous along m (or n) keeps that
// layout in LDS and is transposed by its reads.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "sk_internal.h"

namespace sk {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Bit casts go through by-value helpers: applied directly to an element of
// an ext_vector_type lvalue, __builtin_bit_cast reads element 0 of the vector.
__device__ __forceinline__ uint32_t f2u(float f) { return __builtin_bit_cast(uint32_t, f); }
__device__ __forceinline__ float u2f(uint32_t u) { return __builtin_bit_cast(float, u); }
__device__ __forceinline__ uint64_t d2u(double d) { return __builtin_bit_cast(uint64_t, d); }
__device__ __forceinline__ double u2d(uint64_t u) { return __builtin_bit_cast(double, u); }

// Compile-time loop: f(integral_constant<int, 0>), ..., f(<N-1>).  Used
// where accumulator fragments are indexed, so every index is a constant even
// when the body is too large for the loop unroller.
template <class F, int... Is>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, Is...>) {
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

enum class Dt { F64, F16, BF16, F8 };

template <Dt D> struct DtTraits;
template <> struct DtTraits<Dt::F64> {
    static constexpr int E = 8;     // bytes per element
    using Acc = double;
};
template <> struct DtTraits<Dt::F16> {
    static constexpr int E = 2;
    using Acc = float;
};
template <> struct DtTraits<Dt::BF16> {
    static constexpr int E = 2;
    using Acc = float;
};
template <> struct DtTraits<Dt::F8> {
    static constexpr int E = 1;
    using Acc = float;
};

template <Dt D, int BM_, int BN_, bool AKC_, bool BKC_, bool GROUPED_, int NW_ = 4, int NS_ = 0>
struct Cfg {
    static constexpr Dt DT = D;
    static constexpr bool AKC = AKC_, BKC = BKC_, GROUPED = GROUPED_;
    // waves per workgroup, arranged 2 (along m) x NW/2 (along n); each wave
    // instruction of LDS-DMA staging moves 1 KiB, so one round of all waves
    // moves NW KiB
    static constexpr int NW = NW_, THREADS = 64 * NW_;
    static constexpr int WGM = 2, WGN = NW_ / 2;
    static constexpr int DMA_ROUND = 1024 * NW_;
    static_assert(NW_ == 4 || NW_ == 8, "four or eight waves");
    static constexpr int E = DtTraits<D>::E;
    static constexpr int VEC = 16 / E;          // elements per 16-byte load
    static constexpr int BK = 8 * VEC;          // MAC-loop iteration: 128 bytes of k
    static constexpr int BM = BM_, BN = BN_;
    static constexpr int KROW = 128;            // bytes of k per LDS row
    static constexpr int WTM = BM / WGM, WTN = BN / WGN;   // the wave's block of C
    // the 16-bit and FP8 tiles from 128x128 on keep half-tile buffers
    static constexpr bool HALVES = BM >= 128 && D != Dt::F64;
    static constexpr int MT = 16;               // MFMA block edge
    static constexpr int FM = WTM / MT, FN = WTN / MT;
    static constexpr int FRAG_N = 4;            // accumulators per lane of one block
    static constexpr int A_BYTES = BM * KROW, B_BYTES = BN * KROW;
    static constexpr int STAGE = A_BYTES + B_BYTES;
    // LDS k-tile buffers: what the latency of the loads asks for.  The
    // 64x64 tile's four (two workgroups per CU) serve up to two tiles per CU:
    // 256 tiles of 32 k-tiles 19.6 us with two buffers behind a draining
    // barrier, 12.4 with three, 11.5 with four.  With more tiles than
    // that, more resident workgroups hide the latency better: its
    // kernels are also built with two buffers (NS_; 693 tiles of
    // 20 k-tiles 17.2 us against 18.1 with three and 19.0 with four).  FP64
    // 128x128: 4096^3 2141 us with three and the draining barrier, 2064 and
    // 2005 with three and four without it (1896 since the accumulators stay in
    // VGPRs).
    static constexpr int NSTAGE = NS_ ? NS_ : BM == 64 ? (D == Dt::F64 ? 3 : 4) : D == Dt::F64 ? 4 : 2;
    static constexpr int LDS = NSTAGE * STAGE;
    // the eight-wave 256x256 tiles: the two-group MAC loop (mac_loop_pp)
    static constexpr bool PP = NW == 8;
    // bytes of a half-tile buffer (HALVES; in the order A0 A1 B0 B1 of a stage)
    static constexpr int HALF = STAGE / 4;
    static_assert(!HALVES || (NSTAGE == 2 && BM == BN), "two stages of four halves");
    // first row (column) within the tile of a wave's fragment row i (column
    // j).  HALVES: a wave's block is split over the halves of the tile, so that
    // a quarter of its MFMAs needs one half of A and one half of B.
    __device__ static constexpr int frow(int wm, int i) {
        return HALVES ? (i / (FM / 2)) * (BM / 2) + wm * (WTM / 2) + (i % (FM / 2)) * MT : wm * WTM + i * MT;
    }
    __device__ static constexpr int fcol(int wn, int j) {
        return HALVES ? (j / (FN / 2)) * (BN / 2) + wn * (WTN / 2) + (j % (FN / 2)) * MT : wn * WTN + j * MT;
    }
    // peers whose partial fragments are loaded together in the fixup (the
    // 256x256 tiles have no registers for more than one at a time)
    static constexpr int PEER_BATCH = BM >= 256 ? 1 : 4;
    using Acc = typename DtTraits<D>::Acc;
    using Frag = std::conditional_t<D == Dt::F64, f64x4, f32x4>;
    static constexpr int ACC_N = FM * FN * FRAG_N;     // accumulators per thread
    static constexpr int ACC_CHUNKS = ACC_N * (int)sizeof(Acc) / 16;
    static constexpr int SLOT_BYTES = BM * BN * (int)sizeof(Acc);
    static_assert(BM * BN == THREADS * ACC_N && FM >= 1 && FN >= 1, "accumulator split");
};

// LDS byte offset of 16-byte chunk c of row r (KROW-byte rows, XOR
// swizzle).  The LDS serves a 16-byte-per-lane access 16 lanes per cycle
// across 64 banks (256 bytes): 256/KROW consecutive rows share one bank
// row, so the swizzle key is row/(256/KROW).  Then 16 lanes reading the
// same chunk of 16 consecutive rows all hit distinct banks.
__device__ __forceinline__ uint32_t lds_off(uint32_t row, uint32_t chunk) {
    return row * 128u + (((chunk ^ (row >> 1)) & 7u) << 4);
}

// ---------------------------------------------------------------------------
// global -> LDS staging with LDS-DMA loads
// ---------------------------------------------------------------------------
// Wait for this wave's LDS-DMA loads to land: all of them, or all but the
// newest N (vector-memory loads complete in issue order).
__device__ __forceinline__ void wait_dma() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
template <int N>
__device__ __forceinline__ void wait_dma_but() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    // s_waitcnt encoding: vmcnt[3:0] and [15:14], expcnt [6:4] = 7 and
    // lgkmcnt [11:8] = 15 (no wait on those)
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
    asm volatile("" ::: "memory");
}

// ---------------------------------------------------------------------------
// MFMA operand fragments
//
// 16x16 blocks: lane l feeds row (l % 16) of the A block (and column (l % 16)
// of the B block); lane group g = l / 16 holds a part of the k-step's k:
//  16-bit (16x16x32): 8 values, one 16-byte chunk;
//  FP8 (16x16x128): 32 values, chunks g and g + 4 of the k-tile's eight;
//  FP64 (16x16x4): one value per MFMA; a chunk read gives a lane two
//    consecutive k values (2g and 2g + 1 of an 8-k half of the row) consumed
//    by two MFMAs.
// A and B use the same assignment, so every k of the k-tile meets its partner
// exactly once.  (For the 16-bit and FP8 types the 32x32 forms do the same
// work with half the accumulator reads per k but draw more power, see
// mac_loop_pp, and their chains of additions are twice as long.)
// ---------------------------------------------------------------------------
template <class C>
struct Frag {
    static constexpr int CPM = (C::DT == Dt::F8) ? 2 : 1;          // chunks per lane per operand
    static constexpr int NSUB = C::KROW / 64 / CPM;                // k-steps per k-tile
    u32x4 a[C::FM][CPM], b[C::FN][CPM];
};

__device__ __forceinline__ double lo_d(const u32x4 &x) { return u2d((uint64_t)x[0] | ((uint64_t)x[1] << 32)); }
__device__ __forceinline__ double hi_d(const u32x4 &x) { return u2d((uint64_t)x[2] | ((uint64_t)x[3] << 32)); }

// One fragment pair of one 16x16 block, accumulated.  16-bit and FP8 types:
// D = B_frag * A_frag, the transposed block (see the output layout).
template <class C>
__device__ __forceinline__ void mfma16(typename C::Frag &acc, const u32x4 (&a)[Frag<C>::CPM],
                                       const u32x4 (&b)[Frag<C>::CPM]) {
    if constexpr (C::DT == Dt::F64) {
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(lo_d(a[0]), lo_d(b[0]), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(hi_d(a[0]), hi_d(b[0]), acc, 0, 0, 0);
    } else if constexpr (C::DT == Dt::BF16) {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, b[0]),
                                                      __builtin_bit_cast(bf16x8, a[0]), acc, 0, 0, 0);
    } else if constexpr (C::DT == Dt::F16) {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, b[0]),
                                                     __builtin_bit_cast(f16x8, a[0]), acc, 0, 0, 0);
    } else {
        const i32x8 av = __builtin_shufflevector(__builtin_bit_cast(i32x4, a[0]), __builtin_bit_cast(i32x4, a[1]), 0, 1,
                                                 2, 3, 4, 5, 6, 7);
        const i32x8 bv = __builtin_shufflevector(__builtin_bit_cast(i32x4, b[0]), __builtin_bit_cast(i32x4, b[1]), 0, 1,
                                                 2, 3, 4, 5, 6, 7);
        // formats 0/0 = FP8 e4m3 for both operands; zero scale operands select
        // the unscaled instruction: the per-tensor FP32 scales go into alpha
        acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(bv, av, acc, 0, 0, 0, 0, 0, 0);
    }
}

// One k-step of MFMAs.
template <class C>
__device__ __forceinline__ void mfma_step(typename C::Frag (&acc)[C::FM][C::FN], const Frag<C> &f) {
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
        for (int j = 0; j < C::FN; ++j) mfma16<C>(acc[i][j], f.a[i], f.b[j]);
}

// ---------------------------------------------------------------------------
// MAC loop of the eight-wave 256x256 tiles (PP)
//
// Two waves share each SIMD.  Waves 0-3 (wave row 0) and 4-7 (wave row 1) run
// half a phase apart: while one group issues its MFMAs, the other reads its
// next operand fragments from LDS and issues its next global -> LDS loads.
// A k-tile is four phases of a quarter of the wave's MFMAs each; a phase
// needs one half of A (128 rows) and one half of B (128 columns):
//     phase 0: A0 B0    1: A0 B1    2: A1 B0    3: A1 B1
// and reads one half-tile: A0, B1, A1 and, in phase 3, B0 of the next k-tile.
// Half-tiles are numbered in the order they are read and loaded, B0 A0 B1 A1
// of each k-tile: phase c reads half-tile c + 1 and issues the loads of
// half-tile c + 7, into the buffer of half-tile c - 1.  A wave waits, at the
// end of a phase's loads, for all but its newest five half-tiles, so a load
// has five phases (1.25 k-tiles) to land in two k-tile buffers.
//
// Ordering: phase c's memory part runs in interval 2c for group 0, 2c + 1
// for group 1, its MFMAs in the interval after; a workgroup barrier separates
// intervals.  Half-tile c + 1 has landed for every wave by the end of its
// phase c - 1 (interval 2c - 1 at the latest), before any wave reads it in
// phase c.  Half-tile c - 1, overwritten from interval 2c on, was read in
// phase c - 2, and those reads were waited for (by that phase's MFMAs, or for
// B0 after them) in interval 2c - 2 at the latest.
//
// What bounds it, and what it measured (8192^3, B row-major, N(0,1) inputs,
// one machine): the two-buffer loop with one barrier per k-tile that this
// replaces lost a fifth of its time to the fragment reads behind that barrier;
// BF16 881 us, FP8 (four waves) 583.  Here the length of the memory part
// decides: with the edge tests in every load BF16 took 777 us, without them
// (WHOLE) 727 (1511 TFLOP/s), FP8 397 (2768); with the epilogue below 714 and
// 375 (1540 and 2930).  The 16x16 MFMA forms draw less
// power than the 32x32 ones, and power sets the clock: MFMAs alone from
// registers on N(0,1) values 2064 against 1767 TFLOP/s.  On zero inputs the
// same BF16 kernel takes 565 us; its MFMAs and barriers alone, no loads, 500.
// Measured and dropped: two phases of twice the MFMAs (BF16 782 us, FP8 409,
// both with the tests); loads among the MFMAs (+4 %: a load that cannot issue
// stalls the MFMAs behind it); one barrier per phase with the next fragments
// read a phase ahead (the registers spill); four waves of 128x128 (they
// spill).
// ---------------------------------------------------------------------------

// Chunk swizzle of k-row p of a !KC operand part (HR values per k-row): the
// lanes that one LDS cycle serves hit every bank once -- two 16-lane groups'
// transpose reads, whose k-rows lie 8 (16-bit) or 16 (FP8) apart; FP64: 4
// k-rows two apart x 128 bytes.  The swizzled chunk stays inside its k-row.
template <int E, int HR>
__device__ __forceinline__ int kr_swizzle(int p) {
    constexpr int RB = E * HR;
    static_assert(E == 8 ? RB >= 256 : RB == 64 || RB == 128 || RB == 256, "k-row bytes");
    if constexpr (E == 8) return 8 * ((p >> 1) & 1);
    else if constexpr (RB == 256) return 4 * (p & 3) ^ 2 * ((p >> 3) & 1);                 // 16-bit, 128 rows
    else if constexpr (E == 2) return 2 * ((p >> 1) & 1) ^ 4 * ((p >> 3) & 1);             // 16-bit, 64 rows
    else if constexpr (RB == 128) return 2 * ((p >> 1) & 3) ^ ((p >> 4) & 1);              // FP8, 128 rows
    else return ((p >> 2) & 1) ^ 2 * ((p >> 4) & 1);                                       // FP8, 64 rows
}

// The global -> LDS loads of one operand: NH parts (PP: the two halves) of HR
// rows x BK.  The operand is seen as a matrix X with element (r, p) at
// KC ? r*ld + p : p*ld + r.  Each wave instruction moves 1 KiB: lane L's 16
// bytes land at the wave's LDS block + 16 L, so the XOR swizzles are applied
// by choosing which global chunk each lane fetches.
//  KC (rows x k, k contiguous): the block is 8 rows of 128 bytes in the
//    lds_off layout; lane L fetches row L / 8, chunk (L % 8) ^ swizzle(row).
//  !KC (k x rows, rows contiguous): LDS k-row p holds the part's HR values
//    with 16-byte chunk c at slot c ^ swizzle(p); the block is 1024 / (E HR)
//    k-rows.
// Lanes past the edge of the matrix, and every lane of a k-tile past the
// segment's end, get an offset past the resource range and deposit zeros, so
// the count of loads in flight is constant.
template <class C, bool KC, int HR, int NH>
struct OpDma {
    static constexpr int E = C::E, VEC = C::VEC, BK = C::BK, NW = C::NW, KROW = C::KROW;
    static constexpr int NL = HR * KROW / C::DMA_ROUND;    // loads per wave of one part
    static constexpr int LPR = KROW / 16, RPB = 1024 / KROW;
    static constexpr int CPR = HR * E / 16, KR = 1024 / (HR * E);
    static constexpr int STEP = KC ? NW * RPB : NW * KR;   // rows (KC) or k-rows between a wave's loads
    static constexpr uint32_t OOB = 0x80000000u;
    static_assert(BK * E == KROW && KR >= 1 && NL >= 1, "whole rows per 1 KiB block");
    const char *ub;       // the tile's first row at k = 0
    int64_t ustep;        // bytes from one k-tile to the next
    uint32_t ldb;         // bytes between rows (KC) or k-rows (!KC)
    uint32_t voff[2];     // KC: {whole k-tiles, the last, partial one}; !KC: one per part
    // KC: per load, with the rows past the matrix out of range (the 256x256
    // tile has no registers for them: its edge tiles test every load)
    static constexpr bool PER_LOAD = KC && !C::PP;
    uint32_t vrow[PER_LOAD ? NH * NL : 1];
    int pos;              // the lane's row (KC) or k-row within a load
    int rows;             // valid rows from the tile's first one
    int K;
    uint32_t w1024;       // the wave's 1 KiB block of a round

    __device__ __forceinline__ void init(const void *ptr, int64_t ld, int row0, int rows_total, int k, int tid) {
        const int w = __builtin_amdgcn_readfirstlane(tid >> 6), L = tid & 63;
        K = k;
        w1024 = (uint32_t)w * 1024u;
        ldb = (uint32_t)(ld * E);
        rows = rows_total - row0;
        if constexpr (KC) {
            ub = (const char *)ptr + (int64_t)row0 * ld * E;
            ustep = KROW;
            pos = RPB * w + L / LPR;
            const int c = (L % LPR) ^ ((pos >> 1) & 7);
            voff[0] = pos * ldb + c * 16;
            voff[1] = k / BK * BK + c * VEC < k ? voff[0] : OOB;
            if constexpr (PER_LOAD) {
#pragma unroll
                for (int i = 0; i < NH * NL; ++i)
                    vrow[i] = pos < rows - (i / NL * HR + i % NL * STEP) ? voff[0] : OOB;
            }
        } else {
            ub = (const char *)ptr + (int64_t)row0 * E;
            ustep = (int64_t)BK * ld * E;
            pos = w * KR + L / CPR;
            // (the swizzle is the same STEP k-rows on)
            const int c = (L % CPR) ^ kr_swizzle<E, HR>(pos);
#pragma unroll
            for (int h = 0; h < NH; ++h) voff[h] = h * HR + c * VEC < rows ? pos * ldb + (h * HR * E + c * 16) : OOB;
        }
    }

    __device__ __forceinline__ static i32x4 rsrc(uint64_t base) {
        return i32x4{__builtin_amdgcn_readfirstlane((int)(uint32_t)base),
                     __builtin_amdgcn_readfirstlane((int)((uint32_t)(base >> 32) & 0xffffu)), 0x7fffffff, 0x00020000};
    }
    // One 1 KiB load.  Issued as text: the compiler would otherwise wait,
    // before the reads of one buffer, for loads into others (it keeps too few
    // of them apart).  Its hazard handling does not see into the text: a vector
    // instruction that writes rs or so (the readlane of a spilled register) has
    // to lie five wait states ahead of the load, of which the text holds two.
    // The nearest lies ten ahead, and a test of the built library's machine
    // code holds that; the three more in the text (s_nop 3) cost BF16 8192^3 714 ->
    // 721 us, FP64 4096x4096x2048 962 -> 969, FP16 200x136x520 5.0 -> 5.2.
    __device__ __forceinline__ static void dma(const i32x4 &rs, uint32_t dst, uint32_t vo, uint32_t so) {
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // m0 as clobbered: "reserved register"
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :: "s"(__builtin_amdgcn_readfirstlane(dst)), "v"(vo), "s"(rs), "s"(__builtin_amdgcn_readfirstlane(so))
                     : "memory", "m0");
#pragma clang diagnostic pop
    }
    __device__ __forceinline__ uint32_t dst(char *lds, int i) const {
        return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds + i * C::DMA_ROUND + w1024;
    }

    // The wave's loads of part H of k-tile kt into the buffer `lds`.  WHOLE:
    // the k-tile is not the matrix's last, partial one (PP: and the part lies
    // inside the matrix), and `next` is its base address.
    template <int H, bool WHOLE = false>
    __device__ __forceinline__ void issue(char *lds, int kt, bool live, uint64_t next = 0) const {
        const int krem = K - kt * BK;     // > 0 when live
        const i32x4 rs = rsrc(WHOLE ? next : (uint64_t)ub + kt * ustep);
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const uint32_t so = (KC ? H * HR + i * STEP : i * STEP) * ldb;
            uint32_t vo = PER_LOAD && WHOLE ? vrow[H * NL + i] : voff[KC ? 0 : H];
            if constexpr (!WHOLE) {
                // rows (KC) or k-rows of this load that lie inside the matrix
                const int lim = live ? (KC ? rows - (H * HR + i * STEP) : krem - i * STEP) : 0;
                vo = pos < lim ? (KC && krem < BK ? voff[1] : vo) : OOB;
            }
            dma(rs, dst(lds, i), vo, so);
        }
    }
};

// One MFMA operand fragment of k-step ks from an operand part of HR rows whose
// block starts at row0.  !KC: ds_read_b64_tr_b16 hands lane l of a 16-lane
// group element l%4 of the 4-value runs read by lanes 4e + (l%16)/4, e = 0..3,
// ds_read_b64_tr_b8 byte l%8 of the 8-byte runs read by lanes 2e + (l%16)/8,
// e = 0..7, so source lane s16 reads k-row s16/4 (s16/2) of the group's at rows
// 4(s16%4) (8(s16%2)); two reads give the 8 16-bit values, four the 32 FP8 ones.
// FP64: two 8-byte reads, 16 lanes covering 128 bytes of one k-row.
template <class C, bool KC, int HR>
__device__ __forceinline__ void read_frag(u32x4 (&out)[Frag<C>::CPM], const char *op, int row0, int ks, int lane) {
    const int g = lane >> 4, s16 = lane & 15;
    if constexpr (KC) {
#pragma unroll
        for (int s = 0; s < Frag<C>::CPM; ++s)
            out[s] = *(const u32x4 *)(op + lds_off((uint32_t)(row0 + s16), (uint32_t)(ks * 4 + g + 4 * s)));
    } else if constexpr (C::DT == Dt::F64) {
        constexpr int RB = HR * 8;
        const uint32_t r = (uint32_t)(row0 + s16);
        u32x2 h[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int p = 8 * ks + 2 * g + e;
            h[e] = *(const u32x2 *)(op + (uint32_t)p * RB + (((r >> 1) ^ (uint32_t)kr_swizzle<8, HR>(p)) << 4) + (r & 1) * 8);
        }
        out[0] = u32x4{h[0][0], h[0][1], h[1][0], h[1][1]};
    } else if constexpr (C::DT == Dt::F8) {
        typedef int i32x2 __attribute__((ext_vector_type(2)));
        // (adding 8 h or 64 to the k-row leaves its swizzle alone)
        const int r0 = row0 + 8 * (s16 & 1), p0 = 16 * g + (s16 >> 1);
        const char *const src = op + p0 * HR + (((r0 >> 4) ^ kr_swizzle<1, HR>(p0)) << 4) + (r0 & 15);
        uint32_t v[8];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const i32x2 x = __builtin_amdgcn_ds_read_tr8_b64_v2i32(
                (__attribute__((address_space(3))) i32x2 *)(src + (64 * (h >> 1) + 8 * (h & 1)) * HR));
            v[2 * h] = (uint32_t)x[0];
            v[2 * h + 1] = (uint32_t)x[1];
        }
        out[0] = u32x4{v[0], v[1], v[2], v[3]};
        out[1] = u32x4{v[4], v[5], v[6], v[7]};
    } else {
        typedef short s16x4 __attribute__((ext_vector_type(4)));
        const int r0 = row0 + 4 * (s16 & 3), p0 = 8 * g + (s16 >> 2);
        const char *const src = op + p0 * HR * 2 + (((r0 >> 3) ^ kr_swizzle<2, HR>(p0)) << 4) + (r0 & 7) * 2;
        u32x2 v[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            v[h] = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                                 (__attribute__((address_space(3))) s16x4 *)(src + (32 * ks + 4 * h) * HR * 2)));
        }
        out[0] = u32x4{v[0][0], v[0][1], v[1][0], v[1][1]};
    }
}

template <class C>
struct PpState {
    static constexpr int HM = C::BM / 2, HN = C::BN / 2, FMH = C::FM / 2, FNH = C::FN / 2;
    static constexpr int KS = Frag<C>::NSUB, CPM = Frag<C>::CPM;
    OpDma<C, C::AKC, HM, 2> da;
    OpDma<C, C::BKC, HN, 2> db;
    u32x4 a[FMH][KS][CPM], b[2][FNH][KS][CPM];
    static constexpr int NL = 2;      // loads per wave of one half-tile

    __device__ __forceinline__ void read_a(const char *op, int wm, int lane) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int i = 0; i < FMH; ++i)
                read_frag<C, C::AKC, HM>(a[i][ks], op, wm * (C::WTM / 2) + i * C::MT, ks, lane);
    }
    template <int H>
    __device__ __forceinline__ void read_b(const char *op, int wn, int lane) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int j = 0; j < FNH; ++j)
                read_frag<C, C::BKC, HN>(b[H][j][ks], op, wn * (C::WTN / 2) + j * C::MT, ks, lane);
    }
    template <int HA, int HB>
    __device__ __forceinline__ void mfma(typename C::Frag (&acc)[C::FM][C::FN]) const {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int i = 0; i < FMH; ++i)
#pragma unroll
                for (int j = 0; j < FNH; ++j)
                    mfma16<C>(acc[HA * FMH + i][HB * FNH + j], a[i][ks], b[HB][j][ks]);
    }
};

// a workgroup barrier that neither the compiler nor the scheduler moves
// anything across (it waits for nothing by itself)
__device__ __forceinline__ void plain_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
}

// all but the newest N vector-memory loads, and every LDS access, are done
template <int N>
__device__ __forceinline__ void wait_loads_lds() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (0 << 8) | ((N >> 4) << 14));
    asm volatile("" ::: "memory");
}

// Every LDS access, and all but the newest min(n, MAX) * DPK loads,
// are done.
template <int MAX, int DPK>
__device__ __forceinline__ void wait_newer(int n) {
    if constexpr (MAX > 0) {
        if (n >= MAX) {
            wait_loads_lds<MAX * DPK>();
            return;
        }
        wait_newer<MAX - 1, DPK>(n);
    } else {
        wait_loads_lds<0>();
    }
}

// every LDS access of this wave is done
__device__ __forceinline__ void wait_lds() {
    __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));
    asm volatile("" ::: "memory");
}

// k-tile t in stage S.  WHOLE: the next two k-tiles lie inside the segment
// and the matrices, so their loads need no tests (abase, bbase: the addresses
// of k-tiles t + 1 of A and t + 2 of B, advanced)
template <class C, int S, bool WHOLE>
__device__ __forceinline__ void ktile_pp(PpState<C> &st, typename C::Frag (&acc)[C::FM][C::FN], char *lds,
                                         int t, int t1, int wm, int wn, int lane, uint64_t &abase, uint64_t &bbase) {
    char *const A0 = lds + 4 * S * C::HALF, *const A1 = lds + (4 * S + 1) * C::HALF;
    char *const B0 = lds + (4 * S + 2) * C::HALF, *const B1 = lds + (4 * S + 3) * C::HALF;
    char *const A1n = lds + (4 * (1 - S) + 1) * C::HALF;
    const char *const B0n = lds + (4 * (1 - S) + 2) * C::HALF;
    const bool live1 = t + 1 < t1, live2 = t + 2 < t1;
    static_for<4>([&](auto pp) {
        constexpr int p = decltype(pp)::value;
        if constexpr (p == 0) st.read_a(A0, wm, lane);
        else if constexpr (p == 1) st.template read_b<1>(B1, wn, lane);
        else if constexpr (p == 2) st.read_a(A1, wm, lane);
        else st.template read_b<0>(B0n, wn, lane);
        if constexpr (p == 0) {
            st.da.template issue<1, WHOLE>(A1n, t + 1, live1, abase);
            abase += st.da.ustep;
        } else if constexpr (p == 1) {
            st.db.template issue<0, WHOLE>(B0, t + 2, live2, bbase);
        } else if constexpr (p == 2) {
            st.da.template issue<0, WHOLE>(A0, t + 2, live2, abase);
        } else {
            st.db.template issue<1, WHOLE>(B1, t + 2, live2, bbase);
            bbase += st.db.ustep;
        }
        // all but the newest five half-tiles: half-tile 4 t + p + 2 has landed
        wait_dma_but<5 * PpState<C>::NL>();
        plain_barrier();
        __builtin_amdgcn_s_setprio(1);
        st.template mfma<p / 2, p % 2>(acc);
        __builtin_amdgcn_s_setprio(0);
        if constexpr (p == 3) wait_lds();    // B0's reads: no MFMA of this phase has waited for them
        plain_barrier();
    });
}

template <class C>
__device__ __forceinline__ void mac_loop_pp(const Problem &P, int tm, int tn, int it0, int it1,
                                            typename C::Frag (&acc)[C::FM][C::FN], char *lds, int tid) {
    const int lane = tid & 63, wave = tid >> 6;
    const int uw = __builtin_amdgcn_readfirstlane(wave), wm = uw / C::WGN, wn = uw % C::WGN;
    PpState<C> st;
    st.da.init(P.A, P.lda, tm * C::BM, P.m, P.k, tid);
    st.db.init(P.B, P.ldb, tn * C::BN, P.n, P.k, tid);
    static_for<2>([&](auto ss) {
        constexpr int s = decltype(ss)::value;
        const bool live = it0 + s < it1;
        st.db.template issue<0>(lds + (4 * s + 2) * C::HALF, it0 + s, live);
        st.da.template issue<0>(lds + 4 * s * C::HALF, it0 + s, live);
        st.db.template issue<1>(lds + (4 * s + 3) * C::HALF, it0 + s, live);
        if constexpr (s == 0) st.da.template issue<1>(lds + (4 * s + 1) * C::HALF, it0 + s, live);
    });
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
        for (int j = 0; j < C::FN; ++j) acc[i][j] = typename C::Frag{};
    wait_dma_but<5 * PpState<C>::NL>();      // B0 and A0 of the first k-tile
    plain_barrier();
    st.template read_b<0>(lds + 2 * C::HALF, wn, lane);
    wait_lds();
    if (wm == 1) plain_barrier();            // half a phase behind
    int t = it0;
    uint64_t ab = 0, bb = 0;
    if ((tm + 1) * C::BM <= P.m && (tn + 1) * C::BN <= P.n) {
        const int full = P.k / C::BK < it1 ? P.k / C::BK : it1;
        ab = (uint64_t)st.da.ub + (it0 + 1) * st.da.ustep;
        bb = (uint64_t)st.db.ub + (it0 + 2) * st.db.ustep;
        for (; t + 3 < full; t += 2) {
            ktile_pp<C, 0, true>(st, acc, lds, t, it1, wm, wn, lane, ab, bb);
            ktile_pp<C, 1, true>(st, acc, lds, t + 1, it1, wm, wn, lane, ab, bb);
        }
    }
    for (; t < it1; t += 2) {
        ktile_pp<C, 0, false>(st, acc, lds, t, it1, wm, wn, lane, ab, bb);
        if (t + 1 < it1) ktile_pp<C, 1, false>(st, acc, lds, t + 1, it1, wm, wn, lane, ab, bb);
    }
    if (wm == 0) plain_barrier();
    // the loads past the segment's end still write into the buffers, which
    // the epilogue uses next
    wait_dma();
    __syncthreads();
}

// ---------------------------------------------------------------------------
// MAC loop of the four-wave 128x128 tiles of the 16-bit and FP8 types
//
// Two workgroups share a CU, so no wave grouping is needed; what bounds this
// tile is the latency of its loads.  A k-tile is four phases as in
// mac_loop_pp (A0 B0, A0 B1, A1 B0, A1 B1), but a phase's MFMAs find their
// fragments in registers: phase c reads half-tile c of the order B1 A1 A0' B0'
// (' of the next k-tile) for the phases after it, and issues the loads of
// half-tile c + 6 into the buffer of half-tile c - 2.  Every second phase ends
// with the wait for half-tiles c + 1 and c + 2 (all but the four newest) and a
// barrier: the buffers of half-tiles c - 1 and c, which every wave has read by
// then, are the ones loaded in the two phases after it.  The lead is 1 to 1.25
// k-tiles in the two k-tile buffers whose loads ran 0.75 ahead before.
//
// Measured (against one draining barrier per k-tile): FP8 4096x1024x4096 31.4
// -> 23.4 us, 3072^3 54.5 -> 44.5, FP16 3240x1640x5808 107 -> 98.8, BF16
// 256x256x65536 35.8 -> 28.5, 8192^3 on this tile 1098 -> 979 (with the
// epilogue and fixup below the first now takes 19.9, the fourth 26.7).  A barrier in
// every phase (five half-tiles more in flight): 25.4, 45.6, 104, 28.0, 1000;
// raised wave priority around the MFMAs: 8192^3 1426.
// ---------------------------------------------------------------------------
template <class C>
struct HalfState {
    static constexpr int HR = C::BM / 2;                        // rows of a half
    static constexpr int FA = C::FM / 2, FB = C::FN / 2;        // a wave's fragment rows of an A, a B half
    static constexpr int KS = Frag<C>::NSUB, CPM = Frag<C>::CPM;
    static constexpr int NL = OpDma<C, C::AKC, HR, 2>::NL;      // loads per wave of a half-tile
    OpDma<C, C::AKC, HR, 2> da;
    OpDma<C, C::BKC, HR, 2> db;
    u32x4 a[2][FA][KS][CPM], b[2][FB][KS][CPM];

    // the wave's fragments of half H of operand OP (0: A)
    template <int OP, int H>
    __device__ __forceinline__ void read(const char *op, int w, int lane) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int i = 0; i < (OP == 0 ? FA : FB); ++i) {
                if constexpr (OP == 0) read_frag<C, C::AKC, HR>(a[H][i][ks], op, w * (C::WTM / 2) + i * C::MT, ks, lane);
                else read_frag<C, C::BKC, HR>(b[H][i][ks], op, w * (C::WTN / 2) + i * C::MT, ks, lane);
            }
    }
    template <int HA, int HB>
    __device__ __forceinline__ void mfma(typename C::Frag (&acc)[C::FM][C::FN]) const {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int i = 0; i < FA; ++i)
#pragma unroll
                for (int j = 0; j < FB; ++j) mfma16<C>(acc[HA * FA + i][HB * FB + j], a[HA][i][ks], b[HB][j][ks]);
    }
};

template <class C, int S, bool WHOLE>
__device__ __forceinline__ void ktile_half(HalfState<C> &st, typename C::Frag (&acc)[C::FM][C::FN], char *lds, int t,
                                           int t1, int wm, int wn, int lane, uint64_t &abase, uint64_t &bbase) {
    constexpr int H = C::HALF;
    char *const A0 = lds + 4 * S * H, *const A1 = lds + (4 * S + 1) * H;
    char *const B0 = lds + (4 * S + 2) * H, *const B1 = lds + (4 * S + 3) * H;
    const char *const A0n = lds + 4 * (1 - S) * H, *const B0n = lds + (4 * (1 - S) + 2) * H;
    const bool live2 = WHOLE || t + 2 < t1;
    static_for<4>([&](auto pp) {
        constexpr int p = decltype(pp)::value;
        if constexpr (p == 0) {
            st.template read<1, 1>(B1, wn, lane);
            if (live2) st.da.template issue<0, WHOLE>(A0, t + 2, true, abase);
        } else if constexpr (p == 1) {
            st.template read<0, 1>(A1, wm, lane);
            if (live2) st.db.template issue<0, WHOLE>(B0, t + 2, true, bbase);
        } else if constexpr (p == 2) {
            st.template read<0, 0>(A0n, wm, lane);
            if (live2) st.db.template issue<1, WHOLE>(B1, t + 2, true, bbase);
            if constexpr (WHOLE) bbase += st.db.ustep;
        } else {
            st.template read<1, 0>(B0n, wn, lane);
            if (live2) st.da.template issue<1, WHOLE>(A1, t + 2, true, abase);
            if constexpr (WHOLE) abase += st.da.ustep;
        }
        st.template mfma<p / 2, p % 2>(acc);
        if constexpr (p % 2 == 1) {
            // half-tiles 4 t + p + 1 and + 2 have landed; the segment's last is 4 t1 - 3
            if constexpr (WHOLE) wait_loads_lds<4 * HalfState<C>::NL>();
            else wait_newer<4, HalfState<C>::NL>(4 * (t1 - 1 - t) - p - 1);
            plain_barrier();
        }
    });
}

template <class C>
__device__ __forceinline__ void mac_loop_half(const Problem &P, int tm, int tn, int it0, int it1,
                                              typename C::Frag (&acc)[C::FM][C::FN], char *lds, int tid) {
    const int lane = tid & 63;
    const int uw = __builtin_amdgcn_readfirstlane(tid >> 6), wm = uw / C::WGN, wn = uw % C::WGN;
    constexpr int NL = HalfState<C>::NL;
    HalfState<C> st;
    st.da.init(P.A, P.lda, tm * C::BM, P.m, P.k, tid);
    st.db.init(P.B, P.ldb, tn * C::BN, P.n, P.k, tid);
    static_for<2>([&](auto ss) {
        constexpr int s = decltype(ss)::value;
        if (it0 + s < it1) {
            st.da.template issue<0>(lds + 4 * s * C::HALF, it0 + s, true);
            st.db.template issue<0>(lds + (4 * s + 2) * C::HALF, it0 + s, true);
            st.db.template issue<1>(lds + (4 * s + 3) * C::HALF, it0 + s, true);
            st.da.template issue<1>(lds + (4 * s + 1) * C::HALF, it0 + s, true);
        }
    });
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
        for (int j = 0; j < C::FN; ++j) acc[i][j] = typename C::Frag{};
    const bool one = it0 + 1 >= it1;         // a single k-tile: four half-tiles issued, not eight
    wait_newer<6, NL>(one ? 2 : 6);          // A0 and B0 of the first k-tile
    plain_barrier();
    st.template read<0, 0>(lds, wm, lane);
    st.template read<1, 0>(lds + 2 * C::HALF, wn, lane);
    wait_newer<4, NL>(one ? 0 : 4);          // ... read, and its B1 and A1
    plain_barrier();
    int t = it0;
    uint64_t ab = 0, bb = 0;
    const int full = P.k / C::BK < it1 ? P.k / C::BK : it1;    // k-tiles below need no tests
    ab = (uint64_t)st.da.ub + (it0 + 2) * st.da.ustep;
    bb = (uint64_t)st.db.ub + (it0 + 2) * st.db.ustep;
    for (; t + 3 < full; t += 2) {
        ktile_half<C, 0, true>(st, acc, lds, t, it1, wm, wn, lane, ab, bb);
        ktile_half<C, 1, true>(st, acc, lds, t + 1, it1, wm, wn, lane, ab, bb);
    }
    for (; t < it1; t += 2) {
        ktile_half<C, 0, false>(st, acc, lds, t, it1, wm, wn, lane, ab, bb);
        if (t + 1 < it1) ktile_half<C, 1, false>(st, acc, lds, t + 1, it1, wm, wn, lane, ab, bb);
    }
    __syncthreads();      // every wave is done with the buffers, which the epilogue uses next
}

// ---------------------------------------------------------------------------
// The MAC loop of the other tiles over iterations [it0, it1) of one tile
// (Algorithm 3)
//
// NSTAGE k-tile buffers; the loads run LA k-tiles ahead, into the buffer of
// the k-tile before the running one (NSTAGE - 1).  A k-tile's k-steps run
// with their operand fragments double-buffered in registers (the reads of
// step s + 1 overlap the MFMAs of step s); before the last step's MFMAs the
// wave waits for its reads of this k-tile and its loads of the next one, then
// one barrier, so those MFMAs cover the first fragment reads of the next
// k-tile.  The barrier itself waits for nothing: a __syncthreads would wait
// for every load in flight (they write LDS) and undo the lead.
//
// With two buffers that would leave a load half a k-tile to land.  EARLY: the
// loads follow the barrier, behind which the running k-tile's own buffer is
// free, and have a whole one (64x64 tiles, loads in the first step and behind the
// barrier, us: BF16 1023x2552x4008, 640 of 63 k-tiles, 58.3, 52.1; FP16
// 1749x1328x2760, 588 of 44, 39.5, 35.1; 4000x704x1256, 693 of 20, 18.4, 17.9).
// ---------------------------------------------------------------------------
template <class C>
struct RingState {
    OpDma<C, C::AKC, C::BM, 1> da;
    OpDma<C, C::BKC, C::BN, 1> db;
    static constexpr bool EARLY = C::NSTAGE == 2 && Frag<C>::NSUB > 1;
    static constexpr int LA = EARLY ? C::NSTAGE : C::NSTAGE - 1;
    static constexpr int DPK = OpDma<C, C::AKC, C::BM, 1>::NL + OpDma<C, C::BKC, C::BN, 1>::NL;   // loads per wave per k-tile
};

// a wave's fragments of k-step ks of the k-tile at `st`
template <class C>
__device__ __forceinline__ void read_frags(Frag<C> &f, const char *st, int wm, int wn, int ks, int lane) {
#pragma unroll
    for (int i = 0; i < C::FM; ++i) read_frag<C, C::AKC, C::BM>(f.a[i], st, wm * C::WTM + i * C::MT, ks, lane);
#pragma unroll
    for (int j = 0; j < C::FN; ++j) read_frag<C, C::BKC, C::BN>(f.b[j], st + C::A_BYTES, wn * C::WTN + j * C::MT, ks, lane);
}

// One k-tile: operands at cur, the next k-tile at nx, the loads of k-tile
// t + LA into ld.  WHOLE: that one lies inside the segment and the matrices
// (abase, bbase: its addresses, advanced).
template <class C, bool WHOLE>
__device__ __forceinline__ void ktile_ring(const RingState<C> &st, Frag<C> (&f)[2],
                                           typename C::Frag (&acc)[C::FM][C::FN], const char *cur, const char *nx,
                                           char *ld, int t, int t1, int wm, int wn, int lane, uint64_t &abase,
                                           uint64_t &bbase) {
    constexpr int NSUB = Frag<C>::NSUB, LA = RingState<C>::LA;
    constexpr bool EARLY = RingState<C>::EARLY;
    const bool live = WHOLE || t + LA < t1;
    auto loads = [&](int op) {
        if (op == 0) {
            if (live) st.da.template issue<0, WHOLE>(ld, t + LA, true, abase);
            if constexpr (WHOLE) abase += st.da.ustep;
        } else {
            if (live) st.db.template issue<0, WHOLE>(ld + C::A_BYTES, t + LA, true, bbase);
            if constexpr (WHOLE) bbase += st.db.ustep;
        }
    };
    auto landed = [&]() {
        // k-tile t + 1 has landed; up to NSTAGE - 2 newer ones may be in flight
        if constexpr (WHOLE) wait_loads_lds<(C::NSTAGE - 2) * RingState<C>::DPK>();
        else wait_newer<C::NSTAGE - 2, RingState<C>::DPK>(t1 - 2 - t);
        plain_barrier();
    };
    if constexpr (NSUB == 1) {
        loads(0);
        loads(1);
        mfma_step<C>(acc, f[0]);
        landed();
        read_frags<C>(f[0], nx, wm, wn, 0, lane);
    } else {
        static_assert(NSUB % 2 == 0, "fragment double buffer needs an even step count");
        static_for<NSUB>([&](auto kk) {
            constexpr int ks = decltype(kk)::value;
            if constexpr (ks + 1 == NSUB) landed();
            read_frags<C>(f[(ks + 1) & 1], ks + 1 < NSUB ? cur : nx, wm, wn, (ks + 1) % NSUB, lane);
            if constexpr (ks == (EARLY ? NSUB - 1 : 0)) {
                loads(0);
                loads(1);
            }
            mfma_step<C>(acc, f[ks & 1]);
        });
    }
}

template <class C>
__device__ __forceinline__ void mac_loop(const Problem &P, int tm, int tn, int it0, int it1,
                                         typename C::Frag (&acc)[C::FM][C::FN], char *lds, int tid) {
    constexpr int LA = RingState<C>::LA, RING = C::NSTAGE * C::STAGE;
    const int lane = tid & 63, wave = tid >> 6, wm = wave / C::WGN, wn = wave % C::WGN;
    RingState<C> st;
    st.da.init(P.A, P.lda, tm * C::BM, P.m, P.k, tid);
    st.db.init(P.B, P.ldb, tn * C::BN, P.n, P.k, tid);
    const int full = P.k / C::BK < it1 ? P.k / C::BK : it1;    // k-tiles below need no tests
#pragma unroll
    for (int j = 0; j < LA; ++j) {
        if (it0 + j < it1) {
            st.da.template issue<0>(lds + j * C::STAGE, it0 + j, true);
            st.db.template issue<0>(lds + j * C::STAGE + C::A_BYTES, it0 + j, true);
        }
    }
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
        for (int j = 0; j < C::FN; ++j) acc[i][j] = typename C::Frag{};
    wait_newer<LA - 1, RingState<C>::DPK>(it1 - 1 - it0);
    plain_barrier();
    Frag<C> f[2];
    read_frags<C>(f[0], lds, wm, wn, 0, lane);
    int t = it0;
    int cur = 0, nx = C::STAGE % RING, ld = LA * C::STAGE % RING;   // byte offsets of the buffers in turn
    uint64_t ab = (uint64_t)st.da.ub + (it0 + LA) * st.da.ustep, bb = (uint64_t)st.db.ub + (it0 + LA) * st.db.ustep;
    auto turn = [&]() {
        if constexpr (RingState<C>::EARLY) ld = nx;
        else ld = cur;
        cur = nx;
        nx = nx + C::STAGE == RING ? 0 : nx + C::STAGE;
    };
    if constexpr (C::BM >= 128) {
        // NSTAGE k-tiles at a time: every buffer address a constant
        for (; t + C::NSTAGE - 1 + LA < full; t += C::NSTAGE)
            static_for<C::NSTAGE>([&](auto pp) {
                constexpr int p = decltype(pp)::value;
                ktile_ring<C, true>(st, f, acc, lds + p * C::STAGE, lds + (p + 1) % C::NSTAGE * C::STAGE,
                                    lds + (p + LA) % C::NSTAGE * C::STAGE, t + p, it1, wm, wn, lane, ab, bb);
            });
    } else {
        for (; t + LA < full; ++t) {
            ktile_ring<C, true>(st, f, acc, lds + cur, lds + nx, lds + ld, t, it1, wm, wn, lane, ab, bb);
            turn();
        }
    }
    for (; t < it1; ++t) {
        ktile_ring<C, false>(st, f, acc, lds + cur, lds + nx, lds + ld, t, it1, wm, wn, lane, ab, bb);
        turn();
    }
    __syncthreads();      // every wave is done with the buffers, which the epilogue uses next
}

// ---------------------------------------------------------------------------
// accumulator <-> (row, col) and the epilogue
// ---------------------------------------------------------------------------
// Output layout of a fragment.
// f16/bf16/f8: the MFMAs compute D = B_frag * A_frag, the transposed block, so
// lane l holds C row (l % 16) of the block and, in accumulator register e,
// column 4(l / 16) + e: four consecutive columns, stored as one vector.
// 16x16 f64 blocks: D = A_frag * B_frag; lane l holds column (l % 16) and,
// in register r, row 4r + (l / 16).
// round to nearest even, NaNs quieted: the conversion instruction
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
    return __builtin_bit_cast(uint16_t, (__bf16)f);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
    return __builtin_bit_cast(float, (uint32_t)b << 16);
}

template <int CT, class Acc>
__device__ __forceinline__ Acc load_c(const char *p) {
    if constexpr (CT == SK_F64) return (Acc)(*(const double *)p);
    else if constexpr (CT == SK_F32) return (Acc)(*(const float *)p);
    else if constexpr (CT == SK_F16) return (Acc)(float)(*(const _Float16 *)p);
    else return (Acc)bf16_to_f32(*(const uint16_t *)p);
}

template <int CT, class Acc>
__device__ __forceinline__ void put_c(char *p, Acc v) {
    if constexpr (CT == SK_F64) *(double *)p = (double)v;
    else if constexpr (CT == SK_F32) *(float *)p = (float)v;
    else if constexpr (CT == SK_F16) *(_Float16 *)p = (_Float16)(float)v;
    else *(uint16_t *)p = f32_to_bf16_rne((float)v);
}

template <int CT> struct CBytes { static constexpr int v = CT == SK_F64 ? 8 : (CT == SK_F32 ? 4 : 2); };

// Four consecutive elements of C.
template <int CT, class Acc>
__device__ __forceinline__ void load4(const char *p, Acc (&v)[4]) {
    if constexpr (CT == SK_F64) {
        const f64x4 o = *(const f64x4 *)p;
        for (int e = 0; e < 4; ++e) v[e] = (Acc)o[e];
    } else if constexpr (CT == SK_F32) {
        const u32x4 o = *(const u32x4 *)p;
        for (int e = 0; e < 4; ++e) v[e] = (Acc)u2f(o[e]);
    } else {
        const u32x2 o = *(const u32x2 *)p;
        for (int e = 0; e < 4; ++e) {
            const uint16_t h = (uint16_t)(o[e >> 1] >> ((e & 1) * 16));
            v[e] = (Acc)(CT == SK_F16 ? (float)__builtin_bit_cast(_Float16, h) : bf16_to_f32(h));
        }
    }
}

// Four consecutive outputs of one row, alpha*acc (+ beta*C), rounded once.
template <int CT, class Acc>
__device__ __forceinline__ void put4(char *p, const Acc (&v)[4], Acc beta, bool rd) {
    Acc w[4];
    if (rd) {
        Acc o[4];
        load4<CT, Acc>(p, o);
        for (int e = 0; e < 4; ++e) w[e] = v[e] + beta * o[e];
    } else {
        for (int e = 0; e < 4; ++e) w[e] = v[e];
    }
    if constexpr (CT == SK_F64) {
        *(f64x4 *)p = f64x4{(double)w[0], (double)w[1], (double)w[2], (double)w[3]};
    } else if constexpr (CT == SK_F32) {
        *(u32x4 *)p = u32x4{f2u((float)w[0]), f2u((float)w[1]), f2u((float)w[2]), f2u((float)w[3])};
    } else {
        typedef std::conditional_t<CT == SK_F16, _Float16, __bf16> H;
        typedef H h4 __attribute__((ext_vector_type(4)));
        *(h4 *)p = h4{(H)(float)w[0], (H)(float)w[1], (H)(float)w[2], (H)(float)w[3]};
    }
}

// Partial tiles: thread-fragment order, 16-byte chunk v of thread t at
// slot + (v*THREADS + t)*16, so stores and loads are fully coalesced.
template <class C>
struct PartialLayout {
    static constexpr int PER = 16 / (int)sizeof(typename C::Acc);   // accumulators per chunk
    static constexpr int CPF = C::FRAG_N / PER;                      // chunks per fragment
    __device__ static __forceinline__ int64_t off(int i, int j, int s, int tid) {
        return ((int64_t)((i * C::FN + j) * CPF + s) * C::THREADS + tid) * 16;
    }
};

// One fragment of a partial tile, as a whole vector.
// Cache policy of every partial-tile and flag access: device scope (SC1).
// The eight XCDs have separate L2 caches; accesses with device scope are
// coherent across them by themselves, so publishing a partial tile needs
// neither an L2 write-back on the producer side nor an L2 invalidate on the
// owner side (the agent-scope release/acquire fences would issue both, and
// an invalidate per poll evicts the operand tiles of every other workgroup on
// that XCD).
constexpr int CPOL_DEVICE = 16;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t slot_rsrc(const char *slot, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)slot, (short)0, bytes, 0x00020000);
}

template <class C>
__device__ __forceinline__ typename C::Frag load_partial_frag(const char *slot, int i, int j, int tid) {
    using PL = PartialLayout<C>;
    const __amdgpu_buffer_rsrc_t rs = slot_rsrc(slot, C::SLOT_BYTES);
    u32x4 c[PL::CPF];
#pragma unroll
    for (int s = 0; s < PL::CPF; ++s)
        c[s] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (uint32_t)PL::off(i, j, s, tid),
                                                                             0, CPOL_DEVICE));
    if constexpr (PL::CPF == 1) {
        return __builtin_bit_cast(f32x4, c[0]);
    } else {
        return __builtin_shufflevector(__builtin_bit_cast(f64x2, c[0]), __builtin_bit_cast(f64x2, c[1]), 0, 1, 2, 3);
    }
}

// v + the fragment of the partial tiles in slots [p0, p1], added in
// ascending slot order.
template <class C>
__device__ __forceinline__ typename C::Frag add_peers(typename C::Frag v, const char *slots, int p0, int p1,
                                                      int i, int j, int tid) {
    // PEER_BATCH peers' fragments are loaded before they are added (one
    // memory round trip per batch); the additions keep ascending order
    int peer = p0;
    if constexpr (C::PEER_BATCH > 1) {
        for (; peer + C::PEER_BATCH - 1 <= p1; peer += C::PEER_BATCH) {
            typename C::Frag x[C::PEER_BATCH];
#pragma unroll
            for (int u = 0; u < C::PEER_BATCH; ++u)
                x[u] = load_partial_frag<C>(slots + (int64_t)(peer + u) * C::SLOT_BYTES, i, j, tid);
#pragma unroll
            for (int u = 0; u < C::PEER_BATCH; ++u) v = v + x[u];
        }
    }
    for (; peer <= p1; ++peer)
        v = v + load_partial_frag<C>(slots + (int64_t)peer * C::SLOT_BYTES, i, j, tid);
    return v;
}

// The first peer's partial tile is staged through the (then idle) MAC-loop
// LDS buffers by LDS-DMA loads, in FIX_PH phases, so its fragments are read
// with LDS latency instead of one global round trip each.  Each wave stages
// exactly the chunks its own lanes read back (partial chunk v of thread t
// sits at 16 (THREADS v + t) in both places), so a wave only waits for its own
// loads; a barrier after the epilogue keeps the next unit's DMA away.
template <class C>
struct FixStage {
    static constexpr int PH = (C::SLOT_BYTES + C::LDS - 1) / C::LDS == 1 ? 1 : 2;   // phases
    static constexpr int VPH = C::ACC_CHUNKS / PH;                    // chunks per thread per phase
    static constexpr int ROWS_PH = C::FM / PH;                        // fragment rows per phase
    static constexpr int RB = C::DMA_ROUND;                           // bytes of one chunk of every thread
    static_assert(VPH * RB <= C::LDS && C::FM % PH == 0, "fixup staging fits the LDS");

    // stage chunks [ph*VPH, (ph+1)*VPH) of the slot
    __device__ static __forceinline__ void issue(const char *slot, char *lds, int ph, int tid) {
        const __amdgpu_buffer_rsrc_t rs = slot_rsrc(slot, C::SLOT_BYTES);
        const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
        for (int u = 0; u < VPH; ++u) {
            char *const dst = lds + u * RB + w * 1024;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)dst, 16,
                                                     (uint32_t)tid * 16u, (uint32_t)((ph * VPH + u) * RB), 0,
                                                     CPOL_DEVICE);
        }
    }

    // fragment (i, j) of the staged slot
    __device__ static __forceinline__ typename C::Frag frag(char *lds, int i, int j, int tid) {
        using PL = PartialLayout<C>;
        u32x4 c[PL::CPF];
#pragma unroll
        for (int s = 0; s < PL::CPF; ++s) {
            const int u = (i * C::FN + j) * PL::CPF + s - (i / ROWS_PH) * VPH;
            c[s] = *(const u32x4 *)(lds + u * RB + tid * 16);
        }
        if constexpr (PL::CPF == 1) {
            return __builtin_bit_cast(f32x4, c[0]);
        } else {
            return __builtin_shufflevector(__builtin_bit_cast(f64x2, c[0]), __builtin_bit_cast(f64x2, c[1]), 0, 1, 2,
                                           3);
        }
    }
};

// acc + the peers' partial fragments (i, j), ascending slot order; the first
// peer's fragment comes from the LDS staging.  The accumulator copy is made
// opaque where it is used, so the copies of all fragments are not hoisted
// to the start of the epilogue (which exhausts the VGPRs).
template <class C>
__device__ __forceinline__ typename C::Frag fix_frag(const typename C::Frag &a, const char *slots, int p0, int p1,
                                                     char *lds, int i, int j, int tid) {
    typename C::Frag v = a;
    asm volatile("" : "+v"(v));
    if (p0 <= p1) {
        v = v + FixStage<C>::frag(lds, i, j, tid);
        v = add_peers<C>(v, slots, p0 + 1, p1, i, j, tid);
    }
    return v;
}

// Phase boundary of the staged fixup: stage the phase's chunks of the first
// peer (after this wave's reads of the previous phase) and wait for them.
template <class C>
__device__ __forceinline__ void fix_phase(bool staged, const char *slots, int p0, char *lds, int i,
                                          int tid) {
    if (staged && i % FixStage<C>::ROWS_PH == 0) {
        if (i > 0) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        FixStage<C>::issue(slots + (int64_t)p0 * C::SLOT_BYTES, lds, i / FixStage<C>::ROWS_PH, tid);
        wait_dma();
    }
}

// Epilogue of a tile with no partial sums to add: the fragments pass through
// the idle MAC-loop LDS buffers so that C is written in whole rows.  Straight
// from the MFMA layout a store instruction covers 16 rows with 64 bytes each
// (32 with a 16-bit C), a write request per row; after the transpose a wave's
// instruction covers consecutive bytes: 1 KiB (512 with a 16-bit C), or, where
// C's rows are not 16-byte aligned, 64 consecutive elements of one row.  The
// arithmetic per element is that of store_tile_t: alpha * acc, then + beta *
// C, rounded once.  Bands of 2 x 32 rows (32 per wave row) in two LDS regions
// by turns; chunk c of a row lies at c ^ (row % 16), so the 16 rows of a
// fragment write land in distinct banks.  Rows and columns past the edge of C
// are not stored.
//
// One barrier per band: a band's writes follow the barrier of the band before
// it, which every wave passes with its reads of the band before that done.
// The barriers wait for LDS accesses only: a __syncthreads would have each
// band wait for the stores of the one before to reach memory.
//
// The bands are unrolled, in one form each for interior tiles, for edges and
// for old values of C, and in one for rows that are not aligned.  A tile runs
// this once, so its waits and its instructions are latency: a rolled loop over
// the bands that served edges, old values and unaligned rows at once added 2
// us to a tile (172x192x1072 FP8, four 128x128 tiles, 12.3 us; unrolled 8.0).
// Before (__syncthreads around each band, BF16 rounded in integer steps) and
// now, us: FP16 4096x4096x64 (one 256x256 tile per CU) 13.5, 12.1; BF16 17.2,
// 12.2; BF16 8192x8192x128 70.7, 51.6; FP16 128x128 tiles: 2040x3000x520 17.8,
// 15.4, unaligned rows of FP32 (2041x3001x520) 26.4, 22.5; 8192x8191x128
// 125.5, 80.2.
template <class C, int CT>
__device__ __forceinline__ void store_tile_rows(const Problem &P, int tm, int tn,
                                                const typename C::Frag (&acc)[C::FM][C::FN], int tid, char *lds,
                                                bool interior) {
    using Acc = typename C::Acc;
    constexpr int EB = CBytes<CT>::v;
    constexpr int RS = C::BN * 4;                     // LDS row
    constexpr int Q = C::BN / 4;                      // 16-byte chunks per row
    constexpr int BR = 32, FB = BR / C::MT;           // band rows per wave row, in FB fragment rows
    constexpr int NB = C::FM / FB;                    // bands
    constexpr int NCH = C::WGM * BR * Q / C::THREADS; // chunks per thread per band
    constexpr int RPU = C::THREADS / Q;               // rows between a thread's chunks
    constexpr int REGION = C::WGM * BR * RS;
    static_assert(C::WGM == 2 && 2 * REGION <= C::LDS && Q >= 16, "two bands fit the k-tile buffers");
    static_assert(C::THREADS % Q == 0 && BR % RPU == 0 && NCH % 2 == 0, "whole rows per round");
    const int lane = tid & 63, wave = tid >> 6, wm = wave / C::WGN, wn = wave % C::WGN;
    const Acc alpha = (Acc)P.alpha, beta = (Acc)P.beta;
    const bool rd = P.beta != 0.0;
    // (opaque: its multiples are formed here, not kept in registers through
    // the MAC loops)
    int64_t pitch = (int64_t)P.ldc * EB;
    asm volatile("" : "+s"(pitch));
    auto write_band = [&](auto bb, char *reg) {
        constexpr int i = decltype(bb)::value * FB;
#pragma unroll
        for (int fb = 0; fb < FB; ++fb) {
            char *const wr = reg + (wm * BR + fb * C::MT + lane % C::MT) * RS;
#pragma unroll
            for (int j = 0; j < C::FN; ++j) {
                // an opaque copy where it is used, as in fix_frag: the products
                // of all fragments are not formed ahead
                typename C::Frag f = acc[i + fb][j];
                asm volatile("" : "+v"(f));
                f32x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = alpha * f[e];
                *(f32x4 *)(wr + ((C::fcol(wn, j) / 4 + lane / C::MT) ^ (lane % C::MT)) * 16) = v;
            }
        }
    };
    const int br0 = tid / Q;
    auto staged = [&](const char *reg, int u) {
        return *(const f32x4 *)(reg + (br0 + u * RPU) * RS + ((tid % Q) ^ ((br0 + u * RPU) % 16)) * 16);
    };
    if (P.c_vec) {
        // EDGE: rows and chunks past the edge are left out; RD: C's old
        // values, loaded ahead of the barrier
        auto bands = [&](auto edge, auto read) {
            constexpr bool EDGE = decltype(edge)::value, RD = decltype(read)::value;
            const int row0 = tm * C::BM + br0, col = tn * C::BN + 4 * (tid % Q);
            const int rows = !EDGE ? 0 : col + 4 <= P.n ? P.m - row0 : 0;
            char *const q = (char *)P.C + row0 * pitch + (int64_t)col * EB;
            static_for<NB>([&](auto bb) {
                constexpr int band = decltype(bb)::value;
                char *const reg = lds + (band & 1) * REGION;
                auto row = [](int u) { return C::frow(u / (NCH / 2), band * FB) + u % (NCH / 2) * RPU; };
                Acc old[NCH][4];
                if constexpr (RD) {
#pragma unroll
                    for (int u = 0; u < NCH; ++u)
                        if (!EDGE || row(u) < rows) load4<CT, Acc>(q + row(u) * pitch, old[u]);
                }
                write_band(bb, reg);
                wait_lds();
                plain_barrier();
#pragma unroll
                for (int u = 0; u < NCH; ++u) {
                    const f32x4 v = staged(reg, u);
                    Acc w[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[e] = RD ? v[e] + beta * old[u][e] : v[e];
                    if (!EDGE || row(u) < rows) put4<CT, Acc>(q + row(u) * pitch, w, beta, false);
                }
                if (EDGE && P.n % 4 != 0 && tn * C::BN + C::BN > P.n && col < P.n && col + 4 > P.n) {
                    // the last chunk of a row that ends inside it
#pragma unroll 1
                    for (int u = 0; u < NCH; ++u) {
                        const int r = C::frow(u / (NCH / 2), band * FB) + u % (NCH / 2) * RPU;
                        for (int e = 0; row0 + r < P.m && col + e < P.n; ++e) {
                            const int rr = br0 + u * RPU;
                            const Acc v = *(const float *)(reg + rr * RS + ((tid % Q) ^ (rr % 16)) * 16 + e * 4);
                            char *const qe = q + r * pitch + e * EB;
                            put_c<CT, Acc>(qe, RD ? v + beta * load_c<CT, Acc>(qe) : v);
                        }
                    }
                }
            });
        };
        using Yes = std::integral_constant<bool, true>;
        using No = std::integral_constant<bool, false>;
        if (rd) bands(Yes{}, Yes{});
        else if (interior) bands(No{}, No{});
        else bands(Yes{}, No{});
        wait_lds();
        plain_barrier();                              // LDS free for the next unit's loads
        return;
    }
    // one element per lane: a thread's column stays, a wave's elements lie in
    // one row
    constexpr int RPE = C::THREADS / C::BN, NE = C::WGM * BR / RPE;
    static_assert(C::THREADS % C::BN == 0 && C::BN % 64 == 0 && 16 % RPE == 0, "rows per round");
    const int er = __builtin_amdgcn_readfirstlane(tid / C::BN), e = tid % C::BN;
    const int row0 = tm * C::BM + er, col = tn * C::BN + e;
    const int rows = P.m - row0;
    char *const q = (char *)P.C + row0 * pitch + (int64_t)col * EB;
    static_for<NB>([&](auto bb) {
        constexpr int band = decltype(bb)::value;
        char *const reg = lds + (band & 1) * REGION;
        auto row = [](int u) { return C::frow(u / (NE / 2), band * FB) + u % (NE / 2) * RPE; };
        Acc old[NE];
        if (rd && col < P.n) {
#pragma unroll
            for (int u = 0; u < NE; ++u)
                if (row(u) < rows) old[u] = load_c<CT, Acc>(q + row(u) * pitch);
        }
        write_band(bb, reg);
        wait_lds();
        plain_barrier();
        if (col < P.n) {
#pragma unroll
            for (int u = 0; u < NE; ++u) {
                const int br = er + u * RPE;
                Acc w = *(const float *)(reg + br * RS + ((e / 4) ^ (br % 16)) * 16 + e % 4 * 4);
                if (rd) w = w + beta * old[u];
                if (row(u) < rows) put_c<CT, Acc>(q + row(u) * pitch, w);
            }
        }
    });
    wait_lds();
    plain_barrier();                                  // LDS free for the next unit's loads
}

// C_tile = alpha * (acc + partials of slots [p0, p1]) + beta * C_tile (C read
// only when beta != 0), rounded once to the output type.  The accumulators
// are only read here: each fragment is copied, completed with the peers'
// partial sums and stored, one fragment at a time.  Interior tiles of a C
// whose rows are 16-byte aligned use 4-wide vector accesses; edge tiles test
// every element.
template <class C, int CT>
__device__ __forceinline__ void store_tile_t(const Problem &P, int tm, int tn,
                                             const typename C::Frag (&acc)[C::FM][C::FN], int tid,
                                             const char *slots, int p0, int p1, char *lds) {
    using Acc = typename C::Acc;
    constexpr int EB = CBytes<CT>::v;
    const int lane = tid & 63, wave = tid >> 6, wm = wave / C::WGN, wn = wave % C::WGN;
    const Acc alpha = (Acc)P.alpha, beta = (Acc)P.beta;
    const bool rd = P.beta != 0.0;
    const bool interior = (tm + 1) * C::BM <= P.m && (tn + 1) * C::BN <= P.n;
    const bool fast = P.c_vec && interior;
    if constexpr (C::DT == Dt::F64) {
        // f64: one element per store; a lane group of 16 writes 128
        // consecutive bytes of one row
        const int r0 = tm * C::BM + wm * C::WTM + (lane >> 4);
        const int c0 = tn * C::BN + wn * C::WTN + (lane & 15);
        const bool staged = p0 <= p1;
        static_for<C::FM * C::FN>([&](auto ij) {
            constexpr int i = decltype(ij)::value / C::FN, j = decltype(ij)::value % C::FN;
            if constexpr (j == 0) fix_phase<C>(staged, slots, p0, lds, i, tid);
            const typename C::Frag v = fix_frag<C>(acc[i][j], slots, p0, p1, lds, i, j, tid);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = r0 + i * 16 + 4 * r, col = c0 + j * 16;
                if (interior || (row < P.m && col < P.n)) {
                    char *q = (char *)P.C + ((int64_t)row * P.ldc + col) * EB;
                    Acc w = alpha * v[r];
                    if (rd) w = w + beta * load_c<CT, Acc>(q);
                    put_c<CT, Acc>(q, w);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        return;
    }
    // whole rows through the LDS, edge tiles included (the flags are uniform
    // over the workgroup); not on the 64x64 tile, where it measures even with
    // aligned rows and 5 % slower without
    if (C::BM >= 128 && p0 > p1) {
        store_tile_rows<C, CT>(P, tm, tn, acc, tid, lds, interior);
        return;
    }
    const int rowl = tm * C::BM + C::frow(wm, 0) + (lane % C::MT);
    const int coll = tn * C::BN + C::fcol(wn, 0) + 4 * (lane / C::MT);
    const bool staged = p0 <= p1;
    static_for<C::FM * C::FN>([&](auto ij) {
        constexpr int i = decltype(ij)::value / C::FN, j = decltype(ij)::value % C::FN;
        if constexpr (j == 0) fix_phase<C>(staged, slots, p0, lds, i, tid);
        const int row = rowl + C::frow(0, i);
        char *rp = (char *)P.C + ((int64_t)row * P.ldc + coll) * EB;
        const typename C::Frag f = fix_frag<C>(acc[i][j], slots, p0, p1, lds, i, j, tid);
        constexpr int co = C::fcol(0, j);                 // column offset from coll
        Acc v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = alpha * f[e];
        if (fast) {
            put4<CT, Acc>(rp + co * EB, v, beta, rd);
        } else if (row < P.m) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (coll + co + e < P.n) {
                    char *q = rp + (co + e) * EB;
                    Acc w = v[e];
                    if (rd) w = w + beta * load_c<CT, Acc>(q);
                    put_c<CT, Acc>(q, w);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    });
}

template <class C>
__device__ __forceinline__ void store_tile(const Problem &P, int tm, int tn,
                                           const typename C::Frag (&acc)[C::FM][C::FN], int tid,
                                           const char *slots, int p0, int p1, char *lds) {
    if constexpr (C::DT == Dt::F64) {
        store_tile_t<C, SK_F64>(P, tm, tn, acc, tid, slots, p0, p1, lds);
    } else {
        // the two output types an input type allows
        constexpr int CH = C::DT == Dt::F16 ? SK_F16 : SK_BF16;
        if (P.c_type == SK_F32) store_tile_t<C, SK_F32>(P, tm, tn, acc, tid, slots, p0, p1, lds);
        else store_tile_t<C, CH>(P, tm, tn, acc, tid, slots, p0, p1, lds);
    }
    // the staged fixup used this wave's LDS regions: keep the next unit's
    // loads out until every wave is done with them
    if (p0 <= p1) __syncthreads();
}

template <class C>
__device__ __forceinline__ void store_partial(char *slot, const typename C::Frag (&acc)[C::FM][C::FN], int tid) {
    using PL = PartialLayout<C>;
    const __amdgpu_buffer_rsrc_t rs = slot_rsrc(slot, C::SLOT_BYTES);
    static_for<C::FM * C::FN>([&](auto ij) {
        constexpr int i = decltype(ij)::value / C::FN, j = decltype(ij)::value % C::FN;
        {
#pragma unroll
            for (int s = 0; s < PL::CPF; ++s) {
                u32x4 w;
                if constexpr (PL::PER == 4) {
                    w[0] = f2u(acc[i][j][4 * s + 0]);
                    w[1] = f2u(acc[i][j][4 * s + 1]);
                    w[2] = f2u(acc[i][j][4 * s + 2]);
                    w[3] = f2u(acc[i][j][4 * s + 3]);
                } else {
                    const uint64_t x0 = d2u(acc[i][j][2 * s + 0]);
                    const uint64_t x1 = d2u(acc[i][j][2 * s + 1]);
                    w[0] = (uint32_t)x0; w[1] = (uint32_t)(x0 >> 32);
                    w[2] = (uint32_t)x1; w[3] = (uint32_t)(x1 >> 32);
                }
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, w), rs, (uint32_t)PL::off(i, j, s, tid),
                                                       0, CPOL_DEVICE);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    });
}

// ---------------------------------------------------------------------------
// flags.  Partial tiles and flags are all device-coherent accesses (SC1):
// the producer waits until its partial stores have completed, then one
// thread raises the flag by storing the call's epoch; a waiter polls the
// flags it needs (one lane per flag) and issues its partial loads only after
// it has seen all of them.  Program order plus completion waits order the
// accesses; no cache-wide fence is needed.  A flag is never cleared: a value
// other than this call's epoch (an earlier call's, or zero) means "not yet".
// ---------------------------------------------------------------------------
__device__ __forceinline__ void signal_flag(int32_t *flag, int32_t epoch, int tid) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's partial stores are done
    __syncthreads();
    if (tid == 0) __hip_atomic_store(flag, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Wait until the flags of contributors first..last other than `self` (at
// most MAX_PEERS of them, one per lane of wave 0) all hold `epoch`.
// Contributor c's flag is flags[c], except that contributor `first` uses
// flags[first_flag].  The other waves wait at the barrier.  Bounded in real
// time: once `ticks` of the constant-rate counter have passed (at once if
// ticks <= 0) the error word is set and the wait ends; the partial tiles of a
// contributor that has not arrived are then stale and the call reports
// SK_ERR_TIMEOUT.
__device__ __forceinline__ void wait_flags(const int32_t *flags, int first, int last, int self, int first_flag,
                                           int32_t epoch, int32_t *err, int64_t ticks, int tid) {
    if (tid < 64) {
        const int c = first + tid + (first + tid >= self && self >= first ? 1 : 0);
        const bool mine = c <= last;
        const int fi = c == first ? first_flag : c;
        const int32_t *f = flags + (int64_t)(mine ? fi : first_flag) * FLAG_STRIDE;
        bool seen = !mine;
        const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
        if (ticks > 0) {
            while (true) {
                if (!seen) seen = __hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == epoch;
                if (__all(seen)) break;
                if ((int64_t)(__builtin_amdgcn_s_memrealtime() - t0) > ticks) {
                    seen = false;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        // bounded: give up, report, never hang
        if (!__all(seen) && tid == 0) __hip_atomic_fetch_or(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // the workgroup barrier (with its compiler-level ordering) keeps every
    // wave's partial loads behind the observed flags
    __syncthreads();
}

__device__ __forceinline__ void trace_rec(const Params &p, int wg, int seq, int tile, int k0, int k1,
                                          int role, int last, int extra, int tid) {
    if (p.trace != nullptr && tid == 0) {
        int idx = __hip_atomic_fetch_add(p.trace, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (idx < p.trace_cap) {
            int32_t *rec = p.trace + 8 + (int64_t)idx * 8;
            rec[0] = wg; rec[1] = seq; rec[2] = tile; rec[3] = k0;
            rec[4] = k1; rec[5] = role; rec[6] = last; rec[7] = extra;
        }
    }
}

// ---------------------------------------------------------------------------
// Distributed fixup: every contributor of a split tile stores its partial
// tile, and contributor f + i of the s = l - f + 1 contributors f..l reduces
// chunks [i N / s, (i + 1) N / s) of the tile's N 16-byte partial chunks over
// all s partials, in ascending workgroup order -- the same additions, in the
// same order, as the owner's serial fixup, so both give identical bits --
// then applies alpha / beta and writes those elements of C.  The slices of a
// pass are staged into the (idle) MAC-loop LDS buffers with LDS-DMA loads,
// all contributors' chunks at once, so the reads of one slice take one
// memory round trip instead of one per contributor.
// ---------------------------------------------------------------------------
template <class C>
struct Spread {
    static constexpr int N = C::SLOT_BYTES / 16;                 // chunks per tile
    static constexpr int LDS_CHUNKS = C::LDS / 16;  // staging capacity

    // Elements of chunk c (16 bytes of the thread-fragment order) of tile
    // (tm, tn): alpha * v (+ beta * C), rounded once, masked at the edges.
    template <int CT>
    __device__ static __forceinline__ void put_chunk(const Problem &P, int tm, int tn, int c, const u32x4 &raw) {
        using Acc = typename C::Acc;
        using PL = PartialLayout<C>;
        constexpr int EB = CBytes<CT>::v;
        const int t = c % C::THREADS, vi = c / C::THREADS;
        const int sc = vi % PL::CPF, fij = vi / PL::CPF, fi = fij / C::FN, fj = fij % C::FN;
        const int lane = t & 63, wave = t >> 6, wm = wave / C::WGN, wn = wave % C::WGN;
        const Acc alpha = (Acc)P.alpha, beta = (Acc)P.beta;
        const bool rd = P.beta != 0.0;
        if constexpr (C::DT == Dt::F64) {
            // FP64: the chunk holds rows 4(2 sc) + lane/16 and 4(2 sc + 1) + lane/16 of one column
            const f64x2 v = __builtin_bit_cast(f64x2, raw);
            const int col = tn * C::BN + wn * C::WTN + fj * 16 + (lane & 15);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int row = tm * C::BM + wm * C::WTM + fi * 16 + 4 * (2 * sc + e) + (lane >> 4);
                if (row < P.m && col < P.n) {
                    char *q = (char *)P.C + ((int64_t)row * P.ldc + col) * EB;
                    Acc w = alpha * v[e];
                    if (rd) w = w + beta * load_c<CT, Acc>(q);
                    put_c<CT, Acc>(q, w);
                }
            }
        } else {
            // four consecutive columns of one row
            const f32x4 v = __builtin_bit_cast(f32x4, raw);
            const int row = tm * C::BM + C::frow(wm, fi) + (lane % C::MT);
            const int col = tn * C::BN + C::fcol(wn, fj) + 4 * (lane / C::MT);
            char *rp = (char *)P.C + ((int64_t)row * P.ldc + col) * EB;
            Acc a[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) a[e] = alpha * v[e];
            const bool interior = (tm + 1) * C::BM <= P.m && (tn + 1) * C::BN <= P.n;
            if (P.c_vec && interior) {
                put4<CT, Acc>(rp, a, beta, rd);
            } else if (row < P.m) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (col + e < P.n) {
                        char *q = rp + e * EB;
                        Acc w = a[e];
                        if (rd) w = w + beta * load_c<CT, Acc>(q);
                        put_c<CT, Acc>(q, w);
                    }
                }
            }
        }
    }

    // Element e of chunk c (16 bytes of the thread-fragment order) of tile
    // (tm, tn): alpha * v (+ beta * C), rounded once, masked at the edges.
    template <int CT>
    __device__ static __forceinline__ void put_elem(const Problem &P, int tm, int tn, int c, int e,
                                                    typename C::Acc v) {
        using Acc = typename C::Acc;
        using PL = PartialLayout<C>;
        constexpr int EB = CBytes<CT>::v;
        const int t = c % C::THREADS, vi = c / C::THREADS;
        const int sc = vi % PL::CPF, fij = vi / PL::CPF, fi = fij / C::FN, fj = fij % C::FN;
        const int lane = t & 63, wave = t >> 6, wm = wave / C::WGN, wn = wave % C::WGN;
        int row, col;
        if constexpr (C::DT == Dt::F64) {
            // FP64: the chunk holds rows 4(2 sc) + lane/16 and 4(2 sc + 1) + lane/16 of one column
            row = tm * C::BM + wm * C::WTM + fi * 16 + 4 * (2 * sc + e) + (lane >> 4);
            col = tn * C::BN + wn * C::WTN + fj * 16 + (lane & 15);
        } else {
            // four consecutive columns of one row
            row = tm * C::BM + C::frow(wm, fi) + (lane % C::MT);
            col = tn * C::BN + C::fcol(wn, fj) + 4 * (lane / C::MT) + e;
        }
        if (row < P.m && col < P.n) {
            char *q = (char *)P.C + ((int64_t)row * P.ldc + col) * EB;
            Acc w = (Acc)P.alpha * v;
            if (P.beta != 0.0) w = w + (Acc)P.beta * load_c<CT, Acc>(q);
            put_c<CT, Acc>(q, w);
        }
    }

    template <int CT>
    __device__ static __forceinline__ void reduce_t(const Params &p, const Problem &P, int tm, int tn, int f,
                                                    int l, int x, char *lds, int tid) {
        const int s = l - f + 1, i = x - f;
        const int c0 = (int)((int64_t)N * i / s), c1 = (int)((int64_t)N * (i + 1) / s);
        // chunks per pass: no more than a slice has, and all s contributors'
        // copies of them fit the LDS
        const int pc = LDS_CHUNKS / s < (N + s - 1) / s ? LDS_CHUNKS / s : (N + s - 1) / s;
        const uint32_t region = (uint32_t)(2 * p.g) * (uint32_t)C::SLOT_BYTES;
        const __amdgpu_buffer_rsrc_t rs = slot_rsrc((const char *)p.partials, (int)region);
        const int w = __builtin_amdgcn_readfirstlane(tid >> 6), L = tid & 63;
        for (int cp = c0; cp < c1; cp += pc) {
            const int n = c1 - cp < pc ? c1 - cp : pc;         // chunks this pass
            const int nblk = (s * pc + 63) / 64;              // 1 KiB staging blocks
            __syncthreads();                                   // LDS free (MAC loop / previous pass)
            for (int b = w; b < nblk; b += C::NW) {
                const int k = b * 64 + L;                      // staging index: contributor k / pc, chunk k % pc
                const int cc = k / pc, j = k % pc;
                const int slot = cc == 0 ? p.g + f : f + cc;   // the owner's is its last-segment slot
                const bool ok = cc < s && j < n;
                const uint32_t off = ok ? (uint32_t)slot * (uint32_t)C::SLOT_BYTES + (uint32_t)(cp + j) * 16u
                                        : 0x80000000u;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(lds + b * 1024),
                                                         16, off, 0, 0, CPOL_DEVICE);
            }
            wait_dma();
            __syncthreads();
            using Acc = typename C::Acc;
            constexpr int EPC = 16 / (int)sizeof(Acc);
            if (n >= C::THREADS) {
                // enough chunks for every thread: one 16-byte chunk per
                // thread, vector reads and stores
                for (int j = tid; j < n; j += C::THREADS) {
                    u32x4 raw;
                    if constexpr (sizeof(Acc) == 4) {
                        f32x4 v = *(const f32x4 *)(lds + j * 16);
                        for (int cc = 1; cc < s; ++cc) {
                            const int k = cc * pc + j;
                            v = v + *(const f32x4 *)(lds + k * 16);
                        }
                        raw = __builtin_bit_cast(u32x4, v);
                    } else {
                        f64x2 v = *(const f64x2 *)(lds + j * 16);
                        for (int cc = 1; cc < s; ++cc) {
                            const int k = cc * pc + j;
                            v = v + *(const f64x2 *)(lds + k * 16);
                        }
                        raw = __builtin_bit_cast(u32x4, v);
                    }
                    put_chunk<CT>(P, tm, tn, cp + j, raw);
                }
                continue;
            }
            // a short slice over many contributors: one element per thread
            // (the order of additions is per element, so the elements of a
            // chunk need not share a thread), the contributors' values read
            // eight at a time ahead of their additions, which stay in
            // ascending order
            for (int u = tid; u < n * EPC; u += C::THREADS) {
                const int j = u / EPC, e = u % EPC;
                auto at = [&](int cc) -> Acc {
                    const int k = cc * pc + j;
                    return *(const Acc *)(lds + k * 16 + e * (int)sizeof(Acc));
                };
                Acc v = at(0);
                int cc = 1;
                for (; cc + 8 <= s; cc += 8) {
                    Acc t[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) t[i] = at(cc + i);
#pragma unroll
                    for (int i = 0; i < 8; ++i) v = v + t[i];
                }
                for (; cc < s; ++cc) v = v + at(cc);
                put_elem<CT>(P, tm, tn, cp + j, e, v);
            }
        }
        __syncthreads();                                       // LDS free for the next user
    }

    __device__ static __forceinline__ void reduce(const Params &p, const Problem &P, int tm, int tn, int f, int l,
                                                  int x, char *lds, int tid) {
        if constexpr (C::DT == Dt::F64) {
            reduce_t<SK_F64>(p, P, tm, tn, f, l, x, lds, tid);
        } else {
            constexpr int CH = C::DT == Dt::F16 ? SK_F16 : SK_BF16;
            if (P.c_type == SK_F32) reduce_t<SK_F32>(p, P, tm, tn, f, l, x, lds, tid);
            else reduce_t<CH>(p, P, tm, tn, f, l, x, lds, tid);
        }
    }
};

// ---------------------------------------------------------------------------
// tile lookup
// ---------------------------------------------------------------------------

// Output coordinates of a problem's tile t.  The iteration space is linearised
// tile by tile (m->n->k, section 4); the tile-to-coordinate map is a banded
// raster: bands of `band` tile rows, each walked column by column, so that a
// run of consecutive tiles covers a compact block of C and shares A and B
// panels in cache.  band == 1 is the plain row-major order.
__device__ __forceinline__ void tile_coords(const Problem &P, int t, int band, int &tm, int &tn) {
    if (band <= 1) {
        tm = t / P.tiles_n;
        tn = t % P.tiles_n;
        return;
    }
    const int per = band * P.tiles_n;
    const int m0 = (t / per) * band, r = t % per;
    const int rows = P.tiles_m - m0 < band ? P.tiles_m - m0 : band;
    tm = m0 + r % rows;
    tn = r / rows;
}

// Every field of a unit's problem is the same in all lanes; reading it through
// readfirstlane states that, so buffer resources and loop bounds derived from
// it live in scalar registers (a resource the compiler must assume divergent
// costs a readfirstlane loop around every buffer load).
__device__ __forceinline__ Problem uniform_problem(const Problem &src) {
    static_assert(sizeof(Problem) % 4 == 0, "word copy");
    uint32_t w[sizeof(Problem) / 4];
    __builtin_memcpy(w, &src, sizeof(Problem));
#pragma unroll
    for (int i = 0; i < (int)(sizeof(Problem) / 4); ++i) w[i] = __builtin_amdgcn_readfirstlane(w[i]);
    Problem out;
    __builtin_memcpy(&out, w, sizeof(Problem));
    return out;
}
__device__ __forceinline__ int uniform_int(int v) { return __builtin_amdgcn_readfirstlane(v); }

struct TileRef {
    const Problem *P;
    int tile_local;     // tile index within its problem
    int it_begin;       // global iteration of the tile's first MAC iteration
};

template <bool GROUPED>
__device__ __forceinline__ TileRef tile_of_tile(const Params &p, int tile) {
    if constexpr (!GROUPED) {
        return TileRef{&p.prob, tile, tile * p.prob.iters};
    } else {
        const int32_t *tp = p.group.tile_prefix;
        int lo = 0, hi = p.group.count;
        while (hi - lo > 1) {
            int mid = (lo + hi) >> 1;
            if (tp[mid] <= tile) lo = mid; else hi = mid;
        }
        const Problem *P = p.group.probs + lo;
        int local = tile - tp[lo];
        return TileRef{P, local, p.group.iter_prefix[lo] + local * P->iters};
    }
}

template <bool GROUPED>
__device__ __forceinline__ int tile_of_iter(const Params &p, int it) {
    if constexpr (!GROUPED) {
        return it / p.prob.iters;
    } else {
        const int32_t *ip = p.group.iter_prefix;
        int lo = 0, hi = p.group.count;
        while (hi - lo > 1) {
            int mid = (lo + hi) >> 1;
            if (ip[mid] <= it) lo = mid; else hi = mid;
        }
        return p.group.tile_prefix[lo] + (it - ip[lo]) / p.group.probs[lo].iters;
    }
}

// Data-parallel tiles of a persistent launch after its first wave (tiles
// [0, g) go to workgroups 0..g-1): the tiles [g, dp_tiles) form eight
// contiguous chunks, one per XCD, each taken in order through its own
// counter, so the workgroups of one XCD keep neighbouring tiles (shared A
// and B panels) in flight as a one-workgroup-per-tile launch does, while a
// workgroup that drew short tiles simply takes more of them.  A workgroup
// whose chunk is used up moves on to the next XCDs' chunks.  Thread 0 takes
// a ticket as a tile starts (take) and resolves it after the tile's
// epilogue (resolve), so the atomic's latency hides under the MAC loop.
struct DpQueue {
    // qs: workgroup-shared {chunk tickets are taken from, chunks given up as
    // used up (8: none left)} -- shared memory, so the state costs the
    // persistent loop no registers; ticket: that of the running tile
    __device__ __forceinline__ static int take(const Params &p, const int *qs) {
        return __hip_atomic_fetch_add(p.hdr + HDR_NEXT + qs[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // index into [0, dp_tiles - g) of the next tile, or dp_tiles - g
    __device__ __forceinline__ static int resolve(const Params &p, int *qs, int ticket) {
        const int D = p.dp_tiles - p.g;
        while (qs[1] < XCDS) {
            const int c = qs[0];
            const int lo = (int)((int64_t)D * c / XCDS), hi = (int)((int64_t)D * (c + 1) / XCDS);
            if (ticket < hi - lo) return lo + ticket;
            qs[0] = (c + 1) % XCDS;
            if (++qs[1] < XCDS) ticket = take(p, qs);
        }
        return D;
    }
};

// ---------------------------------------------------------------------------
// the launch's generation
//
// A call's flag value is one more than the generation word, which is advanced
// once per launch, when every workgroup has read it.  The workgroups count
// themselves as having read it in groups, workgroup b in that of b % ARRIVALS:
// atomic additions from all XCDs to one word take about 20 ns each, one after
// the other, and the last of them used to end the launch.  The last of a group
// counts the group, the last group advances the word.  One count at each
// workgroup's end and this, us: BF16 197x106x6680 (424 workgroups) 17.9, 13.9;
// 1024x1024x2048 (512) 16.5, 14.1; 256x256x65536 (256) 27.9, 26.7; FP64
// 384x384x1024 (192) 36.4, 35.8.
// ---------------------------------------------------------------------------
struct Arrival {
    __device__ __forceinline__ static int32_t *word(const Params &p, int b) {
        return p.flags + (2 * MAX_GRID - 1 - 2 * (b % ARRIVALS)) * FLAG_STRIDE + FLAG_STRIDE / 2;
    }
    // order of arrival in the workgroup's group
    __device__ __forceinline__ static int take(const Params &p, int b) {
        return __hip_atomic_fetch_add(word(p, b), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ static void finish(const Params &p, int b, int ticket) {
        if (ticket != (p.g - 1 - b % ARRIVALS) / ARRIVALS) return;
        __hip_atomic_store(word(p, b), 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int groups = p.g < ARRIVALS ? p.g : ARRIVALS;
        if (__hip_atomic_fetch_add(p.hdr + HDR_DONE, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != groups - 1) return;
        __hip_atomic_store(p.hdr + HDR_DONE, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int c = 0; c < XCDS; ++c)
            __hip_atomic_store(p.hdr + HDR_NEXT + c, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(p.hdr + HDR_GEN, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
};

// ---------------------------------------------------------------------------
// the kernel body
// ---------------------------------------------------------------------------
// One workgroup's work is a sequence of units: whole data-parallel tiles
// (j = x, then x+g, x+2g, ... or the per-XCD queues' tiles) and the
// segments of its Stream-K range, in the phase
// order the plan asks for.  Keeping a single MAC-loop / fixup / epilogue site
// keeps the code (and its register allocation) in one piece.
//
// Fixup of a tile split over workgroups f..l (f owns the tile's k = 0):
//  serial (Algorithm 5): f..l-1's successors f+1..l store their partial tiles
//    and raise their flags; f waits for them and adds them to its own
//    accumulators in ascending order inside its epilogue;
//  spread: every contributor stores its partial tile and raises its flag as
//    its segment ends; after its last unit, each contributor waits for the
//    tile's other contributors and reduces its slice (Spread).  Only the
//    first and the last segment of a range can belong to a split tile, so a
//    workgroup has at most two slices to reduce; its partial tiles live in
//    slots x (first segment) and g + x (last segment).
template <class C, bool DP_ONLY>
__device__ __forceinline__ void sk_body(const Params &p) {
    __shared__ __attribute__((aligned(1024))) char lds[C::LDS];   // the k-tile buffers of the MAC loop
    __shared__ int next_dp;     // the next queued data-parallel tile, for all waves
    __shared__ int dp_queue[2]; // DpQueue state (thread 0 only)
    const int tid0 = threadIdx.x;
    const int b = blockIdx.x;
    int x = b;
    if (p.xcd_remap || p.piece_major) {
        // hardware dispatches workgroup b to XCD b % 8; give each XCD a
        // contiguous run of logical ids so Stream-K neighbours share an L2
        const int q8 = p.g >> 3, r8 = p.g & 7, j = b & 7;
        x = j * q8 + (j < r8 ? j : r8) + (b >> 3);
    }
    // this call's flag value: the generation word is only advanced after
    // every workgroup of the launch has read it, so all read the same value;
    // taken up after the first unit's MAC loop, which hides the load
    int32_t epoch = 0, gen = 0;
    if constexpr (!DP_ONLY) gen = __hip_atomic_load(p.hdr + HDR_GEN, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    auto take_epoch = [&]() {
        epoch = uniform_int((int)(((uint32_t)gen & 0x3fffffffu) + 1u));
        asm volatile("" :: "s"(epoch) : "memory");
    };
    const bool spread = !DP_ONLY && p.fixup == FIXUP_SPREAD;
    // Stream-K range of this workgroup: [beg, end) within the SK region
    // (fixed split, Algorithm 4: workgroup x runs piece x mod s of tile
    // x / s, iterations [y ips, min(I, (y+1) ips)) with ips = ceil(I / s) --
    // again one contiguous range of the region, so everything below holds)
    const int fs = DP_ONLY ? 0 : p.split;
    int q = 0, r = 0, beg = 0, end = 0, rq = 0, fI = 1, ips = 1;
    if (!DP_ONLY && p.sk_iters > 0) {
        if (fs > 0) {
            // (a hybrid's region of fewer than g / s tiles leaves the
            // workgroups past s tiles without Stream-K work)
            fI = p.prob.iters;
            ips = (fI + fs - 1) / fs;
            // piece_major: an XCD's run of workgroups takes one piece of
            // neighbouring tiles, which share its panels of A and B (the
            // pieces of one tile share nothing)
            if (p.piece_major) {
                const int t = p.sk_iters / fI;
                x = x % t * fs + x / t;
            }
            const int tl = x / fs, y = x % fs;
            if (tl < p.sk_iters / fI) {
                beg = tl * fI + (y * ips < fI ? y * ips : fI);
                end = tl * fI + ((y + 1) * ips < fI ? (y + 1) * ips : fI);
            } else {
                beg = end = p.sk_iters;
            }
        } else {
            q = p.sk_iters / p.g;
            r = p.sk_iters % p.g;
            beg = x * q + (x < r ? x : r);
            end = beg + q + (x < r ? 1 : 0);
            rq = r * (q + 1);
        }
    }
    // the workgroup holding region-relative iteration i
    auto owner_of = [&](int i) {
        if (fs > 0) return (i / fI) * fs + (i % fI) / ips;
        return i < rq ? i / (q + 1) : r + (i - rq) / q;
    };
    // slices still to reduce (spread fixup): tile, first and last contributor
    int red_tile[2] = {-1, -1}, red_f[2] = {0, 0}, red_l[2] = {0, 0};
    int it = beg;          // next SK iteration
    int j = x;             // next DP tile index
    int phase = 0;         // 0, 1: the two phases; 2: done
    int seq = 0;
    const bool dp_first = DP_ONLY || p.dp_first;
    // data-parallel tiles after the first from the per-XCD queues (DpQueue):
    // thread 0 hands the next one to the workgroup after each epilogue
    const bool dyn = !DP_ONLY && p.dyn_dp;
    int ticket = 0;        // of the running tile; without the queues the arrival's
    if (dyn && tid0 == 0) {
        dp_queue[0] = b % XCDS;
        dp_queue[1] = 0;
    }
    while (true) {
        const bool dp_now = (phase == 0) == dp_first;
        int tile, k0, k1;
        bool started = true, ended = true;
        if (phase >= 2) break;
        if (dp_now) {
            if (j >= p.dp_tiles) { ++phase; continue; }
            tile = j < p.sk_tile_begin ? j : j - p.sk_tile_begin + p.sk_tile_end;
            if (dyn) {
                if (tid0 == 0) ticket = DpQueue::take(p, dp_queue);
            } else {
                j += p.g;
            }
        } else {
            if (DP_ONLY || it >= end) { ++phase; continue; }
            tile = tile_of_iter<C::GROUPED>(p, p.sk_iter_begin + it);
        }
        const TileRef tr = tile_of_tile<C::GROUPED>(p, tile);
        const Problem P = uniform_problem(*tr.P);
        int t0 = 0, t1 = 0;
        if (dp_now) {
            k0 = 0;
            k1 = P.iters;
        } else {
            t0 = uniform_int(tr.it_begin) - p.sk_iter_begin;   // region-relative tile start
            t1 = t0 + P.iters;
            k0 = it - t0;
            k1 = (end < t1 ? end : t1) - t0;
            started = it == t0;
            ended = end >= t1;
            it = t1;
        }
        int tm, tn;
        tile_coords(P, uniform_int(tr.tile_local), p.band, tm, tn);
        // an opaque copy of the thread index: per-thread addresses are
        // recomputed for every unit instead of being hoisted out of this loop
        // and kept live (spilled) across the whole kernel
        int tid = tid0;
        asm volatile("" : "+v"(tid));
        typename C::Frag acc[C::FM][C::FN];
        if constexpr (C::PP) mac_loop_pp<C>(P, tm, tn, k0, k1, acc, lds, tid);
        else if constexpr (C::HALVES) mac_loop_half<C>(P, tm, tn, k0, k1, acc, lds, tid);
        else mac_loop<C>(P, tm, tn, k0, k1, acc, lds, tid);
        if (!DP_ONLY && seq == 0) {
            // every wave has read the generation: the workgroup arrives, with
            // the queues (whose counters the last arrival clears) at its end
            take_epoch();
            plain_barrier();
            if (!dyn && tid0 == 0) ticket = Arrival::take(p, b);
        }
        const int last = ended ? -1 : owner_of(t1 - 1);
        if (!started) {
            // the first segment of this range: partial slot and flag x
            store_partial<C>((char *)p.partials + (int64_t)x * C::SLOT_BYTES, acc, tid);
            signal_flag(p.flags + x * FLAG_STRIDE, epoch, tid);
            trace_rec(p, x, seq++, tile, k0, k1, ROLE_PRODUCER, -1, 0, tid);
            if (spread) {
                red_tile[0] = tile;
                red_f[0] = owner_of(t0);
                red_l[0] = ended ? x : last;
            }
            continue;
        }
        if (!ended && spread) {
            // the last segment of this range owns the tile: partial slot and
            // flag g + x (resp. MAX_GRID + x)
            store_partial<C>((char *)p.partials + (int64_t)(p.g + x) * C::SLOT_BYTES, acc, tid);
            signal_flag(p.flags + (MAX_GRID + x) * FLAG_STRIDE, epoch, tid);
            trace_rec(p, x, seq++, tile, k0, k1, ROLE_OWNER, last, 0, tid);
            red_tile[1] = tile;
            red_f[1] = x;
            red_l[1] = last;
            continue;
        }
        if (!ended) wait_flags(p.flags, x + 1, last, -1, x + 1, epoch, p.err, p.wait_ticks, tid);
        // peers' partial tiles are added in ascending slot order inside the
        // epilogue, fragment by fragment
        store_tile<C>(P, tm, tn, acc, tid, (const char *)p.partials, x + 1, last, lds);
        trace_rec(p, x, seq++, tile, k0, k1, dp_now ? ROLE_DP : (ended ? ROLE_FULL : ROLE_OWNER), last, 0,
                  tid);
        if (dp_now && dyn) {
            if (tid0 == 0) next_dp = DpQueue::resolve(p, dp_queue, ticket);
            __syncthreads();
            j = p.g + next_dp;
            __syncthreads();
        }
    }
    if constexpr (!DP_ONLY) {
        if (spread) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (red_tile[u] < 0) continue;
                const int f = red_f[u], l = red_l[u];
                wait_flags(p.flags, f, l, x, MAX_GRID + f, epoch, p.err, p.wait_ticks, tid0);
                const TileRef tr = tile_of_tile<C::GROUPED>(p, red_tile[u]);
                const Problem P = uniform_problem(*tr.P);
                int tm, tn;
                tile_coords(P, uniform_int(tr.tile_local), p.band, tm, tn);
                const int s = l - f + 1, i = x - f;
                trace_rec(p, x, seq++, red_tile[u], (int)((int64_t)Spread<C>::N * i / s),
                          (int)((int64_t)Spread<C>::N * (i + 1) / s), ROLE_REDUCE, l, f, tid0);
                Spread<C>::reduce(p, P, tm, tn, f, l, x, lds, tid0);
            }
        }
        if (dyn || seq == 0) {
            if (seq == 0) take_epoch();
            __syncthreads();
            if (tid0 == 0) ticket = Arrival::take(p, b);
        }
        if (tid0 == 0) Arrival::finish(p, b, ticket);
    }
}

template <class C>
__global__ __launch_bounds__(C::THREADS) void sk_kernel(Params p) {
    sk_body<C, false>(p);
}

template <class C>
__global__ __launch_bounds__(C::THREADS) void dp_kernel(Params p) {
    sk_body<C, true>(p);
}

template <class C>
int launch_sk(const Params &p, int grid, void *stream) {
    hipLaunchKernelGGL(sk_kernel<C>, dim3(grid), dim3(C::THREADS), 0, (hipStream_t)stream, p);
    return (int)hipGetLastError();
}

template <class C>
int launch_dp(const Params &p, int grid, void *stream) {
    hipLaunchKernelGGL(dp_kernel<C>, dim3(grid), dim3(C::THREADS), 0, (hipStream_t)stream, p);
    return (int)hipGetLastError();
}

template <class C>
int occupancy_sk(int *blocks) {
    return (int)hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, sk_kernel<C>, C::THREADS, 0);
}

}  // namespace sk
