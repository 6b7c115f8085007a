// Stream-K GEMM for gfx950 (MI355X): one persistent kernel serves every
// scheduling policy.  Each workgroup derives its own share of the iteration
// space from a handful of plan numbers (Algorithm 1's range and tile arithmetic), runs the MAC
// loop of each segment on the matrix cores, and either stores the tile, parks an
// fp32 partial in the workspace, or - as the tile's owner - waits for the parked
// partials and adds them in a fixed order (the synchronised reduction that
// Sec. 5.3 names as the alternative to Algorithm 1's atomic adds).
//
// MAC loop data path: A (row-major, k contiguous) and B (row-major, n contiguous)
// tiles go from global memory straight into LDS with 16-byte LDS-DMA loads, into
// a ring of NS stages; the LDS image is XOR-swizzled at 16-byte granularity (the
// swizzle is applied by choosing which global piece each lane fetches) so that
// the matrix-core operand reads are bank-conflict free without padding.  A
// operands are read with 16-byte LDS reads, B operands with the transposing
// 8-byte reads that turn the [k][n] image into k-contiguous lanes.
#pragma once
#include <hip/hip_runtime.h>
#include <atomic>
#include <type_traits>
#include <utility>
#include "streamk_internal.h"


namespace streamk_detail {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16;
typedef __attribute__((address_space(3))) unsigned char lds_byte;
typedef __amdgpu_buffer_rsrc_t buffer_rsrc;
constexpr int BUFFER_RAW = 0x00020000;               // word 3 of a buffer descriptor: raw 32-bit data, no swizzle

struct GemmArgs {
    const void* A;
    const void* B;
    void* D;
    float* partials;       // grid slots of BM*BN floats
    float* image;          // atomic fix-up: fp32 image of D that partial tiles are added into (D itself for fp32 output)
    uint32_t* flags;       // one per workgroup, SK_FLAG_STRIDE bytes apart
    uint32_t* status;      // set non-zero when an owner gives up waiting
    int M, N, K;
    int tiles_m, tiles_n, tiles, ipt, sk_tiles, ipw, grid, sk_iters, tile_order;
    uint32_t spin_limit;
    int out_dtype;
    int dp_first;          // 1: a workgroup runs its data-parallel tiles before its Stream-K iterations
    int xcd_remap;         // which logical workgroup ids share an XCD (see logical_wg)
    int first_ids, other_ids;  // map 1: how many of the first logical ids, and of the others, an XCD runs; together grid / 8
    int k_aligned;         // 1: a workgroup runs the whole tiles of its Stream-K range first, then the head of its last
                           //    tile (k from 0), then the tail of its first one, and the workgroup holding a tile's
                           //    last iteration reduces and stores it
    int stream_b;          // 1: B is read exactly once (one row of tiles) and is large: MAY_STREAM_B tiles request it non-temporally
    // divisors of the index arithmetic: ipt, ipw, tiles_n, SK_GROUP_ROWS * tiles_n, rows of the last (short) band
    sk_fast_div div_ipt, div_ipw, div_tiles_n, div_band, div_last_rows;
    sk_fast_div div_tiles, div_extra;   // of logical_wg: tiles, ipt mod ipw
};

__device__ __forceinline__ uint32_t fast_div(uint32_t n, sk_fast_div f) { return (uint32_t)(((uint64_t)n * f.mul) >> f.shift); }

// ---- matrix-core wrappers ---------------------------------------------------------------------
// One instruction multiplies an MF x KM block (first operand) by a KM x MF block (second operand).
// Lane l holds, for the first operand, row l % MF and the 8 consecutive k starting at
// 8 * (l / MF); for the second, column l % MF and the same k; for the MF x MF result, column
// l % MF and rows (r/4) * (256/MF) + 4 * (l / MF) + r % 4.  Both operands have the same register
// format, so the kernels pass the B block first and the A block second: the instruction then
// produces the transposed block, i.e. lane l holds row l % MF of the D block and, in registers
// 4q .. 4q+3, the four consecutive columns (256/MF) * q + 4 * (l / MF) + {0..3}, which can be
// stored as vectors.
template <int DT, int MF> struct Mfma;
template <> struct Mfma<SK_BF16, 32> {
    typedef f32x16 Acc;
    static __device__ __forceinline__ Acc run(uint4 a, uint4 b, Acc c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
};
template <> struct Mfma<SK_F16, 32> {
    typedef f32x16 Acc;
    static __device__ __forceinline__ Acc run(uint4 a, uint4 b, Acc c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    }
};
template <> struct Mfma<SK_BF16, 16> {
    typedef f32x4 Acc;
    static __device__ __forceinline__ Acc run(uint4 a, uint4 b, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
};
template <> struct Mfma<SK_F16, 16> {
    typedef f32x4 Acc;
    static __device__ __forceinline__ Acc run(uint4 a, uint4 b, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    }
};

// fp8 (e4m3): the scaled 8-bit instruction with both block scales at 2^0 (biased exponent 127);
// per lane 32 consecutive k (8 registers) of row / column l % MF starting at 32 * (l / MF).
template <> struct Mfma<SK_FP8_E4M3, 32> {
    typedef f32x16 Acc;
    static __device__ __forceinline__ Acc run(i32x8 a, i32x8 b, Acc c) {
        return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 127, 0, 127);
    }
};
template <> struct Mfma<SK_FP8_E4M3, 16> {
    typedef f32x4 Acc;
    static __device__ __forceinline__ Acc run(i32x8 a, i32x8 b, Acc c) {
        return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 0, 0, 0, 127, 0, 127);
    }
};

template <int DT_, int BM_, int BN_, int BK_, int WM_, int WN_, int MF_, int NSA_, int NSB_ = NSA_, int FINE_ = 0>
struct Cfg {
    static constexpr int DT = DT_, BM = BM_, BN = BN_, BK = BK_, WM = WM_, WN = WN_, MF = MF_;
    static constexpr int NSA = NSA_, NSB = NSB_;        // LDS ring depth of the A and of the B tiles
    static constexpr int NW = WM * WN, THREADS = 64 * NW;
    static constexpr int WTM = BM / WM, WTN = BN / WN;   // tile of one wave
    static constexpr int MI = WTM / MF, NI = WTN / MF;   // matrix-core blocks per wave tile
    static constexpr bool FP8 = DT == SK_FP8_E4M3;
    static constexpr int ES = FP8 ? 1 : 2;               // bytes per input element
    static constexpr int PE = 16 / ES;                   // elements per 16-byte piece
    static constexpr int KPL = FP8 ? 32 : 8;             // consecutive k per lane per instruction
    static constexpr int APL = KPL / PE;                 // A pieces per lane per instruction
    static constexpr int KG = 64 / MF;                   // groups of KPL k across the lanes
    static constexpr int KM = KPL * KG;                  // k per instruction
    static constexpr int KK = BK / KM;
    static constexpr int ACC = MF * MF / 64;             // accumulator registers per block
    // LDS: a ring of NSA A tiles (BM rows of CPA 16-byte pieces) followed by a ring of NSB B tiles
    // (BK rows of CPB pieces), no padding.  A may be one stage deeper than B: its loads then run
    // two iterations ahead and only the B tile has to arrive within one iteration.
    static constexpr int CPA = BK / PE, CPB = BN / PE;
    static constexpr int A_PIECES = BM * CPA, B_PIECES = BK * CPB;
    static constexpr int A_BYTES = A_PIECES * 16, B_BYTES = B_PIECES * 16;
    static constexpr int B_RING = NSA * A_BYTES;         // byte offset of the B ring
    static constexpr int LDS_BYTES = NSA * A_BYTES + NSB * B_BYTES;
    // one LDS-DMA instruction of one wave fills 64 consecutive pieces
    // (an A tile of fewer pieces than that for every wave is fetched by several waves: the same bytes to the same place)
    static constexpr int A_WAVES = A_PIECES < 64 * NW ? A_PIECES / 64 : NW;
    static constexpr int A_LD = A_PIECES < 64 * NW ? 1 : A_PIECES / (64 * NW), B_LD = B_PIECES / (64 * NW);
    static_assert(A_PIECES % (64 * A_WAVES) == 0 && NW % A_WAVES == 0 && B_PIECES % (64 * NW) == 0, "whole LDS-DMA instructions");
    static constexpr int LPS = A_LD + B_LD;              // LDS-DMA loads per stage per wave
    // register-staged fill (unaligned problems, tiles too small for the DMA split)
    static constexpr int CA = (A_PIECES + THREADS - 1) / THREADS, CB = (B_PIECES + THREADS - 1) / THREADS;
    // Registers of one set of matrix-core operands and of the accumulators.  With 8 waves a lane has
    // 256 registers for everything; with 4 waves 256 plus 256 that can hold the accumulators.
    // PIN_ORDER: there is room to hold two operand sets, so the MAC loop pins "read the next
    // k-step's operands, then multiply the current ones".
    static constexpr int FRAG_REGS = (MI + NI) * (FP8 ? 8 : 4), ACC_REGS = MI * NI * ACC;
    static constexpr bool PIN_ORDER = NW >= 8 ? 2 * FRAG_REGS + ACC_REGS + 64 <= 256 : 2 * FRAG_REGS + 64 <= 192;
    // FINE: the MAC loop is written out instruction by instruction - one matrix-core instruction, then
    // at most a few LDS reads of the next k-step's operands or one LDS-DMA request, and so on - so that
    // a wave that has a SIMD to itself keeps the matrix-core pipe fed while its memory instructions
    // queue up (needs the two operand sets of PIN_ORDER).
    static constexpr bool FINE = FINE_ != 0;
    // the tiles of at most 64 rows (HBM-bound shapes) and the eight-wave 128 x 128 tile can request B non-temporally,
    // decided per launch (GemmArgs::stream_b).  128 x 128 tile, fourteen problems of 65 - 128 rows, B of 128 - 512 MiB:
    // 1.6 - 5 % faster, one without effect (128 x 8192 x 8192: 37.9 -> 37.2 us, 128 x 16384 x 16384: 104.4 -> 99.8).
    // The larger tiles re-use B blocks through the L2 caches, so they carry no such switch
    static constexpr bool MAY_STREAM_B = BM <= 64 || (BM == 128 && BK == 64 && NW == 8);
    static_assert(!FINE || PIN_ORDER, "the instruction-by-instruction order needs two operand sets");
    // register-staged path: a stage's pieces (4 registers each).  STAGED_FINE: the instruction-by-instruction
    // MAC loop with one stage in registers, where the two operand sets leave room for it; the other tiles hold
    // STAGES_HELD stages in registers, about 64 registers of loads in flight.  (The count is an estimate: the compiler
    // spills 6 registers of the eight-wave 256 x 256 kernel, of the one with the shared reduction too, 49 of the four-wave one and 88 of
    // the 8-bit four-wave one.  No trip of a loop holds a spill: they are stored once and reloaded around a segment's loops.)
    static constexpr int PIECES = CA + CB;
    static constexpr bool STAGED_FINE = FINE && KK % 2 == 0 && 2 * FRAG_REGS + (NW >= 8 ? ACC_REGS : 0) + 5 * PIECES + 32 <= 256;
    static constexpr int STAGES_HELD = 2 * FRAG_REGS + (NW >= 8 ? ACC_REGS : 0) + 4 * PIECES + 64 > 256 ? 0 : PIECES <= 5 ? 4 : PIECES <= 8 ? 2 : 1;
    // The other tiles' stages in whole rounds of STAGES_HELD (see mac_loop_staged), but for the tiles of 16 and 32 rows on four waves,
    // which are 1 - 8 % slower with them.  Stage by stage -> rounds, whole tiles, us: 319 x 1021 on 32 x 64, K = 125 / 253 / 1021 / 2043, 4.60 -> 4.30, 5.41 -> 5.12,
    // 10.2 -> 8.8, 16.2 -> 12.8; 639 x 1021 on 64 x 64, K = 509 / 2043, 7.69 -> 7.29, 16.4 -> 16.0 (17 plans 3 % in the mean); 64 x 128 up to eight iterations 1 - 4 %, in
    // 8 bits 2 % in the mean; 8-bit 128 x 128 and 128 x 128 x 32 4 % faster to 3 % slower.  Where whole tiles are slower with them they are taken one
    // by one, see OneByOne; split plans are 6 % faster to 2 % slower.
    static constexpr bool STAGED_ROUNDS = STAGES_HELD > 0 && PIECES != 5;
    // vector stores one wave issues in the epilogue of an unsplit interior tile with 16-bit output (an fp32
    // output issues more): what may still be in flight when the next tile's first stage is waited for
    static constexpr int EPILOGUE_STORES = MI * NI * (MF == 32 ? ACC / 8 : ACC / 4);
    // 16-byte stores from the lanes as the blocks lie, 32 rows of 32 bytes per instruction, instead of store_blocks'
    // exchange, where that costs more than the better pattern gives: the lowest tiles (bound by the length of the chain
    // at the end of the kernel: 23 x 4096 x 8128 to fp32 16.5 us, 16.6 with it) and the four-wave 256 x 256 kernels
    // (nothing runs beside a wave's exchange, 500 instructions or 1 us; the library takes them from 48 k-iterations on, where
    // streamk_whole_tiles_kernel does not apply: fp32 output, 8-bit rows off the 16-byte grid, the longest rows.  Measured with
    // bf16 output before that kernel took those plans: 3840 x 4224 x 4096 109.4 us, 110.0 with it, 4096 x 4032 x 3072 83.4 / 84.9, 8
    // bits 3840 x 4224 x 8192 100.9 / 104.1, 8192^3 no difference).  The other four-wave kernels gain from it at every depth tried.
    static constexpr bool DIRECT_STORES = BM <= 32 || (FINE && NW == 4 && BM == 256 && BN == 256);
    // has a kernel with the shared reduction: slots of 16 bytes per lane (the four-wave 256 x 256 kernels' may be others), and
    // where sk_shared_reduction may ask for it
    static constexpr bool MAY_SHARE = ACC_REGS < 256 && BM * BN >= 4096;
    static_assert(WTM % MF == 0 && WTN % MF == 0 && BK % KM == 0, "tile does not divide");
    static_assert(CPA == 4 || CPA == 8 || CPA == 16, "A swizzle assumes 64/128/256-byte rows");
    static_assert(CPB >= 8, "B swizzle assumes rows of at least 128 bytes");
    static_assert(NSB >= 2 && (NSA == NSB || NSA == NSB + 1) && LDS_BYTES <= 160 * 1024, "LDS budget / ring depths");
    static_assert((NSA - 1) * LPS <= 63, "vmcnt range");
    // Stages requested before the first one is waited for, at the kernel's start; the others of the ring follow once that has
    // landed.  The requests of early workgroups delay the first stage of late ones; a stage that is requested late comes late.  Two instead
    // of three of the ring of four, segments of 2 to 12 k-iterations, operands in caches and not: 64 x 128 in 8 bits 0 - 3 % faster (four
    // iterations, 640 x 2048 x 512 from memory 5.90 us, three 6.04), 32 x 128 in 8 bits 0 - 6 %, the others 2 % faster to 2 % slower.  Not
    // with the small stages (12 KB) of 32 x 64, where three are as fast from caches and faster from memory: 512 x 512 x 256 / 384 / 512 / 768 3.97 / 4.76 / 5.28 /
    // 6.43 -> 3.85 / 4.60 / 5.15 / 6.27.  One, whose successor then comes too late, is 0.1 us slower.
    static constexpr int START = NSA == NSB && NSA > 3 && A_BYTES + B_BYTES >= 16 * 1024 ? 2 : NSA - 1;
    // The last stage of the ring is requested in one go behind the first wait, or slot by slot in the first trip.  In one go is faster by what the
    // slots' checks cost (128 x 128, 4096 x 4096 x 128 .. 832 3 - 6 %), but not in the larger tiles, where the burst, 24 - 32 KB, meets
    // the stores of the tile before.  In one go -> slot by slot, us: 256 x 256, 10656 x 8752 x 192 / 256 / 448 f16 84.8 / 94.7 / 124.2 -> 80.0 /
    // 90.3 / 119.7, 14416 x 5728 x 1008 194.5 -> 183.1, 5120 x 4096 x 256 24.2 -> 24.0; 256 x 128, 2432 x 13424 x 240 to fp32 58.2 -> 55.2, 9248 x 3104 x 320 / 720
    // 35.4 / 62.9 -> 34.2 / 61.2, 11520 x 640 x 624 16.7 -> 16.2, two iterations 1 - 3 % slower (4096 x 4096 x 128 13.8 -> 14.0); 8-bit 128 x 256, 9000 x 9008 x
    // 256 / 384 70.7 / 80.1 -> 67.4 / 77.5, 1040 x 15376 x 368 24.0 -> 23.4, a single iteration 0.7 % slower (4096 x 8192 x 128 17.54 -> 17.66).
    static constexpr bool FILL_FIRST = PIN_ORDER && BM * BN < 256 * 128;
    // LDS-DMA loads that may still be in flight when iteration i starts, if `later` more
    // iterations follow it.  Issue order inside an iteration: B tile of iteration +NSB-1, then A
    // tile of iteration +NSA-1; loads complete in order.
    static constexpr int in_flight(int later) {
        int n = 0;
        if (NSA == NSB) {
            for (int d = 1; d <= NSA - 2; d++) n += later >= d ? LPS : 0;
        } else {
            n += later >= 1 ? A_LD : 0;
            for (int d = 1; d <= NSB - 2; d++) n += (later >= d ? B_LD : 0) + (later >= d + 1 ? A_LD : 0);
        }
        return n;
    }
};

// ---- LDS image --------------------------------------------------------------------------------
// A: piece c of row r sits at position c ^ swz_a(r).  Eight consecutive rows and also sixteen
// consecutive rows then spread the same logical piece over all banks (32- or 64-bank view).
template <int CPA> __device__ __forceinline__ int swz_a(int r) {
    if (CPA == 4) return (r >> 1) & 3;
    return (r & 7) ^ ((r >> 3) & 1);
}
// B: piece c of row k sits at position c ^ swz_b<C::FP8, C::CPB>(k): rows k..k+3, read together by one transposing
// read, land on different 32-byte and different 64-byte bank groups.
// (8-bit elements: one transposing read covers 8 rows; rows k..k+7 go to 8 different 32-byte groups.)
// Rows of 128 bytes (CPB == 8): rows k and k+1 already lie 128 bytes apart, so only every other row moves,
// by 64-byte (16-bit elements; rows 8 apart, read together by the 16-row block, by 32-byte) or 32-byte groups.
template <bool FP8, int CPB> __device__ __forceinline__ int swz_b(int k) {
    if (CPB == 8) return FP8 ? ((k >> 1) & 3) << 1 : ((k >> 1) & 1) << 2 | ((k >> 3) & 1) << 1;
    if (FP8) return (k & 7) << 1;
    const int k0 = k & 1, k1 = (k >> 1) & 1;
    return (k0 << 1) | (k1 << 2) | (k0 << 3);
}

// Source of the pieces that lie beyond K in a ragged last k-iteration.
static __device__ __align__(16) const unsigned char g_zero_piece[16] = {0};

// 16 bytes global -> LDS without passing through registers.  The LDS destination of lane l is
// lds_base + 16 * l; lds_base must be wave-uniform.  Completion is tracked by vmcnt only; the
// compiler is not told that LDS is written: the caller orders the reads with s_waitcnt + barrier.
// m0 is not named as clobbered: it is a reserved register for this compiler (it never holds a value of
// the program across statements; the compiler writes it right before an instruction of its own that
// reads it), and naming a reserved register in a clobber list is rejected as undefined behaviour.
__device__ __forceinline__ void lds_dma16(const void* base, uint32_t byte_off, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(byte_off), "s"(base), "s"(lds_base));
}
// The same load marked non-temporal: for data that is read exactly once and is too large for the caches
// to hold until a later launch (the B operand of a plan with a single row of tiles, see the launcher).
__device__ __forceinline__ void lds_dma16_nt(const void* base, uint32_t byte_off, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(byte_off), "s"(base), "s"(lds_base));
}
__device__ __forceinline__ void lds_dma16_ptr(const void* gptr, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(gptr), "s"(lds_base));
}

template <int N> __device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N <= 63, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);   // lgkmcnt / expcnt not waited
}

// Hardware workgroup ids go round-robin over the 8 XCDs.  Which logical ids (positions in the schedule) an
// XCD runs decides what its L2 can share (sk_plan chooses, see there):
//   1  a contiguous block of logical ids: neighbours in the schedule share tiles and A row-blocks; where only the
//      first ids have work in the last wave of tiles (or at all), a block of those and a block of the others;
//   2  for plans in which several workgroups share every tile: the ids sorted by their piece of the
//      tile's K range, then by tile, and a contiguous block of that - an XCD then reads one slice of K of
//      every tile it touches, and the tiles that share an A row-block or B column-block share its slice in L2;
//   0  the hardware order.
__device__ __forceinline__ int logical_wg(uint32_t hw, const GemmArgs& g) {
    if (g.xcd_remap == 0) return (int)hw;
    const int xcd = (int)(hw % 8), i = (int)(hw / 8);
    if (g.xcd_remap == 1) return sk_spread_id(xcd, i, g.first_ids, g.other_ids);
    const int q = xcd * (g.grid / 8) + i;
    // The ranges of workgroups ceil(t * ipt / ipw) .. ceil((t + 1) * ipt / ipw) - 1 start in tile t: `each` of them or
    // one more; the tiles with one more are t = floor(i * ipw / extra), i = 0, 1, ..., extra = ipt mod ipw.  (By the
    // ranges themselves, not by grid / tiles: ipw is rounded up, and over the tiles that adds up to a slice or more.)
    const int each = (int)fast_div((uint32_t)g.ipt, g.div_ipw);
    if (q >= (int)fast_div((uint32_t)(g.sk_iters + g.ipw - 1), g.div_ipw)) return q;       // an empty range
    int t, j;
    if (q < each * g.tiles) {
        j = (int)fast_div((uint32_t)q, g.div_tiles);
        t = q - j * g.tiles;
    } else {
        j = each;
        t = (int)fast_div((uint32_t)((q - each * g.tiles) * g.ipw), g.div_extra);
    }
    return (int)fast_div((uint32_t)(t * g.ipt + g.ipw - 1), g.div_ipw) + j;
}

// Position of a tile index in the tile grid under the plan's tile order.
__device__ __forceinline__ void tile_position(const GemmArgs& g, int tile, int& tm, int& tn) {
    if (g.tile_order == SK_ORDER_ROW_MAJOR) {
        tm = (int)fast_div((uint32_t)tile, g.div_tiles_n);
        tn = tile - tm * g.tiles_n;
    } else {                                     // bands of 8 tile rows, walked column by column
        const uint32_t per_band = (uint32_t)(SK_GROUP_ROWS * g.tiles_n);
        const uint32_t band = fast_div((uint32_t)tile, g.div_band), within = (uint32_t)tile - band * per_band;
        const int left = g.tiles_m - (int)band * SK_GROUP_ROWS;
        const uint32_t rows = (uint32_t)(left < SK_GROUP_ROWS ? left : SK_GROUP_ROWS);
        tn = (int)(left < SK_GROUP_ROWS ? fast_div(within, g.div_last_rows) : within / (uint32_t)SK_GROUP_ROWS);
        tm = (int)band * SK_GROUP_ROWS + (int)(within - (uint32_t)tn * rows);
    }
}

// 16 bytes whose address is only known to be a multiple of the element size (rows of a matrix whose
// leading dimension is not a multiple of 8 elements start anywhere); the compiler picks the access.
struct __attribute__((packed, aligned(1))) Piece1 { u32x4 v; };
struct __attribute__((packed, aligned(2))) Piece2 { u32x4 v; };

// Element by element: a piece of a matrix of less than 16 bytes, zero beyond its edges.
template <int ES>
__device__ __forceinline__ uint4 load_piece(const unsigned char* __restrict__ base, int row, int col, int rows, int cols) {
    unsigned char e[16];
    const unsigned char* p = base + (size_t)((uint32_t)row * (uint32_t)cols + (uint32_t)col) * ES;
#pragma unroll
    for (int i = 0; i < 16; i++) e[i] = row < rows && col + i / ES < cols ? p[i] : (unsigned char)0;
    return make_uint4(e[0] | (uint32_t)e[1] << 8 | (uint32_t)e[2] << 16 | (uint32_t)e[3] << 24,
                      e[4] | (uint32_t)e[5] << 8 | (uint32_t)e[6] << 16 | (uint32_t)e[7] << 24,
                      e[8] | (uint32_t)e[9] << 8 | (uint32_t)e[10] << 16 | (uint32_t)e[11] << 24,
                      e[12] | (uint32_t)e[13] << 8 | (uint32_t)e[14] << 16 | (uint32_t)e[15] << 24);
}

// Bytes `skip` .. 15 of a piece moved down to byte 0 on, zeros behind them.
__device__ __forceinline__ uint4 shift_piece(uint4 v, uint32_t skip) {
    uint32_t t[4] = {__builtin_amdgcn_alignbyte(v.y, v.x, skip & 3), __builtin_amdgcn_alignbyte(v.z, v.y, skip & 3),
                     __builtin_amdgcn_alignbyte(v.w, v.z, skip & 3), __builtin_amdgcn_alignbyte(0, v.w, skip & 3)};
    if (skip & 4) { t[0] = t[1]; t[1] = t[2]; t[2] = t[3]; t[3] = 0; }
    if (skip & 8) { t[0] = t[2]; t[1] = t[3]; t[2] = 0; t[3] = 0; }
    return make_uint4(t[0], t[1], t[2], t[3]);
}

// Register-staged fill of one stage (same LDS image as the DMA path), piece by piece: fetch a piece
// into registers, and later park it in LDS.  Piece j of thread t is LDS position j * THREADS + t of the
// stage's A or B tile; the swizzle is applied by choosing which global piece goes there, as on the DMA path.
// A piece is one under-aligned 16-byte load.  Rows beyond M and columns beyond N fetch the start of the iteration's
// first row instead - every lane the same aligned 16 bytes, a third of the vector L1's time - and a piece that reaches
// beyond column N - 1 of B runs on into the next row: both only feed output elements that are never stored.
// The k-iterations below `inside` lie wholly inside K with at least one row of B behind them (so that running on
// stays inside B).  The others - the last one, as a rule - are fetched from where 16 bytes still lie inside the matrix
// and cut to what is inside K before they are parked: fetch<CHECKED> and cut() work for every k-iteration of matrices
// of 16 bytes or more.  Short segments run hardly anything else: with element loads here and the checks in every
// slot of the loop, 8-bit problems of one k-iteration took 11.3 us, now 9.1; 12 x 5481 x 8461 67.7, now 35.8;
// 5001 x 5003 x 65 in bf16 40.8, now 28.8.
template <class C> struct StagedFill {
    uint32_t a_off[C::CA], b_off[C::CB];         // byte offsets from A / B at k-iteration 0
    uint32_t a_end, b_end;                       // byte offset of the last 16 bytes of A / B
    int inside;
    int a_col;                                   // column of this lane's A pieces inside the k-iteration (the same for all)
    static_assert(C::THREADS % C::CPA == 0 && (C::THREADS / C::CPA) % 16 == 0, "a thread's A pieces lie in one column");
    static __device__ __forceinline__ bool tiny(const GemmArgs& g) {
        return (uint64_t)g.M * (uint32_t)g.K * C::ES < 16 || (uint64_t)g.N * (uint32_t)g.K * C::ES < 16;
    }
    __device__ __forceinline__ void init(const GemmArgs& g, int m0, int n0) {
        inside = g.N >= C::PE ? (g.K - 1) / C::BK : 0;
        a_end = (uint32_t)g.M * (uint32_t)g.K * C::ES - 16;
        b_end = (uint32_t)g.N * (uint32_t)g.K * C::ES - 16;
        a_col = C::PE * ((threadIdx.x % C::CPA) ^ swz_a<C::CPA>(threadIdx.x / C::CPA));
#pragma unroll
        for (int j = 0; j < C::CA; j++) {
            const int r = (threadIdx.x + j * C::THREADS) / C::CPA;
            a_off[j] = m0 + r < g.M ? ((uint32_t)(m0 + r) * (uint32_t)g.K + (uint32_t)a_col) * C::ES : 0;
        }
#pragma unroll
        for (int j = 0; j < C::CB; j++) {
            const int p = threadIdx.x + j * C::THREADS, k = p / C::CPB, c = (p % C::CPB) ^ swz_b<C::FP8, C::CPB>(k);
            const int col = n0 + C::PE * c;
            b_off[j] = col < g.N ? ((uint32_t)k * (uint32_t)g.N + (uint32_t)col) * C::ES : 0;
        }
    }
    static __device__ __forceinline__ uint4 load16(const char* base, uint32_t off) {
        const u32x4 w = C::ES == 2 ? reinterpret_cast<const Piece2*>(base + off)->v : reinterpret_cast<const Piece1*>(base + off)->v;
        return make_uint4(w[0], w[1], w[2], w[3]);
    }
    // byte offset of piece q at k-iteration kit (modulo 2^32: one beyond the matrix may come out anywhere)
    __device__ __forceinline__ uint32_t offset(const GemmArgs& g, int kit, int q) const {
        const uint32_t it = (uint32_t)kit * (uint32_t)(C::BK * C::ES);
        return q < C::CB ? b_off[q] + it * (uint32_t)g.N : a_off[q - C::CB] + it;
    }
    // piece q of the stage of k-iteration kit: the B pieces first, then the A pieces
    template <bool CHECKED> __device__ __forceinline__ uint4 fetch(const GemmArgs& g, int kit, int q) const {
        const char* m = static_cast<const char*>(q < C::CB ? g.B : g.A);
        if (CHECKED) {
            // (nothing inside K: the start of the matrix, aligned; a little beyond the end of the matrix: its last 16 bytes)
            const uint32_t off = offset(g, kit, q), end = q < C::CB ? b_end : a_end;
            const bool some = (q < C::CB || kit * C::BK + a_col < g.K) && (off <= end || off - end < 16);
            return load16(m, some ? (off < end ? off : end) : 0u);
        }
        if (q < C::CB) return load16(m + (size_t)((uint32_t)kit * (uint32_t)(C::BK * C::ES)) * (uint32_t)g.N, b_off[q]);
        return load16(m + (size_t)((uint32_t)kit * (uint32_t)(C::BK * C::ES)), a_off[q - C::CB]);
    }
    // Before the pieces of a stage that was fetched CHECKED are parked: keep what is inside K.  (A piece with nothing
    // inside K may have come from anywhere: nothing of it is kept.)
    __device__ __forceinline__ void cut(const GemmArgs& g, int kit, uint4 (&st)[C::PIECES]) const {
        if (kit < inside) return;
        int tid = threadIdx.x, col = a_col;      // (opaque: masks and rows are worked out here, not ahead of the loop and kept)
        asm volatile("" : "+v"(tid), "+v"(col));
        uint32_t mask[4];                        // of the bytes of an A piece
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int n = (g.K - kit * C::BK - col) * C::ES - 4 * j;
            mask[j] = n >= 4 ? ~0u : n <= 0 ? 0u : (1u << (8 * n)) - 1u;
        }
#pragma unroll
        for (int q = 0; q < C::PIECES; q++) {
            const uint32_t off = offset(g, kit, q), end = q < C::CB ? b_end : a_end;
            if (off > end && off - end < 16) st[q] = shift_piece(st[q], off - end);
            if (q < C::CB) {
                if (kit * C::BK + (tid + q * C::THREADS) / C::CPB >= g.K) st[q] = make_uint4(0, 0, 0, 0);
            } else {
                st[q] = make_uint4(st[q].x & mask[0], st[q].y & mask[1], st[q].z & mask[2], st[q].w & mask[3]);
            }
        }
    }
    static __device__ __forceinline__ void park(unsigned char* a_stage, unsigned char* b_stage, int q, uint4 v) {
        const int p = threadIdx.x + (q < C::CB ? q : q - C::CB) * C::THREADS;
        if (q < C::CB) {
            if (C::B_PIECES % C::THREADS == 0 || p < C::B_PIECES) reinterpret_cast<uint4*>(b_stage)[p] = v;
        } else {
            if (C::A_PIECES % C::THREADS == 0 || p < C::A_PIECES) reinterpret_cast<uint4*>(a_stage)[p] = v;
        }
    }
    // The stage of k-iteration kit of a problem with a matrix of less than 16 bytes.
    static __device__ __forceinline__ void fill_tiny(const GemmArgs& g, int m0, int n0, int kit, unsigned char* a_stage, unsigned char* b_stage) {
#pragma unroll 1
        for (int p = threadIdx.x; p < C::A_PIECES; p += C::THREADS) {
            const int r = p / C::CPA, c = (p % C::CPA) ^ swz_a<C::CPA>(r);
            reinterpret_cast<uint4*>(a_stage)[p] = load_piece<C::ES>(static_cast<const unsigned char*>(g.A), m0 + r, kit * C::BK + c * C::PE, g.M, g.K);
        }
#pragma unroll 1
        for (int p = threadIdx.x; p < C::B_PIECES; p += C::THREADS) {
            const int k = p / C::CPB, c = (p % C::CPB) ^ swz_b<C::FP8, C::CPB>(k);
            reinterpret_cast<uint4*>(b_stage)[p] = load_piece<C::ES>(static_cast<const unsigned char*>(g.B), kit * C::BK + k, n0 + c * C::PE, g.K, g.N);
        }
    }
};

// Per-tile addressing of the LDS-DMA loads: lane l of this wave's j-th A instruction fills A
// position (j * NW + wave) * 64 + l.  Rows beyond M and columns beyond N are clamped to the last
// valid one: they only feed output elements that are never stored.
template <class C> struct DmaMap {
    uint32_t a_off[C::A_LD > 0 ? C::A_LD : 1];   // byte offsets from A / B at k-iteration 0
    uint32_t b_off[C::B_LD > 0 ? C::B_LD : 1];
    __device__ __forceinline__ void init(const GemmArgs& g, int m0, int n0) {
        const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
#pragma unroll
        for (int j = 0; j < C::A_LD; j++) {
            const int p = (j * C::NW + wave % C::A_WAVES) * 64 + lane;
            const int r = p / C::CPA, c = (p % C::CPA) ^ swz_a<C::CPA>(r);
            int row = m0 + r;
            row = row < g.M ? row : g.M - 1;
            a_off[j] = ((uint32_t)row * (uint32_t)g.K + (uint32_t)(C::PE * c)) * C::ES;
        }
#pragma unroll
        for (int j = 0; j < C::B_LD; j++) {
            const int p = (j * C::NW + wave) * 64 + lane;
            const int k = p / C::CPB, c = (p % C::CPB) ^ swz_b<C::FP8, C::CPB>(k);
            int col = n0 + C::PE * c;
            col = col < g.N ? col : g.N - C::PE;
            b_off[j] = ((uint32_t)k * (uint32_t)g.N + (uint32_t)col) * C::ES;
        }
    }
    // Loads of k-iteration `kit`.  TAIL: the iteration reaches beyond K (K is a multiple of the
    // piece length here); pieces at k >= K are then fetched from a zero piece so that they add nothing.
    template <bool TAIL> __device__ __forceinline__ void issue_a(const GemmArgs& g, int kit, uint32_t lds, int j0 = 0, int j1 = C::A_LD) const {
        const int lane = threadIdx.x % 64;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64) % C::A_WAVES;
        const char* A = static_cast<const char*>(g.A) + (size_t)((uint32_t)kit * (uint32_t)(C::BK * C::ES));
#pragma unroll
        for (int j = 0; j < C::A_LD; j++) {
            if (j < j0 || j >= j1) continue;
            if (!TAIL) {
                lds_dma16(A, a_off[j], lds + (j * C::NW + wave) * 1024);
            } else {
                const int p = (j * C::NW + wave) * 64 + lane;
                const int r = p / C::CPA, c = (p % C::CPA) ^ swz_a<C::CPA>(r);
                const char* src = kit * C::BK + C::PE * c < g.K ? A + a_off[j] : reinterpret_cast<const char*>(g_zero_piece);
                lds_dma16_ptr(src, lds + (j * C::NW + wave) * 1024);
            }
        }
    }
    template <bool TAIL, bool NT = false> __device__ __forceinline__ void issue_b(const GemmArgs& g, int kit, uint32_t lds, int j0 = 0, int j1 = C::B_LD) const {
        const int lane = threadIdx.x % 64;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
        const char* B = static_cast<const char*>(g.B) + (size_t)((uint32_t)kit * (uint32_t)(C::BK * C::ES)) * (uint32_t)g.N;
#pragma unroll
        for (int j = 0; j < C::B_LD; j++) {
            if (j < j0 || j >= j1) continue;
            if (!TAIL) {
                if (NT) lds_dma16_nt(B, b_off[j], lds + (j * C::NW + wave) * 1024);
                else lds_dma16(B, b_off[j], lds + (j * C::NW + wave) * 1024);
            } else {
                const int p = (j * C::NW + wave) * 64 + lane;
                const char* src = kit * C::BK + p / C::CPB < g.K ? B + b_off[j] : reinterpret_cast<const char*>(g_zero_piece);
                lds_dma16_ptr(src, lds + (j * C::NW + wave) * 1024);
            }
        }
    }
};

// k-consecutive elements of one B column out of the row-major [k][n] LDS image.  16-bit: the
// transposing read hands lane j of each 16-lane group column j of a 4 x 16 block whose rows are
// addressed by lanes 4e..4e+3 of the group (4 k per read).  8-bit: an 8 x 16 block whose rows are
// addressed by lanes 2e, 2e+1 (8 k per read).
__device__ __forceinline__ uint2 read_b_tr16(const unsigned char* p) {
    s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p));
    return __builtin_bit_cast(uint2, v);
}
__device__ __forceinline__ i32x2 read_b_tr8(const unsigned char* p) {
    return __builtin_amdgcn_ds_read_tr8_b64_v2i32((i32x2 __attribute__((address_space(3)))*)(p));
}

// Lane-constant parts of the operand addresses inside a stage.
template <class C> struct FragMap {
    uint32_t a_kk[C::KK][C::APL];   // byte offsets of this lane's A piece(s) for k-step kk, block row 0
    uint32_t b_ni[C::NI];           // byte offset of this lane's first B read for block column ni, k-step 0
    __device__ __forceinline__ void init() {
        const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
        const int wm = wave / C::WN, wn = wave % C::WN;
        const int row = wm * C::WTM + lane % C::MF;          // + mi * MF keeps row % 16
#pragma unroll
        for (int kk = 0; kk < C::KK; kk++)
#pragma unroll
            for (int i = 0; i < C::APL; i++)
                a_kk[kk][i] = (row * C::CPA + ((kk * (C::KM / C::PE) + (lane / C::MF) * C::APL + i) ^ swz_a<C::CPA>(row))) * 16;
        // rows of one transposing read: 4 (16-bit) or 8 (8-bit); later reads and k-steps add multiples of that
        const int krow = C::KPL * (lane / C::MF) + (C::FP8 ? (lane % 16) / 2 : (lane % 16) / 4);
#pragma unroll
        for (int ni = 0; ni < C::NI; ni++) {
            const int col = wn * C::WTN + ni * C::MF + 16 * ((lane % C::MF) / 16) + (C::FP8 ? 8 * (lane % 2) : 4 * (lane % 4));
            b_ni[ni] = (krow * C::CPB + ((col / C::PE) ^ swz_b<C::FP8, C::CPB>(krow))) * 16 + (col % C::PE) * C::ES;
        }
    }
};

template <class C, bool FP8 = C::FP8> struct Frags;
template <class C> struct Frags<C, false> {
    uint4 a[C::MI], b[C::NI];
    // The LDS reads of one k-step one at a time, in the order in which the matrix-core work needs
    // them (block row 0, all block columns, the other block rows): read number r of READS.
    static constexpr int READS = C::MI + 2 * C::NI;
    __device__ __forceinline__ void load_one(const unsigned char* a_stage, const unsigned char* b_stage, const FragMap<C>& fm, int kk, int r) {
        if (r == 0 || r > 2 * C::NI) {
            const int mi = r == 0 ? 0 : r - 2 * C::NI;
            a[mi] = *reinterpret_cast<const uint4*>(a_stage + fm.a_kk[kk][0] + mi * C::MF * C::CPA * 16);
        } else {
            const int ni = (r - 1) / 2, h = (r - 1) % 2;
            const uint2 v = read_b_tr16(b_stage + fm.b_ni[ni] + kk * C::KM * C::CPB * 16 + h * 4 * C::CPB * 16);
            if (h == 0) { b[ni].x = v.x; b[ni].y = v.y; } else { b[ni].z = v.x; b[ni].w = v.y; }
        }
    }
    __device__ __forceinline__ void load(const unsigned char* a_stage, const unsigned char* b_stage, const FragMap<C>& fm, int kk) {
#pragma unroll
        for (int mi = 0; mi < C::MI; mi++)
            a[mi] = *reinterpret_cast<const uint4*>(a_stage + fm.a_kk[kk][0] + mi * C::MF * C::CPA * 16);
#pragma unroll
        for (int ni = 0; ni < C::NI; ni++) {
            const unsigned char* p = b_stage + fm.b_ni[ni] + kk * C::KM * C::CPB * 16;
            const uint2 lo = read_b_tr16(p), hi = read_b_tr16(p + 4 * C::CPB * 16);
            b[ni] = make_uint4(lo.x, lo.y, hi.x, hi.y);
        }
    }
};
template <class C> struct Frags<C, true> {
    i32x8 a[C::MI], b[C::NI];
    static constexpr int READS = 2 * C::MI + 4 * C::NI;
    __device__ __forceinline__ void load_one(const unsigned char* a_stage, const unsigned char* b_stage, const FragMap<C>& fm, int kk, int r) {
        if (r < 2 || r >= 2 + 4 * C::NI) {
            const int mi = r < 2 ? 0 : (r - 4 * C::NI) / 2, h = r % 2;
            const uint4 v = *reinterpret_cast<const uint4*>(a_stage + fm.a_kk[kk][h] + mi * C::MF * C::CPA * 16);
            a[mi][4 * h] = (int)v.x; a[mi][4 * h + 1] = (int)v.y; a[mi][4 * h + 2] = (int)v.z; a[mi][4 * h + 3] = (int)v.w;
        } else {
            const int ni = (r - 2) / 4, q = (r - 2) % 4;
            const i32x2 v = read_b_tr8(b_stage + fm.b_ni[ni] + kk * C::KM * C::CPB * 16 + q * 8 * C::CPB * 16);
            b[ni][2 * q] = v[0]; b[ni][2 * q + 1] = v[1];
        }
    }
    __device__ __forceinline__ void load(const unsigned char* a_stage, const unsigned char* b_stage, const FragMap<C>& fm, int kk) {
#pragma unroll
        for (int mi = 0; mi < C::MI; mi++) {
            const uint4 lo = *reinterpret_cast<const uint4*>(a_stage + fm.a_kk[kk][0] + mi * C::MF * C::CPA * 16);
            const uint4 hi = *reinterpret_cast<const uint4*>(a_stage + fm.a_kk[kk][1] + mi * C::MF * C::CPA * 16);
            a[mi] = i32x8{(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
        }
#pragma unroll
        for (int ni = 0; ni < C::NI; ni++) {
            const unsigned char* p = b_stage + fm.b_ni[ni] + kk * C::KM * C::CPB * 16;
            const i32x2 q0 = read_b_tr8(p), q1 = read_b_tr8(p + 8 * C::CPB * 16);
            const i32x2 q2 = read_b_tr8(p + 16 * C::CPB * 16), q3 = read_b_tr8(p + 24 * C::CPB * 16);
            b[ni] = i32x8{q0[0], q0[1], q1[0], q1[1], q2[0], q2[1], q3[0], q3[1]};
        }
    }
};

__device__ __forceinline__ u16 to_bf16_bits(float f) {
    return __builtin_bit_cast(u16, (__bf16)f);     // round to nearest even (one hardware instruction on gfx950)
}

template <class C, int LATER, int EXTRA = 0> __device__ __forceinline__ void wait_stage(int later) {
    // wait until the loads of the wanted stage have landed, given how many stages follow it; EXTRA:
    // vector-memory instructions that this wave is known to have issued after those loads besides the
    // later stages' loads (the counter retires in issue order, so they may stay in flight)
    if (LATER == 0 || later >= LATER) wait_vmcnt<(C::in_flight(LATER) + EXTRA < 63 ? C::in_flight(LATER) + EXTRA : 63)>();
    else wait_stage<C, (LATER > 0 ? LATER - 1 : 0), EXTRA>(later);
}

// The matrix-core work of one k-step.
// TR: pass the B block first and the A block second, which yields the transposed result block.
template <class C, bool TR>
__device__ __forceinline__ void mma_step(const Frags<C>& f, typename Mfma<C::DT, C::MF>::Acc (&acc)[C::MI][C::NI]) {
#pragma unroll
    for (int mi = 0; mi < C::MI; mi++)
#pragma unroll
        for (int ni = 0; ni < C::NI; ni++)
            acc[mi][ni] = TR ? Mfma<C::DT, C::MF>::run(f.b[ni], f.a[mi], acc[mi][ni]) : Mfma<C::DT, C::MF>::run(f.a[mi], f.b[ni], acc[mi][ni]);
}

// All k-steps of one stage, for the register-staged path: the operands of step kk+1 are read from
// LDS while the matrix cores work on step kk.
template <class C, bool TR>
__device__ __forceinline__ void mac_stage(const unsigned char* a_stage, const unsigned char* b_stage, const FragMap<C>& fm,
                                          typename Mfma<C::DT, C::MF>::Acc (&acc)[C::MI][C::NI]) {
    Frags<C> f[2];
    f[0].load(a_stage, b_stage, fm, 0);
#pragma unroll
    for (int kk = 0; kk < C::KK; kk++) {
        if (kk + 1 < C::KK) f[(kk + 1) & 1].load(a_stage, b_stage, fm, kk + 1);
        mma_step<C, TR>(f[kk & 1], acc);
    }
}

// Slice `step` of `steps` of request batch j of a segment (k-iterations k_begin .. k_begin + nk - 1 of a
// tile): the B tile of stage j + NSB, then the A tile of stage j + NSA, into ring slots slot_b / slot_a.
// STEADY: the caller knows that both stages exist and lie entirely inside K.
template <class C, bool STEADY, bool NT>
__device__ __forceinline__ void issue_requests(const GemmArgs& g, const DmaMap<C>& dm, uint32_t lds0, int k_begin, int nk, int full_k,
                                               int j, int slot_a, int slot_b, int step, int steps) {
    const int ib = j + C::NSB, ia = j + C::NSA;
    const int q0 = step * C::LPS / steps, q1 = (step + 1) * C::LPS / steps;
    const int b0 = q0 < C::B_LD ? q0 : C::B_LD, b1 = q1 < C::B_LD ? q1 : C::B_LD;
    const int a0 = q0 > C::B_LD ? q0 - C::B_LD : 0, a1 = q1 > C::B_LD ? q1 - C::B_LD : 0;
    if ((STEADY || (ib >= 0 && ib < nk)) && b1 > b0) {
        const uint32_t lds = lds0 + C::B_RING + slot_b * C::B_BYTES;
        if (STEADY || k_begin + ib < full_k) dm.template issue_b<false, NT>(g, k_begin + ib, lds, b0, b1);
        else dm.template issue_b<true, NT>(g, k_begin + ib, lds, b0, b1);
    }
    if ((STEADY || (ia >= 0 && ia < nk)) && a1 > a0) {
        const uint32_t lds = lds0 + slot_a * C::A_BYTES;
        if (STEADY || k_begin + ia < full_k) dm.template issue_a<false>(g, k_begin + ia, lds, a0, a1);
        else dm.template issue_a<true>(g, k_begin + ia, lds, a0, a1);
    }
}

// The first requests of a segment on the LDS-DMA path: of the batches that NSA stages before the first would have
// requested, numbers FIRST .. LAST - 1.  The ring must be free: no
// wave may still read operands of the previous segment.  All but the last batch are called for either at the start of the MAC loop
// (in two parts, see Cfg::START) or - for the segment after the current one - before the current tile's fix-up and epilogue, so that
// the first loads travel while the tile is stored; the last one once the first stage has landed.
template <class C, bool NT, int FIRST = 0, int LAST = C::NSA - 1>
__device__ __forceinline__ void mac_prefetch(const GemmArgs& g, int k_begin, int k_end, unsigned char* smem, const DmaMap<C>& dm) {
    const uint32_t lds0 = (uint32_t)(size_t)(lds_byte*)smem;
    const int nk = k_end - k_begin, full_k = g.K / C::BK;
#pragma unroll
    for (int j = FIRST - C::NSA; j < LAST - C::NSA; j++)
        issue_requests<C, false, NT>(g, dm, lds0, k_begin, nk, full_k, j, (j + C::NSA) % C::NSA, (j + 2 * C::NSB) % C::NSB, 0, 1);
}

// MAC loop of one segment on the register-staged path (rows of A or B that do not start on 16-byte
// boundaries: the LDS-DMA loads need aligned addresses).  Two LDS slots, stage s in slot s & 1.
//
// STAGED_FINE: the pipeline of the DMA path with registers in place of the deeper ring.  Trip i =
// [barrier that hands over stage i+1, one k-step before stage i ends] [last k-step of stage i, k-steps
// 0 .. KK-2 of stage i+1], written out slot by slot: one matrix-core instruction, its share of the next
// k-step's LDS reads, and one piece parked (stage i+2, into the slot that the barrier has freed) whose
// registers then take the same piece of stage i+3.  A load therefore has a whole trip to land.
// What bounds it is not settled: under-aligned 16-byte loads move about 25 bytes per clock and CU where
// aligned ones move 52 (a microbenchmark of this access pattern), and a 256 x 256 x 64 stage is 64 KB: 2600 clocks,
// against 2050 of matrix-core work.  3841 x 4225 x 4097 looks up 63 million cache lines in the vector L1 where the aligned
// neighbour looks up 19 (counters); its matrix cores are busy a third of the time, 0.63 there.  But loads widened to aligned
// ones, with half the look-ups, took longer (174 -> 187 us), and loads that wait for less changed nothing; a row's 128 bytes
// of A straddle two lines, so a stage fills 106 KB from L2.
template <class C, bool TR>
__device__ __forceinline__ void mac_loop_staged(const GemmArgs& g, int m0, int n0, int k_begin, int k_end, unsigned char* smem,
                                                const FragMap<C>& fm, typename Mfma<C::DT, C::MF>::Acc (&acc)[C::MI][C::NI]) {
    const int nk = k_end - k_begin;
    auto a_slot = [&](int s) { return smem + (s & 1) * C::A_BYTES; };
    auto b_slot = [&](int s) { return smem + C::B_RING + (s & 1) * C::B_BYTES; };
    if (StagedFill<C>::tiny(g)) {                // (K is at most 15 then: a single k-iteration)
        for (int k = k_begin; k < k_end; k++) {
            StagedFill<C>::fill_tiny(g, m0, n0, k, a_slot(0), b_slot(0));
            __syncthreads();
            mac_stage<C, TR>(a_slot(0), b_slot(0), fm, acc);
            __syncthreads();
        }
        return;
    }
    StagedFill<C> sf;
    sf.init(g, m0, n0);
    const int inside = sf.inside;
    if constexpr (C::STAGED_FINE) {
        constexpr int NM = C::MI * C::NI, SLOTS = C::KK * NM, PS = SLOTS * 7 / 8 > 0 ? SLOTS * 7 / 8 : 1;
        uint4 st[C::PIECES];
#pragma unroll
        for (int q = 0; q < C::PIECES; q++) st[q] = sf.template fetch<true>(g, k_begin, q);
        sf.cut(g, k_begin, st);
#pragma unroll
        for (int q = 0; q < C::PIECES; q++) sf.park(a_slot(0), b_slot(0), q, st[q]);
        if (nk > 1) {
#pragma unroll
            for (int q = 0; q < C::PIECES; q++) st[q] = sf.template fetch<true>(g, k_begin + 1, q);
        }
        Frags<C> f[2];
        // Kinds of trips: STEADY parks a stage and fetches one that is inside, CHECKED any, PARK has none left to fetch, QUIET none to park.
        // (Which it is is known at compile time: behind a branch the compiler waits for every load in flight, not only for
        // the piece that is parked, and the first and last trips of a segment took twice a steady one's time.  us: 1279 x 2045 on 128 x 128,
        // K = 253 / 509 / 2043, 8.7 -> 7.4, 11.4 -> 9.8, 25.6 -> 24.1; 256 x 128, 1535 x 2045 x 509 16.3 -> 14.1; 3841 x 4225 x 4097 161 -> 156.)
        enum { STEADY, CHECKED, PARK, QUIET };
        auto step = [&](int i, int k_step, auto read, const Frags<C>& cur, Frags<C>& nxt, int kk_next, auto kind) {
            constexpr int R = Frags<C>::READS, NRS = NM * 3 / 4 > 0 ? NM * 3 / 4 : 1, KIND = decltype(kind)::value;
#pragma unroll
            for (int s = 0; s < NM; s++) {
                const int mi = s / C::NI, ni = s % C::NI, slot = k_step * NM + s;
                acc[mi][ni] = TR ? Mfma<C::DT, C::MF>::run(cur.b[ni], cur.a[mi], acc[mi][ni]) : Mfma<C::DT, C::MF>::run(cur.a[mi], cur.b[ni], acc[mi][ni]);
                if (decltype(read)::value && s < NRS) {
#pragma unroll
                    for (int r = s * R / NRS; r < (s + 1) * R / NRS; r++) nxt.load_one(a_slot(i + 1), b_slot(i + 1), fm, kk_next, r);
                }
                if (KIND != QUIET && slot < PS) {
#pragma unroll
                    for (int q = slot * C::PIECES / PS; q < (slot + 1) * C::PIECES / PS; q++) {
                        sf.park(a_slot(i), b_slot(i), q, st[q]);
                        if (KIND != PARK) st[q] = sf.template fetch<KIND != STEADY>(g, k_begin + i + 3, q);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto trip = [&](int i, auto next, auto kind) {
            constexpr bool NEXT = decltype(next)::value;
            constexpr int KIND = decltype(kind)::value;
            if (NEXT) __syncthreads();
            if (KIND == CHECKED || KIND == PARK) sf.cut(g, k_begin + i + 2, st);
            __builtin_amdgcn_sched_barrier(0);
            step(i, 0, std::integral_constant<bool, NEXT>(), f[1], f[0], 0, kind);
            if (NEXT) {
#pragma unroll
                for (int kk = 0; kk < C::KK - 1; kk++) step(i, kk + 1, std::true_type(), f[kk & 1], f[(kk + 1) & 1], kk + 1, kind);
            }
        };
        // trips 0 .. n_steady-1 fetch a stage that exists and is inside: no checks in their body
        const int n_steady = (inside - k_begin < nk ? inside - k_begin : nk) - 3;
        f[1] = Frags<C>{};                       // trip -1 multiplies zeros: the other checked trips run its code
        int i = -1;
        while (i < nk - 3) {
            trip(i, std::true_type(), std::integral_constant<int, CHECKED>());
            i++;
            for (; i < n_steady; i++) trip(i, std::true_type(), std::integral_constant<int, STEADY>());
        }
        if (nk > 1) trip(nk - 3, std::true_type(), std::integral_constant<int, PARK>());
        trip(nk - 2, std::true_type(), std::integral_constant<int, QUIET>());
        trip(nk - 1, std::false_type(), std::integral_constant<int, QUIET>());
    } else {
        // The other tiles: HELD stages in registers, requested HELD k-iterations ahead of their use (HELD = 0: the
        // two operand sets leave no room, a stage is requested right before it is parked).
        constexpr int HELD = C::STAGES_HELD, H = HELD > 0 ? HELD : 1;
        uint4 st[H][C::PIECES];
        auto fetch_stage = [&](int kit, uint4 (&dst)[C::PIECES]) {
#pragma unroll
            for (int q = 0; q < C::PIECES; q++) dst[q] = sf.template fetch<true>(g, kit, q);
        };
        // whole rounds of H stages whose requests are all inside, then the rest
        auto consume = [&](int s, uint4 (&src)[C::PIECES], auto steady) {
            constexpr bool STEADY = decltype(steady)::value;
            if (HELD == 0) fetch_stage(k_begin + s, src);
            if (!STEADY) sf.cut(g, k_begin + s, src);
#pragma unroll
            for (int q = 0; q < C::PIECES; q++) sf.park(a_slot(s), b_slot(s), q, src[q]);
            if (HELD > 0) {
                if (STEADY) {
#pragma unroll
                    for (int q = 0; q < C::PIECES; q++) src[q] = sf.template fetch<false>(g, k_begin + s + H, q);
                } else if (s + H < nk) {
                    fetch_stage(k_begin + s + H, src);
                }
            }
            __syncthreads();      // also: every wave is done with the other slot (stage s-1)
            mac_stage<C, TR>(a_slot(s), b_slot(s), fm, acc);
        };
        if constexpr (!C::STAGED_ROUNDS) {
            if (HELD > 0) {
#pragma unroll
                for (int h = 0; h < H; h++)
                    if (h < nk) fetch_stage(k_begin + h, st[h]);
            }
            const int n_steady = HELD == 0 ? 0 : (inside - k_begin < nk ? inside - k_begin : nk) - H;
            int s = 0;
            for (; s + H <= n_steady; s += H) {
#pragma unroll
                for (int h = 0; h < H; h++) consume(s + h, st[h], std::true_type());
            }
            for (; s < nk; s += H) {
#pragma unroll
                for (int h = 0; h < H; h++)
                    if (s + h < nk) consume(s + h, st[h], std::false_type());
            }
        } else {
            // The first round filled up with `pad` stages in front that do not exist; each round fetches the next one's stages, the
            // last one none.  Padding in front, and fetching in the first round where nothing is multiplied, leaves the same loads in
            // flight behind a stage's own whatever the number of stages: where that depends on a branch the compiler waits
            // for every load in flight before a stage is parked.
            const int rounds = (nk + H - 1) / H, pad = rounds * H - nk;
            auto round = [&](int r, int skip, auto checked, auto more) {
#pragma unroll
                for (int h = 0; h < H; h++) {
                    const int s = r * H + h - pad;
                    if (!decltype(checked)::value || h >= skip) {
                        if (decltype(checked)::value) sf.cut(g, k_begin + s, st[h]);
#pragma unroll
                        for (int q = 0; q < C::PIECES; q++) sf.park(a_slot(s), b_slot(s), q, st[h][q]);
                    }
                    if (decltype(more)::value) {
#pragma unroll
                        for (int q = 0; q < C::PIECES; q++) st[h][q] = sf.template fetch<decltype(checked)::value>(g, k_begin + s + H, q);
                    }
                    if (!decltype(checked)::value || h >= skip) {
                        __syncthreads();
                        mac_stage<C, TR>(a_slot(s), b_slot(s), fm, acc);
                    }
                }
            };
#pragma unroll
            for (int h = 0; h < H; h++)
                if (h >= pad) fetch_stage(k_begin + h - pad, st[h]);
            // rounds 1 .. n_steady-1 multiply and fetch stages that are inside
            const int n_steady = ((inside - k_begin < nk ? inside - k_begin : nk) + pad) / H - 1;
            int r = 0;
            while (r < rounds - 1) {
                round(r, r == 0 ? pad : 0, std::true_type(), std::true_type());
                r++;
                for (; r < n_steady; r++) round(r, 0, std::false_type(), std::true_type());
            }
            round(r, r == 0 ? pad : 0, std::true_type(), std::false_type());
        }
    }
    __syncthreads();                             // all reads done before the next segment refills
}

// MAC loop of one segment (Algorithm 1's MAC-loop call): k-iterations [k_begin, k_end) of one tile.
//
// Software pipeline of the LDS-DMA path.  Stage s (one k-iteration) lives in A ring slot s % NSA and
// B ring slot s % NSB.  The barrier that hands stage i+1 to the waves sits one k-step *before* the
// end of stage i: by then every wave has read the operands of stage i's last k-step into registers,
// so (1) stage i's slots can be refilled at once (with stages i+NSB / i+NSA), (2) the operands of
// stage i+1's first k-step are read while the matrix cores still work on stage i's last one, and
// (3) the time a wave spends at the barrier is covered by matrix-core work already queued.
// prefetched / stores_in_flight (LDS-DMA path only): prefetched says that mac_prefetch has already been
// called for this segment; stores_in_flight that this wave has since issued exactly C::EPILOGUE_STORES (or
// more) other vector-memory instructions, which the first wait may leave in flight.  (The per-tile
// addressing is worked out again here rather than kept from the prefetch: kept in registers across the
// epilogue it gets spilled, and a reload pending at the loop's entry makes the compiler wait for every
// outstanding load inside the steady-state trips.)
template <class C, bool ALIGNED, bool TR, bool NT>
__device__ __forceinline__ void mac_loop(const GemmArgs& g, int m0, int n0, int k_begin, int k_end,
                                         unsigned char* smem, const FragMap<C>& fm,
                                         typename Mfma<C::DT, C::MF>::Acc (&acc)[C::MI][C::NI],
                                         bool prefetched, bool stores_in_flight) {
    const int nk = k_end - k_begin;
    if constexpr (ALIGNED) {
        static_assert(C::KK % 2 == 0, "operand double buffering assumes an even number of k-steps");
        const uint32_t lds0 = (uint32_t)(size_t)(lds_byte*)smem;
        const int full_k = g.K / C::BK;             // iterations below this index are entirely inside K
        DmaMap<C> dm;
        dm.init(g, m0, n0);
        if (!prefetched) mac_prefetch<C, NT, 0, C::START>(g, k_begin, k_end, smem, dm);
        // request batch j (issued after the barrier of stage j): B tile of stage j+NSB, then A tile of
        // stage j+NSA, into the slots of stage j; step / steps select a slice of the batch
        // (steady: 1, nothing to check; 0: see issue_requests; -1: a trip that requests nothing)
        auto issue_batch = [&](int j, int slot_a, int slot_b, int step, int steps, auto steady) {
            if (decltype(steady)::value >= 0) issue_requests<C, decltype(steady)::value == 1, NT>(g, dm, lds0, k_begin, nk, full_k, j, slot_a, slot_b, step, steps);
        };
        Frags<C> f[2];
        int ca = C::NSA - 1, cb = C::NSB - 1;        // ring slots of stage i (i = -1: the slots batch -1 fills)
        // one trip = [barrier that hands over stage i+1] [operands of stage i+1's first k-step]
        //            [requests of batch i, sliced over the k-steps] [last k-step of stage i]
        //            [k-steps 0 .. KK-2 of stage i+1, each preceded by the operand reads of the next one].
        // FIRST: i = -1, no stage i yet.  NEXT: whether a stage i+1 exists.  Where registers allow two
        // operand sets (PIN_ORDER), NEXT is a compile-time fact - the steady-state loop body then has
        // no joins between the LDS reads and the matrix-core work (the compiler's wait-count
        // bookkeeping merges conservatively at joins) - and scheduling barriers keep the reads of
        // k-step kk+1 ahead of the matrix-core work of k-step kk.  Otherwise the compiler is left
        // to order reads and matrix-core work so that one operand set suffices.
        // FINE: one k-step written out slot by slot.  Slot s = [matrix-core instruction s of the k-step
        // on operand set `cur`] [its share of the LDS reads that fill `nxt` with the operands of k-step
        // kk_next of stage i+1: the reads go into the first three quarters of the slots, so that the
        // last of them has long landed when the k-step ends] [its share of request batch i, spread
        // evenly over all slots of the trip].  A scheduling barrier after every slot keeps that order:
        // a wave that has a SIMD to itself issues about five other instructions in the shadow of one
        // matrix-core instruction, and issued in a block they would drain the matrix-core pipe.
        auto fine_step = [&](int i, int step, auto mma, auto read, const Frags<C>& cur, Frags<C>& nxt,
                             const unsigned char* a_next, const unsigned char* b_next, int kk_next, auto steady) {
            constexpr int NM = C::MI * C::NI, R = Frags<C>::READS, NRS = NM * 3 / 4 > 0 ? NM * 3 / 4 : 1;
#pragma unroll
            for (int s = 0; s < NM; s++) {
                const int mi = s / C::NI, ni = s % C::NI;
                if (decltype(mma)::value)
                    acc[mi][ni] = TR ? Mfma<C::DT, C::MF>::run(cur.b[ni], cur.a[mi], acc[mi][ni]) : Mfma<C::DT, C::MF>::run(cur.a[mi], cur.b[ni], acc[mi][ni]);
                if (decltype(read)::value && s < NRS) {
#pragma unroll
                    for (int r = s * R / NRS; r < (s + 1) * R / NRS; r++) nxt.load_one(a_next, b_next, fm, kk_next, r);
                }
                issue_batch(i, ca, cb, step * NM + s, C::KK * NM, steady);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        // Wait for the segment's first stage and request the rest of the ring, all of which is free (the last one: FILL_FIRST).
        auto wait_first = [&]() {
            if (!prefetched) {
                wait_stage<C, C::START - 1>(nk - 1);
                mac_prefetch<C, NT, C::START, C::NSA - 1>(g, k_begin, k_end, smem, dm);
            } else if (stores_in_flight) {
                wait_stage<C, C::NSA - 1, C::EPILOGUE_STORES>(nk - 1);
            } else {
                wait_stage<C, C::NSA - 1>(nk - 1);
            }
            if (C::FILL_FIRST) mac_prefetch<C, NT, C::NSA - 1, C::NSA>(g, k_begin, k_end, smem, dm);
        };
        auto trip = [&](int i, auto first, auto next, auto steady) {
            constexpr bool FIRST = decltype(first)::value;
            constexpr bool STEADY = decltype(steady)::value == 1;   // batch i's stages exist and need no K-tail handling, and at least NSA - 1 stages follow stage i + 1
            constexpr int NEXT = decltype(next)::value;          // 1 / 0: known, -1: decided at run time
            const bool has_next = NEXT < 0 ? i + 1 < nk : NEXT == 1;
            const int na = ca + 1 == C::NSA ? 0 : ca + 1, nb = cb + 1 == C::NSB ? 0 : cb + 1;   // slots of stage i+1
            const unsigned char* a_next = smem + na * C::A_BYTES;
            const unsigned char* b_next = smem + C::B_RING + nb * C::B_BYTES;
            if constexpr (C::FINE) {
                static_assert(!C::FINE || NEXT >= 0, "known at compile time under PIN_ORDER");
                if (NEXT) {
                    if (STEADY) wait_vmcnt<C::in_flight(C::NSA - 1)>();
                    else if (FIRST) wait_first();
                    else wait_stage<C, C::NSA - 1>(nk - 2 - i);
                    __syncthreads();
                }
                __builtin_amdgcn_sched_barrier(0);
                // last k-step of stage i, with the reads of stage i+1's first k-step
                fine_step(i, 0, std::integral_constant<bool, !FIRST>(), std::integral_constant<bool, NEXT == 1>(), f[1], f[0], a_next, b_next, 0, steady);
                if (NEXT) {
#pragma unroll
                    for (int kk = 0; kk < C::KK - 1; kk++)
                        fine_step(i, kk + 1, std::true_type(), std::true_type(), f[kk & 1], f[(kk + 1) & 1], a_next, b_next, kk + 1, steady);
                }
                ca = na;
                cb = nb;
                return;
            }
            if (has_next) {
                if (STEADY) wait_vmcnt<C::in_flight(C::NSA - 1)>();
                else if (FIRST) wait_first();
                else wait_stage<C, C::NSA - 1>(nk - 2 - i);   // stage i+1 has landed (this wave's share)
                __syncthreads();                         // ... and everybody's; stage i's slots are free
                f[0].load(a_next, b_next, fm, 0);
            }
            issue_batch(i, ca, cb, 0, C::KK, steady);
            if (C::PIN_ORDER) __builtin_amdgcn_sched_barrier(0);
            if (!FIRST) mma_step<C, TR>(f[1], acc);          // last k-step of stage i
            if (has_next) {
#pragma unroll
                for (int kk = 0; kk < C::KK - 1; kk++) {
                    if (C::PIN_ORDER) __builtin_amdgcn_sched_barrier(0);
                    f[(kk + 1) & 1].load(a_next, b_next, fm, kk + 1);
                    issue_batch(i, ca, cb, kk + 1, C::KK, steady);
                    if (C::PIN_ORDER) __builtin_amdgcn_sched_barrier(0);
                    mma_step<C, TR>(f[kk & 1], acc);
                }
            }
            ca = na;
            cb = nb;
        };
        typedef std::integral_constant<int, 1> Yes;
        typedef std::integral_constant<int, 0> No;
        typedef std::integral_constant<int, -1> AtRunTime;
        // Trips 0 .. n_steady-1 request stages that exist and lie inside K: their body carries neither
        // range checks nor the K-tail variant of the requests, and waits with a constant count.  The first trip (where wait_first
        // has filled the ring) and those from nk - NSB on request nothing, and a copy of the trip without requests serves them: slot by
        // slot the checks cost 0.05 - 0.2 us a trip, NSA of them per segment.  With START, us: 512^3 f16 4.71 -> 4.42, 1280 x 2048 x 256
        // on 128 x 128 6.36 -> 5.89, 640 x 1024 x 512 on 64 x 64 5.49 -> 5.01, 1472 x 1936 x 144 6.26 -> 5.64, 1008 x 1200 x 1040 9.43 -> 9.19.
        int n_steady = (full_k - k_begin < nk ? full_k - k_begin : nk) - C::NSA;
        if (n_steady < 0) n_steady = 0;
        typedef std::integral_constant<int, -1> Quiet;
        if constexpr (C::PIN_ORDER) {
            trip(-1, std::true_type(), Yes(), std::conditional_t<C::FILL_FIRST, Quiet, No>());
            int i = 0;
            for (; i < n_steady; i++) trip(i, std::false_type(), Yes(), Yes());
            for (; i < nk - C::NSB; i++) trip(i, std::false_type(), Yes(), No());
            for (; i < nk - 1; i++) trip(i, std::false_type(), Yes(), Quiet());
            trip(nk - 1, std::false_type(), No(), Quiet());
        } else {
            // (The one tile whose accumulators leave no room for a second operand set, 8-bit 256 x 256 on eight waves, has no
            // copy of the trip without requests: with one the compiler keeps accumulators in scratch, 14464 x 1632 x 6432 172 us ->
            // 1595.)
            trip(-1, std::true_type(), AtRunTime(), No());
            int i = 0;
            for (; i < n_steady; i++) trip(i, std::false_type(), Yes(), Yes());
            for (; i < nk; i++) trip(i, std::false_type(), AtRunTime(), No());
        }
        __syncthreads();                             // all reads done before the next segment refills
    } else {
        mac_loop_staged<C, TR>(g, m0, n0, k_begin, k_end, smem, fm, acc);
    }
}

// Wait until `count` contributors have raised their flags: workgroups first, first + stride, ...
// The lanes of the calling wave watch up to 64 flags at a time, one flag each, so the wait costs one
// round trip however many flags there are.  A lane that has seen its flag takes it down again:
// every flag is watched by exactly one lane of one waiting workgroup, so all flags are back at zero
// when the kernel ends and the next launch (or a replay of a captured launch) starts from the same
// state.  The wait is bounded: after spin_limit unsuccessful polls it is recorded in the status word
// and given up.
__device__ __forceinline__ void wait_flags(const GemmArgs& g, int first, int count, int stride) {
    const int lane = threadIdx.x % 64;
    uint32_t polls = 0;
    for (int base = 0; base < count; base += 64) {
        const bool mine = base + lane < count;
        uint32_t* flag = g.flags + (size_t)(first + (mine ? base + lane : 0) * stride) * (SK_FLAG_STRIDE / 4);
        bool seen = !mine;
        while (true) {
            if (!seen && __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) {
                seen = true;
                __hip_atomic_store(flag, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (__all(seen)) break;
            if (polls++ >= g.spin_limit) {
                if (lane == 0) __hip_atomic_store(g.status, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            __builtin_amdgcn_s_sleep(2);
        }
    }
}

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>)
template <int N, class F, int... I>
__device__ __forceinline__ void for_each_below_impl(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>()), ...); }
template <int N, class F>
__device__ __forceinline__ void for_each_below(F&& f) { for_each_below_impl<N>(f, std::make_integer_sequence<int, N>()); }

// A workgroup's slot of the workspace: the partial tile in register order, 16 bytes per lane side by side: registers 4q .. 4q + 3
// of block b of all lanes are at ((b * ACC / 4 + q) * THREADS + thread) * 16.  Accessed at device scope (sc1), as the flags
// are: coherent across the XCDs' L2 caches without a write-back or an invalidation.  The slot is addressed by a descriptor
// in scalar registers (64-bit addresses per lane do not fit beside the accumulators of the large tiles).
// WIDE: as above; otherwise register r of block b at ((b * ACC + r) * THREADS + thread) * 4 (the register-staged four-wave
// 256 x 256 kernels, whose accumulators fill the accumulation registers: in groups of four they spilled 510 registers, in 8 bits 940).
template <class C, bool WIDE> struct Slot {
    static constexpr int DEVICE_SCOPE = 16;      // sc1, among the cache policy bits of the instruction
    buffer_rsrc rsrc;
    // An offset that is put into its register where it is used: left alone the compiler loads all of them at the kernel's start,
    // more than there are scalar registers, and every launch waits for that.
    static __device__ __forceinline__ int here(int offset) {
        if (offset) asm volatile("" : "+s"(offset));
        return offset;
    }
    // !WIDE: four accesses share an offset register, what lies between them is in the instructions.  With an offset register
    // each the moves bound the round trips: 507 x 1021 x 4093 on 32 workgroups a tile 105.4 us, 90.7 now, 256 x 256 x 32 tiles 96.1 / 81.0,
    // 8 bits x 8189 111.5 / 97.3.  (The lane's offset is taken anew for each block, or the compiler adds ahead of the loops and
    // keeps four registers.)
    static __device__ __forceinline__ int lane_here() {
        int offset = (int)threadIdx.x * 4;
        asm volatile("" : "+v"(offset));
        return offset;
    }
    __device__ __forceinline__ explicit Slot(const float* start)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(start), 0, C::BM * C::BN * 4, BUFFER_RAW)) {}
    template <class Acc> __device__ __forceinline__ void park(int block, const Acc& acc) const {
        if constexpr (WIDE) {
#pragma unroll
            for (int q = 0; q < C::ACC / 4; q++)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]}),
                                                       rsrc, (int)threadIdx.x * 16, here((block * (C::ACC / 4) + q) * C::THREADS * 16), DEVICE_SCOPE);
        } else {
            const int lane = lane_here();
#pragma unroll
            for (int q = 0; q < C::ACC / 4; q++) {
                const int at = here((block * (C::ACC / 4) + q) * C::THREADS * 16);
#pragma unroll
                for (int e = 0; e < 4; e++)
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[4 * q + e]), rsrc, lane + e * C::THREADS * 4, at, DEVICE_SCOPE);
            }
        }
    }
    template <class Acc> __device__ __forceinline__ void fetch(int block, Acc& v) const {
        if constexpr (WIDE) {
#pragma unroll
            for (int q = 0; q < C::ACC / 4; q++) {
                const f32x4 w = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)threadIdx.x * 16, here((block * (C::ACC / 4) + q) * C::THREADS * 16), DEVICE_SCOPE));
#pragma unroll
                for (int e = 0; e < 4; e++) v[4 * q + e] = w[e];
            }
        } else {
            const int lane = lane_here();
#pragma unroll
            for (int q = 0; q < C::ACC / 4; q++) {
                const int at = here((block * (C::ACC / 4) + q) * C::THREADS * 16);
#pragma unroll
                for (int e = 0; e < 4; e++)
                    v[4 * q + e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, lane + e * C::THREADS * 4, at, DEVICE_SCOPE));
            }
        }
    }
};

template <class C, bool TR> constexpr bool WIDE_SLOT = TR || C::ACC_REGS < 256;

// Blocks FIRST .. FIRST + N - 1 of a wave tile: blks += their share of the parked partial tiles src, src + stride, ...
// (`count` of them), in that order, one contributor per round trip.
template <class C, bool WIDE, int FIRST, int N>
__device__ __forceinline__ void add_block_partials(typename Mfma<C::DT, C::MF>::Acc (&blks)[N], const float* src, int count, ptrdiff_t stride) {
#pragma unroll 1
    for (int c = 0; c < count; c++, src += stride) {
        typename Mfma<C::DT, C::MF>::Acc v[N];
        const Slot<C, WIDE> slot(src);
#pragma unroll
        for (int b = 0; b < N; b++) slot.fetch(FIRST + b, v[b]);
        __builtin_amdgcn_sched_barrier(0);     // all loads of the round trip in flight before the first addition waits for one
#pragma unroll
        for (int b = 0; b < N; b++)
#pragma unroll
            for (int r = 0; r < C::ACC; r++) blks[b][r] += v[b][r];
    }
}

// sum += the parked partial tiles src, src + stride, ... (`count` of them, this lane's share), in
// that order.  Tiles with at most 64 accumulators per lane: a contributor's whole share is
// fetched at once and G contributors per round trip (about 64 registers of loads in flight).
// The 256 x 256 tile: what bounds an owner is the chain of its round trips, each of which fetches what the registers beside the
// accumulators hold.  SUM_BLOCKS blocks of one contributor each, four round trips for a tile with one contributor, the commonest
// case where the tiles are deep; one block of two contributors each were eight of them.  With that and 16 bytes per lane and
// access instead of 4 (all tiles), us, before -> two blocks -> and 16 bytes: 4608 x 4608 x 1024 65.6 -> 54.3 -> 52.9 (all tiles split),
// 256 x 512 x 16384 101 -> 84 -> 76 (127 contributors), 3848 x 4232 x 4104 136 -> 126 -> 125, 6144 x 4096 x 2048 105 -> 93 -> 93;
// 128 x 8192 x 8192 with 128 x 128 tiles 37.0 -> 36.1, 1 x 4096 x 4096 9.81 -> 9.69.  Four blocks spill 46 registers and more.
template <class C> constexpr int SUM_BLOCKS = 2;
template <class C, bool WIDE>
__device__ __forceinline__ void add_partials(typename Mfma<C::DT, C::MF>::Acc (&sum)[C::MI][C::NI], const float* src, int count, ptrdiff_t stride) {
    typedef typename Mfma<C::DT, C::MF>::Acc Acc;
    if constexpr (C::ACC_REGS > 64) {
        constexpr int N = SUM_BLOCKS<C>;
        for_each_below<C::MI * C::NI / N>([&](auto chunk) {
            constexpr int first = decltype(chunk)::value * N;
            Acc blks[N];
#pragma unroll
            for (int b = 0; b < N; b++) blks[b] = sum[(first + b) / C::NI][(first + b) % C::NI];
            add_block_partials<C, WIDE, first, N>(blks, src, count, stride);
#pragma unroll
            for (int b = 0; b < N; b++) sum[(first + b) / C::NI][(first + b) % C::NI] = blks[b];
            __builtin_amdgcn_sched_barrier(0);
        });
    } else {
    constexpr int G = 64 / C::ACC_REGS < 8 ? 64 / C::ACC_REGS : 8;
    auto add_group = [&](const float* p, auto cnt) {
        constexpr int CNT = decltype(cnt)::value;
        Acc v[CNT][C::MI * C::NI];
#pragma unroll
        for (int j = 0; j < CNT; j++) {
            const Slot<C, WIDE> slot(p + j * stride);
#pragma unroll
            for (int b = 0; b < C::MI * C::NI; b++) slot.fetch(b, v[j][b]);
        }
        __builtin_amdgcn_sched_barrier(0);     // all loads of the round trip in flight before the first addition waits for one
#pragma unroll
        for (int j = 0; j < CNT; j++)
#pragma unroll
            for (int mi = 0; mi < C::MI; mi++)
#pragma unroll
                for (int ni = 0; ni < C::NI; ni++)
#pragma unroll
                    for (int r = 0; r < C::ACC; r++) sum[mi][ni][r] += v[j][mi * C::NI + ni][r];
    };
    int c = 0;
    for (; c + G <= count; c += G, src += G * stride) add_group(src, std::integral_constant<int, G>());
    // the 1 .. G-1 contributors left over: one round trip for all of them (the order of the additions is
    // the same whatever the grouping)
    for_each_below<G>([&](auto r) {
        if (decltype(r)::value > 0 && count - c == decltype(r)::value) add_group(src, std::integral_constant<int, decltype(r)::value < 1 ? 1 : decltype(r)::value>());
    });
    }
}

// Two fp32 values -> one register of two 16-bit values, round to nearest even (gfx950 converts a
// pair to bf16 with one instruction).
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{lo, hi}), bf16x2));
}
__device__ __forceinline__ uint32_t pack_f16(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{lo, hi}), f16x2));
}

// The other 8-lane half of a lane's 16-lane row.
__device__ __forceinline__ uint32_t swap_lane8(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128 /* row_ror:8 */, 0xf, 0xf, true);
}

// Convert and store NB accumulator blocks that lie side by side (the transposed blocks in pairs where a wave has an
// even number of them, see STORE_BLOCKS).
// TR (transposed blocks; used when rows of D start on 16-byte boundaries and N is a multiple of 8):
// lane l holds row `row` (= block row l % MF) and in registers 4q..4q+3 the columns
// col0 + 4*KG*q + {0..3}, col0 already including 4 * (l / MF).  A group of 4 (8) columns
// starting at a multiple of 4 (8) is then inside N as a whole or not at all.
// 32 x 32 blocks are packed into 16 bytes per lane and group (16-bit outputs exchange register pairs between lanes
// l and l + 32 for that), and the groups are exchanged between the 16-lane rows and the 8-lane halves so that
// one store instruction writes 8 rows of 128 bytes.  What that is for: the same bytes written as 32 rows of 32 bytes,
// 16 of 64, 8 of 128 or 4 of 256 reach 2.6 / 3.9 / 5.2 / 5.6 TB/s (a kernel that only stores 256 x 256 tiles of an
// 8192 x 8192 16-bit matrix).  A single 32-column block of 16-bit values only has 64 bytes per row.
// Not TR: lane l holds column `col0` (= block column l % MF) and in register r the row
// row + 4*KG*(r/4) + r%4, `row` already including 4 * (l / MF); stored element by element, the
// lanes of one store instruction side by side in a row of D.
template <class C, int OUT, bool TR> constexpr int STORE_BLOCKS = TR && C::MF == 32 && OUT != SK_F32 && C::NI % 2 == 0 ? 2 : 1;
template <class C, int OUT, bool EDGE, bool TR, int NB>
__device__ __forceinline__ void store_blocks(const GemmArgs& g, int row, int col0, const typename Mfma<C::DT, C::MF>::Acc (&blks)[NB]) {
    constexpr int Q = C::ACC / 4, QS = 4 * C::KG;    // register groups per lane, distance between their rows / columns
    if constexpr (!TR) {
        static_assert(NB == 1, "pairs of transposed blocks only");
#pragma unroll
        for (int r = 0; r < C::ACC; r++) {
            const int rr = row + (r / 4) * QS + r % 4;
            if (!EDGE || (rr < g.M && col0 < g.N)) {
                const size_t o = (size_t)((uint32_t)rr * (uint32_t)g.N + (uint32_t)col0);
                if (OUT == SK_F32) static_cast<float*>(g.D)[o] = blks[0][r];
                else if (OUT == SK_BF16) static_cast<u16*>(g.D)[o] = to_bf16_bits(blks[0][r]);
                else static_cast<_Float16*>(g.D)[o] = (_Float16)blks[0][r];
            }
        }
        return;
    }
    auto pack = [](float lo, float hi) { return OUT == SK_BF16 ? pack_bf16(lo, hi) : pack_f16(lo, hi); };
    if constexpr (C::MF == 32) {
        // v[i]: 16 bytes of row l % 32 at 16-byte slot (l / 32) + 2 * i of its 64 or 128 bytes
        constexpr int ES = OUT == SK_F32 ? 4 : 2, COLS = 16 / ES, G = OUT == SK_F32 ? 4 : 2 * NB;
        u32x4 v[G];
#pragma unroll
        for (int i = 0; i < G; i++) {
            if constexpr (OUT == SK_F32) {
                v[i] = __builtin_bit_cast(u32x4, f32x4{blks[0][4 * i], blks[0][4 * i + 1], blks[0][4 * i + 2], blks[0][4 * i + 3]});
            } else {
                const auto& blk = blks[i / 2];
                const int q = 8 * (i % 2);
                const u32x2 d0 = __builtin_amdgcn_permlane32_swap(pack(blk[q], blk[q + 1]), pack(blk[q + 4], blk[q + 5]), false, false);
                const u32x2 d1 = __builtin_amdgcn_permlane32_swap(pack(blk[q + 2], blk[q + 3]), pack(blk[q + 6], blk[q + 7]), false, false);
                v[i] = u32x4{d0[0], d1[0], d0[1], d1[1]};
            }
        }
        const int lane = threadIdx.x % 64;
        if constexpr (C::DIRECT_STORES) {
#pragma unroll
            for (int i = 0; i < G; i++) {
                const int col = col0 - 4 * (lane / 32) + COLS * (lane / 32 + 2 * i);
                if (!EDGE || (row < g.M && col < g.N))
                    *reinterpret_cast<u32x4*>(static_cast<char*>(g.D) + (size_t)((uint32_t)row * (uint32_t)g.N + (uint32_t)col) * ES) = v[i];
            }
            return;
        }
        const bool upper8 = (lane & 8) != 0;
        // w[h][i]: row 16 * h + l % 16 at slot (l / 32) + 2 * (l / 16 % 2) + 4 * i
        u32x4 w[2][G / 2];
#pragma unroll
        for (int i = 0; i < G / 2; i++)
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const u32x2 x = __builtin_amdgcn_permlane16_swap(v[2 * i][e], v[2 * i + 1][e], false, false);
                w[0][i][e] = x[0];
                w[1][i][e] = x[1];
            }
        constexpr int ROWS = G == 4 ? 8 : 16;                // rows of one store instruction
        const int slot = lane / 32 + 2 * (lane / 16 % 2) + (G == 4 ? 4 * (lane / 8 % 2) : 0);
        const int first = row - lane % 32 + lane % ROWS, col = col0 - 4 * (lane / 32) + COLS * slot;
        auto put = [&](int r, const u32x4& x) {
            if (!EDGE || (r < g.M && col < g.N))
                *reinterpret_cast<u32x4*>(static_cast<char*>(g.D) + (size_t)((uint32_t)r * (uint32_t)g.N + (uint32_t)col) * ES) = x;
        };
#pragma unroll
        for (int h = 0; h < 2; h++) {
            if constexpr (G == 4) {
                u32x4 lo, hi;                                // rows 16 * h + l % 8 and 8 further down, slot + 4 in the upper lanes
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const uint32_t got = swap_lane8(upper8 ? w[h][0][e] : w[h][1][e]);
                    lo[e] = upper8 ? got : w[h][0][e];
                    hi[e] = upper8 ? w[h][1][e] : got;
                }
                put(first + 16 * h, lo);
                put(first + 16 * h + 8, hi);
            } else {
                put(first + 16 * h, w[h][0]);
            }
        }
    } else {
        static_assert(NB == 1, "pairs of 32 x 32 blocks only");
        const bool row_ok = !EDGE || row < g.M;
        const uint32_t row_off = (uint32_t)row * (uint32_t)g.N;
#pragma unroll
        for (int q = 0; q < Q; q++) {
            const int col = col0 + q * QS;
            const auto& blk = blks[0];
            if (row_ok && (!EDGE || col < g.N)) {
                if constexpr (OUT == SK_F32)
                    *reinterpret_cast<f32x4*>(static_cast<float*>(g.D) + (size_t)(row_off + (uint32_t)col)) =
                        f32x4{blk[4 * q], blk[4 * q + 1], blk[4 * q + 2], blk[4 * q + 3]};
                else
                    *reinterpret_cast<u32x2*>(static_cast<u16*>(g.D) + (size_t)(row_off + (uint32_t)col)) =
                        u32x2{pack(blk[4 * q], blk[4 * q + 1]), pack(blk[4 * q + 2], blk[4 * q + 3])};
            }
        }
    }
}

// Epilogue of a tile's owner (or of an unsplit tile, n_contrib = 0): add the parked partials of the
// contributors part0, part0 + part_stride, ... (a fixed order: away from the owner in k), convert and store.  OUT selects the
// output type, EDGE adds the bounds checks, TR says that the blocks are transposed (see store_blocks).
// row0 / col0: the lane's (first) row and (first) column in the wave's first block.  The big tiles
// work one block (or pair of blocks) at a time, which keeps their register need flat.
template <class C, int OUT, bool EDGE, bool TR>
__device__ __forceinline__ void reduce_and_store(const GemmArgs& g, int row0, int col0, const float* part0, int n_contrib,
                                                 ptrdiff_t part_stride, const typename Mfma<C::DT, C::MF>::Acc (&acc)[C::MI][C::NI]) {
    typedef typename Mfma<C::DT, C::MF>::Acc Acc;
    constexpr int NB = STORE_BLOCKS<C, OUT, TR>;
    // Tiles with few accumulators per lane fetch a contributor's whole share at once (one round trip
    // per contributor instead of one per block and contributor); the big tiles have no registers for that.
    constexpr bool WHOLE = C::ACC_REGS <= 64, WIDE = WIDE_SLOT<C, TR>;
    Acc sum[WHOLE ? C::MI : 1][WHOLE ? C::NI : 1];
    if constexpr (WHOLE) {
#pragma unroll
        for (int mi = 0; mi < C::MI; mi++)
#pragma unroll
            for (int ni = 0; ni < C::NI; ni++) sum[mi][ni] = acc[mi][ni];
        add_partials<C, WIDE>(sum, part0, n_contrib, part_stride);
    }
    // (unrolled by instantiation: written as loops the four-wave kernels' bodies exceed the compiler's limit for
    // unrolling, and accumulators indexed at run time would live in memory)
    if constexpr (WHOLE) {
        for_each_below<C::MI * C::NI / NB>([&](auto index) {
            constexpr int mi = decltype(index)::value * NB / C::NI, ni = decltype(index)::value * NB % C::NI;
            Acc blks[NB];
#pragma unroll
            for (int b = 0; b < NB; b++) blks[b] = sum[mi][ni + b];
            store_blocks<C, OUT, EDGE, TR, NB>(g, row0 + mi * C::MF, col0 + ni * C::MF, blks);
            __builtin_amdgcn_sched_barrier(0);
        });
    } else {
        constexpr int N = SUM_BLOCKS<C>;
        static_assert(N % NB == 0 && C::MI * C::NI % N == 0, "whole chunks of blocks, of whole pairs");
        for_each_below<C::MI * C::NI / N>([&](auto chunk) {
            constexpr int first = decltype(chunk)::value * N;
            Acc sums[N];
#pragma unroll
            for (int b = 0; b < N; b++) sums[b] = acc[(first + b) / C::NI][(first + b) % C::NI];
            add_block_partials<C, WIDE, first, N>(sums, part0, n_contrib, part_stride);
            for_each_below<N / NB>([&](auto index) {
                constexpr int b0 = decltype(index)::value * NB, mi = (first + b0) / C::NI, ni = (first + b0) % C::NI;
                Acc blks[NB];
#pragma unroll
                for (int b = 0; b < NB; b++) blks[b] = sums[b0 + b];
                store_blocks<C, OUT, EDGE, TR, NB>(g, row0 + mi * C::MF, col0 + ni * C::MF, blks);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    }
}

// ---- shared reduction -----------------------------------------------------------------------
// Fix-up of plans in which many workgroups share every tile and nothing follows the Stream-K work (sk_shared_reduction): each
// workgroup of a tile, its owner too, parks its piece and counts itself in; once all have, each fetches the same share
// of all pieces, adds them up and stores that share of D.  What bounds the exchange otherwise is the owner's CU, which takes the
// partial tiles of all contributors through one port (about 107 bytes per ns); here a tile's pieces go to as many CUs as made
// them.  The order of the additions is the owner's (and, from 2 * SK_TREE_GROUP contributors on, the group leaders'): the
// results are the same bit for bit, whoever takes a share (see sk_leave_tile).
struct TileLine {
    uint32_t* word;
    __device__ __forceinline__ TileLine(const GemmArgs& g, int tile) : word(g.flags + (size_t)tile * SK_LINE_WORDS) {}
    __device__ __forceinline__ uint32_t load(int i = 0) const { return __hip_atomic_load(word + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ uint32_t add(uint32_t v) const { return __hip_atomic_fetch_add(word, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ void give_up(int j) const {
        uint32_t before = __hip_atomic_fetch_or(word + 1 + j / 32, 1u << j % 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("" : "+v"(before) : : "memory");      // waits for the answer: the bit is there before the count says so
    }
    __device__ __forceinline__ bool is_given_up(int j) const { return load(1 + j / 32) >> j % 32 & 1; }
    __device__ __forceinline__ void clear(int i = 0) const { __hip_atomic_store(word + i, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
};
// Where a workgroup's piece of a tile is parked: in the workgroup's slot - but the owner's, whose slot holds its piece of
// the next tile if its range goes on there, then behind the workgroups' slots.
__device__ __forceinline__ int owner_slot(const GemmArgs& g, int tile, int wg) {
    const int end = (wg + 1) * g.ipw < g.sk_iters ? (wg + 1) * g.ipw : g.sk_iters;
    return end > (tile + 1) * g.ipt ? g.grid + tile : wg;
}

// Four consecutive values of a lane: of a row (TR) or of a column (see store_blocks).
template <int OUT, bool TR>
__device__ __forceinline__ void store_four(const GemmArgs& g, int row, int col, f32x4 v) {
    if (col >= g.N) return;
    if constexpr (TR) {
        if (row >= g.M) return;
        const size_t o = (size_t)((uint32_t)row * (uint32_t)g.N + (uint32_t)col);
        if constexpr (OUT == SK_F32) *reinterpret_cast<f32x4*>(static_cast<float*>(g.D) + o) = v;
        else if constexpr (OUT == SK_BF16) *reinterpret_cast<u32x2*>(static_cast<u16*>(g.D) + o) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
        else *reinterpret_cast<u32x2*>(static_cast<u16*>(g.D) + o) = u32x2{pack_f16(v[0], v[1]), pack_f16(v[2], v[3])};
    } else {
#pragma unroll
        for (int e = 0; e < 4; e++) {
            if (row + e >= g.M) return;
            const size_t o = (size_t)((uint32_t)(row + e) * (uint32_t)g.N + (uint32_t)col);
            if constexpr (OUT == SK_F32) static_cast<float*>(g.D)[o] = v[e];
            else if constexpr (OUT == SK_BF16) static_cast<u16*>(g.D)[o] = to_bf16_bits(v[e]);
            else static_cast<_Float16*>(g.D)[o] = (_Float16)v[e];
        }
    }
}

// A workgroup's share of one split tile: units [begin, end) of the tile's pieces.  A unit is the 1 KB that one register group
// of one wave takes in a slot.
template <class C> struct Share {
    static constexpr int Q = C::ACC / 4, BLOCKS = C::MI * C::NI, UNITS = C::NW * BLOCKS * Q;
    int tile, last_wg, n_all, j, begin, end;     // the tile, its owner, the number of its contributors, which share
    __device__ __forceinline__ void init(const GemmArgs& g, int x, int t) {
        tile = t;
        const int first_wg = (int)fast_div((uint32_t)(t * g.ipt), g.div_ipw);
        last_wg = (int)fast_div((uint32_t)(t * g.ipt + g.ipt - 1), g.div_ipw);
        n_all = last_wg - first_wg;
        take(last_wg - x);
    }
    __device__ __forceinline__ void take(int share) {
        j = share;
        begin = sk_share_begin(UNITS, j, n_all + 1);
        end = sk_share_begin(UNITS, j + 1, n_all + 1);
    }
};

// One unit of a tile: all its pieces added up, 16 contributors per round trip, and stored.
template <class C, bool TR>
__device__ __forceinline__ void store_unit(const GemmArgs& g, const buffer_rsrc& rsrc, const Share<C>& share, int unit, int lane) {
    constexpr int Q = Share<C>::Q, BLOCKS = Share<C>::BLOCKS, AT_ONCE = 2 * SK_TREE_GROUP;
    constexpr uint32_t SLOT_BYTES = C::BM * C::BN * 4;
    const int n_all = share.n_all;
    const int w = unit / (BLOCKS * Q), b = unit / Q % BLOCKS, q = unit % Q;
    const int at = ((b * Q + q) * C::NW + w) * 1024 + lane * 16;
    auto fetch = [&](int slot) {
        return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, at, (int)((uint32_t)slot * SLOT_BYTES), 16 /* sc1 */));
    };
    f32x4 sum = fetch(owner_slot(g, share.tile, share.last_wg));
    for (int c = 1; c <= n_all; c += AT_ONCE) {
        f32x4 part[AT_ONCE];
#pragma unroll
        for (int e = 0; e < AT_ONCE; e++) {
            part[e] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (c + e <= n_all) part[e] = fetch(share.last_wg - c - e);
        }
        if (n_all >= AT_ONCE) {                  // the order of the two-level reduction
#pragma unroll
            for (int h = 0; h < AT_ONCE; h += SK_TREE_GROUP) {
                f32x4 group = part[h];
#pragma unroll
                for (int e = 1; e < SK_TREE_GROUP; e++) group += part[h + e];
                sum += group;
            }
        } else {
#pragma unroll
            for (int e = 0; e < AT_ONCE; e++) sum += part[e];
        }
    }
    int tm, tn;
    tile_position(g, share.tile, tm, tn);
    const int wm = w / C::WN, wn = w % C::WN, mi = b / C::NI, ni = b % C::NI;
    const int row = tm * C::BM + wm * C::WTM + mi * C::MF + (TR ? lane % C::MF : 4 * (lane / C::MF) + q * 4 * C::KG);
    const int col = tn * C::BN + wn * C::WTN + ni * C::MF + (TR ? 4 * (lane / C::MF) + q * 4 * C::KG : lane % C::MF);
    if (g.out_dtype == SK_BF16) store_four<SK_BF16, TR>(g, row, col, sum);
    else if (g.out_dtype == SK_F16) store_four<SK_F16, TR>(g, row, col, sum);
    else store_four<SK_F32, TR>(g, row, col, sum);
}

// This workgroup's shares of the one or two tiles of its range, all of them split (the range is shorter than a tile): both
// counts are waited for at once, and a wave takes every NW-th unit of the two shares together.
template <class C, bool TR>
__device__ __forceinline__ void store_shares(const GemmArgs& g, int x, unsigned char* smem) {
    int thread = threadIdx.x;
    asm volatile("" : "+s"(x), "+v"(thread));        // (what follows from them is worked out here and not ahead of the MAC loop)
    const int begin = x * g.ipw, end = begin + g.ipw < g.sk_iters ? begin + g.ipw : g.sk_iters;
    if (begin >= end) return;
    const int lane = thread % 64, wave = __builtin_amdgcn_readfirstlane(thread / 64);
    Share<C> s0, s1;
    s0.init(g, x, (int)fast_div((uint32_t)begin, g.div_ipt));
    const int last = (int)fast_div((uint32_t)end - 1, g.div_ipt);
    s1 = s0;
    if (last > s0.tile) s1.init(g, x, last);
    else s1.end = s1.begin;
    // lane i of the first wave watches and leaves tile i; the other waves learn through LDS, which is free by now, which shares
    // are taken (bits 0 and 1), and whether some were given up (bit 2); what it mostly says is there before the wait
    const bool mine = wave == 0 && lane <= last - s0.tile, second_lane = lane == 1;
    const TileLine line(g, second_lane ? s1.tile : s0.tile);
    const uint32_t n = (uint32_t)(second_lane ? s1.n_all : s0.n_all) + 1;
    volatile int* told = reinterpret_cast<volatile int*>(smem);
    bool with_share = true;
    uint32_t word = 0;
    if (wave == 0) {
        if (lane == 0) told[0] = 3;
        with_share = !mine || (second_lane ? s1.end - s1.begin : s0.end - s0.begin) == 0;
        for (uint32_t polls = 0;; polls++) {
            if (!with_share) {
                word = line.load();
                with_share = sk_arrived(word) == n;
            }
            if (__all(with_share) || polls >= g.spin_limit) break;
            __builtin_amdgcn_s_sleep(1);
        }
        if (__any(!with_share || sk_given_up(word) > 0)) {
            const int taken = (int)(__ballot(with_share) & 3);
            if (lane == 0) told[0] = taken | 4;
        }
    }
    __syncthreads();
    word = 0;
    if (mine) word = sk_leave_tile(line, second_lane ? s1.j : s0.j, with_share);
    const int state = __builtin_amdgcn_readfirstlane(told[0]);
    const buffer_rsrc rsrc = __builtin_amdgcn_make_buffer_rsrc(g.partials, 0, (uint32_t)(g.grid + g.tiles) * (uint32_t)(C::BM * C::BN * 4), BUFFER_RAW);
    int len0 = state & 1 ? s0.end - s0.begin : 0, len1 = state & 2 ? s1.end - s1.begin : 0;
    // The last one to leave a tile takes its line down, after the shares that others gave up.  All waves work at these where the first one
    // knew of some before it left; of those given up right then it alone learns.  (One loop for them and the workgroup's own: with a copy of
    // the unit's code for each the 8-bit 256 x 256 kernel spilled 11 registers instead of 7 and took 3 % longer.)
    const bool all_waves = (state & 4) != 0;
    int rest = 0, stride = C::NW, j = 0;
    for (int t = -1;;) {
        for (int i = wave; i < len0 + len1; i += stride) {
            const bool second = i >= len0;
            store_unit<C, TR>(g, rsrc, second ? s1 : s0, second ? s1.begin + i - len0 : s0.begin + i, lane);
        }
        if (t < 0) {
            const bool last_out = mine && sk_left(word) == n;
            if (last_out && sk_given_up(word) == 0) line.clear();
            rest = (int)(__ballot(last_out && sk_given_up(word) > 0) & 3);
            if (all_waves) {
                if (thread == 0) told[1] = rest;
                __syncthreads();
                rest = __builtin_amdgcn_readfirstlane(told[1]);
            } else {
                stride = 1;
            }
            if (rest == 0) return;
            t = 0;
        }
        // the next share given up, of tile t or the one after it
        for (; t < 2; t++, j = 0) {
            if (!(rest >> t & 1)) continue;
            const TileLine left(g, t == 0 ? s0.tile : s1.tile);
            const int n_all = t == 0 ? s0.n_all : s1.n_all;
            while (j <= n_all && !__builtin_amdgcn_readfirstlane((int)left.is_given_up(j))) j++;
            if (j <= n_all) break;
            if (all_waves) __syncthreads();
            if (wave == 0 && lane < SK_LINE_WORDS) left.clear(lane);
        }
        if (t == 2) return;
        len0 = len1 = 0;
        if (t == 0) {
            s0.take(j++);
            len0 = s0.end - s0.begin;
        } else {
            s1.take(j++);
            len1 = s1.end - s1.begin;
        }
    }
}

// Atomic fix-up (the accumulation step of Algorithm 1): a segment that covers only part of the tile's
// K-iterations adds its accumulators into the zero-initialised fp32 image with atomic adds; a
// segment that covers the whole tile stores them.  Blocks are not transposed here: the lanes of
// one atomic instruction then sit side by side in a row of the image (two cache lines per
// instruction instead of 32).
template <class C, bool EDGE>
__device__ __forceinline__ void add_to_image(const GemmArgs& g, int row0, int col0, bool partial,
                                             const typename Mfma<C::DT, C::MF>::Acc (&acc)[C::MI][C::NI]) {
#pragma unroll
    for (int mi = 0; mi < C::MI; mi++)
#pragma unroll
        for (int ni = 0; ni < C::NI; ni++) {
            const int col = col0 + ni * C::MF;
#pragma unroll
            for (int r = 0; r < C::ACC; r++) {
                const int row = row0 + mi * C::MF + (r / 4) * (4 * C::KG) + r % 4;
                if (!EDGE || (row < g.M && col < g.N)) {
                    float* p = g.image + (size_t)((uint32_t)row * (uint32_t)g.N + (uint32_t)col);
                    if (partial) unsafeAtomicAdd(p, acc[mi][ni][r]);
                    else *p = acc[mi][ni][r];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
}

// How the pieces of a split tile come together: OWNER: one of its workgroups waits for the partial tiles of the others and adds them
// up; SHARED: all of them, a share each, which a kernel of its own does (in one kernel the two cost the small problems 0.1 - 0.2 us:
// 512^3 4.74 -> 4.85), all of whose segments are pieces of split tiles; ATOMIC: atomic adds into an image of D.
enum FixUp { OWNER, SHARED, ATOMIC_ADDS };
template <class C, bool ALIGNED, FixUp FIXUP = OWNER>
__global__ __launch_bounds__(C::THREADS) void streamk_gemm_kernel(GemmArgs g) {
    extern __shared__ __align__(1024) unsigned char smem[];
    typedef typename Mfma<C::DT, C::MF>::Acc Acc;
    const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
    const int wm = wave / C::WN, wn = wave % C::WN;
    const int x = logical_wg(blockIdx.x, g);
    // transposed accumulator blocks (vector stores) where D's rows are 16-byte aligned; the atomic
    // fix-up and the element-wise stores of unaligned problems want the lanes side by side in a row
    constexpr bool ATOMIC = FIXUP == ATOMIC_ADDS, TR = ALIGNED && !ATOMIC;
    FragMap<C> fm;
    fm.init();

    // Algorithm 1 (clamped): this workgroup's share of the Stream-K iterations
    int it = x * g.ipw, it_end = it + g.ipw;
    if (it > g.sk_iters) it = g.sk_iters;
    if (it_end > g.sk_iters) it_end = g.sk_iters;
    int dp_tile = g.sk_tiles + x;   // data-parallel tiles come after the Stream-K work
    // k-aligned order: a share that contains a tile boundary is run as its whole tiles first, then
    // the head piece of its last tile (k from 0), then the tail piece of its first tile.  Whole
    // tiles and head pieces then start at k = 0 at multiples of a tile's duration in every workgroup,
    // whatever its offset in the iteration space, which keeps the operand blocks that neighbouring
    // tiles share in L2; and the tail piece, whose workgroup owns the tile, comes last, when the
    // pieces before it in k have long been parked.
    int next_b = it_end, next_e = it_end, last_b = it_end, last_e = it_end;     // the sub-ranges after [it, it_end)
    if (g.k_aligned && it < it_end) {
        const int first_full = (int)fast_div((uint32_t)it + (uint32_t)g.ipt - 1, g.div_ipt) * g.ipt;
        const int last_full = (int)fast_div((uint32_t)it_end, g.div_ipt) * g.ipt;
        if (first_full <= last_full) {
            next_b = last_full; next_e = it_end;     // head piece (may be empty)
            last_b = it; last_e = first_full;        // tail piece (may be empty)
            it = first_full; it_end = last_full;     // whole tiles (may be none)
        }
    }
    // The next segment of this workgroup: tile index, k-iterations and the tile's origin; false when the work is done.
    auto next_segment = [&](int& tile, int& k_begin, int& k_end, int& m0, int& n0) -> bool {
        if (it >= it_end) { it = next_b; it_end = next_e; next_b = last_b; next_e = last_e; last_b = last_e; }
        if (it >= it_end) { it = next_b; it_end = next_e; next_b = last_b; next_e = last_e; last_b = last_e; }
        const bool dp_now = dp_tile < g.tiles && (g.dp_first || it >= it_end);
        if (!dp_now && it < it_end) {            // Algorithm 1: cut the share at tile boundaries
            tile = (int)fast_div((uint32_t)it, g.div_ipt);
            const int tile_first = tile * g.ipt;
            k_begin = it - tile_first;
            const int stop = it_end < tile_first + g.ipt ? it_end : tile_first + g.ipt;
            k_end = stop - tile_first;
            it = stop;
        } else if (dp_now) {
            tile = dp_tile; k_begin = 0; k_end = g.ipt;
            dp_tile += g.grid;
        } else {
            return false;
        }
        int tm, tn;
        tile_position(g, tile, tm, tn);
        m0 = tm * C::BM;
        n0 = tn * C::BN;
        return true;
    };

    // Fix-up and epilogue of one finished segment.  Returns true if every wave has issued exactly the
    // stores of an unsplit interior tile (C::EPILOGUE_STORES for 16-bit outputs, more for fp32) and no
    // other vector-memory instruction.
    auto finish_segment = [&](int tile, int k_begin, int k_end, int m0, int n0, Acc (&acc)[C::MI][C::NI]) -> bool {
        if (ATOMIC) {
            int row0 = m0 + wm * C::WTM + 4 * (lane / C::MF), col0 = n0 + wn * C::WTN + lane % C::MF;
            asm volatile("" : "+v"(row0), "+v"(col0));
            const bool partial = k_begin > 0 || k_end < g.ipt;
            if (m0 + C::BM > g.M || n0 + C::BN > g.N) add_to_image<C, true>(g, row0, col0, partial, acc);
            else add_to_image<C, false>(g, row0, col0, partial, acc);
            return false;
        }
        if constexpr (FIXUP == SHARED) {
            int wg = x;
            asm volatile("" : "+s"(wg));
            const Slot<C, true> slot(g.partials + (size_t)(k_end < g.ipt ? wg : owner_slot(g, tile, wg)) * (C::BM * C::BN));
#pragma unroll
            for (int mi = 0; mi < C::MI; mi++)
#pragma unroll
                for (int ni = 0; ni < C::NI; ni++) {
                    slot.park(mi * C::NI + ni, acc[mi][ni]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            wait_vmcnt<0>();                      // every lane's part of the piece has reached memory
            __syncthreads();
            if (tid == 0) TileLine(g, tile).add(SK_ARRIVES);
            return false;
        }

        // ---- fix-up
        // Tiles shared by many workgroups are reduced in two levels: every SK_TREE_GROUP-th contributor first
        // adds the partials of the contributors behind it to its own accumulators, so the owner
        // collects one partial per group.  The order of the additions stays fixed.
        // The owner of a split tile is the workgroup holding its first iteration, the contributors
        // are the workgroups after it (dir = +1); in the k-aligned order the one holding its last
        // iteration, which finishes last, and the contributors are the workgroups before it (dir = -1).
        // (wg, from_end: x and g.k_aligned, taken anew here; what follows from them - addresses, conditions - would otherwise be
        // worked out at the kernel's start and kept, 40 instructions and 10 to 15 spilled scalars of the 400 and 25 ahead of the
        // first request.  With the offsets above, us: 512^3 4.80 -> 4.77, 1 x 4096 x 4096 9.80 -> 9.67, 16 x 8192 x 8192 25.3 -> 25.2,
        // 1008 x 1200 x 1040 9.68 -> 9.63, 256 x 512 x 16384 to fp32 14.86 -> 14.73.  Issuing the first requests ahead of the lanes' LDS
        // addresses as well, another 90 instructions, made 512^3 4.92.  Not on the register-staged path of the 64 x 64 x 128 tile, eight k-steps
        // of one block: the reads of its MAC loop, whose order is the compiler's, then run no longer ahead of the matrix-core work,
        // 1083 x 1021 x 4093 53.2 us, 50.7 without, 500 x 700 x 5001 30.5 / 28.6; below five k-iterations 0.1 us the other way.  The
        // staged path of the other tiles gains from it, 32 x 128 4 %.)
        int wg = x, from_end = g.k_aligned, thread = tid;
        if constexpr (ALIGNED || C::MI * C::NI > 1 || C::KK < 8) asm volatile("" : "+s"(wg), "+s"(from_end), "+v"(thread));
        const bool split = k_begin > 0 || k_end < g.ipt;
        const bool contributor = from_end ? k_end < g.ipt : k_begin > 0;
        const int dir = from_end ? -1 : 1;
        int j = 0, n_all = 0;                                           // distance from the tile's owner, the tile's number of contributors
        if (split) {                                                    // (only split tiles; ipw is 0 in a plan without Stream-K work)
            const int first_wg = (int)fast_div((uint32_t)(tile * g.ipt), g.div_ipw);
            const int last_wg = (int)fast_div((uint32_t)(tile * g.ipt + g.ipt - 1), g.div_ipw);
            n_all = last_wg - first_wg;
            j = from_end ? last_wg - wg : wg - first_wg;
        }
        const bool two_level = n_all >= 2 * SK_TREE_GROUP;
        const ptrdiff_t slot_stride = (ptrdiff_t)dir * (C::BM * C::BN);
        if (contributor) {
            if (two_level && (j - 1) % SK_TREE_GROUP == 0) {            // group leader: members j+1 .. j+GROUP-1
                const int members = (j + SK_TREE_GROUP - 1 <= n_all ? j + SK_TREE_GROUP - 1 : n_all) - j;
                if (thread < 64) wait_flags(g, wg + dir, members, dir);
                __syncthreads();
                add_partials<C, WIDE_SLOT<C, TR>>(acc, g.partials + (ptrdiff_t)(wg + dir) * (C::BM * C::BN), members, slot_stride);
            }
            // park the accumulators, then signal
            const Slot<C, WIDE_SLOT<C, TR>> slot(g.partials + (size_t)wg * (C::BM * C::BN));
#pragma unroll
            for (int mi = 0; mi < C::MI; mi++)
#pragma unroll
                for (int ni = 0; ni < C::NI; ni++) {
                    slot.park(mi * C::NI + ni, acc[mi][ni]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            wait_vmcnt<0>();                      // every lane's part of the partial tile has reached memory
            __syncthreads();
            if (thread == 0)
                __hip_atomic_store(g.flags + (size_t)wg * (SK_FLAG_STRIDE / 4), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
        int n_contrib = 0;
        ptrdiff_t part_stride = slot_stride;
        if (split) {
            // owner: the contributors are the n_all workgroups next to it in direction dir - or, with
            // two levels, their group leaders.  Wait for all of them; the epilogue adds their
            // partials in a fixed order, so the result does not depend on timing.
            const int step = two_level ? SK_TREE_GROUP : 1;
            n_contrib = two_level ? (n_all + SK_TREE_GROUP - 1) / SK_TREE_GROUP : n_all;
            part_stride *= step;
            if (thread < 64) wait_flags(g, wg + dir, n_contrib, step * dir);
            __syncthreads();
        }

        // ---- epilogue: fp32 accumulators -> D
        int row0 = m0 + wm * C::WTM + (TR ? lane % C::MF : 4 * (lane / C::MF));
        int col0 = n0 + wn * C::WTN + (TR ? 4 * (lane / C::MF) : lane % C::MF);
        asm volatile("" : "+v"(row0), "+v"(col0));
        const float* part0 = g.partials + (ptrdiff_t)(wg + dir) * (C::BM * C::BN);
        const bool edge = m0 + C::BM > g.M || n0 + C::BN > g.N;
        if (g.out_dtype == SK_BF16) {
            if (edge) reduce_and_store<C, SK_BF16, true, TR>(g, row0, col0, part0, n_contrib, part_stride, acc);
            else reduce_and_store<C, SK_BF16, false, TR>(g, row0, col0, part0, n_contrib, part_stride, acc);
        } else if (g.out_dtype == SK_F16) {
            if (edge) reduce_and_store<C, SK_F16, true, TR>(g, row0, col0, part0, n_contrib, part_stride, acc);
            else reduce_and_store<C, SK_F16, false, TR>(g, row0, col0, part0, n_contrib, part_stride, acc);
        } else {
            if (edge) reduce_and_store<C, SK_F32, true, TR>(g, row0, col0, part0, n_contrib, part_stride, acc);
            else reduce_and_store<C, SK_F32, false, TR>(g, row0, col0, part0, n_contrib, part_stride, acc);
        }
        return TR && !split && !edge;
    };

    // On the LDS-DMA path the first requests of the next segment go out before the current tile's
    // fix-up and epilogue (the ring is free once the MAC loop has ended): the loads travel while the
    // tile is stored, and the first wait of the next MAC loop leaves the epilogue's stores in flight.
    constexpr bool PREFETCH = ALIGNED, MAY_NT = ALIGNED && C::MAY_STREAM_B;
    int tile, k_begin, k_end, m0, n0;
    bool have = next_segment(tile, k_begin, k_end, m0, n0);
    bool prefetched = false, stores_in_flight = false;
    while (have) {
        Acc acc[C::MI][C::NI];
#pragma unroll
        for (int mi = 0; mi < C::MI; mi++)
#pragma unroll
            for (int ni = 0; ni < C::NI; ni++) acc[mi][ni] = Acc{};
        // B requested non-temporally or not: decided once per launch, two copies of the loop in the tiles that may
        // (the register-staged path has no such requests, so its kernels carry one copy)
        if (MAY_NT && g.stream_b) mac_loop<C, ALIGNED, TR, MAY_NT>(g, m0, n0, k_begin, k_end, smem, fm, acc, prefetched, stores_in_flight);
        else mac_loop<C, ALIGNED, TR, false>(g, m0, n0, k_begin, k_end, smem, fm, acc, prefetched, stores_in_flight);

        // this segment's numbers for the fix-up and the epilogue; then look ahead
        const int cur_tile = tile, cur_k_begin = k_begin, cur_k_end = k_end, cur_m0 = m0, cur_n0 = n0;
        have = next_segment(tile, k_begin, k_end, m0, n0);
        prefetched = PREFETCH && have;
        stores_in_flight = false;
        if (prefetched) {
            DmaMap<C> ahead;
            ahead.init(g, m0, n0);
            if (MAY_NT && g.stream_b) mac_prefetch<C, MAY_NT>(g, k_begin, k_end, smem, ahead);
            else mac_prefetch<C, false>(g, k_begin, k_end, smem, ahead);
        }
        stores_in_flight = finish_segment(cur_tile, cur_k_begin, cur_k_end, cur_m0, cur_n0, acc) && prefetched;
    }
    if constexpr (FIXUP == SHARED) store_shares<C, TR>(g, x, smem);
}

// ---- kernel table entries --------------------------------------------------------------------
typedef void (*kernel_fn)(GemmArgs);
struct KernelEntry {
    int dtype, bm, bn, bk, variant, fixup;
    int whole_tiles_choice = 0;          // > 0: the library launches this variant instead of variant 0 for plans without split
                                         // tiles whose tiles have at least this many k-iterations
    kernel_fn aligned, generic;
    kernel_fn across = nullptr;          // the MAC loop that runs on across the tiles of a workgroup (streamk_whole_tiles.h), and the fewest
    int across_iters = 0;                // k-iterations per tile that it takes; for plans without split tiles, aligned, with 16-bit output
    kernel_fn shared_aligned = nullptr, shared_generic = nullptr;    // with the shared reduction
    kernel_fn generic_one_by_one = nullptr;                          // for plans without split tiles, see takes_one_by_one
    int threads, lds_bytes, piece_elems;
    std::atomic<int> max_resident{-1};   // co-resident workgroups on the device, -1 = not yet asked
    std::atomic<int> max_shared{0};      // ... of the kernels with the shared reduction
    KernelEntry(int d, int m, int n, int k, int v, int fx, kernel_fn a, kernel_fn g, int t, int l, int pe)
        : dtype(d), bm(m), bn(n), bk(k), variant(v), fixup(fx), aligned(a), generic(g), threads(t), lds_bytes(l), piece_elems(pe) {}
};

// A tile whose register-staged path takes its stages one by one instead of in rounds, for plans of whole tiles.  A round
// that is not inside in all its stages pays for the checks of all, and the first one counts as such; in return no load is waited for
// early, which is worth more the longer the loads take and the more of them there are.  Rounds -> one by one, us:
//  - 32 x 64: 5 - 8 iterations, N up to 1022, 4 to 512 tiles, 1 - 5 % faster (319 x 1021, 6 iterations, 6.04 -> 5.93, 103 x 334 5.85 -> 5.62, 1022 x 1020
//    10.35 -> 9.98); a wider B, less of which is read twice, 5 - 7 to N = 2630 2 - 3 % faster, 31 x 1533 with 8 6 % slower, 32 x 8191 2 - 8 %; up to 48
//    tiles, or N = 510, 9 iterations level to 2 % faster, and with the rows of A or of B 4-byte aligned, which arrive sooner, 9 - 14 1 - 5 % (103 x 334, 12, 7.17 ->
//    6.92; 1302 x 273 x 610 6.87 -> 6.68; 690 x 244 with 16 2 - 4 % faster, 95 x 508 with 17 10 % slower); otherwise slower: 3 and 4 iterations 3 - 4 %, 160
//    tiles, N = 1021, of 10 / 12 / 20 5 / 10 / 19 %, split plans 2 - 6 %;
//  - 64 x 128, 12 to 400 tiles: 9 - 24 iterations 5 % faster to 2 % slower (383 x 1021, 10 / 12 / 16, 8.81 / 10.43 / 11.70 -> 8.56 / 10.16 / 11.41; 288 plans of all
//    alignments 0.9 % in the mean), 7 and from 33 on level to 2 % slower (379 x 1022 x 2110 17.0 -> 17.3);
//  - 8-bit 128 x 256, 12 to 400 tiles: from 8 iterations on 2 % faster to level (767 x 2045, 8 / 18, 17.43 / 29.30 -> 17.17 / 28.80), from 44 on level, below 8 1 - 4 % slower.
template <class C> struct OneByOne : C { static constexpr bool STAGED_ROUNDS = false; };
template <class C> constexpr bool MAY_TAKE_ONE_BY_ONE = C::FP8 ? C::BM == 128 && C::BN == 256 : (C::BM == 32 && C::BN == 64) || (C::BM == 64 && C::BN == 128 && C::NW == 8);
inline bool takes_one_by_one(const sk_plan_header& h) {
    const int ipt = h.iters_per_tile;
    if (h.blk_n == 256) return ipt >= 8 && ipt < 44;
    if (h.blk_n == 128) return ipt >= 9 && ipt <= 24;
    const int near = h.tiles > 48 && h.tiles_n > 8 ? 8 : h.N % 2 && h.K % 2 ? 9 : 14;
    return ipt >= 5 && ipt <= (h.tiles_n > 64 ? 0 : h.tiles_n > 16 ? 7 : near);
}

template <class C, bool ATOMIC = false> KernelEntry* make_entry(int variant = 0, int whole_tiles_choice = 0) {
    KernelEntry* e = new KernelEntry(C::DT, C::BM, C::BN, C::BK, variant, ATOMIC ? SK_FIXUP_ATOMIC : SK_FIXUP_FLAGS,
                                     streamk_gemm_kernel<C, true, ATOMIC ? ATOMIC_ADDS : OWNER>, streamk_gemm_kernel<C, false, ATOMIC ? ATOMIC_ADDS : OWNER>,
                                     C::THREADS, C::LDS_BYTES, C::PE);
    e->whole_tiles_choice = whole_tiles_choice;
    if constexpr (C::MAY_SHARE && !ATOMIC) {
        e->shared_aligned = streamk_gemm_kernel<C, true, SHARED>;
        e->shared_generic = streamk_gemm_kernel<C, false, SHARED>;
    }
    if constexpr (MAY_TAKE_ONE_BY_ONE<C> && !ATOMIC) e->generic_one_by_one = streamk_gemm_kernel<OneByOne<C>, false>;
    return e;
}

// Tile shapes with a kernel: <dtype, BM, BN, BK, waves along M, waves along N, matrix-core block,
// A ring depth[, B ring depth[, instruction-by-instruction MAC loop]]>.  Variant 0 of a shape is the
// one sk_gemm uses; other variants are alternative wave layouts of the same shape, selectable with
// sk_plan_set_kernel_variant for tuning runs.  ATOMIC selects the atomic-add fix-up (sk_fixup).
// The three compute-bound shapes have two kernels that the library itself chooses between: four
// waves (one per SIMD, twice the tile per wave: a quarter less LDS read traffic, +1.5 - 3 % on problems
// of whole tiles) for plans without split tiles, eight waves for plans with split tiles (twice as
// many lanes fetch and add the partial tiles: 10 - 25 % faster there with 256 x 256 tiles).  Variant 3
// is the eight-wave kernel under a number of its own (variant 0 means "the library's choice").
template <int DT, bool ATOMIC = false> void add_16bit_tiles(KernelEntry** t, int* n) {
    // The 128- and 64-row tiles run 8 waves (2 x 4), two per SIMD, like the large ones: with one wave
    // per SIMD (2 x 2) nothing overlaps a wave's waits (128 x 128 x 64: +8 - 12 % on 512 x 8192 x 8192
    // and 4096^3; 64 x 128 x 64: +4 % on the HBM-bound M = 64 shape, +12 - 20 % on small problems).
    // The three compute-bound shapes run the instruction-by-instruction MAC loop (+5 % on 8192^3 with
    // 256 x 256, +8 % on 4096^3 with 128 x 128, +2 - 3 % with 256 x 128; the 64-row tile loses 7 % with it).
    t[(*n)++] = make_entry<Cfg<DT, 128, 128, 32, 2, 4, 32, 4>, ATOMIC>();
    t[(*n)++] = make_entry<Cfg<DT, 128, 128, 64, 2, 4, 32, 3, 3, 1>, ATOMIC>();
    t[(*n)++] = make_entry<Cfg<DT, 256, 128, 64, 4, 2, 32, 3, 3, 1>, ATOMIC>();
    t[(*n)++] = make_entry<Cfg<DT, 256, 256, 64, 2, 4, 32, 3, 2, 1>, ATOMIC>();
    if constexpr (!ATOMIC) {  // (the atomic fix-up exists for the layouts above only)
        t[(*n)++] = make_entry<Cfg<DT, 256, 128, 64, 2, 2, 32, 3, 3, 1>>(1, 16);
        t[(*n)++] = make_entry<Cfg<DT, 256, 128, 64, 4, 2, 32, 3, 3, 1>>(3);
        t[(*n)++] = make_entry<Cfg<DT, 256, 256, 64, 2, 2, 32, 3, 2, 1>>(1, 48);
        t[(*n)++] = make_entry<Cfg<DT, 256, 256, 64, 2, 4, 32, 3, 2>>(2);
        t[(*n)++] = make_entry<Cfg<DT, 256, 256, 64, 2, 4, 32, 3, 2, 1>>(3);      // variant 0's kernel under a number of its own
        t[(*n)++] = make_entry<Cfg<DT, 256, 256, 32, 2, 2, 32, 4>>();
        t[(*n)++] = make_entry<Cfg<DT, 128, 128, 64, 2, 2, 32, 3, 3, 1>>(1, 1);
        t[(*n)++] = make_entry<Cfg<DT, 128, 128, 64, 2, 4, 32, 3, 3, 1>>(3);
    }
}

// The tiles of at most 64 rows.  What bounds them outside the HBM-bound shapes is the rate at which a CU
// takes operand bytes into LDS (about 90 bytes per ns with rows on 128-byte boundaries, 60 off them), so they
// matter where the larger tiles leave CUs idle: 1024^3 on 256 tiles of 64 x 64 7.0 us (128 of 64 x 128: 8.2,
// 256 of 32 x 128: 7.2), 1 x 4096 x 4096 on 16 x 128 10.9 us from cold
// operands (32 x 128: 12.4; 32 x 64: 10.7, and at 1 x 4096 x 8192 16.3 against 18.2, which the cost model has behind it).
template <int DT, bool ATOMIC = false> void add_16bit_low_tiles(KernelEntry** t, int* n) {
    t[(*n)++] = make_entry<Cfg<DT, 64, 128, 64, 2, 4, 32, 4>, ATOMIC>();
    t[(*n)++] = make_entry<Cfg<DT, 32, 128, 64, 1, 4, 32, 4>, ATOMIC>();
    t[(*n)++] = make_entry<Cfg<DT, 16, 128, 64, 1, 4, 16, 4>, ATOMIC>();
    if constexpr (!ATOMIC) {
        t[(*n)++] = make_entry<Cfg<DT, 64, 128, 64, 2, 2, 32, 4>>(1);
    }
    t[(*n)++] = make_entry<Cfg<DT, 64, 64, 128, 2, 2, 32, 4>, ATOMIC>();
    t[(*n)++] = make_entry<Cfg<DT, 32, 64, 64, 1, 2, 32, 4>, ATOMIC>();
}

// One or two functions per input type, each in its own translation unit (so that they compile in parallel);
// it appends that type's kernels to the table.
void register_bf16(KernelEntry** t, int* n);
void register_f16(KernelEntry** t, int* n);
void register_fp8(KernelEntry** t, int* n);
void register_bf16_low(KernelEntry** t, int* n);
void register_f16_low(KernelEntry** t, int* n);
void register_fp8_low(KernelEntry** t, int* n);
// ... and these add the MAC loop that runs on across tiles to the kernels it belongs to.
void add_across_bf16(KernelEntry** t, int n);
void add_across_f16(KernelEntry** t, int n);
void add_across_fp8(KernelEntry** t, int n);
// 256 rows of N 16-bit values have to stay below 2^31 bytes there (32-bit offsets inside a tile's rows).
constexpr int64_t SK_ACROSS_MAX_N = 1 << 22;
void register_bf16_atomic(KernelEntry** t, int* n);
void register_f16_atomic(KernelEntry** t, int* n);
void register_fp8_atomic(KernelEntry** t, int* n);

}  // namespace streamk_detail
