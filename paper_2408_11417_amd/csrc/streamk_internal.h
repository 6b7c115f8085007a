// Internal definitions shared by the host planner and the HIP launcher.
#pragma once
#include <cstdint>
#include <cstddef>
#include "streamk.h"

struct sk_plan_t {
    sk_plan_header h;
    void* workspace = nullptr;      // caller-owned device memory
    size_t workspace_bytes = 0;
    uint32_t spin_limit = 1u << 24;
    int needs_fixup = 0;            // 1 if any tile is split over several workgroups
    int fixup = SK_FIXUP_FLAGS;     // how split tiles are combined
    int dp_first = 0;               // 1: data-parallel tiles before the Stream-K iterations
    int k_aligned = 1;              // 1: head piece of a Stream-K range first, last workgroup of a tile owns it
    int kernel_variant = 0;         // which compiled wave layout of the tile's kernel to launch (0 = the library's choice)
};

// Workspace layout: [grid flag lines of SK_FLAG_STRIDE bytes][status line][partials]
constexpr size_t SK_FLAG_STRIDE = 128;
constexpr int SK_GROUP_ROWS = 8;   // tile rows per band of the grouped tile order
constexpr int SK_TREE_GROUP = 8;   // contributors per group in the two-level reduction of tiles shared by many workgroups
inline size_t sk_ws_status_offset(int grid) { return (size_t)grid * SK_FLAG_STRIDE; }
inline size_t sk_ws_partials_offset(int grid) { return ((size_t)grid + 1) * SK_FLAG_STRIDE + 384; }

// Size of the device array behind sk_gemm_static: the flag and status lines of 256 workgroups plus
// 256 partial tiles of 256 x 256 fp32 (the largest tile), i.e. every plan on the default grid.
constexpr size_t SK_STATIC_WORKSPACE_MAX = (256 + 1) * SK_FLAG_STRIDE + 384 + (size_t)256 * 256 * 256 * 4;

// Division of a number below 2^31 by a divisor that is fixed for a launch: with shift = 31 + ceil(log2 d)
// and mul = ceil(2^shift / d) (which fits 32 bits), n / d == (n * mul) >> shift for every n < 2^31, because
// the error n * (mul * d - 2^shift) stays below 2^shift.  The kernels' index arithmetic (Algorithm 1's
// iteration -> tile and tile -> workgroup maps) sits ahead of a workgroup's first load and inside the
// fix-up chain, and a division by a run-time value costs about 300 cycles of dependent instructions there.
struct sk_fast_div { uint32_t mul, shift; };
inline sk_fast_div sk_make_fast_div(uint32_t d) {
    if (d == 0) return sk_fast_div{0u, 0u};          // never divided by (e.g. no Stream-K iterations)
    uint32_t log2_up = 0;
    while ((1ull << log2_up) < d) log2_up++;
    const uint32_t shift = 31 + log2_up;
    return sk_fast_div{(uint32_t)(((1ull << shift) + d - 1) / d), shift};
}
inline uint32_t sk_fast_div_apply(uint32_t n, sk_fast_div f) { return (uint32_t)(((uint64_t)n * f.mul) >> f.shift); }

#ifdef __HIPCC__
#define SK_HOST_DEVICE __host__ __device__
#else
#define SK_HOST_DEVICE
#endif

// Map 1 of the workgroups: the logical id that workgroup i of an XCD runs, where the first 8 * first_ids ids and the 8 * other_ids others are
// dealt out in a block of each per XCD.
SK_HOST_DEVICE inline int sk_spread_id(int xcd, int i, int first_ids, int other_ids) {
    return i < first_ids ? xcd * first_ids + i : 7 * first_ids + xcd * other_ids + i;
}
// How many of the first ids are dealt out so (0: one contiguous block per XCD).
int sk_first_ids(const sk_plan_header& h);

// ---- shared reduction: who adds up and stores which part of a split tile, and when -----------------
// The n workgroups of a tile park their pieces and count themselves in at the tile's flag line.  Then each waits for the others, for a
// bounded time, and leaves: with its share of the tile where all have arrived by then, and otherwise giving the share up, which it
// notes in the line's other words.  The last one to leave, by whose time all have arrived, takes what was given up.  So nobody
// depends on a workgroup that has not started: the launch ends whatever part of the device it gets, and only the split of the
// work depends on it.  (tests/host/shared_reduction.cpp runs these functions on threads.)
// The line's first word: three counts of ten bits, of the workgroups that have arrived, have left, have given their share up.
constexpr uint32_t SK_ARRIVES = 1, SK_LEAVES = 1u << 10, SK_GIVES_UP = 1u << 20;
SK_HOST_DEVICE inline uint32_t sk_arrived(uint32_t word) { return word & 1023; }
SK_HOST_DEVICE inline uint32_t sk_left(uint32_t word) { return word >> 10 & 1023; }
SK_HOST_DEVICE inline uint32_t sk_given_up(uint32_t word) { return word >> 20; }
// ... and a bit per workgroup in the other words.
constexpr int SK_LINE_WORDS = (int)(SK_FLAG_STRIDE / 4), SK_MAX_SHARERS = 32 * (SK_LINE_WORDS - 1);
// How often a workgroup polls for the others: a little longer than they are apart on an idle device, which is a part of the time that
// their iterations take.  Least number without a loss, 256 x 256 tiles: 8 iterations 64, 12 of 8 bits 112, 118 about 800;
// 64 x 128: 34 64, 54 - 94 about 100; smaller ones 2 - 32.
inline uint32_t sk_share_polls(const sk_plan_header& h) {
    return 64 + (uint32_t)h.iters_per_wg * (2 + (uint32_t)(h.blk_m * h.blk_n) / 8192);
}
// Leave the tile, with share j or giving it up.  Returns the first word as it is then.
// Line: add(v), the word before it; give_up(j), which is done when it returns.
template <class Line> SK_HOST_DEVICE inline uint32_t sk_leave_tile(const Line& line, int j, bool with_share) {
    if (!with_share) line.give_up(j);
    const uint32_t step = with_share ? SK_LEAVES : SK_LEAVES + SK_GIVES_UP;
    return line.add(step) + step;
}
// Share j of n of a tile of `units` units.
SK_HOST_DEVICE inline int sk_share_begin(int units, int j, int n) { return (int)((uint32_t)units * (uint32_t)j / (uint32_t)n); }

// Does the plan's fix-up share the reduction of a tile among all its workgroups (where its kernel can and the workspace suffices)?
bool sk_shared_reduction(const sk_plan_t* plan);
// The workspace that a plan cannot do without; sk_workspace_bytes adds what the shared reduction needs.
size_t sk_ws_least_bytes(const sk_plan_t* plan);
// Does the GEMM launcher hold a kernel for this configuration?
bool sk_kernel_available(int in_dtype, int blk_m, int blk_n, int blk_k);
// Bytes of the fp32 image of D that the atomic fix-up accumulates into (0 if D itself serves).
inline size_t sk_ws_image_bytes(const sk_plan_t* p) {
    return p->fixup == SK_FIXUP_ATOMIC && p->h.out_dtype != SK_F32 ? (size_t)p->h.M * (size_t)p->h.N * sizeof(float) : 0;
}
