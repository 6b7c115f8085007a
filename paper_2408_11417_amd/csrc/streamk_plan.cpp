// Host-side scheduler: turns (M, N, K, policy, tile, grid) into the numbers the
// persistent kernel walks, and expands them into the canonical segment list.
// Integer arithmetic only; no device contact.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <new>
#include <vector>
#include "streamk_internal.h"

namespace {

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Stream-K batches of a policy: 0..6, or -1 for "every tile is split" (Sec. 3.2).
int batches_of(int policy) {
    switch (policy) {
    case SK_POLICY_ALL_SK: return -1;
    case SK_POLICY_SK6_DP_EXT: return 6;
    default: return policy;   // DP .. SK5_DP carry their batch count as enum value
    }
}

// Tiles of a policy's Stream-K region (Sec. 3.2, Sec. 4.1).
int64_t sk_tile_count(int policy, int64_t tiles, int64_t grid) {
    const int b = batches_of(policy);
    if (b < 0) return tiles;
    if (b == 0) return 0;
    return std::min(tiles % grid + (int64_t)(b - 1) * grid, tiles);
}
// Is a tile split, i.e. does some workgroup's range end strictly inside one?
bool splits_tiles(int64_t sk_iters, int64_t iters_per_wg, int64_t iters_per_tile) {
    return sk_iters > iters_per_wg && iters_per_wg % iters_per_tile != 0;
}

bool dtype_in_ok(int d) { return d == SK_F16 || d == SK_BF16 || d == SK_FP8_E4M3; }
bool dtype_out_ok(int d) { return d == SK_F16 || d == SK_BF16 || d == SK_F32; }

// Segments of workgroup x, appended in execution order.
void expand_wg(const sk_plan_header& h, int x, std::vector<sk_segment>* out, sk_wg_range* range, bool dp_first = false,
               bool k_aligned = false) {
    const int64_t ipt = h.iters_per_tile;
    int64_t it = x * (int64_t)h.iters_per_wg;
    int64_t end = it + h.iters_per_wg;
    if (it > h.sk_iters) it = h.sk_iters;
    if (end > h.sk_iters) end = h.sk_iters;
    if (range) { range->sk_iter_begin = it; range->sk_iter_end = end; }
    const size_t at = out ? out->size() : 0;     // where this workgroup's segments start
    auto role_of = [&](const sk_segment& s) {
        if (s.k_begin == 0 && s.k_end == ipt) return SK_ROLE_FULL;
        const bool contributor = k_aligned ? s.k_end < ipt : s.k_begin > 0;
        return contributor ? SK_ROLE_CONTRIB : SK_ROLE_OWNER;
    };
    // a range that contains a tile boundary runs, in the k-aligned order, its whole tiles, then the
    // head piece of its last tile, then the tail piece of its first tile
    int64_t sub[3][2] = {{it, end}, {end, end}, {end, end}};
    if (k_aligned && it < end) {
        const int64_t first_full = ceil_div(it, ipt) * ipt, last_full = end / ipt * ipt;
        if (first_full <= last_full) {
            sub[0][0] = first_full; sub[0][1] = last_full;
            sub[1][0] = last_full;  sub[1][1] = end;
            sub[2][0] = it;         sub[2][1] = first_full;
        }
    }
    for (const auto& r : sub) {
        // Algorithm 1, outer loop: one segment per tile the range touches
        for (int64_t i = r[0]; i < r[1];) {
            const int64_t tile = i / ipt;
            const int64_t tile_first = tile * ipt;
            const int64_t stop = (r[1] < tile_first + ipt) ? r[1] : tile_first + ipt;
            sk_segment s;
            s.wg = x;
            s.tile = (int32_t)tile;
            s.k_begin = (int32_t)(i - tile_first);
            s.k_end = (int32_t)(stop - tile_first);
            s.role = role_of(s);
            if (out) out->push_back(s);
            i = stop;
        }
    }
    // data-parallel tiles follow the Stream-K work (Sec. 4.1) - or precede it (Sec. 3.2's earlier hybrid)
    int32_t count = 0;
    for (int64_t t = (int64_t)h.sk_tiles + x; t < h.tiles; t += h.grid) {
        if (out) {
            const sk_segment s{x, (int32_t)t, 0, (int32_t)ipt, SK_ROLE_FULL};
            if (dp_first) out->insert(out->begin() + (std::ptrdiff_t)(at + count), s);
            else out->push_back(s);
        }
        ++count;
    }
    if (range) {
        range->dp_tile_count = count;
        range->dp_tile_first = count ? h.sk_tiles + x : h.tiles;
    }
}

// Cost model shared by the tile dispatcher and sk_plan_estimate_us.  The constants - per kernel the rate of
// its MAC loop with the grid full and the microseconds a tile takes outside the loop (first loads, drain,
// store), and for the exchange of partial tiles a latency per level, the rate of one owner's chain of fetches
// and the rate of all partial traffic together - were fitted to timings of every tile shape and schedule on 397
// of the first 400 of 500 seeded problem sizes, 72 with at most 128 rows and 40 with few tiles and deep K on
// MI355X; sizes 400 .. 499 are the selector's held-out split and stay out of the fit (fit_tile_model.py; the
// fit optimises the dispatcher's pick of tile and policy, not the predicted times).  Time of the pick over the
// fastest of all tiles and schedules, geometric mean: 16 bits 1.015 / 1.020 / 1.028 on the three sets (the six shapes
// and constants of before: 1.047 / 1.110 / 1.097), 8 bits 1.011 / 1.008 / 1.016 (two shapes: 1.59 / 2.29 / 2.44).
// (per_cu: workgroups of the tile's kernel that fit a compute unit side by side - 160 KB of LDS)
struct TileCost { int bm, bn, bk; double tflops, tile_us; int per_cu; };
const TileCost tile_costs16[] = {{256, 256, 64, 1590., 10.40, 1}, {256, 128, 64, 1307., 5.61, 1}, {128, 128, 64, 1062., 4.33, 1},
                                 {64, 128, 64, 745., 2.91, 1}, {32, 128, 64, 478., 2.73, 2}, {16, 128, 64, 287., 2.68, 2},
                                 {64, 64, 128, 500., 3.08, 1}, {32, 64, 64, 364., 2.76, 3}};
// (the large 8-bit tile moves the bytes of the large 16-bit one with twice the k at twice the rate: its constants)
const TileCost tile_costs8[] = {{256, 256, 128, 3180., 10.40, 1}, {128, 256, 128, 2821., 4.75, 1}, {128, 128, 128, 1919., 2.61, 1},
                                {64, 128, 128, 1467., 2.45, 1},  {32, 128, 128, 915., 2.48, 2}};
constexpr int N_COSTS16 = 8, N_COSTS8 = 5;
constexpr int MODEL_GRID = 256;
constexpr double MODEL_LEVEL_US = 1.68, MODEL_FETCH_BYTES_PER_US = 107e3, MODEL_TRAFFIC_BYTES_PER_US = 6.953e6;

double model_iter_us(const TileCost& c, int bk) {          // one k-iteration of every workgroup of a full grid
    return 2.0 * c.bm * c.bn * bk * MODEL_GRID / (c.tflops * 1e12) * 1e6;
}

// Workgroups that park a partial tile: those whose range ends inside a tile (as many as start inside one).
// ipw iterations per workgroup, `workgroups` ranges that are not empty; every ipt / gcd(ipt, ipw)-th ends on a boundary.
int64_t model_contributors(int64_t workgroups, int64_t ipt, int64_t ipw) {
    int64_t a = ipt, b = ipw;
    while (b) { const int64_t r = a % b; a = b; b = r; }
    return workgroups - 1 - (workgroups - 1) / (ipt / a);
}

// Rows of A or B off the 16-byte grid: the register-staged kernels, whose first two stages arrive one after the other and
// whose D leaves element by element.  Counting 1.6 times the microseconds outside the loop took the 16-bit picks on 69 odd
// sizes from 1.050 of the fastest to 1.035; scaling the loop as well did not help.  With the kernels as they are, time of
// the picked tile and schedule over the fastest of all on 70 odd sizes, 40 of at most 128 rows and 40 of short K: 16 bits
// 1.023 / 1.069 / 1.002, 8 bits 1.016 / 1.073 / 1.002 (8-bit problems on the two large shapes only: 1.88 / 2.52 / 1.52).
constexpr double MODEL_STAGED_TILE = 1.6;
bool model_staged(int64_t N, int64_t K, int in_dtype) {
    const int piece = in_dtype == SK_FP8_E4M3 ? 16 : 8;
    return N % piece != 0 || K % piece != 0;
}

// Microseconds of a schedule: sk_tiles tiles split evenly over the grid, the rest in whole-tile waves.
double model_us(const TileCost& c, int bk, int64_t ipt, int64_t tiles, int64_t sk_tiles, int grid, bool staged) {
    const double t_iter = model_iter_us(c, bk), tile_us = staged ? MODEL_STAGED_TILE * c.tile_us : c.tile_us;
    double t = (double)ceil_div(tiles - sk_tiles, grid) * (ipt * t_iter + tile_us);
    if (sk_tiles == 0) return t;
    const int64_t iters = sk_tiles * ipt, ipw = ceil_div(iters, grid);
    const bool split_tiles = ipw % ipt != 0 && iters > ipw;
    const double waves = split_tiles ? (double)sk_tiles / grid : (double)(ipw / ipt);       // tiles a workgroup stores
    t += ipw * t_iter + tile_us * (waves > 1 ? waves : 1.0);
    if (split_tiles) {
        // about `split` workgroups share a tile: the partials an owner (or a group leader) fetches one after the
        // other - all of them up to 16 workgroups per tile, beyond that the two-level reduction with groups of 8 -
        // and the traffic of all of them together, which shares the memory system
        const double split = ipt > ipw ? (double)ipt / ipw : 1.0;
        const bool tree = split >= 16;
        t += MODEL_LEVEL_US * (tree ? 2 : 1) + (tree ? 8 + split / 8 : split) * c.bm * c.bn * 4 / MODEL_FETCH_BYTES_PER_US;
        t += (double)model_contributors(ceil_div(iters, ipw), ipt, ipw) * c.bm * c.bn * 8 / MODEL_TRAFFIC_BYTES_PER_US;
    }
    return t;
}

const TileCost* model_costs(int in_dtype, int* count) {
    const bool fp8 = in_dtype == SK_FP8_E4M3;
    *count = fp8 ? N_COSTS8 : N_COSTS16;
    return fp8 ? tile_costs8 : tile_costs16;
}
// The constants of a tile shape: the entry with its blk_m and blk_n.  A tile's rate hardly depends on blk_k, so the
// tiles of 128 columns (8 bits: of 128 rows) and more answer for any; the smaller ones for their own and, where that
// is 64, for less.  8 bits: 256 x 128, which has no kernel, as 128 x 256.
const TileCost* model_constants(int bm, int bn, int bk, int in_dtype) {
    int n;
    const TileCost* t = model_costs(in_dtype, &n);
    const bool fp8 = in_dtype == SK_FP8_E4M3;
    if (fp8 && bm == 256 && bn == 128) std::swap(bm, bn);
    for (int i = 0; i < n; i++)
        if (t[i].bm == bm && t[i].bn == bn && ((fp8 ? bm : bn) >= 128 || t[i].bk == bk || (t[i].bk == 64 && bk < 64))) return &t[i];
    return nullptr;
}

// Which logical workgroups an XCD runs (sk_plan_header.xcd_remap; the three maps are logical_wg's).  Measured on
// 1667 (size, tile) pairs whose tiles are all split, 16 and 8 bits, under each map, and on more under 1 and 2:
//  - the contiguous map (1) is the fastest in general: the workgroups of a tile then exchange their partials
//    inside one L2 (64 x 128 tiles of 8 workgroups, 512 x 512 x 8192: 14.4 us against 18.3 with either other map);
//  - with at least 4 workgroups per tile each XCD reads the whole K range of its few tiles, so operand blocks
//    shared with other XCDs' tiles are fetched once per XCD; sorted by K slice (2) they are fetched once.
//    Where that saves 20 MB or more in all it pays for the longer exchange: 2408 pairs under 1 and 2, tiles of at most
//    64 rows 4 - 18 % at 20 - 40 MB, 17 - 36 % above, larger tiles level at 20 - 40 MB, 3 - 17 % above (384 x 240 x
//    52832, 64 x 128 tiles: 48.1 -> 31.6 us; 512 x 240 x 63792, 64 x 128 8-bit tiles: 51.2 -> 26.8); below 20 MB it
//    loses 2 - 13 %.  Where the contiguous map
//    gives every XCD whole tiles, it keeps the exchange inside one L2 altogether, and what is saved has to be twice the
//    bytes of the partials (written and fetched) as well.  On 1939 such (size, tile) pairs the contiguous map is 10 %
//    faster up to once those bytes, 4 % up to twice, level up to three times, and the sorted one 6 - 20 % beyond
//    (1024 x 1024 x 8192, 128 x 256 8-bit tiles: 29.0 us, sorted 41.3);
//  - a single row of low 16-bit tiles over a large B streams B once and shares only the small A: the hardware
//    order (0), neighbouring column blocks on different XCDs, gains 2 - 6 % from 48 MB of B on (32 rows and
//    less: from 16 MB on) and loses 2 - 20 % below.  8-bit tiles lose 3 - 20 % with it at any size.
int choose_remap(const sk_plan_header& h) {
    const double es = h.in_dtype == SK_FP8_E4M3 ? 1 : 2;
    if (h.tiles_m == 1 && h.blk_m <= 64 && es == 2) {
        const double b_bytes = (double)h.K * (double)h.N * es;
        if (b_bytes >= (h.blk_m <= 32 ? 16e6 : 48e6)) return 0;
    }
    if (h.dp_tiles == 0 && h.tiles <= h.grid && h.grid <= 4096 && h.grid % 8 == 0 && 4ll * h.iters_per_wg <= h.iters_per_tile) {
        const double per_xcd = h.grid / 8.0 * h.iters_per_wg / h.iters_per_tile;   // tiles of one XCD under the contiguous map
        const double all = (double)h.tiles_m * h.blk_m + (double)h.tiles_n * h.blk_n;      // operand rows and columns
        double fetched;
        if (per_xcd >= 1) {
            double rows = per_xcd < SK_GROUP_ROWS ? per_xcd : SK_GROUP_ROWS;
            if (rows > h.tiles_m) rows = h.tiles_m;
            double cols = std::ceil(per_xcd / rows);
            if (cols > h.tiles_n) cols = h.tiles_n;
            fetched = 8 * std::min(rows * h.blk_m + cols * h.blk_n, all);
        } else {
            fetched = (double)h.tiles * (h.blk_m + h.blk_n);
        }
        const double saved = (fetched - all) * (double)h.K * es;
        // (tiles * ipt == grid * ipw: the ranges fill the tiles evenly; then an XCD's grid / 8 ranges may be whole tiles)
        const bool exchange_inside = h.total_iters == (int64_t)h.grid * h.iters_per_wg && (int64_t)(h.grid / 8) * h.iters_per_wg % h.iters_per_tile == 0;
        const double partials = (double)(h.grid - h.tiles) * h.blk_m * h.blk_n * 8;
        if (saved >= 20e6 && !(exchange_inside && saved < 2 * partials)) return 2;
    }
    return 1;
}

}  // namespace

extern "C" int sk_plan_estimate_us(const sk_plan_t* plan, double* microseconds) {
    if (!plan || !microseconds) return SK_ERR_INVALID_ARG;
    const sk_plan_header& h = plan->h;
    const TileCost* c = model_constants(h.blk_m, h.blk_n, h.blk_k, h.in_dtype);
    if (!c) return SK_ERR_UNSUPPORTED;
    *microseconds = model_us(*c, h.blk_k, h.iters_per_tile, h.tiles, h.sk_tiles, h.grid, model_staged(h.N, h.K, h.in_dtype));
    return SK_OK;
}

namespace {

// Dispatcher: the tile shape whose best schedule - whole tiles in waves, the remainder wave split, or every
// tile split - the cost model estimates the cheapest.  given: blk_m, blk_n, blk_k that the caller fixes (0 = free);
// then only shapes that agree with them and, with the given blk_k, have a kernel count.  False if there is none.
// policy, grid: those of the plan the tile is for.  On more workgroups than CUs a plan that splits tiles can only be
// launched if several workgroups fit a CU, so there a shape that can run goes before one that cannot, unless the
// model has it 1.4 times slower or more (a plan may also be meant for the atomic fix-up, which runs any grid).
bool pick_tile(int64_t M, int64_t N, int64_t K, int in_dtype, const int32_t* given, int policy, int64_t grid, int32_t* out_blk) {
    int n;
    const TileCost* costs = model_costs(in_dtype, &n);
    const bool free = !given[0] && !given[1] && !given[2];
    const bool staged = model_staged(N, K, in_dtype);
    const int64_t most = std::numeric_limits<int32_t>::max();
    double best_t = 0, runs_t = 0;
    int best = -1, runs = -1;
    auto bk_of = [&](const TileCost& c) { return given[2] ? given[2] : c.bk; };
    for (int i = 0; i < n; i++) {
        const TileCost& c = costs[i];
        const int bk = bk_of(c);
        if (!free && ((given[0] && given[0] != c.bm) || (given[1] && given[1] != c.bn) || !sk_kernel_available(in_dtype, c.bm, c.bn, bk))) continue;
        const int64_t ipt = ceil_div(K, bk), tiles_m = ceil_div(M, c.bm), tiles_n = ceil_div(N, c.bn);
        // beyond what sk_plan accepts: any answer will do, the first (largest) shape
        if (ipt > most || tiles_m > most || tiles_n > most || tiles_m * tiles_n > most || tiles_m * tiles_n > std::numeric_limits<int64_t>::max() / ipt) continue;
        const int64_t tiles = tiles_m * tiles_n;
        double t = model_us(c, bk, ipt, tiles, 0, MODEL_GRID, staged);
        t = std::min(t, model_us(c, bk, ipt, tiles, tiles, MODEL_GRID, staged));
        t = std::min(t, model_us(c, bk, ipt, tiles, tiles % MODEL_GRID, MODEL_GRID, staged));
        if (best < 0 || t < best_t) { best = i; best_t = t; }
        const int64_t iters = sk_tile_count(policy, tiles, grid) * ipt;
        if ((grid <= MODEL_GRID * c.per_cu || !splits_tiles(iters, ceil_div(iters, grid), ipt)) && (runs < 0 || t < runs_t)) { runs = i; runs_t = t; }
    }
    if (best < 0 && !free) return false;
    if (best < 0) best = 0;
    else if (runs >= 0 && runs_t < 1.4 * best_t) best = runs;
    out_blk[0] = costs[best].bm; out_blk[1] = costs[best].bn; out_blk[2] = bk_of(costs[best]);
    return true;
}

}  // namespace

extern "C" int sk_default_tile(int64_t M, int64_t N, int64_t K, int in_dtype, int32_t* out_blk) {
    if (!out_blk || M < 1 || N < 1 || K < 1 || !dtype_in_ok(in_dtype)) return SK_ERR_INVALID_ARG;
    const int32_t none[3] = {0, 0, 0};
    pick_tile(M, N, K, in_dtype, none, SK_POLICY_DP, MODEL_GRID, out_blk);
    return SK_OK;
}

extern "C" int sk_plan(int64_t M, int64_t N, int64_t K, int policy, const sk_config* cfg, sk_plan_t** out) {
    if (!out || M < 1 || N < 1 || K < 1) return SK_ERR_INVALID_ARG;
    if (policy < 0 || policy > SK_POLICY_SK6_DP_EXT) return SK_ERR_INVALID_ARG;
    sk_config c{};
    if (cfg) c = *cfg;
    if (c.blk_m < 0 || c.blk_n < 0 || c.blk_k < 0 || c.grid < 0 || c.tile_order < 0) return SK_ERR_INVALID_ARG;
    const int in_dtype = c.in_dtype ? c.in_dtype - 1 : SK_BF16;
    if (!dtype_in_ok(in_dtype)) return SK_ERR_INVALID_ARG;
    const int out_dtype = c.out_dtype ? c.out_dtype - 1 : (in_dtype == SK_FP8_E4M3 ? SK_BF16 : in_dtype);
    if (!dtype_out_ok(out_dtype)) return SK_ERR_INVALID_ARG;
    int order = c.tile_order ? c.tile_order - 1 : -1;   // -1: decided below, once the split is known
    if (order != -1 && order != SK_ORDER_ROW_MAJOR && order != SK_ORDER_GROUPED) return SK_ERR_INVALID_ARG;
    int32_t blk[3] = {c.blk_m, c.blk_n, c.blk_k};
    const int grid = c.grid ? c.grid : 256;
    if (!blk[0] || !blk[1] || !blk[2]) {
        // the rest of a partly given shape: from a shape that has a kernel with the given fields, else from the default
        int32_t def[3];
        if (!pick_tile(M, N, K, in_dtype, blk, policy, grid, def)) sk_default_tile(M, N, K, in_dtype, def);
        for (int i = 0; i < 3; i++) if (!blk[i]) blk[i] = def[i];
    }

    sk_plan_header h{};
    h.M = M; h.N = N; h.K = K; h.policy = policy;
    h.blk_m = blk[0]; h.blk_n = blk[1]; h.blk_k = blk[2]; h.grid = grid;
    h.in_dtype = in_dtype; h.out_dtype = out_dtype;
    // Algorithm 1: iterations per tile, total iterations
    const int64_t tiles_m = ceil_div(M, blk[0]), tiles_n = ceil_div(N, blk[1]);
    const int64_t ipt = ceil_div(K, blk[2]);
    const int64_t tiles = tiles_m * tiles_n;
    const int64_t imax = std::numeric_limits<int32_t>::max();
    if (tiles_m > imax || tiles_n > imax || tiles > imax - grid || ipt > imax) return SK_ERR_INVALID_ARG;
    if (tiles > std::numeric_limits<int64_t>::max() / ipt) return SK_ERR_INVALID_ARG;
    h.tiles_m = (int32_t)tiles_m; h.tiles_n = (int32_t)tiles_n; h.tiles = (int32_t)tiles;
    h.iters_per_tile = (int32_t)ipt;
    h.total_iters = tiles * ipt;
    const int64_t sk_tiles = sk_tile_count(policy, tiles, grid);     // Stream-K / data-parallel split
    // Default tile order: the one under which the tiles that an XCD's workgroups hold at the same
    // time touch fewer operand rows and columns (A row-blocks x blk_m + B column-blocks x blk_n,
    // averaged over the XCDs): that is what the XCD's L2 has to keep per k-iteration.  The
    // workgroups of the grid hold the first min(tiles, grid) tile indices at once, an eighth of
    // them (consecutive indices) per XCD.  Picking by this figure loses 0.4 - 0.7 % against the
    // faster order of each size on a 500-size sweep (either order alone: 0.5 - 3 %, up to 1.5x).
    if (order < 0) {
        auto footprint = [&](int ord) {
            const int64_t active = tiles < grid ? tiles : grid;
            const int64_t per_xcd = active / 8 > 0 ? active / 8 : 1;
            double total = 0;
            int chunks = 0;
            for (int64_t c = 0; c < active; c += per_xcd, ++chunks) {
                std::vector<int64_t> row, col;
                for (int64_t t = c; t < c + per_xcd && t < active; t++) {
                    int64_t tm, tn;
                    if (ord == SK_ORDER_ROW_MAJOR) {
                        tm = t / tiles_n; tn = t % tiles_n;
                    } else {
                        const int64_t per_band = SK_GROUP_ROWS * tiles_n, first = t / per_band * SK_GROUP_ROWS;
                        const int64_t band_rows = tiles_m - first < SK_GROUP_ROWS ? tiles_m - first : SK_GROUP_ROWS;
                        tm = first + t % per_band % band_rows; tn = t % per_band / band_rows;
                    }
                    row.push_back(tm);
                    col.push_back(tn);
                }
                std::sort(row.begin(), row.end());
                std::sort(col.begin(), col.end());
                const auto rows = std::unique(row.begin(), row.end()) - row.begin();
                const auto cols = std::unique(col.begin(), col.end()) - col.begin();
                total += (double)rows * blk[0] + (double)cols * blk[1];
            }
            return total / chunks;
        };
        try {
            order = footprint(SK_ORDER_GROUPED) < footprint(SK_ORDER_ROW_MAJOR) ? SK_ORDER_GROUPED : SK_ORDER_ROW_MAJOR;
        } catch (const std::bad_alloc&) {
            return SK_ERR_NOMEM;
        }
    }
    h.tile_order = order;
    h.fixup = SK_FIXUP_FLAGS;
    h.batch_order = SK_STREAMK_FIRST;
    h.segment_order = SK_SEGMENTS_K_ALIGNED;
    h.sk_tiles = (int32_t)sk_tiles;
    h.dp_tiles = (int32_t)(tiles - sk_tiles);
    h.sk_iters = sk_tiles * ipt;
    const int64_t ipw = ceil_div(h.sk_iters, grid);   // Algorithm 1: iterations per workgroup, on the split region
    if (ipw > imax) return SK_ERR_INVALID_ARG;
    h.iters_per_wg = (int32_t)ipw;
    h.xcd_remap = choose_remap(h);
    h.dp_waves = (int32_t)ceil_div(h.dp_tiles, grid);
    h.has_kernel = sk_kernel_available(in_dtype, blk[0], blk[1], blk[2]) ? 1 : 0;

    sk_plan_t* p = new (std::nothrow) sk_plan_t;
    if (!p) return SK_ERR_NOMEM;
    p->h = h;
    p->needs_fixup = splits_tiles(h.sk_iters, ipw, ipt) ? 1 : 0;
    *out = p;
    return SK_OK;
}

extern "C" int sk_plan_info(const sk_plan_t* plan, sk_plan_header* out) {
    if (!plan || !out) return SK_ERR_INVALID_ARG;
    *out = plan->h;
    return SK_OK;
}

extern "C" int sk_plan_ranges(const sk_plan_t* plan, sk_wg_range* out) {
    if (!plan || !out) return SK_ERR_INVALID_ARG;
    for (int x = 0; x < plan->h.grid; x++) expand_wg(plan->h, x, nullptr, &out[x]);
    return SK_OK;
}

extern "C" int sk_plan_segments(const sk_plan_t* plan, sk_segment* out, size_t cap, size_t* n) {
    if (!plan || !n || (!out && cap)) return SK_ERR_INVALID_ARG;
    std::vector<sk_segment> segs;
    try {
        for (int x = 0; x < plan->h.grid; x++) expand_wg(plan->h, x, &segs, nullptr, plan->dp_first != 0, plan->k_aligned != 0);
    } catch (const std::bad_alloc&) {
        return SK_ERR_NOMEM;
    }
    *n = segs.size();
    if (segs.size() > cap) return SK_ERR_INVALID_ARG;
    if (!segs.empty()) std::memcpy(out, segs.data(), segs.size() * sizeof(sk_segment));
    return SK_OK;
}

extern "C" int sk_plan_tile_coords(const sk_plan_t* plan, int32_t tile, int32_t* tile_m, int32_t* tile_n) {
    if (!plan || !tile_m || !tile_n || tile < 0 || tile >= plan->h.tiles) return SK_ERR_INVALID_ARG;
    const sk_plan_header& h = plan->h;
    if (h.tile_order == SK_ORDER_ROW_MAJOR) {
        *tile_m = tile / h.tiles_n;
        *tile_n = tile % h.tiles_n;
    } else {
        // bands of SK_GROUP_ROWS tile rows, walked column by column
        const int per_band = SK_GROUP_ROWS * h.tiles_n;
        const int band_row = (tile / per_band) * SK_GROUP_ROWS;
        const int rows = h.tiles_m - band_row < SK_GROUP_ROWS ? h.tiles_m - band_row : SK_GROUP_ROWS;
        const int within = tile % per_band;
        *tile_m = band_row + within % rows;
        *tile_n = within / rows;
    }
    return SK_OK;
}

extern "C" int bloom_shape_key(const sk_plan_t* plan, uint32_t* key) {
    if (!plan || !key) return SK_ERR_INVALID_ARG;
    const sk_plan_header& h = plan->h;
    uint32_t waves = (uint32_t)(h.tiles / h.grid);
    if (waves > 3) waves = 3;
    const uint32_t rem = (uint32_t)(h.tiles % h.grid);
    const uint32_t fill = (4 * rem + (uint32_t)h.grid - 1) / (uint32_t)h.grid;   // 0 = no remainder wave, 1..4 quarters
    uint32_t lg = 0;
    for (uint32_t v = (uint32_t)h.iters_per_tile; v > 1; v >>= 1) lg++;
    if (lg > 12) lg = 12;
    key[0] = (uint32_t)h.blk_m << 16 | ((uint32_t)h.blk_n & 0xFFFFu);
    key[1] = waves << 8 | fill;
    key[2] = lg << 16 | ((uint32_t)h.blk_k & 0xFFFFu);
    return SK_OK;
}

// Map 1 of logical_wg (streamk_kernels.h): how many logical ids, the first ones, are dealt to the XCDs evenly because the others have no work
// in the last wave of tiles, or none at all (0: no such two kinds).  Contiguous blocks would leave whole XCDs idle there and crowd the
// others, which costs what their CUs share: an L2's bandwidth, the fabric port and, most of all, the clock of an XCD
// whose 32 CUs all run the matrix cores.  Neighbours that an XCD's L2 served together are taken apart, which costs something where few
// are left.  Contiguous -> spread, 256 workgroups, per cent of the time; 1200 plans, 4 to 40 iterations per tile, 16 bits unless said:
//  - less than one wave of whole tiles.  256 x 256 (8 bits too), 20 - 160 tiles -5 .. -26 (K = 2048, 128 tiles, 54.7 -> 40.3 us), 190 - 232 -1 .. -14; 256 x 128 and 8-bit
//    128 x 256 -4 .. -21 to 190 tiles, 0 .. -7 above (one of 32 plans +2.5); 128 x 128 -2 .. -12 to 190, 0 .. -3 above (20 tiles of 40 iterations
//    +2 .. +4); 64 x 128 -1 .. -11 to 17 iterations, +4 .. -6 at 40, nearly a wave of 16 and more +1 .. -2; 32 x 128 at 17 iterations 0 .. -19, below 16
//    level, at 40 +3 .. -14; 16 x 128 from 32 iterations on +1 .. -13, below level; fewer than 16 tiles of any shape are level to slower, tiles of
//    64 columns lose as often as they gain;
//  - the last of several waves, where the full ones then hold two blocks of tiles per XCD.  Behind one wave, a last one of 4 - 8 tiles: 256 x 256 +1 .. +4, 256 x 128 and
//    8-bit 128 x 256 +2 .. +7, 128 x 128 +1 .. +5; of 16 - 24 +4 .. -3; of 32 - 154 256 x 256 0 .. -13, 256 x 128 0 .. -8, 8-bit 128 x 256 0 .. -7, 128 x 128 of 32 - 52 +3 .. -5,
//    64 - 154 +2 .. -4; 256 x 256 behind two waves, 8 tiles +1 .. +5, 28 - 148 from 8 iterations on 0 .. -11, below +6 .. -2, behind any number from 32
//    iterations on -1 .. -7; the others behind two, and tiles of at most 64 rows anywhere, lose up to 4 as often as they gain;
//  - Stream-K plans with empty ranges: all tiles 0 .. -26 (182 plans, four of them +1 .. +4) while 32 to 240 workgroups are busy; fewer, all of one
//    tile, +1 .. +5; 16-row tiles that 17 to 36 workgroups share -6 .. +8 (5 x 893 x 3328 8.4 -> 7.9 us, 70 x 120 x 4096 6.6 -> 7.0);
//  - not where nearly all workgroups have work: 3840 x 4224 x 4096, 255 tiles, 107.1 -> 107.9 us.
int sk_first_ids(const sk_plan_header& h) {
    if (h.xcd_remap != 1 || h.blk_n < 128) return 0;
    const int most = h.grid - h.grid / 16;
    if (h.sk_tiles > 0) {
        if (h.dp_tiles > 0) return 0;
        const int busy = (int)((h.sk_iters + h.iters_per_wg - 1) / h.iters_per_wg);
        return busy >= 32 && busy <= most ? busy : 0;
    }
    const int last = h.tiles % h.grid, full = h.tiles / h.grid, ipt = h.iters_per_tile, area = h.blk_m * h.blk_n;
    if (last > most) return 0;
    if (full == 0) return last >= 16 && (h.blk_m >= 64 || h.blk_m * (int64_t)ipt >= 512) ? last : 0;
    if (area < 128 * 128 || 8ll * last < (area >= 256 * 128 ? 1 : 2) * h.grid) return 0;
    const bool few = 8ll * last <= 5ll * h.grid;
    if (area >= 256 * 256) return (few && (full == 1 || (full == 2 && ipt >= 8))) || ipt >= 32 ? last : 0;
    return full == 1 && few ? last : 0;
}

// Where the shared reduction (store_shares in streamk_kernels.h) is the faster fix-up: the owner's chain of fetches, n - 1 partial
// tiles through one CU, has to be longer than what sharing adds: the owner's own piece is parked and waited for too.  A range that goes
// on into the next tile ends with shares of two tiles, and the piece parked first is fetched last; that costs most where neighbours
// share an XCD, whose L2 then serves the owner (map 1 or 0 of the workgroups; sorted by K slice, map 2, the owner fetches from
// all XCDs).  n = ipt / ipw, owner alone -> shared, same build, 16 bits unless said; 450 plans, per cent of the time:
//  - ranges that end with the tiles, or map 2: from n = 4.5 on 256 x 256 -7 .. -42, 256 x 128 and 128 x 256 -5 .. -44, 128 x 128 -3 .. -25, and
//    below 4.5 level to slower (n = 3: 384 x 3584 x 1536 on 128 x 128 12.1 -> 13.6 us); 64 x 128 from 7 on -7 .. -21; 32 x 128 and 64 x 64 from
//    7.6 on -1 .. -24 (one plan at 7.1 and one at 7.3 +4, +2);
//  - straddling ranges otherwise: 128 x 128 (8 bits too) n = 4.5 .. 6.4 +1 .. +18, from 7.4 on -8 .. -27; 256 x 128 4.7 .. 6.4 +9 .. -4, from
//    7.4 on -6 .. -36; 8-bit 128 x 256 4.5 .. 5.5 +4 .. +15, 5.6 .. 6.4 +2 .. -6; 256 x 256 4.7 .. 5.4 +1 .. +6, 6.2 -3, 6.4 -7, in 8 bits -2 .. -14 from
//    4.7 on; 64 x 128 (8 bits too) from 7.3 on -1 .. -19; 32 x 128 (8 bits too) and 64 x 64 7.3 .. 8.4 +7 .. 0, 9.1 .. 10.4 +2 .. -3, 11.5 .. 16.3 0 .. -7,
//    18 .. 20 +6 .. -4;
//  - more than 1.25 workgroups per 1 KB unit of the tile: 64 x 128, n = 57: +3, 32 x 128, n = 40: +3; tiles of 8 KB, 16 x 128 and 32 x 64, +2 .. +25 at any n.
// Only where nothing follows the Stream-K work, whose workgroups would otherwise wait with tiles of their own left to do.
bool sk_shared_reduction(const sk_plan_t* plan) {
    const sk_plan_header& h = plan->h;
    if (plan->fixup != SK_FIXUP_FLAGS || !plan->needs_fixup || !plan->k_aligned || h.dp_tiles > 0 || h.grid > 4096) return false;
    const int64_t tile_kb = (int64_t)h.blk_m * h.blk_n / 256, ipt = h.iters_per_tile, ipw = h.iters_per_wg;
    if (ipt > (SK_MAX_SHARERS - 2) * ipw) return false;      // at most ceil(ipt / ipw) + 1 workgroups
    int64_t least = tile_kb >= 64 ? 18 : 28, most = 5 * tile_kb;   // workgroups per tile, in quarters
    if (ipt % ipw != 0 && h.xcd_remap != 2) {
        if (tile_kb >= 256) least = h.in_dtype == SK_FP8_E4M3 ? 18 : 24;
        else if (tile_kb >= 64) least = 26;
        else if (tile_kb < 32) least = 36, most = 4 * (tile_kb + 1);
    }
    return tile_kb >= 16 && 4 * ipt >= least * ipw && 4 * ipt <= most * ipw;
}

size_t sk_ws_least_bytes(const sk_plan_t* plan) {
    const sk_plan_header& h = plan->h;
    if (plan->fixup == SK_FIXUP_ATOMIC) return sk_ws_partials_offset(h.grid) + sk_ws_image_bytes(plan);
    return sk_ws_partials_offset(h.grid) + (size_t)h.grid * h.blk_m * h.blk_n * sizeof(float);
}

extern "C" size_t sk_workspace_bytes(const sk_plan_t* plan) {
    if (!plan) return 0;
    // a slot per tile for owners whose range goes on into the next tile
    const sk_plan_header& h = plan->h;
    const bool more = sk_shared_reduction(plan) && h.iters_per_tile % h.iters_per_wg != 0;
    return sk_ws_least_bytes(plan) + (more ? (size_t)h.tiles * h.blk_m * h.blk_n * sizeof(float) : 0);
}

extern "C" int sk_plan_set_fixup(sk_plan_t* plan, int fixup) {
    if (!plan || (fixup != SK_FIXUP_FLAGS && fixup != SK_FIXUP_ATOMIC) || plan->workspace) return SK_ERR_INVALID_ARG;
    plan->fixup = fixup;
    plan->h.fixup = fixup;
    return SK_OK;
}

extern "C" int sk_plan_set_batch_order(sk_plan_t* plan, int batch_order) {
    if (!plan || (batch_order != SK_STREAMK_FIRST && batch_order != SK_DATA_PARALLEL_FIRST)) return SK_ERR_INVALID_ARG;
    plan->dp_first = batch_order == SK_DATA_PARALLEL_FIRST;
    plan->h.batch_order = batch_order;
    return SK_OK;
}

extern "C" int sk_plan_set_segment_order(sk_plan_t* plan, int segment_order) {
    if (!plan || (segment_order != SK_SEGMENTS_ASCENDING && segment_order != SK_SEGMENTS_K_ALIGNED)) return SK_ERR_INVALID_ARG;
    plan->k_aligned = segment_order == SK_SEGMENTS_K_ALIGNED;
    plan->h.segment_order = segment_order;
    return SK_OK;
}

extern "C" int sk_plan_set_spin_limit(sk_plan_t* plan, uint32_t polls) {
    if (!plan) return SK_ERR_INVALID_ARG;
    plan->spin_limit = polls;
    return SK_OK;
}

extern "C" int sk_plan_set_kernel_variant(sk_plan_t* plan, int variant) {
    if (!plan || variant < 0) return SK_ERR_INVALID_ARG;
    plan->kernel_variant = variant;
    return SK_OK;
}

extern "C" void sk_plan_destroy(sk_plan_t* plan) { delete plan; }

extern "C" const char* sk_status_str(int status) {
    switch (status) {
    case SK_OK: return "ok";
    case SK_ERR_INVALID_ARG: return "invalid argument";
    case SK_ERR_UNSUPPORTED: return "unsupported configuration";
    case SK_ERR_WORKSPACE: return "workspace missing or too small";
    case SK_ERR_HIP: return "HIP runtime error";
    case SK_ERR_NOMEM: return "out of host memory";
    case SK_ERR_TIMEOUT: return "tile owner timed out waiting for a partial tile";
    default: return "unknown status";
    }
}
