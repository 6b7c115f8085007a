// Host-only run of the shared reduction's protocol (sk_leave_tile and the counts of a tile's line, streamk_internal.h): threads
// stand for the workgroups that are on the device at once, SLOTS per XCD, and take the launch's workgroups in hardware order, as a
// device does of which the launch gets only a part.  Whatever the part: the run ends, every unit of every split tile is stored
// once, after all pieces of the tile have been parked, and the lines are back at zero.
// usage: shared_reduction M N K BLK_M BLK_N BLK_K GRID SLOTS POLLS ORDER   (ORDER: 0 hardware, 1 contiguous, 2 shuffled)
#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <numeric>
#include <random>
#include <thread>
#include <vector>
#include "streamk.h"
#include "streamk_internal.h"

bool sk_kernel_available(int, int, int, int) { return true; }

#define FAIL(...) do { fprintf(stderr, __VA_ARGS__); fprintf(stderr, "\n"); return 1; } while (0)

struct Line {
    std::atomic<uint32_t>* word;
    uint32_t load(int i = 0) const { return word[i].load(); }
    uint32_t add(uint32_t v) const { return word->fetch_add(v); }
    void give_up(int j) const { word[1 + j / 32].fetch_or(1u << j % 32); }
    bool is_given_up(int j) const { return load(1 + j / 32) >> j % 32 & 1; }
    void clear(int i = 0) const { word[i].store(0); }
};

int main(int argc, char** argv) {
    if (argc != 11) FAIL("usage: shared_reduction M N K BLK_M BLK_N BLK_K GRID SLOTS POLLS ORDER");
    sk_config cfg{};
    cfg.blk_m = atoi(argv[4]); cfg.blk_n = atoi(argv[5]); cfg.blk_k = atoi(argv[6]); cfg.grid = atoi(argv[7]);
    const int slots = atoi(argv[8]), polls_limit = atoi(argv[9]), order = atoi(argv[10]);
    sk_plan_t* plan = nullptr;
    if (sk_plan(atoll(argv[1]), atoll(argv[2]), atoll(argv[3]), SK_POLICY_ALL_SK, &cfg, &plan) != SK_OK) FAIL("sk_plan failed");
    if (!sk_shared_reduction(plan)) FAIL("the plan has no shared reduction");
    sk_plan_header h;
    sk_plan_info(plan, &h);
    std::vector<sk_wg_range> ranges(h.grid);
    sk_plan_ranges(plan, ranges.data());

    const int units = h.blk_m * h.blk_n / 256, ipt = h.iters_per_tile, ipw = h.iters_per_wg;
    std::vector<int> logical(h.grid);
    std::iota(logical.begin(), logical.end(), 0);
    if (order == 1) for (int i = 0; i < h.grid; i++) logical[i] = i % 8 * (h.grid / 8) + i / 8;
    if (order == 2) std::shuffle(logical.begin(), logical.end(), std::mt19937(5));

    std::vector<std::atomic<uint32_t>> words((size_t)h.grid * SK_LINE_WORDS);
    std::vector<std::atomic<int>> parked(h.tiles), stored((size_t)h.tiles * units);
    std::atomic<int> too_early{0}, given_up{0}, next[8] = {};
    auto line_of = [&](int tile) { return Line{&words[(size_t)tile * SK_LINE_WORDS]}; };
    struct Share { int tile, last_wg, n, j; };
    auto share_of = [&](int x, int tile) {
        const int first = tile * ipt / ipw, last = (tile * ipt + ipt - 1) / ipw;
        return Share{tile, last, last - first + 1, last - x};
    };
    auto store = [&](const Share& s, int j) {
        for (int u = sk_share_begin(units, j, s.n); u < sk_share_begin(units, j + 1, s.n); u++) {
            too_early += parked[s.tile] != s.n;
            stored[(size_t)s.tile * units + u]++;
        }
    };
    auto workgroup = [&](int x) {
        const int begin = (int)ranges[x].sk_iter_begin, end = (int)ranges[x].sk_iter_end;
        if (begin >= end) return;
        std::vector<Share> mine;
        for (int tile = begin / ipt; tile <= (end - 1) / ipt; tile++) mine.push_back(share_of(x, tile));
        std::vector<int> with_share(mine.size());
        for (size_t i = mine.size(); i-- > 0;) { parked[mine[i].tile]++; line_of(mine[i].tile).add(SK_ARRIVES); }
        for (size_t i = 0; i < mine.size(); i++) with_share[i] = sk_share_begin(units, mine[i].j, mine[i].n) == sk_share_begin(units, mine[i].j + 1, mine[i].n);
        for (int polls = 0;; polls++) {
            bool all = true;
            for (size_t i = 0; i < mine.size(); i++) {
                if (!with_share[i]) with_share[i] = sk_arrived(line_of(mine[i].tile).load()) == (uint32_t)mine[i].n;
                all = all && with_share[i];
            }
            if (all || polls >= polls_limit) break;
            std::this_thread::yield();
        }
        std::vector<uint32_t> word(mine.size());
        for (size_t i = 0; i < mine.size(); i++) { word[i] = sk_leave_tile(line_of(mine[i].tile), mine[i].j, with_share[i]); given_up += !with_share[i]; }
        for (size_t i = 0; i < mine.size(); i++) if (with_share[i]) store(mine[i], mine[i].j);
        for (size_t i = 0; i < mine.size(); i++) {
            if (sk_left(word[i]) != (uint32_t)mine[i].n) continue;
            const Line line = line_of(mine[i].tile);
            if (sk_given_up(word[i]) > 0) for (int j = 0; j < mine[i].n; j++) if (line.is_given_up(j)) store(mine[i], j);
            for (int w = 0; w < SK_LINE_WORDS; w++) line.clear(w);
        }
    };
    std::vector<std::thread> threads;
    for (int t = 0; t < 8 * slots; t++)
        threads.emplace_back([&, xcd = t % 8] {
            for (int i = next[xcd]++; i * 8 + xcd < h.grid; i = next[xcd]++) workgroup(logical[i * 8 + xcd]);
        });
    for (auto& t : threads) t.join();

    if (too_early) FAIL("%d units were stored before all pieces of their tile were parked", too_early.load());
    for (size_t u = 0; u < stored.size(); u++) if (stored[u] != 1) FAIL("unit %zu stored %d times", u, stored[u].load());
    for (size_t w = 0; w < words.size(); w++) if (words[w]) FAIL("word %zu left at %u", w, words[w].load());
    printf("ok %d tiles, at most %d workgroups of a tile, %d shares given up\n", h.tiles, share_of(0, 0).n, given_up.load());
    sk_plan_destroy(plan);
    return 0;
}
