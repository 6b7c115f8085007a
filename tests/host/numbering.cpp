// Host-only: which logical ids the workgroups of a launch run where the first ones are dealt to the XCDs evenly (sk_spread_id, sk_first_ids).
// usage: numbering bijection              every grid and every number of first ids: the ids 0 .. grid - 1, each once, the first ones spread
//        numbering M N K POLICY BLK_M BLK_N BLK_K GRID DTYPE     prints sk_first_ids of that plan
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>
#include "streamk.h"
#include "streamk_internal.h"

bool sk_kernel_available(int, int, int, int) { return true; }

#define FAIL(...) do { fprintf(stderr, __VA_ARGS__); fprintf(stderr, "\n"); return 1; } while (0)

int main(int argc, char** argv) {
    if (argc == 2 && !strcmp(argv[1], "bijection")) {
        for (int grid = 8; grid <= 4096; grid += grid < 1024 ? 8 : 512)
            for (int first = 0; first <= grid / 8; first++) {
                std::vector<int> seen(grid, 0);
                for (int hw = 0; hw < grid; hw++) {
                    const int id = sk_spread_id(hw % 8, hw / 8, first, grid / 8 - first);
                    if (id < 0 || id >= grid || seen[id]++) FAIL("grid %d, %d first ids per XCD: workgroup %d runs id %d", grid, first, hw, id);
                    if ((id < 8 * first) != (hw / 8 < first)) FAIL("grid %d, %d first ids per XCD: id %d on workgroup %d", grid, first, id, hw);
                }
            }
        printf("ok\n");
        return 0;
    }
    if (argc != 10) FAIL("usage: numbering bijection | M N K POLICY BLK_M BLK_N BLK_K GRID DTYPE");
    sk_config cfg{};
    cfg.blk_m = atoi(argv[5]); cfg.blk_n = atoi(argv[6]); cfg.blk_k = atoi(argv[7]); cfg.grid = atoi(argv[8]); cfg.in_dtype = atoi(argv[9]) + 1;
    sk_plan_t* plan = nullptr;
    if (sk_plan(atoll(argv[1]), atoll(argv[2]), atoll(argv[3]), atoi(argv[4]), &cfg, &plan) != SK_OK) FAIL("sk_plan failed");
    sk_plan_header h;
    sk_plan_info(plan, &h);
    printf("%d\n", sk_first_ids(h));
    sk_plan_destroy(plan);
    return 0;
}
