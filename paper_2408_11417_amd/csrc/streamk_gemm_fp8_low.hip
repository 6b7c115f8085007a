// fp8 (e4m3) kernels of the Stream-K GEMM: the tiles for problems that fill few tiles of 256 columns (see
// streamk_kernels.h).  64 x 8192 x 8192: 16.9 us on 64 x 128 tiles, 29.3 on 128 x 256 (whose second 64 rows are padding
// and whose partial tiles are four times as large); 2048^3 12.1 us on 128 x 128, 18.3 on 128 x 256; 1024^3 5.2 us on
// 32 x 128, 12.8 on 128 x 256.  256-column tiles of 64 and 32 rows were slower on every size tried (64 x 8192 x 8192:
// 27.7 and 18.2 us): twice as many workgroups share a tile.
#include "streamk_kernels.h"
namespace streamk_detail {
template <bool ATOMIC> void add_tiles(KernelEntry** t, int* n) {
    t[(*n)++] = make_entry<Cfg<SK_FP8_E4M3, 128, 128, 128, 2, 4, 32, 3>, ATOMIC>();
    t[(*n)++] = make_entry<Cfg<SK_FP8_E4M3, 64, 128, 128, 2, 4, 32, 4>, ATOMIC>();
    t[(*n)++] = make_entry<Cfg<SK_FP8_E4M3, 32, 128, 128, 1, 4, 32, 4>, ATOMIC>();
}
void register_fp8_low(KernelEntry** t, int* n) {
    add_tiles<false>(t, n);
    add_tiles<true>(t, n);
}
}  // namespace streamk_detail
