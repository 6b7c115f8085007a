// fp8 (e4m3) kernel of the Stream-K GEMM for plans of whole tiles (see streamk_whole_tiles.h).
#include "streamk_whole_tiles.h"
namespace streamk_detail {
void add_across_fp8(KernelEntry** t, int n) { add_across<Cfg<SK_FP8_E4M3, 256, 256, 128, 2, 2, 32, 3, 2, 1>>(t, n); }
}  // namespace streamk_detail
