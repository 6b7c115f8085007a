// bf16 kernel of the Stream-K GEMM for plans of whole tiles (see streamk_whole_tiles.h).
#include "streamk_whole_tiles.h"
namespace streamk_detail {
void add_across_bf16(KernelEntry** t, int n) { add_across<Cfg<SK_BF16, 256, 256, 64, 2, 2, 32, 3, 2, 1>>(t, n); }
}  // namespace streamk_detail
