// bf16 kernels of the Stream-K GEMM: tiles of at most 64 rows (see streamk_kernels.h).
#include "streamk_kernels.h"
namespace streamk_detail {
void register_bf16_low(KernelEntry** t, int* n) { add_16bit_low_tiles<SK_BF16>(t, n); }
}  // namespace streamk_detail
