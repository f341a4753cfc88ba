// BF16 verified GEMM in 256 x 256 tiles, B stored N x K.
#include "gemm16_fast.h"
namespace vabft {
int gemm16_launch_bf16_nt(const GemmArgs& a, int mode, int form, hipStream_t st) {
    return gemm16_fast_launch_tb<bf16_t, 1>(a, mode, form, st);
}
}  // namespace vabft
