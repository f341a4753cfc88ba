// FP16 verified GEMM in 256 x 256 tiles, B stored K x N.
#include "gemm16_fast.h"
namespace vabft {
int gemm16_launch_f16_nn(const GemmArgs& a, int mode, int form, hipStream_t st) {
    return gemm16_fast_launch_tb<f16_t, 0>(a, mode, form, st);
}
}  // namespace vabft
