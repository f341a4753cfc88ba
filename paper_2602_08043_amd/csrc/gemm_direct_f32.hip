// FP32 verified GEMM of any shape, alignment and layout of B (direct kernels).
#include "gemm_direct.h"
namespace vabft {
int gemm_direct_launch_f32(const DirectArgs& d, int shape, int transB, hipStream_t st) {
    return gemm_direct_launch_t<false, float>(d, shape, transB, st);
}
}  // namespace vabft
