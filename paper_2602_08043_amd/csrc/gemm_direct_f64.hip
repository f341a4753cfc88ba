// FP64 verified GEMM of any shape, alignment and layout of B (direct kernels).
#include "gemm_direct.h"
namespace vabft {
int gemm_direct_launch_f64(const DirectArgs& d, int shape, int transB, hipStream_t st) {
    return gemm_direct_launch_t<false, double>(d, shape, transB, st);
}
}  // namespace vabft
