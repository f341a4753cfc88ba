// BF16 verified GEMM with position-weighted row sums, of any shape, alignment and layout of B (direct kernels).
#include "gemm_direct.h"
namespace vabft {
int gemm_direct_launch_w_bf16(const DirectArgs& d, int shape, int transB, hipStream_t st) {
    return gemm_direct_launch_t<true, bf16_t>(d, shape, transB, st);
}
}  // namespace vabft
