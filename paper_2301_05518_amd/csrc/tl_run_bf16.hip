// Whole-run kernels and the Laplacian stored in BF16: every link form (two-links or one-links, 18
// or 12 reals).
#include "tl_laplacian.h"
#include "tl_run.h"

namespace tl {

hipError_t launch_run_bf16(const RunConfig& cfg, const RunArgs& args, double alpha, double beta, hipStream_t stream) {
  return launch_run_p<BF16>(cfg, args, alpha, beta, stream);
}

hipError_t run_attributes_bf16() { return run_attributes<BF16>(); }

hipError_t launch_laplacian_bf16(const char* W, int64_t w_mu_stride, int Vp, const int32_t L[4], int hop, bool w12,
                               const void* in, void* out, double alpha, double beta, hipStream_t stream) {
  return launch_laplacian_p<BF16>(W, w_mu_stride, Vp, L, hop, w12, in, out, alpha, beta, stream);
}

}  // namespace tl
