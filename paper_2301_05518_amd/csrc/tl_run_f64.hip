// Whole-run kernels and the Laplacian stored in F64: every link form (two-links or one-links, 18
// or 12 reals).
#include "tl_laplacian.h"
#include "tl_run.h"

namespace tl {

hipError_t launch_run_f64(const RunConfig& cfg, const RunArgs& args, double alpha, double beta, hipStream_t stream) {
  return launch_run_p<F64>(cfg, args, alpha, beta, stream);
}

hipError_t run_attributes_f64() { return run_attributes<F64>(); }

hipError_t launch_laplacian_f64(const char* W, int64_t w_mu_stride, int Vp, const int32_t L[4], int hop, bool w12,
                               const void* in, void* out, double alpha, double beta, hipStream_t stream) {
  return launch_laplacian_p<F64>(W, w_mu_stride, Vp, L, hop, w12, in, out, alpha, beta, stream);
}

}  // namespace tl
