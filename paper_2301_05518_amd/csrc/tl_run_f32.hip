// Whole-run kernels stored in F32: every link form (two-links or one-links, 18 or 12 reals).
#include "tl_run.h"

namespace tl {

hipError_t launch_run_f32(const RunConfig& cfg, const RunArgs& args, double alpha, double beta, hipStream_t stream) {
  return launch_run_p<F32>(cfg, args, alpha, beta, stream);
}

hipError_t run_attributes_f32() { return run_attributes<F32>(); }

}  // namespace tl
