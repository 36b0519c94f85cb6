// Whole-run kernels stored in F64: every link form (two-links or one-links, 18 or 12 reals).
#include "tl_run.h"

namespace tl {

hipError_t launch_run_f64(const RunConfig& cfg, const RunArgs& args, double alpha, double beta, hipStream_t stream) {
  return launch_run_p<F64>(cfg, args, alpha, beta, stream);
}

hipError_t run_attributes_f64() { return run_attributes<F64>(); }

}  // namespace tl
