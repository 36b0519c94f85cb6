// Whole-run kernels stored in F16S: every link form (two-links or one-links, 18 or 12 reals).
#include "tl_run.h"

namespace tl {

hipError_t launch_run_f16s(const RunConfig& cfg, const RunArgs& args, double alpha, double beta, hipStream_t stream) {
  return launch_run_p<F16S>(cfg, args, alpha, beta, stream);
}

hipError_t run_attributes_f16s() { return run_attributes<F16S>(); }

}  // namespace tl
