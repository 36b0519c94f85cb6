// Whole-run kernels stored in BF16: every link form (two-links or one-links, 18 or 12 reals).
#include "tl_run.h"

namespace tl {

hipError_t launch_run_bf16(const RunConfig& cfg, const RunArgs& args, double alpha, double beta, hipStream_t stream) {
  return launch_run_p<BF16>(cfg, args, alpha, beta, stream);
}

hipError_t run_attributes_bf16() { return run_attributes<BF16>(); }

}  // namespace tl
