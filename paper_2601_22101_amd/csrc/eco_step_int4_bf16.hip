// Instantiations of the fused ECO step kernel: INT4 codes, bfloat16 optimizer state.
#include "eco_step_resident.hpp"

namespace eco {
hipError_t launch_step_int4_bf16(const KernelVariant &kv, const StepLaunch &sl, hipStream_t stream) {
  return launch_step_variants<FMT_INT4, true>(kv, sl, stream);
}
}  // namespace eco
