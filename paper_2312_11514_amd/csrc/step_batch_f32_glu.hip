#include "lif_step1.h"

namespace lif {
hipError_t launch_step_batch_f32_glu(const StepArgs& a, int grid, size_t lds, bool allow, hipStream_t s) {
    return launch_step_batch_as<float, true, false, false>(a, grid, lds, allow, s);
}
}  // namespace lif
