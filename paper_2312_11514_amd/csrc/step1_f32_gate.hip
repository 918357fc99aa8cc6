#include "lif_step1.h"

namespace lif {
void launch_step1_f32_gate(const StepArgs& a, int grid, hipStream_t s) { launch_step1_as<float, false, true>(a, grid, s); }
}  // namespace lif
