#include "lif_step1.h"

namespace lif {
void launch_step1_f16_gate(const StepArgs& a, int grid, hipStream_t s) { launch_step1_as<_Float16, false, true>(a, grid, s); }
}  // namespace lif
