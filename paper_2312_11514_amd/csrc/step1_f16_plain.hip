#include "lif_step1.h"

namespace lif {
void launch_step1_f16_plain(const StepArgs& a, int grid, hipStream_t s) { launch_step1_as<_Float16, false, false>(a, grid, s); }
}  // namespace lif
