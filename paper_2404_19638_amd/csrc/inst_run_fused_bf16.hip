// Explicit instantiation: run-family fused kernels on bf16 rows.
#include "run.h"

namespace spc3d {

template void launch_run<bf16_t, 8, true>(SPC3D_RUN_LAUNCH_ARGS);

}  // namespace spc3d
