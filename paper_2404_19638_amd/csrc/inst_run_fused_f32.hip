// Explicit instantiation: run-family fused kernels on f32 rows.
#include "run.h"

namespace spc3d {

template void launch_run<float, 4, true>(SPC3D_RUN_LAUNCH_ARGS);

}  // namespace spc3d
