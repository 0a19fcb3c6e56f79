// Explicit instantiation: run-family SpMM kernels on f32 rows.
#include "run.h"

namespace spc3d {

template void launch_run<float, 4, false>(SPC3D_RUN_LAUNCH_ARGS);

}  // namespace spc3d
