// Explicit instantiation: run-family SpMM kernels on bf16 rows.
#include "run.h"

namespace spc3d {

template void launch_run<bf16_t, 8, false>(SPC3D_RUN_LAUNCH_ARGS);

}  // namespace spc3d
