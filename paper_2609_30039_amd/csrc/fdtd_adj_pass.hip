// fdtd_adj_pass.hip -- the single-pass adjoint step (fdtd_adj_pass.h) in FP32.
#include "fdtd_adj_pass.h"

template void fdtd::launch_adj_pass<float>(const fdtd::LaunchCfg&, const void*, int, int, hipStream_t);
template void fdtd::launch_adj_grad<float>(const fdtd::LaunchCfg&, const void*, int, int, int, hipStream_t);
