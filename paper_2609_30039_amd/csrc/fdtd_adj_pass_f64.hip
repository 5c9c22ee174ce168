// fdtd_adj_pass_f64.hip -- the single-pass adjoint step (fdtd_adj_pass.h) in FP64.
#include "fdtd_adj_pass.h"

template void fdtd::launch_adj_pass<double>(const fdtd::LaunchCfg&, const void*, int, int, hipStream_t);
template void fdtd::launch_adj_grad<double>(const fdtd::LaunchCfg&, const void*, int, int, int, hipStream_t);
