// dmm_pipe.hip - one (lanes per chain, labels per lane) tile of the pipelined chain sweeps,
// built once per tile with -DDM_PIPE_G=<lanes> -DDM_PIPE_L=<labels per lane>.
#if !defined(DM_PIPE_G) || !defined(DM_PIPE_L)
#error "DM_PIPE_G and DM_PIPE_L must be defined"
#endif

#include "dmm_pipe.h"

namespace dm {
template hipError_t launch_pipe<DM_PIPE_G, DM_PIPE_L>(const SweepArgs&, dm_dtype, hipStream_t);
}  // namespace dm
