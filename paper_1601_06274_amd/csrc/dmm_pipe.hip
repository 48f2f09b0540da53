// dmm_pipe.hip - one (lanes per chain, labels per lane) tile of the pipelined chain sweeps,
// built once per tile with -DDM_PIPE_G=<lanes> -DDM_PIPE_L=<labels per lane> and
// -DDM_PIPE_SCAN=<0: direct window messages, single and batched, 1: scan messages>.
#if !defined(DM_PIPE_G) || !defined(DM_PIPE_L) || !defined(DM_PIPE_SCAN)
#error "DM_PIPE_G, DM_PIPE_L and DM_PIPE_SCAN must be defined"
#endif

#include "dmm_pipe.h"

namespace dm {
template hipError_t launch_pipe<DM_PIPE_G, DM_PIPE_L, DM_PIPE_SCAN != 0>(const SweepArgs&, dm_dtype, hipStream_t);
#if !DM_PIPE_SCAN
template hipError_t launch_batched_pipe<DM_PIPE_G, DM_PIPE_L>(const BatchLaunch&, bool, dm_dtype, hipStream_t);
#endif
}  // namespace dm
