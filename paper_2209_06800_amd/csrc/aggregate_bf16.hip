// Aggregation kernels for bf16 tables (16 bytes per lane; element by element below that width), fp32 accumulation.
#include "aggregate_kernels.h"

namespace mgg {

hipError_t launch_aggregate_bf16(const AggArgs &a, bool gcn, int vec, dim3 grid, int wpb, hipStream_t stream, int lpr, int ch, bool lds, bool team)
{
    if (vec == 8) return dispatch_shape<true, 8>(a, gcn, grid, wpb, stream, lpr, ch, lds, team);
    return launch_cfg<Cfg<true, 1, 8, 1>>(a, gcn, grid, wpb, stream, lds, team);      // rows shorter than a vector
}

}  // namespace mgg
