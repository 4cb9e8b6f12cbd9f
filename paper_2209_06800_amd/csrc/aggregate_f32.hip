// Aggregation kernels for fp32 tables (16 bytes per lane; element by element below that width).
#include "aggregate_kernels.h"

namespace mgg {

hipError_t launch_aggregate_f32(const AggArgs &a, bool gcn, int vec, dim3 grid, int wpb, hipStream_t stream, int lpr, int ch, bool lds, bool team)
{
    if (vec == 4) return dispatch_shape<false, 4>(a, gcn, grid, wpb, stream, lpr, ch, lds, team);
    return launch_cfg<Cfg<false, 1, 4, 1>>(a, gcn, grid, wpb, stream, lds, team);      // rows shorter than a vector
}

}  // namespace mgg
