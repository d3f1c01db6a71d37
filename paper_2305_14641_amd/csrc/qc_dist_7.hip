// Instantiations of the counting search that also write the distance rows,
// 7 bit-planes of the level (levels up to 126). Up to 4 quads: batches of 32
// sources; above: 16.
#include "qc_count.h"

namespace qc {

hipError_t launch_dist_7(int nq, int nqn, const GraphDev *graphs, const BfsJob *jobs, int n_jobs,
                         hipStream_t stream)
{
    const dim3 grid(n_jobs), block(1024);
    switch (nq * 100 + nqn) {
    case 101: hipLaunchKernelGGL((k_count<1, 1024, 1, 7, 1>), grid, block, 0, stream, graphs, jobs); break;
    case 102: hipLaunchKernelGGL((k_count<1, 1024, 1, 7, 2>), grid, block, 0, stream, graphs, jobs); break;
    case 202: hipLaunchKernelGGL((k_count<2, 1024, 1, 7, 2>), grid, block, 0, stream, graphs, jobs); break;
    case 203: hipLaunchKernelGGL((k_count<2, 1024, 1, 7, 3>), grid, block, 0, stream, graphs, jobs); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace qc
