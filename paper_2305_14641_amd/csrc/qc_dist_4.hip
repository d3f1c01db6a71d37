// Instantiations of the counting search that also write the distance rows,
// 4 bit-planes of the level (levels up to 14). Up to 4 quads: batches of 32
// sources; above: 16.
#include "qc_count.h"

namespace qc {

hipError_t launch_dist_4(int nq, int nqn, const GraphDev *graphs, const BfsJob *jobs, int n_jobs,
                         hipStream_t stream)
{
    const dim3 grid(n_jobs), block(1024);
    switch (nq * 100 + nqn) {
    case 101: hipLaunchKernelGGL((k_count<1, 1024, 1, 4, 1>), grid, block, 0, stream, graphs, jobs); break;
    case 102: hipLaunchKernelGGL((k_count<1, 1024, 1, 4, 2>), grid, block, 0, stream, graphs, jobs); break;
    case 202: hipLaunchKernelGGL((k_count<2, 1024, 1, 4, 2>), grid, block, 0, stream, graphs, jobs); break;
    case 203: hipLaunchKernelGGL((k_count<2, 1024, 1, 4, 3>), grid, block, 0, stream, graphs, jobs); break;
    case 303: hipLaunchKernelGGL((k_count<3, 1024, 1, 4, 3>), grid, block, 0, stream, graphs, jobs); break;
    case 304: hipLaunchKernelGGL((k_count<3, 1024, 1, 4, 4>), grid, block, 0, stream, graphs, jobs); break;
    case 404: hipLaunchKernelGGL((k_count<4, 1024, 1, 4, 4>), grid, block, 0, stream, graphs, jobs); break;
    case 405: hipLaunchKernelGGL((k_count<4, 1024, 1, 4, 5>), grid, block, 0, stream, graphs, jobs); break;
    case 505: hipLaunchKernelGGL((k_count<5, 1024, 2, 4, 5>), grid, block, 0, stream, graphs, jobs); break;
    case 506: hipLaunchKernelGGL((k_count<5, 1024, 2, 4, 6>), grid, block, 0, stream, graphs, jobs); break;
    case 606: hipLaunchKernelGGL((k_count<6, 1024, 2, 4, 6>), grid, block, 0, stream, graphs, jobs); break;
    case 607: hipLaunchKernelGGL((k_count<6, 1024, 2, 4, 7>), grid, block, 0, stream, graphs, jobs); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace qc
