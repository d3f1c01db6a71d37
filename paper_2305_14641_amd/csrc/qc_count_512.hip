// Counting-search instantiations of 512 threads (batches of 32 sources).
#include "qc_count.h"

namespace qc {

hipError_t launch_count_512(int nq, const GraphDev *graphs, const BfsJob *jobs, int n_jobs, hipStream_t stream)
{
    const dim3 grid(n_jobs), block(512);
    switch (nq) {
    case 5: hipLaunchKernelGGL((k_count<5, 512, 1, 0, 0>), grid, block, 0, stream, graphs, jobs); break;
    case 6: hipLaunchKernelGGL((k_count<6, 512, 1, 0, 0>), grid, block, 0, stream, graphs, jobs); break;
    case 7: hipLaunchKernelGGL((k_count<7, 512, 1, 0, 0>), grid, block, 0, stream, graphs, jobs); break;
    case 8: hipLaunchKernelGGL((k_count<8, 512, 1, 0, 0>), grid, block, 0, stream, graphs, jobs); break;
    case 9: hipLaunchKernelGGL((k_count<9, 512, 1, 0, 0>), grid, block, 0, stream, graphs, jobs); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace qc
