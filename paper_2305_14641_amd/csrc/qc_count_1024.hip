// Counting-search instantiations of 1,024 threads (batches of 32 and 16
// sources), and the histograms of the nodes the search leaves out.
#include "qc_count.h"

namespace qc {

static hipError_t launch_count_1024(int nq, const GraphDev *graphs, const BfsJob *jobs, int n_jobs,
                                    hipStream_t stream)
{
    const dim3 grid(n_jobs), block(1024);
    switch (nq) {
    case 1: hipLaunchKernelGGL((k_count<1, 1024, 1, 0, 0>), grid, block, 0, stream, graphs, jobs); break;
    case 2: hipLaunchKernelGGL((k_count<2, 1024, 1, 0, 0>), grid, block, 0, stream, graphs, jobs); break;
    case 5: hipLaunchKernelGGL((k_count<5, 1024, 1, 0, 0>), grid, block, 0, stream, graphs, jobs); break;
    case 6: hipLaunchKernelGGL((k_count<6, 1024, 1, 0, 0>), grid, block, 0, stream, graphs, jobs); break;
    case 7: hipLaunchKernelGGL((k_count<7, 1024, 1, 0, 0>), grid, block, 0, stream, graphs, jobs); break;
    case 8: hipLaunchKernelGGL((k_count<8, 1024, 1, 0, 0>), grid, block, 0, stream, graphs, jobs); break;
    case 9: hipLaunchKernelGGL((k_count<9, 1024, 1, 0, 0>), grid, block, 0, stream, graphs, jobs); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

static hipError_t launch_count_x2(int nq, const GraphDev *graphs, const BfsJob *jobs, int n_jobs,
                                  hipStream_t stream)
{
    const dim3 grid(n_jobs), block(1024);
    switch (nq) {
    case 10: hipLaunchKernelGGL((k_count<10, 1024, 2, 0, 0>), grid, block, 0, stream, graphs, jobs); break;
    case 11: hipLaunchKernelGGL((k_count<11, 1024, 2, 0, 0>), grid, block, 0, stream, graphs, jobs); break;
    case 12: hipLaunchKernelGGL((k_count<12, 1024, 2, 0, 0>), grid, block, 0, stream, graphs, jobs); break;
    case 14: hipLaunchKernelGGL((k_count<14, 1024, 2, 0, 0>), grid, block, 0, stream, graphs, jobs); break;
    case 16: hipLaunchKernelGGL((k_count<16, 1024, 2, 0, 0>), grid, block, 0, stream, graphs, jobs); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_count(int nq, int threads, int per, const GraphDev *graphs, const BfsJob *jobs,
                        int n_jobs, hipStream_t stream)
{
    if (n_jobs <= 0) return hipSuccess;
    if (threads == 512 && per == 1) return launch_count_512(nq, graphs, jobs, n_jobs, stream);
    if (threads == 1024 && per == 1) return launch_count_1024(nq, graphs, jobs, n_jobs, stream);
    if (threads == 1024 && per == 2) return launch_count_x2(nq, graphs, jobs, n_jobs, stream);
    return hipErrorInvalidValue;
}

// Histogram rows of the nodes the search leaves out (32 per workgroup, one
// thread per bin; a few rows of 4 K bytes each, bound by latency):
//   a leaf v with neighbour u: d(v, x) = 1 + d(u, x) for every x != v, so
//     h[v][0] = 1, h[v][k] = h[u][k - 1], less v itself at k = 2 (v is at
//     distance 1 from u);
//   both ends of an isolated edge: one node at distance 0, one at 1;
//   a node without edges: itself.
// The last bin of a neighbour's row has no place in the leaf's; the largest
// distance (status[0]) still covers it, so a caller sees rows too short.
template <int K>
__device__ __forceinline__ void hist_rest(const GraphDev &G, int r0)
{
    const RowsDev &R = G.rows;
    int far = 0;
    for (int i = (int)threadIdx.x; i < 32 * K; i += (int)blockDim.x) {
        const int r = r0 + i / K, k = i % K;
        if (r >= R.n_rest) break;
        const uint32_t e = R.rest[r];
        const int v = (int)(e & 0xFFFFu), u = (int)(e >> 16);
        int h;
        if (r < R.n_rest_leaf) {
            const int32_t *const hu = G.hist + (int64_t)u * K;
            h = (k == 0) ? 1 : hu[k - 1] - (k == 2 ? 1 : 0);
            if (k == K - 1 && hu[k]) far = K;
        } else {
            h = (k == 0 || (k == 1 && r < R.n_rest_leaf + R.n_rest_pair)) ? 1 : 0;
        }
        G.hist[(int64_t)v * K + k] = h;
        if (h) far = max(far, k);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) far = max(far, __shfl_xor(far, off));
    if ((threadIdx.x & 63) == 0 && far > 0) {
        atomicMax(&G.status[0], far);
        if (far > kMaxDist) atomicOr(&G.status[1], 1);
    }
}

template <int K>
__global__ void k_hist_rest(const GraphDev *__restrict__ graphs, const NodeJob *__restrict__ jobs)
{
    const NodeJob job = jobs[blockIdx.x];
    hist_rest<K>(graphs[job.g], job.i0);
}

hipError_t launch_hist_rest(int K, const GraphDev *graphs, const NodeJob *jobs, int n_jobs, int waves,
                            hipStream_t stream)
{
    if (n_jobs <= 0) return hipSuccess;
    const dim3 grid(n_jobs), block(64 * waves);
    switch (K) {
    case 32: hipLaunchKernelGGL(k_hist_rest<32>, grid, block, 0, stream, graphs, jobs); break;
    case 64: hipLaunchKernelGGL(k_hist_rest<64>, grid, block, 0, stream, graphs, jobs); break;
    case 128: hipLaunchKernelGGL(k_hist_rest<128>, grid, block, 0, stream, graphs, jobs); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Distance rows of the nodes the search leaves out, one workgroup each
// (streamed: n bytes read and n written per leaf): a leaf's row is its
// neighbour's plus one, unreached bytes (all ones) as they are, itself 0.
// (The first workgroups also make the histogram rows, 32 each.)
template <int K>
__global__ __launch_bounds__(256) void k_dist_rest(const GraphDev *__restrict__ graphs)
{
    const GraphDev &G = graphs[0];
    const RowsDev &R = G.rows;
    const int r = (int)blockIdx.x;
    if (r * 32 < R.n_rest) hist_rest<K>(G, r * 32);
    const uint32_t e = R.rest[r];
    const int v = (int)(e & 0xFFFFu), u = (int)(e >> 16);
    const bool leaf = r < R.n_rest_leaf, pair = !leaf && r < R.n_rest_leaf + R.n_rest_pair;
    int8_t *const dst = G.dist + (int64_t)v * G.ld;
    const int8_t *const from = G.dist + (int64_t)u * G.ld;
    const int n = G.n;
    // stores aligned to 16 bytes, the neighbour's bytes at whatever alignment
    const int head = min(n, (int)((16 - ((uintptr_t)dst & 15)) & 15));
    const int chunks = (n - head) / 16;
    auto one = [&](int x) -> int8_t {
        if (x == v) return 0;
        if (pair) return x == u ? 1 : -1;
        const int8_t d = leaf ? from[x] : (int8_t)-1;
        return d < 0 ? d : (int8_t)(d + 1);
    };
    typedef uint32_t __attribute__((aligned(1))) u32_any;
    for (int c = (int)threadIdx.x; c < chunks; c += 256) {
        const int x0 = head + c * 16;
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t x = leaf ? *(const u32_any *)(from + x0 + 4 * i) : ~0u;
            x += (~x >> 7) & 0x01010101u;
            const int a = v - (x0 + 4 * i), b = u - (x0 + 4 * i);
            if (pair && b >= 0 && b < 4) x = (x & ~(0xFFu << (8 * b))) | 1u << (8 * b);
            if (a >= 0 && a < 4) x &= ~(0xFFu << (8 * a));
            w[i] = x;
        }
        *(uint4 *)(dst + x0) = make_uint4(w[0], w[1], w[2], w[3]);
    }
    for (int x = (int)threadIdx.x; x < n; x += 256)
        if (x < head || x >= head + chunks * 16) dst[x] = one(x);
}

hipError_t launch_dist_rest(int K, const GraphDev *graph, int n_rest, hipStream_t stream)
{
    if (n_rest <= 0) return hipSuccess;
    const dim3 grid(n_rest), block(256);
    switch (K) {
    case 32: hipLaunchKernelGGL(k_dist_rest<32>, grid, block, 0, stream, graph); break;
    case 64: hipLaunchKernelGGL(k_dist_rest<64>, grid, block, 0, stream, graph); break;
    case 128: hipLaunchKernelGGL(k_dist_rest<128>, grid, block, 0, stream, graph); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace qc
