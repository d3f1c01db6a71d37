// Shortest paths under real edge weights (Section 3.1: a path's length is the
// sum of its edges' weights), a few sources per workgroup, and the conversion
// of a dense FP64 potential into the resident layout the descent reads.
//
// A path's length is summed in binary32 from the source outward, each partial
// sum rounded to nearest, and d(s, v) is the least such sum over all paths.
// The workgroup keeps its S sources' tentative lengths side by side in LDS
// (the bits of a non-negative float order like the float, so an unsigned min
// is a float min) and works in rounds of two kinds:
//
//   push   while few nodes dropped in the previous round: they stand in a
//          queue, 8 lanes per node (32 while that leaves none waiting) offer
//          d(v) + w along its out-edges, and a drop (LDS min) puts the head into the next queue
//          (a bit per node keeps it from being there twice; it is cleared
//          before the node's length is read);
//   sweep  while many did: every node takes the least d(u) + w over its
//          in-edges, in place, and a bit per node says whether that dropped.
//          The in-edges come as rows of 64 lanes (two neighbours a lane),
//          each wavefront's in one stream, so the loads are coalesced and
//          run a block ahead, a gather fetches all S sources' lengths at
//          once, and no min is atomic but those of nodes whose list is cut
//          into parts.
//
// The search ends after a round in which nothing dropped. The least sum is
// what any such order reaches: a round only ever produces the sum of an actual
// path, and once nothing drops, every node on a least path holds at most that
// path's partial sum (rounding is monotone), so the order inside a round and
// the kind of the rounds do not change the result.
//
// Measured (19,717 nodes, 88,726 entries, all sources): 14.2 -> 3.2 ms against
// one source per workgroup, every active node's edges walked by its own
// thread (184 us a source on its CU: the uncoalesced 8-byte edge loads, one
// line each, two serial loads per round, and atomics for every relaxation).
// Now 75 us for two sources: 5-6 sweeps of 10 us, 5-7 pushes of 2.5 us, 4 us
// of output. A sweep runs the LDS gathers (half of their cycles bank
// conflicts) and the VALU at 40 % each, with the rows at 58 GB/s per CU from
// L2. Counting the sweep's drops as it goes instead of from the marks: 88 ->
// 77 us; 32 lanes per node in the small pushes: 3 -> 2.5 us.
#include <hip/hip_runtime.h>

#include "qc_internal.h"

namespace qc {

namespace {

constexpr uint32_t kInfBits = 0x7F800000u;   // +infinity: unreached
constexpr int kPushChunk = 2;                // edges a lane of a push has in flight

// Two in-edges: the tails' slots and the two weights.
struct Pair {
    uint32_t x, y, z;
};

template <int S> struct Lengths {
    uint32_t x[S];
};

// S lengths of a node with one LDS read.
template <int S>
__device__ __forceinline__ Lengths<S> lengths(const uint32_t *d, int v)
{
    typedef uint32_t V __attribute__((ext_vector_type(S == 1 ? 2 : S)));
    Lengths<S> r;
    if constexpr (S == 1) {
        r.x[0] = d[v];
    } else {
        const V y = *(const V *)(d + S * v);
#pragma unroll
        for (int k = 0; k < S; ++k) r.x[k] = y[k];
    }
    return r;
}

template <int S>
__device__ __forceinline__ void set_lengths(uint32_t *d, int v, const Lengths<S> &x)
{
    if constexpr (S == 1) {
        d[v] = x.x[0];
    } else {
        typedef uint32_t V __attribute__((ext_vector_type(S)));
        V y;
#pragma unroll
        for (int k = 0; k < S; ++k) y[k] = x.x[k];
        *(V *)(d + S * v) = y;
    }
}

__device__ __forceinline__ uint32_t longer(uint32_t d, uint32_t w)
{
    return __float_as_uint(__uint_as_float(d) + __uint_as_float(w));
}

template <int S, int T, int MAXN, int CAP>
__global__ __launch_bounds__(T) void k_sssp(SsspDev t, float *__restrict__ dist, int64_t ld, int src0, int src1)
{
    static_assert(MAXN % 64 == 0 && MAXN <= 65472, "whole rows, 16-bit slots");
    constexpr int kWords = MAXN / 32;
    __shared__ __attribute__((aligned(16))) uint32_t d[(MAXN + 1) * S];
    __shared__ __attribute__((aligned(8))) uint32_t mark[kWords];
    __shared__ uint16_t queue[2][CAP];
    __shared__ int dropped[3], filled;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = t.n, n_slots = (n + 63) & ~63, nw = n_slots / 32;
    const int s0 = src0 + (int)blockIdx.x * S;
    // (slots past the last node, and the one that pads lists, stay unreached)
    for (int i = tid; i < (n_slots + 1) * S; i += T) d[i] = kInfBits;
    for (int i = tid; i < nw; i += T) mark[i] = 0u;
    if (tid < 3) dropped[tid] = tid == 0 ? min(S, src1 - s0) : 0;
    __syncthreads();
    if (tid < S && s0 + tid < src1) {
        const int v = t.slot[s0 + tid];
        d[v * S + tid] = 0u;
        queue[0][tid] = (uint16_t)v;
        __hip_atomic_fetch_or(&mark[v >> 5], 1u << (v & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __syncthreads();
    // (block ranges and codes through the scalar cache: the host wrote them
    // before the launch)
    typedef const __attribute__((address_space(4))) int32_t *Ints;
    typedef const __attribute__((address_space(4))) uint64_t *Codes;
    const int first_block = ((Ints)t.wave_block)[wave], n_blocks = ((Ints)t.wave_block)[wave + 1] - first_block;
    const Pair *const my_rows = (const Pair *)t.rows + (size_t)first_block * (kSsspBlockRows * 64) + lane;
    const Codes codes = (Codes)t.codes + first_block;

    for (int round = 0;; ++round) {
        const int now = dropped[round % 3];
        int *const next = &dropped[(round + 1) % 3];
        if (now == 0) break;
        if (now <= CAP) {
            if (tid == 0) dropped[(round + 2) % 3] = 0;
            const uint16_t *const q = queue[round & 1];
            uint16_t *const nq = queue[(round + 1) & 1];
            const int lg = now <= T / 32 ? 5 : 3, lanes = 1 << lg, l = tid & (lanes - 1);
            for (int j = tid >> lg; j < now; j += T >> lg) {
                const int u = q[j];
                const int e0 = t.row_ptr[u], e1 = t.row_ptr[u + 1];
                if (l == 0)
                    __hip_atomic_fetch_and(&mark[u >> 5], ~(1u << (u & 31)), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                asm volatile("" ::: "memory");
                const Lengths<S> du = lengths<S>(d, u);
                for (int e = e0 + l; e < e1; e += kPushChunk * lanes) {
                    uint2 x[kPushChunk];
#pragma unroll
                    for (int k = 0; k < kPushChunk; ++k) x[k] = t.edges[min(e + k * lanes, e1 - 1)];
#pragma unroll
                    for (int k = 0; k < kPushChunk; ++k) {
                        const int v = (int)x[k].x;
                        const Lengths<S> dv = lengths<S>(d, v);
                        bool drops = false;
#pragma unroll
                        for (int s = 0; s < S; ++s) {
                            const uint32_t c = longer(du.x[s], x[k].y);
                            if (c < dv.x[s])
                                drops |= c < __hip_atomic_fetch_min(&d[v * S + s], c, __ATOMIC_RELAXED,
                                                                    __HIP_MEMORY_SCOPE_WORKGROUP);
                        }
                        if (drops) {
                            const uint32_t bit = 1u << (v & 31);
                            if (!(__hip_atomic_fetch_or(&mark[v >> 5], bit, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_WORKGROUP) & bit)) {
                                const int at =
                                    __hip_atomic_fetch_add(next, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                                if (at < CAP) nq[at] = (uint16_t)v;
                            }
                        }
                    }
                }
            }
            __syncthreads();
            continue;
        }
        // A sweep. The marks that it does not write whole are those of the
        // nodes whose lists are cut.
        for (int i = tid; i < t.n_cut / 32; i += T) mark[i] = 0u;
        if (tid == 0) {
            dropped[(round + 2) % 3] = 0;
            filled = 0;
        }
        __syncthreads();
        if (n_blocks > 0) {
            constexpr int R = kSsspBlockRows;
            int n_drops = 0;
            Lengths<S> best;
#pragma unroll
            for (int s = 0; s < S; ++s) best.x[s] = kInfBits;
            auto load = [&](Pair (&x)[R], int i) {
                const Pair *const p = my_rows + (size_t)min(i, n_blocks - 1) * (R * 64);
#pragma unroll
                for (int r = 0; r < R; ++r) x[r] = p[64 * r];
            };
            auto block = [&](const Pair (&x)[R], uint64_t code) {
                Lengths<S> lo[R], hi[R];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    lo[r] = lengths<S>(d, (int)(x[r].x & 0xFFFFu));
                    hi[r] = lengths<S>(d, (int)(x[r].x >> 16));
                }
#pragma unroll
                for (int r = 0; r < R; ++r) {
#pragma unroll
                    for (int s = 0; s < S; ++s)
                        best.x[s] = min(best.x[s], min(longer(lo[r].x[s], x[r].y), longer(hi[r].x[s], x[r].z)));
                    const uint32_t c = (uint32_t)(code >> (16 * r)) & 0xFFFFu;
                    if (!c) continue;
                    bool drops = false;
                    if (c >> 14 == kSsspEnd) {
                        // the last row of 64 nodes' lists
                        const int v = (int)(c & 0x3FFFu) * 64 + lane;
                        const Lengths<S> own = lengths<S>(d, v);
#pragma unroll
                        for (int s = 0; s < S; ++s) {
                            drops |= best.x[s] < own.x[s];
                            best.x[s] = min(best.x[s], own.x[s]);
                        }
                        set_lengths<S>(d, v, best);
                        const uint64_t all = __ballot(drops);
                        if (lane == 0) *(uint64_t *)&mark[v >> 5] = all;
                        n_drops += __popcll(all);
                    } else {
                        // the row that names the nodes whose parts these were
                        const int v = (int)(x[r].x & 0xFFFFu);
#pragma unroll
                        for (int s = 0; s < S; ++s)
                            if (best.x[s] < lo[r].x[s])
                                drops |= best.x[s] < __hip_atomic_fetch_min(&d[v * S + s], best.x[s], __ATOMIC_RELAXED,
                                                                            __HIP_MEMORY_SCOPE_WORKGROUP);
                        if (drops) {
                            const uint32_t bit = 1u << (v & 31);
                            drops = !(__hip_atomic_fetch_or(&mark[v >> 5], bit, __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_WORKGROUP) & bit);
                        }
                        n_drops += __popcll(__ballot(drops));
                    }
#pragma unroll
                    for (int s = 0; s < S; ++s) best.x[s] = kInfBits;
                }
            };
            // two blocks in flight behind the one that is looked up (past the
            // end: the last one again, whose codes the loop does not reach)
            Pair a[R], b[R], c[R];
            load(a, 0);
            load(b, 1);
            uint64_t code = codes[0];
            for (int i = 0;;) {
                uint64_t next_code = codes[i + 1];
                load(c, i + 2);
                block(a, code);
                if (++i == n_blocks) break;
                code = codes[i + 1];
                load(a, i + 2);
                block(b, next_code);
                if (++i == n_blocks) break;
                next_code = codes[i + 1];
                load(b, i + 2);
                block(c, code);
                if (++i == n_blocks) break;
                code = next_code;
            }
            if (lane == 0 && n_drops)
                __hip_atomic_fetch_add(next, n_drops, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        __syncthreads();
        const int count = *next;
        if (count > 0 && count <= CAP) {
            uint16_t *const nq = queue[(round + 1) & 1];
            for (int i = tid; i < nw; i += T) {
                uint32_t bits = mark[i];
                if (!bits) continue;
                int at = __hip_atomic_fetch_add(&filled, __popc(bits), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                for (; bits; bits &= bits - 1u) nq[at++] = (uint16_t)(32 * i + __builtin_ctz(bits));
            }
            __syncthreads();
        }
    }
    for (int v = tid; v < n; v += T) {
        const Lengths<S> x = lengths<S>(d, t.slot[v]);
#pragma unroll
        for (int s = 0; s < S; ++s)
            if (s0 + s < src1) dist[(int64_t)(s0 + s) * ld + v] = __uint_as_float(x.x[s]);
    }
}

// v32[v_index(n, s, i)] = (float)v64[s * n + i]: the descent's FP32 copy of a
// potential, sigma groups of kVGroup interleaved by node.
__global__ __launch_bounds__(256) void k_v_resident(const double *__restrict__ v64, int n, int n_sigmas,
                                                    float *__restrict__ v32)
{
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= (int64_t)n * n_sigmas) return;
    const int s = (int)(k / n), i = (int)(k % n);
    v32[v_index(n, s, i)] = (float)v64[k];
}

template <int S, int T, int MAXN, int CAP>
hipError_t launch_sssp_t(const SsspDev &t, float *dist, int64_t ld, int src0, int count, hipStream_t stream)
{
    hipLaunchKernelGGL((k_sssp<S, T, MAXN, CAP>), dim3((count + S - 1) / S), dim3(T), 0, stream, t, dist, ld, src0,
                       src0 + count);
    return hipGetLastError();
}

}  // namespace

// Sources per workgroup: as many as their lengths fit the LDS that a workgroup
// has (the row loads and the gathers' instructions serve them all): 4 up to
// 9,920 nodes, 2 up to 19,840 (4,500 nodes 1,291 -> 716 us, 9,000: 4.0 -> 1.7
// ms, 19,717: 17.1 -> 5.4 ms a call), one beyond (30,000 nodes: 43.9 -> 14.9
// ms). Small graphs take fewer so that there are workgroups for every CU (500
// nodes 122 -> 119 us, 2,000: 424 -> 311), and workgroups small enough that
// several share a CU.
int sssp_waves(int n) { return n <= 2432 ? 4 : n <= 4928 ? 8 : 16; }

hipError_t launch_sssp(const SsspDev &t, float *dist, int64_t ld, int src0, int count, hipStream_t stream)
{
    const int n = t.n;
    if (n < 1 || n > kSsspMaxNodes || src0 < 0 || count < 0 || src0 + count > n || ld < n)
        return hipErrorInvalidValue;
    if (count == 0) return hipSuccess;
    if (n <= 1024) return launch_sssp_t<1, 256, 1024, 128>(t, dist, ld, src0, count, stream);
    if (n <= 2432) return launch_sssp_t<2, 256, 2432, 128>(t, dist, ld, src0, count, stream);
    if (n <= 4928) return launch_sssp_t<4, 512, 4928, 512>(t, dist, ld, src0, count, stream);
    if (n <= 9920) return launch_sssp_t<4, 1024, 9920, 512>(t, dist, ld, src0, count, stream);
    if (n <= 19840) return launch_sssp_t<2, 1024, 19840, 512>(t, dist, ld, src0, count, stream);
    return launch_sssp_t<1, 1024, 32768, 1024>(t, dist, ld, src0, count, stream);
}

hipError_t launch_v_resident(const double *v64, int n, int n_sigmas, float *v32, hipStream_t stream)
{
    const int64_t total = (int64_t)n * n_sigmas;
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_v_resident, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, v64, n,
                       n_sigmas, v32);
    return hipGetLastError();
}

}  // namespace qc
