// Graph Gradient Descent and its centres (Algorithms 2 and 3) of one graph and
// one sigma in one workgroup: potentials, parents and pointer jumping in LDS.
#include <float.h>

#include "qc_internal.h"

namespace qc {

namespace {

// Near ties of one (graph, sigma) that LDS keeps, of either kind (the others
// go to the parents' table, which this path has no other use for).
constexpr int kTieQueue = 1024;

// On-demand canonical FP64 V (potentials without a resident FP64 table): the
// products and sums of the potential kernel, in its order.
__device__ __noinline__ double canonical_node_v(const GraphDev &G, int s, int node)
{
#pragma clang fp contract(off)
    const int32_t *__restrict__ h = G.hist + (int64_t)node * G.K;
    const double *__restrict__ w = G.w64 + (int64_t)s * G.K;
    double s2 = 0.0, s1 = 0.0;
    for (int k = 0; k <= G.dmax; ++k) {
        const double hk = (double)h[k];
        s2 = s2 + hk * w[k];
        s1 = s1 + ((double)(k * k) * hk) * w[k];
    }
    return G.inv_a[s] * (s1 / s2);
}

__device__ __forceinline__ double node_v64(const GraphDev &G, int s, int node)
{
    return G.v64 ? G.v64[(int64_t)s * G.n + node] : canonical_node_v(G, s, node);
}

// The lowest and the second lowest V among neighbours, and whose the lowest
// is. Entries that pad a list name node n, whose V is FLT_MAX.
struct Low {
    float m1 = FLT_MAX, m2 = FLT_MAX;
    int j1 = -1;
    __device__ __forceinline__ void take(const float *V, int j)
    {
        const float v = V[j];
        const bool lower = v < m1;
        m2 = __builtin_amdgcn_fmed3f(m1, m2, v);
        m1 = lower ? v : m1;
        j1 = lower ? j : j1;
    }
    __device__ __forceinline__ void take2(const float *V, uint32_t word)
    {
        take(V, (int)(word & 0xFFFFu));
        take(V, (int)(word >> 16));
    }
};

// f(i) of every i = tid, tid + T, ... below n, U of them in flight: load(i)
// of all U, then store(i, value).
template <int U, int T, class Load, class Store>
__device__ __forceinline__ void strided(int n, int tid, Load &&load, Store &&store)
{
    using X = decltype(load(0));
    for (int i0 = tid; i0 < n; i0 += U * T) {
        X x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = load(min(i0 + u * T, n - 1));
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * T < n) store(i0 + u * T, x[u]);
    }
}

// A list of more than kLong neighbours, and a near tie among more than
// 2 * kChunk, is shared by kShare threads.
constexpr int kLong = 32, kShare = 16;
constexpr int kChunk = 4;   // words (pairs of neighbours) in flight per thread

// One workgroup per (graph, sigma): the sigma's FP32 V of every node and the
// parents (16-bit ids) in LDS. The descent through global memory
// (k_ggd_parent, k_jump) gathers V from L2, one cache line per neighbour, and
// waits for a serial chain of such gathers wherever a list is long or a near
// tie is re-decided; here a gather is an LDS read, a list longer than kLong is
// shared by kShare threads, near ties are set aside and re-decided together,
// and the parents never leave the chip. What bounds it: for one large graph
// the LDS gathers of its one CU (19,717 nodes: 5 us of loads, 20 the short
// lists, 10 the long ones, 7 the jumps), for many graphs the same on all CUs.
// Measured against the two kernels it replaces, which gathered a list in
// thread order whatever its length: 2,708 nodes and one sigma 17 -> 11 us,
// 19,717 nodes 65 -> 50 us; a batch of 64 graphs of 1,000-20,000 nodes and 32
// sigmas 0.74 -> 0.3 ms of its step. Tried: ties through a 2,048-entry queue
// and a scan for the rest (275 us where a small sigma ties one node in five),
// lists of 32-bit ids with a test per entry (28 us for the short lists).
template <int CAP>
__global__ __launch_bounds__(1024, CAP <= kDescendHalfNodes ? 8 : 4) void k_descend(
    int tie_mode, const GraphDev *__restrict__ graphs, const NodeJob *__restrict__ jobs, int sigma_base,
    int32_t *labels_base, int64_t labels_ld, bool store_count)
{
    constexpr int T = 1024, kWaves = T / 64, kGroups = T / kShare;
    constexpr uint16_t kUndecided = 0xFFFF;
    __shared__ float V[CAP + 1];
    static_assert(CAP % 4 == 0, "parents are read four at a time");
    __shared__ uint64_t par4[CAP / 4];
    uint16_t *const par = (uint16_t *)par4;
    __shared__ uint16_t queue[2][kTieQueue];
    __shared__ int queued[2], again[3];
    const NodeJob job = jobs[blockIdx.y];
    const GraphDev &G = graphs[job.g];
    const int n = G.n, tid = (int)threadIdx.x;
    const int s = sigma_base + (int)blockIdx.x;
    if (s >= G.n_labels || n > CAP) return;
    const int32_t *__restrict__ order = G.order, *__restrict__ sdeg = G.sell_deg, *__restrict__ soff = G.sell_off;
    const uint32_t *__restrict__ scol = G.sell_col;
    int32_t *const spill = G.parent + (int64_t)s * n;
    // The tables' lines into this XCD's L2 all at once, so that the scans'
    // dependent loads wait for it and not for memory (up to kTouch lines of
    // the lists per thread).
    uint32_t touched = 0;
    {
        constexpr int kLine = 32, kTouch = 6;   // words
        const int n_words = (int)(G.nnz / 2);   // (at least)
        if (tid * kLine < n) touched = sdeg[tid * kLine] ^ order[tid * kLine];
#pragma unroll
        for (int u = 0; u < kTouch; ++u) touched ^= scol[min((u * T + tid) * kLine, n_words)];
    }
    if (tid < 2) queued[tid] = 0;
    if (tid < 3) again[tid] = 0;
    if (tid == 0) V[n] = FLT_MAX;
    if (tid < (-n & 3)) par[n + tid] = (uint16_t)(n + tid);
    // (float)v64 is the resident FP32 V wherever the FP64 one is resident
    if (G.v64) {
        const double *__restrict__ v64 = G.v64 + (int64_t)s * n;
        strided<8, T>(n, tid, [&](int i) { return v64[i]; }, [&](int i, double v) { V[i] = (float)v; });
    } else {
        const float *__restrict__ v32 = G.v;
        strided<8, T>(n, tid, [&](int i) { return v32[v_index(n, s, i)]; }, [&](int i, float v) { V[i] = v; });
    }
    asm volatile("" ::"v"(touched));
    __syncthreads();
    // slot t's parent from its neighbours' lowest, or its place in a queue
    auto settle = [&](int t, int node, int deg, const Low &low) {
        const float vi = V[node];
        int parent = node;
        if (low.j1 >= 0) {
            const float hi = fmaxf(low.m1, vi), lo = fminf(low.m1, vi);
            bool tie = (hi - lo <= kTieTau * hi);
            // which neighbour is lowest matters only when the node moves
            if (low.m1 < vi && low.m2 - low.m1 <= kTieTau * low.m2) tie = true;
            if (tie) {
                parent = kUndecided;
                const int many = deg > 2 * kChunk;
                const int q =
                    __hip_atomic_fetch_add(&queued[many], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (q < kTieQueue) queue[many][q] = (uint16_t)t;
                else spill[many ? n - 1 - q : q] = t;
            } else if (low.m1 < vi) {
                parent = low.j1;
            }
        }
        par[node] = (uint16_t)parent;
    };
    {
        // Lists of at most kLong neighbours: a thread each, slices of 64
        // slots per wavefront, dealt to the wavefronts to and fro (a slice's
        // lists are about equally long, each window's longest first). The
        // next words of the slice, or the first ones of the wavefront's next
        // slice, are in flight while these are looked up.
        const int lane = tid % 64, wave = __builtin_amdgcn_readfirstlane(tid / 64), n_slices = (n + 63) / 64;
        auto slice = [&](int it) { return it * kWaves + ((it & 1) ? kWaves - 1 - wave : wave); };
        auto deg_of = [&](int w) { return 64 * w + lane < n ? sdeg[64 * w + lane] : 0; };
        auto node_of = [&](int w) { return order[min(64 * w + lane, n - 1)]; };
        auto base_of = [&](int w) { return scol + soff[min(w, n_slices - 1)] + lane; };
        // words of the longest list of the slice that one thread scans
        auto rows_of = [&](int deg) {
            const int longs = __popcll(__ballot(deg > kLong));
            return longs < 64 ? (__builtin_amdgcn_readlane(deg, longs) + 1) >> 1 : 0;
        };
        auto load = [&](uint32_t (&c)[kChunk], const uint32_t *base, int r, int rows) {
#pragma unroll
            for (int u = 0; u < kChunk; ++u) c[u] = base[64 * max(min(r + u, rows - 1), 0)];
        };
        int it = 0, w = slice(0), r = 0;
        uint32_t c[kChunk];
        int deg = deg_of(w), node = node_of(w), rows = rows_of(deg);
        const uint32_t *base = base_of(w);
        load(c, base, 0, rows);
        int w1 = slice(1), deg1 = deg_of(w1), node1 = node_of(w1);
        const uint32_t *base1 = base_of(w1);
        Low low;
        while (w < n_slices) {
            const bool last = r + kChunk >= rows;
            uint32_t c1[kChunk];
            int rows1 = 0;
            if (last) {
                rows1 = rows_of(deg1);
                load(c1, base1, 0, rows1);
            } else {
                load(c1, base, r + kChunk, rows);
            }
#pragma unroll
            for (int u = 0; u < kChunk; ++u)
                if (r + u < rows) low.take2(V, c[u]);
            if (last) {
                if (deg <= kLong && 64 * w + lane < n) settle(64 * w + lane, node, deg, low);
                low = Low();
                w = w1;
                deg = deg1;
                node = node1;
                base = base1;
                rows = rows1;
                r = 0;
                w1 = slice(++it + 1);
                deg1 = deg_of(w1);
                node1 = node_of(w1);
                base1 = base_of(w1);
            } else {
                r += kChunk;
            }
#pragma unroll
            for (int u = 0; u < kChunk; ++u) c[u] = c1[u];
        }
    }
    const int group = tid / kShare, gl = tid % kShare;
    // Longer lists (each window's first slots), the next slot's head in flight.
    for (int w0 = 0; w0 < n; w0 += kOrderWindow) {
        const int end = min(n, w0 + kOrderWindow);
        int t = min(w0 + group, n - 1), deg = sdeg[t], off = soff[t >> 6], node = order[t];
        for (t = w0 + group; t < end && deg > kLong; t += kGroups) {
            const int t1 = min(t + kGroups, n - 1), deg1 = sdeg[t1], off1 = soff[t1 >> 6], node1 = order[t1];
            const uint32_t *const base = scol + off + (t & 63);
            const int rows = (deg + 1) >> 1;
            Low low;
            for (int r = gl; r < rows; r += kChunk * kShare) {
                uint32_t c[kChunk];
#pragma unroll
                for (int u = 0; u < kChunk; ++u) c[u] = base[64 * min(r + u * kShare, rows - 1)];
#pragma unroll
                for (int u = 0; u < kChunk; ++u)
                    if (r + u * kShare < rows) low.take2(V, c[u]);
            }
            // (which of equal lowest ones is named does not matter: a node
            // that could move to either is re-decided)
#pragma unroll
            for (int d = 1; d < kShare; d *= 2) {
                const float m1 = __shfl_xor(low.m1, d), m2 = __shfl_xor(low.m2, d);
                const int j1 = __shfl_xor(low.j1, d);
                low.m2 = fminf(fmaxf(low.m1, m1), fminf(low.m2, m2));
                if (m1 < low.m1) {
                    low.m1 = m1;
                    low.j1 = j1;
                }
            }
            if (gl == 0) settle(t, node, deg, low);
            deg = deg1;
            off = off1;
            node = node1;
        }
    }
    __syncthreads();
    // Near ties: among the neighbours whose FP32 V lies within the bound of
    // the lowest, the lowest canonical FP64 V (the first of equal ones, in
    // CSR order), compared with the node's own.
    auto moves = [&](double bv, int best, double vi, int node) {
        return bv < vi || (tie_mode != 0 && bv == vi && best < node);
    };
    const int n_few = queued[0], n_many = queued[1];
    for (int q = tid; q < n_few; q += T) {
        const int t = q < kTieQueue ? (int)queue[0][q] : spill[q];
        const int node = order[t], deg = sdeg[t];
        const uint32_t *const base = scol + soff[t >> 6] + (t & 63);
        uint32_t c[kChunk];
#pragma unroll
        for (int u = 0; u < kChunk; ++u) c[u] = base[64 * min(u, (deg - 1) >> 1)];
        const double vi = node_v64(G, s, node);
        // (entries past the list repeat its last word and change no minimum)
        float m1 = FLT_MAX;
#pragma unroll
        for (int u = 0; u < kChunk; ++u) m1 = fminf(m1, fminf(V[c[u] & 0xFFFFu], V[c[u] >> 16]));
        double bv = DBL_MAX;
        int best = -1;
        auto near = [&](int j) {
            const float vj = V[j];
            return vj - m1 <= kTieTau * vj;
        };
        auto lower = [&](double d, int j) {
            if (d < bv) {
                bv = d;
                best = j;
            }
        };
        if (G.v64) {
            const double *__restrict__ v64 = G.v64 + (int64_t)s * n;
            double d[2 * kChunk];
#pragma unroll
            for (int k = 0; k < 2 * kChunk; ++k) {
                const int j = (k & 1) ? (int)(c[k / 2] >> 16) : (int)(c[k / 2] & 0xFFFFu);
                d[k] = near(j) ? v64[j] : DBL_MAX;
            }
#pragma unroll
            for (int k = 0; k < 2 * kChunk; ++k)
                lower(d[k], (k & 1) ? (int)(c[k / 2] >> 16) : (int)(c[k / 2] & 0xFFFFu));
        } else {
            for (int k = 0; k < deg; ++k) {
                const uint32_t x = base[64 * (k >> 1)];
                const int j = (k & 1) ? (int)(x >> 16) : (int)(x & 0xFFFFu);
                if (near(j)) lower(canonical_node_v(G, s, j), j);
            }
        }
        par[node] = (uint16_t)(moves(bv, best, vi, node) ? best : node);
    }
    for (int q = group; q < n_many; q += kGroups) {
        const int t = q < kTieQueue ? (int)queue[1][q] : spill[n - 1 - q];
        const int node = order[t], deg = sdeg[t], rows = (deg + 1) >> 1;
        const uint32_t *const base = scol + soff[t >> 6] + (t & 63);
        const double vi = node_v64(G, s, node);
        float m1 = FLT_MAX;
        for (int r = gl; r < rows; r += kShare) {
            const uint32_t x = base[64 * r];
            m1 = fminf(m1, fminf(V[x & 0xFFFFu], V[x >> 16]));
        }
#pragma unroll
        for (int d = 1; d < kShare; d *= 2) m1 = fminf(m1, __shfl_xor(m1, d));
        double bv = DBL_MAX;
        int best = -1, at = 0x7FFFFFFF;
        for (int r = gl; r < rows; r += kShare) {
            const uint32_t x = base[64 * r];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int j = k ? (int)(x >> 16) : (int)(x & 0xFFFFu);
                const float vj = V[j];
                const double d = (vj - m1 <= kTieTau * vj) ? node_v64(G, s, j) : DBL_MAX;
                if (d < bv) {
                    bv = d;
                    best = j;
                    at = 2 * r + k;
                }
            }
        }
#pragma unroll
        for (int d = 1; d < kShare; d *= 2) {
            const double ov = __shfl_xor(bv, d);
            const int oj = __shfl_xor(best, d), oa = __shfl_xor(at, d);
            if (ov < bv || (ov == bv && oa < at)) {
                bv = ov;
                best = oj;
                at = oa;
            }
        }
        if (gl == 0) par[node] = (uint16_t)(moves(bv, best, vi, node) ? best : node);
    }
    if (tid == 0) {
        const unsigned long long ties = (unsigned long long)(n_few + n_many);
        if (store_count) *G.recheck = ties;
        else if (ties) atomicAdd(G.recheck, ties);
    }
    __syncthreads();
    // Algorithm 3 for every node: pointer jumping until every node points at
    // a root. Parents only ever point to strictly lower (V, id) nodes, so
    // the forest has no cycles; updates in place are safe because every value
    // written is an ancestor on the same path.
    for (int round = 0; round < 64; ++round) {
        bool changed = false;
        for (int i0 = 4 * tid; i0 < n; i0 += 4 * T) {
            const uint64_t four = __hip_atomic_load(&par4[i0 / 4], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            uint16_t p[4], q[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                p[u] = (uint16_t)(four >> (16 * u));
                q[u] = __hip_atomic_load(&par[p[u]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (q[u] != p[u]) {
                    __hip_atomic_store(&par[i0 + u], q[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    changed = true;
                }
        }
        // (a flag per round, cleared two rounds ahead of its next use: a
        // workgroup reduction costs several barriers)
        if (changed) again[round % 3] = 1;
        if (tid == 0) again[(round + 1) % 3] = 0;
        __syncthreads();
        if (!again[round % 3]) break;
    }
    int32_t *const out = labels_base + (int64_t)blockIdx.x * labels_ld + job.out_off;
    for (int i = tid; i < n; i += T) out[i] = par[i];
}

}  // namespace

hipError_t launch_descend(int tie_mode, const GraphDev *graphs, const NodeJob *jobs, int n_jobs, int sigma_base,
                          int n_sig, int32_t *labels_base, int64_t labels_ld, int max_n, hipStream_t stream,
                          bool store_count)
{
    if (n_jobs <= 0 || n_sig <= 0) return hipSuccess;
    if (max_n > kDescendNodes || (store_count && (n_jobs > 1 || n_sig > 1))) return hipErrorInvalidValue;
    const dim3 grid(n_sig, n_jobs), block(1024);
    if (max_n <= kDescendHalfNodes)   // two workgroups per CU
        hipLaunchKernelGGL(k_descend<kDescendHalfNodes>, grid, block, 0, stream, tie_mode, graphs, jobs, sigma_base,
                           labels_base, labels_ld, store_count);
    else
        hipLaunchKernelGGL(k_descend<kDescendNodes>, grid, block, 0, stream, tie_mode, graphs, jobs, sigma_base,
                           labels_base, labels_ld, store_count);
    return hipGetLastError();
}

}  // namespace qc
