// Counting search: the per-source distance histograms of a graph straight
// from a multi-source breadth-first search, without the distance matrix
// (instantiated per launch shape by qc_count_<threads>.hip).
//
// h[i][k] is the number of nodes at distance k from i, i.e. the number of
// nodes the search from i reaches for the first time at level k, so the
// search only has to count its new (node, source) pairs level by level.
//
// One workgroup searches a batch of BW sources at once, one bit per (node,
// source). The nodes sit in LDS in an order of their own ("positions", by
// decreasing number of entries; qc_rows.cpp builds it), and every lane owns
// quads of 4 consecutive positions: it gathers the frontier bits of its
// nodes' in-neighbours, ORs them and keeps what its `seen` registers do not
// hold yet. Nothing is delivered by atomics except the partial ORs of rows of
// many entries (hub rows), which are cut into units of 8 entries that any
// lane may take. Nodes of one entry (leaves, undirected graphs) have no
// position: nothing reaches a node through a leaf, no leaf is a source (its
// histogram follows from its neighbour's, k_hist_rest), and a leaf is new
// exactly one level after its neighbour, so a level only gathers and counts
// its neighbour's frontier bits. A level:
//   A. units of the hub rows (atomic OR into hacc[hub]); the leaves; then the
//      wavefront's quads, 256 positions of (nearly) one row length each,
//      their entries streamed as 16-bit positions one quad ahead; a lane
//      whose 4 nodes every source has reached gathers nothing, and a quad
//      whose 256 nodes are all reached is skipped, loads included;
//   B. (after a barrier) hub owners take hacc, every owner writes its new
//      bits as the next frontier and adds them to `seen`; the wavefront
//      counts its new bits per source (bit-sliced sums, then a bit transpose
//      across lanes) and adds the counts to the level's LDS counters;
//   C. (after a barrier) every wavefront reads the counters: the search ends
//      once every source has reached its whole component, or nothing is new.
//
// Why: the matrix search (qc_bfs.h) writes n^2 bytes, the histogram pass reads
// them back, and both only served these counts; its pull also spends 10
// operations per edge on merging and delivering runs, where a row's owner
// spends 2 (an address and an OR). What bounds it: the LDS gathers (their
// bank conflicts double them) and the fixed work per level (counts, barriers,
// the latency of the first entries), each about 40 % of the time. n = 19,717
// with 88,726 entries: 104 us against 426 + 114 us (search + histogram pass);
// a step over 64 graphs of 1,000 to 20,000 nodes x 32 widths: 4.71 -> 1.88 ms
// with the descent of the time (1.58 with today's).
//
// With P > 0 the search also writes its sources' distance rows: P bit-planes
// of the level per owned word (as in qc_bfs.h), permuted from the positions'
// owners to the nodes' through LDS at the end and transposed to bytes there.
// The planes fill the registers (one workgroup of 16 wavefronts per CU), and
// the last workgroups' rows leave at HBM speed; n = 19,717, matrix, histograms
// and all: 250 us against 521 (qc_bfs.h's search and the histogram pass).
#pragma once

#include "qc_internal.h"

namespace qc {

// Per-lane roles of the bit transpose below. The lane pairs of its four
// stages are lane ^ 8, ^ 7, ^ 2 and ^ 1 within a row of 16 lanes (the DPP
// patterns row_ror:8, row_half_mirror, quad_perm), so the roles are the dual
// basis of these four patterns over the lane bits.
struct ColumnRoles {
    uint32_t sh8, sh4, sh2, sh1;   // 0 or the stage's shift
    uint32_t perm8;                // byte selector of the first stage
    int column;                    // the column (mod 16) the lane ends with
    __device__ __forceinline__ explicit ColumnRoles(int lane)
    {
        const int b0 = lane & 1, b1 = (lane >> 1) & 1, b2 = (lane >> 2) & 1, b3 = (lane >> 3) & 1;
        const int r4 = b2, r2 = b1 ^ b2, r1 = b0 ^ b2;
        sh8 = b3 ? 8u : 0u;
        sh4 = r4 ? 4u : 0u;
        sh2 = r2 ? 2u : 0u;
        sh1 = r1 ? 1u : 0u;
        // own bytes 0, 2 and the partner's 0, 2 (or 1, 3 of both):
        // v_perm selects 0-3 from its second operand, 4-7 from its first
        perm8 = b3 ? 0x07030501u : 0x06020400u;
        column = b3 * 8 + r4 * 4 + r2 * 2 + r1;
    }
};

// One transpose stage: columns whose bit `s` equals the lane's role, own
// rows' bits at the column's low place, the partner's `s` places up.
template <int S, int CTRL>
__device__ __forceinline__ uint32_t column_stage(uint32_t x, uint32_t sh, uint32_t mask)
{
    const uint32_t p = (uint32_t)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xF, 0xF, true);
    return ((x >> sh) & mask) | ((p << (S - sh)) & ~mask);
}

// x: 32 columns (bits) of this lane's row. After the four stages the low
// half word holds column r.column of the 16 lanes of the DPP row, the high
// half word column r.column + 16.
__device__ __forceinline__ uint32_t gather_columns(uint32_t x, const ColumnRoles &r)
{
    const uint32_t p = (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x128, 0xF, 0xF, true);  // row_ror:8
    x = __builtin_amdgcn_perm(p, x, r.perm8);
    x = column_stage<4, 0x141>(x, r.sh4, 0x0F0F0F0Fu);   // row_half_mirror: lane ^ 7
    x = column_stage<2, 0x4E>(x, r.sh2, 0x33333333u);    // quad_perm: lane ^ 2
    x = column_stage<1, 0xB1>(x, r.sh1, 0x55555555u);    // quad_perm: lane ^ 1
    return x;
}

// Bit-sliced sum of N words, per bit column: out[w] receives the bits of
// weight 2^w (full adders, two operations each).
template <int N, int W, int M>
__device__ __forceinline__ void add_columns(const uint32_t (&x)[N], uint32_t (&out)[M])
{
    static_assert(W < M, "not enough sum bits");
    uint32_t s = x[0];
    if constexpr (N > 1) {
        constexpr int C = N / 2;
        uint32_t c[C];
#pragma unroll
        for (int i = 1, k = 0; i < N; i += 2, ++k) {
            if (i + 1 < N) {
                const uint32_t a = x[i], b = x[i + 1];
                c[k] = (s & a) | (s & b) | (a & b);
                s = s ^ a ^ b;
            } else {
                c[k] = s & x[i];
                s ^= x[i];
            }
        }
        out[W] = s;
        add_columns<C, W + 1, M>(c, out);
    } else {
        out[W] = s;
#pragma unroll
        for (int w = W + 1; w < M; ++w) out[w] = 0u;
    }
}

constexpr int sum_bits(int n) { return n < 2 ? 1 : 1 + sum_bits(n / 2); }

// s, a, b -> s + a + b per bit column: the sum stays in s, the carry returns.
__device__ __forceinline__ uint32_t carry_add(uint32_t &s, uint32_t a, uint32_t b)
{
    const uint32_t c = (s & a) | (s & b) | (a & b);
    s = s ^ a ^ b;
    return c;
}

// Transpose the 8 x 8 bit matrix in each byte lane of a[0..7]: afterwards
// bit 8j + p of a[k] is what bit 8j + k of a[p] was.
__device__ __forceinline__ void transpose_bytes(uint32_t (&a)[8])
{
    constexpr uint32_t kMask[3] = {0x0F0F0F0Fu, 0x33333333u, 0x55555555u};
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const int s = 4 >> r;
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            if (p & s) continue;
            const uint32_t x = a[p], y = a[p + s], m = kMask[r];
            a[p] = (x & m) | ((y << s) & ~m);
            a[p + s] = ((x >> s) & m) | (y & ~m);
        }
    }
}

// NQ quads (4 positions) per lane, KT threads, PER positions per 32-bit word
// (1: batches of 32 sources, 2: 16). P > 0: the distance rows of the sources
// too, from P bit-planes of the level in registers (levels up to 2^P - 2;
// all ones: not reached), NQN quads of consecutive nodes per lane. The small
// counting shapes are held to 64 registers, so that two workgroups of 1,024
// threads share a CU (two quads: 6 registers go to scratch; 79,000 sources of
// 4,000 to 8,000 nodes 567 -> 471 us, the step above 1.63 -> 1.58 ms).
template <int NQ, int KT, int PER, int P, int NQN>
__global__ __launch_bounds__(KT, KT == 1024 && NQ <= 2 && P == 0 ? 8 : 4) void k_count(
    const GraphDev *__restrict__ graphs, const BfsJob *__restrict__ jobs)
{
    constexpr int QW = 4 / PER;             // words per quad
    constexpr int NW = NQ * QW;             // words per lane
    constexpr int BW = 32 / PER;
    constexpr int HUB = rows_hub_cap(NQ, KT);
    constexpr int kHubQuads = (HUB + 4 * KT - 1) / (4 * KT);   // quads per lane that may hold hubs
    // bits of a lane's count: at most NW + 4 + 65,535 / KT
    constexpr int CB = KT >= 1024 ? 7 : KT >= 512 ? 8 : 9;
    constexpr int PA = P > 0 ? P : 1;
    // `seen` in registers, or the planes' disjunction where they fill them
    constexpr bool kSeenReg = P == 0 || NW * (P + 1) <= 64;
    // With planes, two frontier fields: a quad's new bits go straight to the
    // next frontier instead of waiting in registers for the barrier (the
    // planes leave no registers, and one workgroup per CU leaves LDS).
    constexpr bool kTwo = P > 0;
    constexpr int kHold = kTwo ? kHubQuads * QW : NW;   // words held over the barrier
    // registers to load a quad's third and fourth rows ahead too
    constexpr bool kWide = P == 0 && NW <= 28;
    constexpr uint32_t kFull = PER == 1 ? ~0u : 0xFFFFu;
    constexpr uint32_t kAbsent = 0x80000000u;         // an offset past any table: loads nothing
    typedef const __attribute__((address_space(4))) uint32_t *const_u32;

    __shared__ __attribute__((aligned(16))) uint32_t fields[(kTwo ? 2 : 1) * NW * KT];
    __shared__ __attribute__((aligned(16))) uint32_t hacc[HUB];
    __shared__ uint32_t hdone[HUB / 32];
    __shared__ uint32_t cnt[3][16];   // counts of a level
    __shared__ uint32_t batch[2][BW + 1];   // the sources' first and third words; how many

    const BfsJob job = jobs[blockIdx.x];
    const GraphDev &G = graphs[job.g];
    const int tid = (int)threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_pos = G.rows.n_pos;
    const int nb = min(BW, G.rows.n_search - job.s0);
    const uint4 *__restrict__ src = (const uint4 *)G.rows.src + job.s0;

    uint32_t *const front = fields;
    // own words of quad g
    auto own = [&](int g) { return (g * KT + tid) * QW; };
    auto clear_front = [&] {
#pragma unroll
        for (int g = 0; g < NQ; ++g)
#pragma unroll
            for (int i = 0; i < QW; ++i) front[own(g) + i] = 0u;
    };
    auto put = [&](uint32_t p, int b) {
        __hip_atomic_fetch_or(&front[PER == 1 ? p : p >> 1], 1u << (PER == 1 ? b : (int)(p & 1) * 16 + b),
                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    clear_front();
    for (int i = tid; i < HUB; i += KT) hacc[i] = 0u;
    for (int i = tid; i < HUB / 32; i += KT) hdone[i] = 0u;
    if (tid < 48) cnt[tid / 16][tid % 16] = 0u;
    if (tid == 0) batch[0][BW] = (uint32_t)nb;
    __syncthreads();
    if (tid < nb) {   // level 0: the sources
        const uint4 s = src[tid];
        put(s.x >> 16, tid);
        batch[0][tid] = s.x;
        batch[1][tid] = s.z;
    }
    __syncthreads();
    uint32_t seen_r[kSeenReg ? NW : 1], plane[NW][PA];
    // bits of word w that are reached (or that stand for nothing)
    auto seen_of = [&](int w) -> uint32_t {
        if constexpr (kSeenReg) {
            return seen_r[w];
        } else {
            uint32_t u = plane[w][0];
#pragma unroll
            for (int p = 1; p < PA; ++p) u &= plane[w][p];
            return ~u;
        }
    };
    // word w's new bits at a level
    auto reach = [&](int w, uint32_t bits, int level) {
        if constexpr (kSeenReg) seen_r[w] |= bits;
        if constexpr (P > 0) {
#pragma unroll
            for (int p = 0; p < PA; ++p)
                if (!((level >> p) & 1)) plane[w][p] &= ~bits;   // uniform branch
        }
    };
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        if constexpr (kSeenReg) seen_r[w] = 0u;
#pragma unroll
        for (int p = 0; p < PA; ++p) plane[w][p] = ~0u;
    }
    const uint32_t pad_bits = (nb < BW) ? ~((1u << nb) - 1u) & kFull : 0u;
#pragma unroll
    for (int g = 0; g < NQ; ++g)
#pragma unroll
        for (int i = 0; i < QW; ++i)
            reach(g * QW + i, front[own(g) + i] | pad_bits | (PER == 1 ? 0u : pad_bits << 16), 0);
    clear_front();
    __syncthreads();
    {   // level 1: their neighbours, along the sources' rows
        constexpr int kTps = KT / BW;
        const int b = tid / kTps, part = tid % kTps;
        if (b < nb) {
            const uint4 s = src[b];
            const uint16_t *__restrict__ col = G.rows.col_pos + s.y;
            for (int e = part; e < (int)(s.z >> 16); e += kTps) put(col[e], b);
        }
    }
    __syncthreads();

    // this lane's view of source `lane` (every wavefront keeps one)
    const uint4 my = (lane < nb) ? src[lane] : make_uint4(0u, 0u, 0u, 1u);
    const uint32_t my_deg = my.z & 0xFFFFu;
    uint32_t left = my.w - 1u - my_deg;      // nodes of its component not yet reached
    int32_t *const hist = G.hist + (int64_t)(my.x & 0xFFFFu) * G.K;
    const int K = G.K;
    if (wave == 0 && lane < nb) {
        hist[0] = 1;
        hist[1] = (int32_t)my_deg;
    }
    int last = __ballot(my_deg != 0u) ? 1 : 0;

    uint32_t act = 0u;                       // quads with a node left to reach
#pragma unroll
    for (int g = 0; g < NQ; ++g) {
        uint32_t all = ~0u;
#pragma unroll
        for (int i = 0; i < QW; ++i) {
            reach(g * QW + i, front[own(g) + i], 1);
            // (a position that holds no node counts as reached)
            uint32_t none = 0u;
#pragma unroll
            for (int h = 0; h < PER; ++h) {
                const int p = (g * KT + tid) * 4 + i * PER + h;
                if (p >= n_pos) none |= kFull << (16 * h);
            }
            reach(g * QW + i, none, 0);
            all &= seen_of(g * QW + i);
        }
        if (__ballot(all != ~0u)) act |= 1u << g;
    }
    const uint32_t voff = (uint32_t)lane * 16u;
    // The graph's descriptor through an address the compiler cannot see
    // through: what a level reads of it is loaded again (scalar loads) instead
    // of being held in scalar registers, which have no room for all of it. An
    // instance of 16 quads with 101 scalar registers spilled (to lanes of two
    // vector registers) and 37 vector ones lost counts; nothing in the source
    // explains it (every value a level branches on is the wavefront's or the
    // workgroup's own, from ballots, scalar loads and LDS after a barrier), and
    // no spill in its listing is stored under a narrower mask than it is
    // loaded. Whatever the cause, the build refuses an instance that spills a
    // scalar register (build.py).
    typedef const __attribute__((address_space(4))) GraphDev *const_graph;
    auto descriptor = [&]() -> const_graph {
        uint64_t a = (uint64_t)(uintptr_t)&G;
        asm volatile("" : "+s"(a));
        return (const_graph)a;
    };
    int pulled = 0;
    bool overflow = false;
    auto ent_rsrc = [&](const_graph D) {
        return __builtin_amdgcn_make_buffer_rsrc((void *)D->rows.ent, 0, (int)D->rows.ent_bytes, kBufferWord3);
    };
    auto row_of = [&](const __amdgpu_buffer_rsrc_t &ent, uint32_t r, bool on) -> u32x4 {
        return __builtin_amdgcn_raw_buffer_load_b128(ent, (int)(voff | (on ? 0u : kAbsent)), (int)r, 0);
    };
    auto unit_ent = [&](const_graph D, int u) { return ((global_u4)D->rows.units)[(int64_t)u * 80 + lane]; };
    auto unit_tgt = [&](const_graph D, int u) {
        return ((const __attribute__((address_space(1))) uint32_t *)((global_u4)D->rows.units + (int64_t)u * 80 +
                                                                     64))[lane];
    };
    // One level; true when the search ends.
    auto run_level = [&](int level) __attribute__((always_inline)) -> bool {
        const uint32_t *const from = fields + (kTwo ? (level & 1) * NW * KT : 0);
        uint32_t *const to = fields + (kTwo ? (1 - (level & 1)) * NW * KT : 0);
        auto gather = [&](uint32_t p) -> uint32_t {
            if constexpr (PER == 1) return from[p];
            else return ((const uint16_t *)from)[p];
        };
        ++pulled;
        const const_graph D = descriptor();
        const __amdgpu_buffer_rsrc_t ent = ent_rsrc(D);
        const int n_hub = D->rows.n_hub;
        uint32_t any = 0u;
        uint32_t cl[CB];   // the lane's new bits per source, bit-sliced
#pragma unroll
        for (int p = 0; p < CB; ++p) cl[p] = 0u;
        auto count4 = [&](uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3) {
            const uint32_t t0 = carry_add(cl[0], x0, x1), t1 = carry_add(cl[0], x2, x3);
            uint32_t c = carry_add(cl[1], t0, t1);
#pragma unroll
            for (int p = 2; p < CB; ++p) {
                const uint32_t d = cl[p] & c;
                cl[p] ^= c;
                c = d;
            }
        };
        // quad g's new bits: the next frontier, `seen`, the planes
        auto settle = [&](int g, uint32_t *y) {
            uint32_t all = ~0u;
#pragma unroll
            for (int i = 0; i < QW; ++i) {
                to[own(g) + i] = y[i];
                reach(g * QW + i, y[i], level);
                any |= y[i];
                all &= seen_of(g * QW + i);
            }
            if (!__ballot(all != ~0u)) act &= ~(1u << g);
            if (g < kHubQuads && (g * KT + wave * 64) * 4 < n_hub) {
                // which hubs are done: bit (i, lane) of the quad's 256 positions
                uint32_t v = 0u;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t s = (seen_of(g * QW + i / PER) >> (16 * (i % PER))) & kFull;
                    const uint64_t o = __ballot(s == kFull);
                    if (lane == 2 * i) v = (uint32_t)o;
                    if (lane == 2 * i + 1) v = (uint32_t)(o >> 32);
                }
                if (lane < 8) hdone[(g * KT + wave * 64) / 8 + lane] = v;
            }
        };
        // A. hub units: 8 entries per lane, the next unit's in flight
        const int u0 = (int)((const_u32)D->rows.wave_unit)[wave], u1 = (int)((const_u32)D->rows.wave_unit)[wave + 1];
        if (u0 < u1) {
            u32x4 e = unit_ent(D, u0);
            uint32_t t = unit_tgt(D, u0);
            for (int u = u0; u < u1; ++u) {
                const int un = min(u + 1, u1 - 1);
                const u32x4 en = unit_ent(D, un);
                const uint32_t tn = unit_tgt(D, un);
                if (!((hdone[t >> 21] >> ((t >> 16) & 31)) & 1u)) {
                    uint32_t x[8];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        x[2 * k] = gather(e[k] & 0xFFFFu);
                        x[2 * k + 1] = gather(e[k] >> 16);
                    }
                    const uint32_t acc = (x[0] | x[1] | x[2]) | (x[3] | x[4] | x[5]) | (x[6] | x[7]);
                    if (acc)
                        __hip_atomic_fetch_or(&hacc[t & 0xFFFFu], acc, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                e = en;
                t = tn;
            }
        }
        // leaves: 4 per lane and step, added to the lane's count
        const int n_leaf = D->rows.n_leaf;
        for (int l = tid * 4; l < n_leaf; l += KT * 4) {
            const u32x2 e = ((const __attribute__((address_space(1))) u32x2 *)D->rows.leaf)[l >> 2];
            const uint32_t x0 = gather(e.x & 0xFFFFu), x1 = gather(e.x >> 16);
            const uint32_t x2 = gather(e.y & 0xFFFFu), x3 = gather(e.y >> 16);
            if constexpr (PER == 1) count4(x0, x1, x2, x3);
            else count4(x0 | x1 << 16, x2 | x3 << 16, 0u, 0u);
        }
        // the quads, their first two rows of entries loaded one quad ahead
        uint32_t hold[kHold];
        u32x4 ra[2], rb[2];
        uint32_t wd[2], rx[2], row = ((const_u32)D->rows.wave_row)[wave] * 1024u;
        auto issue = [&](int g) {
            const uint32_t w = ((const_u32)D->rows.codes)[wave * NQ + g];
            const uint32_t on = ((act >> g) & 1u) ? w : 0u;
            ra[g & 1] = row_of(ent, row, on > 0u);
            rb[g & 1] = row_of(ent, row + 1024u, on > 2u);
            wd[g & 1] = on;
            rx[g & 1] = row + 2048u;
            row += ((w + 1u) >> 1) * 1024u;
        };
        issue(0);
#pragma unroll
        for (int g = 0; g < NQ; ++g) {
            const uint32_t w = wd[g & 1], xr = rx[g & 1];
            const u32x4 a = ra[g & 1], b = rb[g & 1];
            u32x4 c, d;
            if constexpr (kWide) {
                c = row_of(ent, xr, w > 4u);
                d = row_of(ent, xr + 1024u, w > 6u);
            }
            if (g + 1 < NQ) issue(g + 1);
            uint32_t x[4] = {0u, 0u, 0u, 0u};
            // one entry of each of the 4 positions
            auto slot = [&](uint32_t e0, uint32_t e1) {
                x[0] |= gather(e0 & 0xFFFFu);
                x[1] |= gather(e0 >> 16);
                x[2] |= gather(e1 & 0xFFFFu);
                x[3] |= gather(e1 >> 16);
            };
            auto pair = [&](const u32x4 &r) {
                const uint32_t p0 = gather(r.x & 0xFFFFu), p1 = gather(r.x >> 16), p2 = gather(r.y & 0xFFFFu),
                               p3 = gather(r.y >> 16), q0 = gather(r.z & 0xFFFFu), q1 = gather(r.z >> 16),
                               q2 = gather(r.w & 0xFFFFu), q3 = gather(r.w >> 16);
                x[0] |= p0 | q0;
                x[1] |= p1 | q1;
                x[2] |= p2 | q2;
                x[3] |= p3 | q3;
            };
            if (w) {
                uint32_t all = ~0u;
#pragma unroll
                for (int i = 0; i < QW; ++i) all &= seen_of(g * QW + i);
                if (all != ~0u) {
                    if (w >= 2u) pair(a);
                    else slot(a.x, a.y);
                    if (w >= 4u) pair(b);
                    else if (w == 3u) slot(b.x, b.y);
                    if (w > 4u) {
                        if constexpr (!kWide) {
                            c = row_of(ent, xr, true);
                            d = row_of(ent, xr + 1024u, w > 6u);
                        }
                        if (w >= 6u) pair(c);
                        else slot(c.x, c.y);
                        if (w >= 8u) pair(d);
                        else if (w == 7u) slot(d.x, d.y);
                        if (w > 8u) {
                            // longer rows: two entries per step, the next two in flight
                            uint32_t r = xr + 2048u;
                            u32x4 z = row_of(ent, r, true);
                            for (uint32_t k = 8u; k < w; k += 2u) {
                                r += (k + 2u < w) ? 1024u : 0u;
                                const u32x4 zn = row_of(ent, r, true);
                                if (k + 1u < w) pair(z);
                                else slot(z.x, z.y);
                                z = zn;
                            }
                        }
                    }
                }
            }
            uint32_t y[QW];
#pragma unroll
            for (int i = 0; i < QW; ++i)
                y[i] = ((PER == 1) ? x[i] : (x[2 * i] | x[2 * i + 1] << 16)) & ~seen_of(g * QW + i);
            if (!kTwo || g < kHubQuads) {
#pragma unroll
                for (int i = 0; i < QW; ++i) hold[g * QW + i] = y[i];
            } else {
                settle(g, y);
                if constexpr (PER == 1) count4(y[0], y[1], y[QW > 2 ? 2 : 0], y[QW > 3 ? 3 : 0]);
                else count4(y[0], y[1], 0u, 0u);
            }
        }
        __syncthreads();
        // B. hub rows; the held quads' next frontier
#pragma unroll
        for (int g = 0; g < kHubQuads; ++g) {
            if ((g * KT + wave * 64) * 4 < n_hub) {
                uint4 *const h = (uint4 *)hacc + (g * KT + tid);
                const uint4 a = *h;
                *h = make_uint4(0u, 0u, 0u, 0u);
                const uint32_t v[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
                for (int i = 0; i < QW; ++i)
                    hold[g * QW + i] |=
                        ((PER == 1) ? v[i] : (v[2 * i] | v[2 * i + 1] << 16)) & ~seen_of(g * QW + i);
            }
        }
#pragma unroll
        for (int g = 0; g < kHold / QW; ++g) settle(g, hold + g * QW);
        uint32_t *const lc = cnt[level % 3];
#pragma unroll
        for (int p = 0; p < CB; ++p) any |= cl[p];
        if (__ballot(any != 0u)) {
            uint32_t sum[CB];
            add_columns<kHold, 0, CB>(hold, sum);
            if (kTwo || n_leaf) {
                uint32_t c = 0u;
#pragma unroll
                for (int p = 0; p < CB; ++p) c = carry_add(sum[p], cl[p], c);
            }
            int lane_now = lane;    // (recomputed per level instead of held in registers)
            asm volatile("" : "+v"(lane_now));
            const ColumnRoles roles(lane_now);
            uint32_t lo = 0u, hi = 0u;
#pragma unroll
            for (int p = CB - 1; p >= 0; --p) {
                lo <<= 1;
                hi <<= 1;
                if (p < 2 || __ballot(sum[p] != 0u)) {
                    const uint32_t t = gather_columns(sum[p], roles);
                    lo += (uint32_t)__popc(t & 0xFFFFu);
                    hi += (uint32_t)__popc(t >> 16);
                }
            }
            // (at most 65,535 new pairs per source and level: the halves
            // never carry into one another)
            const uint32_t v = (PER == 1) ? (lo | hi << 16) : lo + hi;
            if (v)
                __hip_atomic_fetch_add(&lc[roles.column], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        __syncthreads();
        // C. the level's counts
        uint32_t c = 0u;
        if (lane < BW) {
            c = lc[lane & 15];
            if constexpr (PER == 1) c = (lane < 16) ? (c & 0xFFFFu) : (c >> 16);
        }
        // the counters of the level after next: last read after the previous
        // level's last barrier, next added to after this level's successor's
        if (tid < 16) cnt[(level + 2) % 3][tid] = 0u;
        if (!__ballot(c != 0u)) return true;   // nothing new: every search ended
        last = level;
        if (level > kMaxDist) {
            overflow = true;
            return true;
        }
        if (wave == 0 && lane < nb && level < K) hist[level] = (int32_t)c;
        left -= c;
        return !__ballot(left != 0u);
    };
    if (__ballot(left != 0u)) {
        for (int level = 2;; ++level)
            if (run_level(level)) break;
    }
    // The histograms' ends and the status. Before the distance rows where the
    // planes fill the registers (fewer spills: 4 quads, 5 planes, 295 -> 285 us
    // for 19,717 nodes), else after them, where no wavefront waits for it.
    auto finish = [&] {
        // (everything anew from the descriptor and LDS: held over the levels, it
        // took scalar registers that the smaller shapes do not have)
        int tid_now = (int)threadIdx.x;
        asm volatile("" : "+v"(tid_now));
        if (__builtin_amdgcn_readfirstlane(tid_now >> 6) == 0) {
            const const_graph D = descriptor();
            const int l = tid_now & 63, rows = D->K, mine = (int)batch[0][BW];
            const uint32_t node = (l < mine) ? batch[0][l] & 0xFFFFu : 0u, z = (l < mine) ? batch[1][l] : 0u;
            int32_t *const h = D->hist + (int64_t)node * rows;
            if (l < mine)
                for (int k = max(last, 1) + 1; k < rows; ++k) h[k] = 0;
            // A source's leaves are not searched from and lie one further from what
            // the source reaches last; counted here where that passes the rows' (or
            // the library's) last distance, so that the status is final before
            // anything reads the histograms.
            int far = last;
            if (last == rows - 1 || last == kMaxDist) {
                const bool further = l < mine && last < rows && (z & 0xFFFFu) > (z >> 16) && h[last] != 0;
                if (__ballot(further)) far = last + 1;
            }
            if (l == 0) {
                atomicMax(&D->status[0], far);
                if (overflow || far > kMaxDist) atomicOr(&D->status[1], 1);
            }
            unsigned long long *const visits = D->visits;
            if (visits) {
                // the search's work, as the levels cover it: every entry per
                // pulled level (what the skipped rows leave out included), and the
                // sources' own entries
                uint32_t deg = z & 0xFFFFu;
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) deg += (uint32_t)__shfl_xor((int)deg, off);
                if (l == 0) {
                    const unsigned long long v =
                        (unsigned long long)pulled * (unsigned long long)D->nnz_bfs + deg;
                    atomicAdd(&visits[0], v);
                    atomicAdd(&visits[1], v * 4ull);
                }
            }
        }
    };
    if constexpr (P > 0 && !kSeenReg) finish();
    if constexpr (P > 0) {
        // The distance rows. The planes go from the positions' owners to the
        // nodes' (quads of 4 consecutive nodes per lane) through the frontier's
        // LDS, one plane at a time: a node reads its position's word, a leaf its
        // neighbour's, to which it adds one.
        constexpr int NN = NQN * QW;
        typedef __attribute__((address_space(1))) int8_t gbyte;
        typedef uint32_t __attribute__((aligned(1))) u32_any;   // rows need not be 4-byte aligned
        typedef __attribute__((address_space(1))) u32_any gu32;
        const int n = G.n;
        gbyte **const rows = (gbyte **)hacc;                    // (HUB >= 256 words)
        __syncthreads();
        if (tid < nb) rows[tid] = (gbyte *)G.dist + (int64_t)(src[tid].x & 0xFFFFu) * G.ld;
        const uint2 *__restrict__ node_pos = (const uint2 *)G.rows.node_pos;
        auto gather = [&](int f, uint32_t p) -> uint32_t {
            const uint32_t *const x = fields + f * NW * KT;
            if constexpr (PER == 1) return x[p];
            else return ((const uint16_t *)x)[p];
        };
        // plane p of the positions into field p % 2
        auto publish = [&](int p) {
#pragma unroll
            for (int g = 0; g < NQ; ++g)
#pragma unroll
                for (int i = 0; i < QW; ++i) fields[(p & 1) * NW * KT + own(g) + i] = plane[g * QW + i][p];
        };
        // planes p0.. of node quad g from the fields into d[][p0..]
        uint32_t d[NN][PA];
        auto fetch = [&](int g, int p0, int count) {
            const int v0 = (g * KT + tid) * 4;
            const uint2 e = (v0 < n) ? node_pos[v0 >> 2] : make_uint2(0u, 0u);
#pragma unroll
            for (int q = 0; q < count; ++q) {
                const int p = p0 + q;
                const uint32_t x0 = gather(p & 1, e.x & 0xFFFFu), x1 = gather(p & 1, e.x >> 16);
                const uint32_t x2 = gather(p & 1, e.y & 0xFFFFu), x3 = gather(p & 1, e.y >> 16);
                if constexpr (PER == 1) {
                    d[4 * g + 0][p] = x0;
                    d[4 * g + 1][p] = x1;
                    d[4 * g + 2][p] = x2;
                    d[4 * g + 3][p] = x3;
                } else {
                    d[2 * g + 0][p] = x0 | x1 << 16;
                    d[2 * g + 1][p] = x2 | x3 << 16;
                }
            }
        };
        // all but the last (one or two) planes into registers; the last are
        // fetched quad by quad below, so the quads' registers die one by one
        constexpr int kLate = 2 - (PA & 1);
#pragma unroll
        for (int p0 = 0; p0 + kLate < PA; p0 += 2) {
            __syncthreads();
            publish(p0);
            publish(p0 + 1);
            __syncthreads();
#pragma unroll
            for (int g = 0; g < NQN; ++g) fetch(g, p0, 2);
        }
        __syncthreads();
#pragma unroll
        for (int p = PA - kLate; p < PA; ++p) publish(p);
        __syncthreads();
        const uint32_t *__restrict__ flags = G.rows.node_flags;
#pragma unroll
        for (int g = 0; g < NQN; ++g) {
            const int v0 = (g * KT + tid) * 4;
            if (v0 >= n) continue;
            fetch(g, PA - kLate, kLate);
            // per node 2 bits: 1 leaf (one more than its neighbour), 2 no edges
            const uint32_t f = flags[v0 >> 4] >> (2 * (v0 & 15));
            uint32_t a[QW][8];
#pragma unroll
            for (int i = 0; i < QW; ++i) {
                uint32_t leaf = 0u, alone = 0u;
#pragma unroll
                for (int h = 0; h < PER; ++h) {
                    const uint32_t b = f >> (2 * (i * PER + h));
                    if (b & 1u) leaf |= kFull << (16 * h);
                    if (b & 2u) alone |= kFull << (16 * h);
                }
                uint32_t u = d[g * QW + i][0];
#pragma unroll
                for (int p = 1; p < PA; ++p) u &= d[g * QW + i][p];
                u |= alone;
                uint32_t c = leaf & ~u;
#pragma unroll
                for (int p = 0; p < PA; ++p) {
                    const uint32_t t = d[g * QW + i][p];
                    a[i][p] = (t ^ c) | u;
                    c &= t;
                }
#pragma unroll
                for (int p = PA; p < 8; ++p) a[i][p] = u;
                transpose_bytes(a[i]);
            }
            // byte j of a[i][k]: PER 1: node v0 + i, source 8j + k; PER 2: node
            // v0 + 2i + j / 2, source 8 (j % 2) + k
            auto quad = [&](int k, uint32_t (&o)[4 / PER]) {
                if constexpr (PER == 1) {
                    const uint32_t t0 = __builtin_amdgcn_perm(a[1][k], a[0][k], 0x05010400u);
                    const uint32_t t1 = __builtin_amdgcn_perm(a[1][k], a[0][k], 0x07030602u);
                    const uint32_t t2 = __builtin_amdgcn_perm(a[3][k], a[2][k], 0x05010400u);
                    const uint32_t t3 = __builtin_amdgcn_perm(a[3][k], a[2][k], 0x07030602u);
                    o[0] = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
                    o[1] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
                    o[2] = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
                    o[3] = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
                } else {
                    o[0] = __builtin_amdgcn_perm(a[1][k], a[0][k], 0x06040200u);
                    o[1] = __builtin_amdgcn_perm(a[1][k], a[0][k], 0x07050301u);
                }
            };
            if (v0 + 3 < n && nb == BW) {
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    uint32_t o[4 / PER];
                    quad(k, o);
#pragma unroll
                    for (int j = 0; j < 4 / PER; ++j) *(gu32 *)(rows[8 * j + k] + v0) = o[j];
                }
            } else {
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    uint32_t o[4 / PER];
                    quad(k, o);
#pragma unroll
                    for (int j = 0; j < 4 / PER; ++j)
                        if (8 * j + k < nb)
                            for (int i = 0; i < 4 && v0 + i < n; ++i)
                                rows[8 * j + k][v0 + i] = (int8_t)((o[j] >> (8 * i)) & 0xFFu);
                }
            }
        }
    }
    if constexpr (P == 0 || kSeenReg) finish();
}

}  // namespace qc
