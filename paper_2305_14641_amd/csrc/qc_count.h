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
// with 88,726 entries: 119 us against 426 + 114 us (search + histogram pass);
// 64 graphs of 1,000 to 20,000 nodes x 32 widths as one batch: 1.88 ms
// against 4.71.
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

// NQ quads (4 positions) per lane, KT threads, PER positions per 32-bit word
// (1: batches of 32 sources, 2: 16).
template <int NQ, int KT, int PER>
__global__ __launch_bounds__(KT) void k_count(const GraphDev *__restrict__ graphs,
                                              const BfsJob *__restrict__ jobs)
{
    constexpr int QW = 4 / PER;             // words per quad
    constexpr int NW = NQ * QW;             // words per lane
    constexpr int BW = 32 / PER;
    constexpr int HUB = rows_hub_cap(NQ, KT);
    constexpr int kHubQuads = (HUB + 4 * KT - 1) / (4 * KT);   // quads per lane that may hold hubs
    constexpr uint32_t kFull = PER == 1 ? ~0u : 0xFFFFu;
    constexpr uint32_t kAbsent = 0x80000000u;         // an offset past any table: loads nothing
    // bits of a lane's count: at most NW + 4 + 65,535 / KT
    constexpr int P = KT >= 1024 ? 7 : KT >= 512 ? 8 : 9;
    typedef const __attribute__((address_space(4))) uint32_t *const_u32;

    __shared__ __attribute__((aligned(16))) uint32_t front[NW * KT];
    __shared__ __attribute__((aligned(16))) uint32_t hacc[HUB];
    __shared__ uint32_t hdone[HUB / 32];
    __shared__ uint32_t cnt[3][16];

    const BfsJob job = jobs[blockIdx.x];
    const GraphDev &G = graphs[job.g];
    const int tid = (int)threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_pos = G.rows.n_pos;
    const int nb = min(BW, G.rows.n_search - job.s0);
    const int n_hub = G.rows.n_hub;
    const uint4 *__restrict__ src = (const uint4 *)G.rows.src + job.s0;

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
    __syncthreads();
    if (tid < nb) put(src[tid].x >> 16, tid);   // level 0: the sources
    __syncthreads();
    uint32_t seen[NW], y[NW];
    const uint32_t pad_bits = (nb < BW) ? ~((1u << nb) - 1u) & kFull : 0u;
#pragma unroll
    for (int g = 0; g < NQ; ++g)
#pragma unroll
        for (int i = 0; i < QW; ++i)
            seen[g * QW + i] = front[own(g) + i] | pad_bits | (PER == 1 ? 0u : pad_bits << 16);
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
            uint32_t s = seen[g * QW + i] | front[own(g) + i];
            // (a position past the last node counts as reached)
#pragma unroll
            for (int h = 0; h < PER; ++h)
                if ((g * KT + tid) * 4 + i * PER + h >= n_pos) s |= kFull << (16 * h);
            seen[g * QW + i] = s;
            all &= s;
        }
        if (__ballot(all != ~0u)) act |= 1u << g;
    }
    const ColumnRoles roles(lane);
    const const_u32 codes = (const_u32)G.rows.codes + wave * NQ;
    const uint32_t row0 = ((const_u32)G.rows.wave_row)[wave] * 1024u;
    const int u0 = (int)((const_u32)G.rows.wave_unit)[wave];
    const int u1 = (int)((const_u32)G.rows.wave_unit)[wave + 1];
    const int n_leaf = G.rows.n_leaf;
    const __amdgpu_buffer_rsrc_t ent =
        __builtin_amdgcn_make_buffer_rsrc((void *)G.rows.ent, 0, (int)G.rows.ent_bytes, kBufferWord3);
    const uint32_t voff = (uint32_t)lane * 16u;
    auto gather = [&](uint32_t p) -> uint32_t {
        if constexpr (PER == 1) return front[p];
        else return ((const uint16_t *)front)[p];
    };
    auto row_of = [&](uint32_t row, bool on) -> u32x4 {
        return __builtin_amdgcn_raw_buffer_load_b128(ent, (int)(voff | (on ? 0u : kAbsent)), (int)row, 0);
    };

    int pulled = 0;
    bool overflow = false;
    for (int level = 2; __ballot(left != 0u); ++level) {
        ++pulled;
        // A. hub units: 8 entries per lane, the next unit's in flight
        if (u0 < u1) {
            const global_u4 ue = (global_u4)(const void *)G.rows.units;
            auto ent_of = [&](int u) { return ue[(int64_t)u * 80 + lane]; };
            auto tgt_of = [&](int u) {
                return ((const __attribute__((address_space(1))) uint32_t *)(ue + (int64_t)u * 80 + 64))[lane];
            };
            u32x4 e = ent_of(u0);
            uint32_t t = tgt_of(u0);
            for (int u = u0; u < u1; ++u) {
                const int un = min(u + 1, u1 - 1);
                const u32x4 en = ent_of(un);
                const uint32_t tn = tgt_of(un);
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
        uint32_t cl[P];
#pragma unroll
        for (int p = 0; p < P; ++p) cl[p] = 0u;
        for (int l = tid * 4; l < n_leaf; l += KT * 4) {
            const uint2 e = ((const uint2 *)G.rows.leaf)[l >> 2];
            const uint32_t x0 = gather(e.x & 0xFFFFu), x1 = gather(e.x >> 16);
            const uint32_t x2 = gather(e.y & 0xFFFFu), x3 = gather(e.y >> 16);
            uint32_t c;
            if constexpr (PER == 1) {
                const uint32_t t0 = carry_add(cl[0], x0, x1), t1 = carry_add(cl[0], x2, x3);
                c = carry_add(cl[1], t0, t1);
            } else {
                const uint32_t t0 = carry_add(cl[0], x0 | x1 << 16, x2 | x3 << 16);
                c = cl[1] & t0;
                cl[1] ^= t0;
            }
#pragma unroll
            for (int p = 2; p < P; ++p) {
                const uint32_t d = cl[p] & c;
                cl[p] ^= c;
                c = d;
            }
        }
        // the quads, their first two rows of entries loaded one quad ahead
        u32x4 ra[2], rb[2];
        uint32_t wd[2], rx[2];
        uint32_t row = row0;
        auto issue = [&](int g) {
            const uint32_t w = codes[g];
            const uint32_t on = ((act >> g) & 1u) ? w : 0u;
            ra[g & 1] = row_of(row, on > 0u);
            rb[g & 1] = row_of(row + 1024u, on > 2u);
            wd[g & 1] = on;
            rx[g & 1] = row + 2048u;
            row += ((w + 1u) >> 1) * 1024u;
        };
        issue(0);
#pragma unroll
        for (int g = 0; g < NQ; ++g) {
            const uint32_t w = wd[g & 1], xr = rx[g & 1];
            const u32x4 a = ra[g & 1], b = rb[g & 1];
            const u32x4 c = row_of(xr, w > 4u), d = row_of(xr + 1024u, w > 6u);
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
                for (int i = 0; i < QW; ++i) all &= seen[g * QW + i];
                if (all != ~0u) {
                    if (w >= 2u) pair(a);
                    else slot(a.x, a.y);
                    if (w >= 4u) pair(b);
                    else if (w == 3u) slot(b.x, b.y);
                    if (w > 4u) {
                        if (w >= 6u) pair(c);
                        else slot(c.x, c.y);
                        if (w >= 8u) pair(d);
                        else if (w == 7u) slot(d.x, d.y);
                        if (w > 8u) {
                            // longer rows: two entries per step, the next two in flight
                            uint32_t r = xr + 2048u;
                            u32x4 z = row_of(r, true);
                            for (uint32_t k = 8u; k < w; k += 2u) {
                                r += (k + 2u < w) ? 1024u : 0u;
                                const u32x4 zn = row_of(r, true);
                                if (k + 1u < w) pair(z);
                                else slot(z.x, z.y);
                                z = zn;
                            }
                        }
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < QW; ++i) {
                const uint32_t v = (PER == 1) ? x[i] : (x[2 * i] | x[2 * i + 1] << 16);
                y[g * QW + i] = v & ~seen[g * QW + i];
            }
        }
        __syncthreads();
        // B. hub rows, then the next frontier
#pragma unroll
        for (int g = 0; g < kHubQuads; ++g) {
            if ((g * KT + wave * 64) * 4 < n_hub) {
                uint4 *const h = (uint4 *)hacc + (g * KT + tid);
                const uint4 a = *h;
                *h = make_uint4(0u, 0u, 0u, 0u);
                const uint32_t v[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
                for (int i = 0; i < QW; ++i)
                    y[g * QW + i] |= ((PER == 1) ? v[i] : (v[2 * i] | v[2 * i + 1] << 16)) & ~seen[g * QW + i];
            }
        }
        uint32_t any = 0u;
#pragma unroll
        for (int p = 0; p < P; ++p) any |= cl[p];
#pragma unroll
        for (int g = 0; g < NQ; ++g) {
            uint32_t all = ~0u;
#pragma unroll
            for (int i = 0; i < QW; ++i) {
                front[own(g) + i] = y[g * QW + i];
                seen[g * QW + i] |= y[g * QW + i];
                any |= y[g * QW + i];
                all &= seen[g * QW + i];
            }
            if (!__ballot(all != ~0u)) act &= ~(1u << g);
            if (g < kHubQuads && (g * KT + wave * 64) * 4 < n_hub) {
                // which hubs are done: bit (i, lane) of the quad's 256 positions
                uint32_t v = 0u;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t s = (PER == 1) ? seen[g * QW + i / PER] : (seen[g * QW + i / PER] >> (16 * (i % PER))) & 0xFFFFu;
                    const uint64_t o = __ballot(s == kFull);
                    if (lane == 2 * i) v = (uint32_t)o;
                    if (lane == 2 * i + 1) v = (uint32_t)(o >> 32);
                }
                if (lane < 8) hdone[(g * KT + wave * 64) / 8 + lane] = v;
            }
        }
        uint32_t *const lc = cnt[level % 3];
        if (__ballot(any != 0u)) {
            uint32_t plane[P];
            add_columns<NW, 0, P>(y, plane);
            if (n_leaf) {
                uint32_t c = 0u;
#pragma unroll
                for (int p = 0; p < P; ++p) c = carry_add(plane[p], cl[p], c);
            }
            uint32_t lo = 0u, hi = 0u;
#pragma unroll
            for (int p = P - 1; p >= 0; --p) {
                lo <<= 1;
                hi <<= 1;
                if (p < 2 || __ballot(plane[p] != 0u)) {
                    const uint32_t t = gather_columns(plane[p], roles);
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
        // the counters of the level after next: last read before this
        // level's first barrier, next added to after the next level's
        if (tid < 16) cnt[(level + 2) % 3][tid] = 0u;
        if (!__ballot(c != 0u)) break;     // nothing new: every search ended
        last = level;
        if (level > kMaxDist) {
            overflow = true;
            break;
        }
        if (wave == 0 && lane < nb && level < K) hist[level] = (int32_t)c;
        left -= c;
    }
    if (wave == 0) {
        if (lane < nb)
            for (int k = max(last, 1) + 1; k < K; ++k) hist[k] = 0;
        if (lane == 0) {
            atomicMax(&G.status[0], last);
            if (overflow) atomicOr(&G.status[1], 1);
        }
        if (G.visits) {
            // the search's work, as the levels cover it: every entry per
            // pulled level (what the skipped rows leave out included), and the
            // sources' own entries
            uint32_t deg = my_deg;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) deg += (uint32_t)__shfl_xor((int)deg, off);
            if (lane == 0) {
                const unsigned long long v =
                    (unsigned long long)pulled * (unsigned long long)G.nnz_bfs + deg;
                atomicAdd(&G.visits[0], v);
                atomicAdd(&G.visits[1], v * 4ull);
            }
        }
    }
}

}  // namespace qc
