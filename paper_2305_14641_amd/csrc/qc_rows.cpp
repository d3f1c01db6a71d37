// Launch plan and tables of the counting search (see qc_rows.h, qc_count.h).
#include "qc_rows.h"

#include <algorithm>
#include <numeric>

#include "qc_internal.h"

namespace qc {

RowsPlan plan_rows(int32_t n_pos)
{
    // one position more than needed, which stays zero (unused entries point there)
    const int32_t need = n_pos < 65536 ? n_pos + 1 : n_pos;
    RowsPlan p;
    auto fits = [&](int nq, int threads, int per) {
        p.nq = nq;
        p.threads = threads;
        p.per = per;
        return need <= p.capacity();
    };
    if (fits(1, 1024, 1) || fits(2, 1024, 1)) return p;
    for (int nq = 5; nq <= 9; ++nq)
        if (fits(nq, 512, 1)) return p;
    for (int nq = 5; nq <= 9; ++nq)
        if (fits(nq, 1024, 1)) return p;
    for (int nq : {10, 11, 12, 14})
        if (fits(nq, 1024, 2)) return p;
    (void)fits(16, 1024, 2);
    return p;
}

RowsDistPlan plan_rows_dist(int32_t n, int32_t n_pos, int32_t dmax)
{
    RowsDistPlan d;
    d.planes = dmax <= 14 ? 4 : dmax <= 30 ? 5 : 7;
    d.rows.threads = 1024;
    // (a graph whose nodes all have positions can fill its shape: build_rows
    // then lets unused entries gather the row's own bits)
    const int32_t need = n_pos < n ? n_pos + 1 : n_pos;
    // About 16 words x 4 planes are what the registers hold: larger shapes
    // spill more than they gain (qc_dist_*.hip have the same list). What no
    // shape holds stays with the matrix search (qc_bfs.h). So do 5 planes above
    // 16,384 nodes while it takes 32 sources at a time and the row owners only
    // 16 (nodes of 3 neighbours, 5 planes, 17,000 nodes: 489 against 524 us; but
    // with 4 planes, 5 neighbours, 345 against 327; at 18,400 nodes 514 against 508,
    // and above 18,432, both at 16, 951 against 538).
    struct Shape { int nq, per; };
    static const Shape kShapes[] = {{1, 1}, {2, 1}, {3, 1}, {4, 1}, {5, 2}, {6, 2}};
    const int most = d.planes == 4 ? 6 : d.planes == 5 ? 5 : 2;
    for (const Shape &x : kShapes) {
        if (x.nq > most) break;
        if (d.planes == 5 && x.per > 1 && n <= 18200) break;
        if (need > x.nq * 4096) continue;
        for (int nqn = x.nq; nqn <= x.nq + 1; ++nqn)
            if (n <= nqn * 4096) {
                d.rows.nq = x.nq;
                d.rows.per = x.per;
                d.nqn = nqn;
                return d;
            }
    }
    return d;
}

std::vector<uint8_t> rows_kinds(int32_t n, const std::vector<int32_t> &rp,
                                const std::vector<int32_t> &col, bool leaves)
{
    std::vector<uint8_t> k(n, kRowsCore);
    if (!leaves) {
        std::vector<uint8_t> any(n, 0);
        for (int32_t c : col) any[c] = 1;
        for (int32_t v = 0; v < n; ++v)
            if (!any[v] && rp[v] == rp[v + 1]) k[v] = kRowsAlone;
        return k;
    }
    for (int32_t v = 0; v < n; ++v) {
        const int32_t d = rp[v + 1] - rp[v];
        if (d == 0) {
            k[v] = kRowsAlone;
        } else if (d == 1) {
            const int32_t u = col[rp[v]];
            k[v] = rp[u + 1] - rp[u] == 1 ? kRowsPair : kRowsLeaf;
        }
    }
    return k;
}

RowsTables build_rows(int32_t n, const std::vector<int32_t> &rp, const std::vector<int32_t> &col,
                      bool directed, const std::vector<int32_t> &comp_size,
                      const std::vector<uint8_t> &kind, const RowsPlan &plan)
{
    RowsTables t;
    t.plan = plan;
    const int waves = plan.threads / 64, nq = plan.nq;
    const int hub_cap = rows_hub_cap(plan.nq, plan.threads);
    // in-neighbours: the CSR itself when undirected, else its transpose
    std::vector<int32_t> irp, icol;
    if (directed) {
        irp.assign(n + 1, 0);
        for (int32_t c : col) ++irp[c + 1];
        for (int32_t v = 0; v < n; ++v) irp[v + 1] += irp[v];
        icol.resize(col.size());
        std::vector<int32_t> at(irp.begin(), irp.end() - 1);
        for (int32_t v = 0; v < n; ++v)
            for (int32_t e = rp[v]; e < rp[v + 1]; ++e) icol[at[col[e]]++] = v;
    }
    const std::vector<int32_t> &R = directed ? irp : rp, &C = directed ? icol : col;
    // a core node's entries: its in-neighbours that are core nodes
    std::vector<int32_t> len(n, 0);
    int32_t largest = 0, maxlen = 0, n_pos = 0;
    for (int32_t v = 0; v < n; ++v) {
        if (kind[v] != kRowsCore) continue;
        int32_t d = 0;
        for (int32_t e = R[v]; e < R[v + 1]; ++e) d += kind[C[e]] == kRowsCore;
        len[v] = d;
        ++n_pos;
        largest = std::max(largest, comp_size[v]);
        maxlen = std::max(maxlen, d);
    }
    t.n_pos = n_pos;
    std::vector<int32_t> count(maxlen + 2, 0);
    for (int32_t v = 0; v < n; ++v)
        if (kind[v] == kRowsCore) ++count[len[v]];
    // rows longer than `cut` are hub rows
    int32_t cut = 8;
    for (;; cut += 8) {
        int32_t hubs = 0;
        for (int32_t d = maxlen; d > cut; --d) hubs += count[d];
        if (hubs <= hub_cap) {
            t.n_hub = hubs;
            break;
        }
    }
    // positions: the hubs, then by decreasing number of entries, those of the
    // largest component first (counting sort)
    std::vector<int32_t> by_pos(n_pos, -1);
    t.pos.assign(n, 0);
    {
        auto key = [&](int32_t v) {   // smaller first
            if (len[v] > cut) return maxlen - len[v];
            return (comp_size[v] == largest ? 0 : maxlen + 1) + maxlen - len[v];
        };
        std::vector<int32_t> start(2 * (maxlen + 1) + 1, 0);
        for (int32_t v = 0; v < n; ++v)
            if (kind[v] == kRowsCore) ++start[key(v) + 1];
        std::partial_sum(start.begin(), start.end(), start.begin());
        for (int32_t v = 0; v < n; ++v)
            if (kind[v] == kRowsCore) {
                const int32_t p = start[key(v)]++;
                t.pos[v] = (uint16_t)p;
                by_pos[p] = v;
            }
    }
    // out-entries (the first level is pushed along them)
    t.first.assign(n + 1, 0u);
    t.col_pos.reserve(col.size());
    for (int32_t v = 0; v < n; ++v) {
        for (int32_t e = rp[v]; e < rp[v + 1]; ++e)
            if (kind[col[e]] == kRowsCore) t.col_pos.push_back(t.pos[col[e]]);
        t.first[v + 1] = (uint32_t)t.col_pos.size();
    }
    // an unused entry gathers the position past the last node, whose bits are
    // always zero, or (a graph that fills its shape) the row's own, whose
    // bits the row has seen
    const bool spare = n_pos < plan.capacity();
    const uint16_t zero_pos = (uint16_t)(spare ? n_pos : 0);

    t.codes.assign((size_t)waves * nq, 0u);
    t.wave_row.assign(waves, 0u);
    size_t rows = 0;
    for (int w = 0; w < waves; ++w) {
        t.wave_row[w] = (uint32_t)rows;
        for (int g = 0; g < nq; ++g) {
            const int32_t p0 = (g * plan.threads + w * 64) * 4;
            int32_t wd = 0;
            for (int32_t p = std::max(p0, t.n_hub); p < std::min(n_pos, p0 + 256); ++p)
                if (by_pos[p] >= 0) wd = std::max(wd, len[by_pos[p]]);
            t.codes[(size_t)w * nq + g] = (uint32_t)wd;
            rows += (size_t)(wd + 1) / 2;
        }
    }
    t.ent.assign(rows * 512, zero_pos);
    size_t row = 0;
    for (int w = 0; w < waves; ++w)
        for (int g = 0; g < nq; ++g) {
            const uint32_t wd = t.codes[(size_t)w * nq + g];
            uint16_t *const base = t.ent.data() + row * 512;
            const int32_t p0 = (g * plan.threads + w * 64) * 4;
            if (!spare)
                for (uint32_t k = 0; k < (wd + 1) / 2 * 2; ++k)
                    for (int32_t i = 0; i < 256; ++i)
                        base[(k / 2) * 512 + (i / 4) * 8 + (k % 2) * 4 + i % 4] = (uint16_t)(p0 + i);
            for (int32_t p = std::max(p0, t.n_hub); p < std::min(n_pos, p0 + 256); ++p) {
                const int32_t v = by_pos[p], i = p - p0;
                if (v < 0) continue;
                uint16_t *const mine = base + (i / 4) * 8 + i % 4;
                int32_t k = 0;
                for (int32_t e = R[v]; e < R[v + 1]; ++e)
                    if (kind[C[e]] == kRowsCore) {
                        mine[(k / 2) * 512 + (k % 2) * 4] = t.pos[C[e]];
                        ++k;
                    }
            }
            row += (wd + 1) / 2;
        }
    // hub units, longest hub first, 64 per slice; a unit's target: the hub's
    // position and the place of its bit in the done flags
    std::vector<uint16_t> ue;
    std::vector<uint32_t> ut;
    for (int32_t p = 0; p < t.n_hub; ++p) {
        const int32_t v = by_pos[p];
        int k = 0;
        for (int32_t e = R[v]; e < R[v + 1]; ++e) {
            if (kind[C[e]] != kRowsCore) continue;
            if (k % 8 == 0)
                ut.push_back((uint32_t)p | (uint32_t)((p / 256) * 256 + (p % 4) * 64 + (p % 256) / 4) << 16);
            ue.push_back(t.pos[C[e]]);
            ++k;
        }
        for (; k % 8; ++k) ue.push_back(spare ? zero_pos : (uint16_t)p);
    }
    while (ut.size() % 64) {
        for (int k = 0; k < 8; ++k) ue.push_back(zero_pos);   // (hub 0's own position without a spare)
        ut.push_back(0u);
    }
    const size_t nu = ut.size() / 64;
    t.units.resize(nu * 320);
    for (size_t u = 0; u < nu; ++u) {
        for (size_t l = 0; l < 64; ++l) {
            for (size_t k = 0; k < 4; ++k)
                t.units[u * 320 + l * 4 + k] = (uint32_t)ue[(u * 64 + l) * 8 + 2 * k] |
                                               (uint32_t)ue[(u * 64 + l) * 8 + 2 * k + 1] << 16;
            t.units[u * 320 + 256 + l] = ut[u * 64 + l];
        }
    }
    std::vector<double> load(waves, 0.0);
    for (int w = 0; w < waves; ++w)
        for (int g = 0; g < nq; ++g) load[w] += 4.0 * t.codes[(size_t)w * nq + g] + 8.0;
    std::vector<uint32_t> share(waves, 0u);
    for (size_t u = 0; u < nu; ++u) {
        const size_t w = (size_t)(std::min_element(load.begin(), load.end()) - load.begin());
        load[w] += 12.0;
        ++share[w];
    }
    t.wave_unit.assign(waves + 1, 0u);
    for (int w = 0; w < waves; ++w) t.wave_unit[w + 1] = t.wave_unit[w] + share[w];
    // leaves, in the order of their neighbours' positions
    for (int32_t p = 0; p < n_pos; ++p) {
        const int32_t v = by_pos[p];
        if (directed || v < 0 || len[v] == rp[v + 1] - rp[v]) continue;
        for (int32_t k = len[v]; k < rp[v + 1] - rp[v]; ++k) t.leaf.push_back((uint16_t)p);
    }
    while (t.leaf.size() % 4) t.leaf.push_back(zero_pos);   // (leaves leave a spare position)
    t.n_leaf = (int32_t)t.leaf.size();
    return t;
}

std::vector<uint32_t> rest_table(int32_t n, const std::vector<int32_t> &rp, const std::vector<int32_t> &col,
                                 const std::vector<uint8_t> &kind, int32_t &n_leaf, int32_t &n_pair)
{
    std::vector<uint32_t> t;
    for (const RowsKind k : {kRowsLeaf, kRowsPair, kRowsAlone}) {
        if (k == kRowsPair) n_leaf = (int32_t)t.size();
        if (k == kRowsAlone) n_pair = (int32_t)t.size() - n_leaf;
        for (int32_t v = 0; v < n; ++v)
            if (kind[v] == k) t.push_back((uint32_t)v | (k == kRowsAlone ? 0u : (uint32_t)col[rp[v]] << 16));
    }
    return t;
}

}  // namespace qc
