// The counting search on a graph handle: its tables, histograms without the
// distance matrix, and the same search writing distance rows.
#include <stdlib.h>
#include <string.h>

#include <algorithm>

#include "qc_handle.h"

namespace qc {

bool can_count(qc_graph g) { return !g->weighted && !getenv("QC_BFS_SHAPE"); }

bool small_deep(qc_graph g)
{
    const int levels = g->dmax >= 0 ? g->dmax : g->dist_bound >= 0 ? g->dist_bound : kMaxDist;   // (at most)
    return g->n <= 512 && levels > std::max(24, g->n / 6);
}

bool may_have_rows(qc_graph g)
{
    // the sweeps' bound is at most twice the largest distance (and above 126
    // where it is none); nodes of one neighbour at most may need no position
    if (!g->ecc_order) return true;
    const int least = (g->dist_bound >= 0 ? g->dist_bound + 1 : kMaxDist + 2) / 2;
    int32_t n_core = 0;
    for (int32_t v = 0; v < g->n; ++v) n_core += g->row_ptr[v + 1] - g->row_ptr[v] > 1;
    return plan_rows_dist(g->n, n_core, least).rows.nq > 0;
}

// The sources in the handle's order, with what the search needs of each.
static std::vector<uint32_t> source_table(qc_graph g, const RowsState &r)
{
    std::vector<uint32_t> t;
    t.reserve(4 * (size_t)r.dev.n_search);
    const std::vector<int32_t> &rp = g->row_ptr;
    for (int32_t v : g->src_order) {
        if (r.kind[v] != kRowsCore) continue;
        t.push_back((uint32_t)v | (uint32_t)r.pos[v] << 16);
        t.push_back(r.first[v]);
        t.push_back((uint32_t)(rp[v + 1] - rp[v]) | (r.first[v + 1] - r.first[v]) << 16);
        t.push_back((uint32_t)g->comp_size[v]);
    }
    return t;
}

void free_rows(qc_graph g, RowsState &r)
{
    gfree(g, r.d_base);
    r.d_src = nullptr;
    r.d_jobs = nullptr;
    r.d_rest_jobs = nullptr;
    r.dev = RowsDev{};
    r.ready = false;
}

// Build and upload r's tables; with `dist`, those of the search that writes
// distance rows (nothing is built when no shape holds the graph).
static qc_status make_rows(qc_graph g, RowsState &r, bool dist)
{
    const std::vector<int32_t> &rp = g->row_ptr, &col = g->col;
    // With the sources in node order (QC_SOURCE_ORDER=identity, a switch for
    // measurements and tests) every node is searched.
    // So is it for the distance rows of a graph whose batches all find a CU
    // several times over: a launch for the left-out nodes' rows would wait for
    // the search (a binary tree of 1,000 nodes 36 -> 28 us, 1,000 nodes with
    // 117 leaves 25 -> 20, 2,000 with 476 29 -> 26; from 3,000 nodes on it is
    // the other way round as often). Not where most nodes are left out (a star
    // of 4,000 leaves 20 -> 24).
    const char *so = getenv("QC_SOURCE_ORDER");
    r.kind = rows_kinds(g->n, rp, col, !g->directed);
    const bool all = dist && g->n <= 2048 &&
                     2 * std::count(r.kind.begin(), r.kind.end(), (uint8_t)kRowsCore) >= g->n;
    if (all || (so && strcmp(so, "identity") == 0))
        r.kind.assign(g->n, kRowsCore);
    const int32_t n_core = (int32_t)std::count(r.kind.begin(), r.kind.end(), (uint8_t)kRowsCore);
    if (dist) {
        const RowsDistPlan p = plan_rows_dist(g->n, n_core, g->dmax);
        r.planes = p.rows.nq ? p.planes : 0;
        r.nqn = p.nqn;
        r.plan = p.rows;
        if (!r.planes) {
            r.ready = true;
            return QC_OK;
        }
    } else {
        r.plan = plan_rows(n_core);
    }
    const RowsTables t = build_rows(g->n, rp, col, g->directed, g->comp_size, r.kind, r.plan);
    r.pos = t.pos;
    r.first = t.first;
    r.dev = RowsDev{};
    r.dev.n_search = n_core;
    r.dev.n_pos = t.n_pos;
    r.dev.n_hub = t.n_hub;
    r.dev.n_leaf = t.n_leaf;
    r.dev.ent_bytes = (uint32_t)(t.ent.size() * sizeof(uint16_t));
    const std::vector<uint32_t> rest = rest_table(g->n, rp, col, r.kind, r.dev.n_rest_leaf, r.dev.n_rest_pair);
    r.dev.n_rest = (int32_t)rest.size();
    const std::vector<uint32_t> src = source_table(g, r);
    std::vector<uint16_t> node_pos;
    std::vector<uint32_t> node_flags;
    if (dist) {
        node_pos.assign((size_t)(g->n + 3) / 4 * 4, 0);
        node_flags.assign((size_t)(g->n + 15) / 16, 0u);
        for (int32_t v = 0; v < g->n; ++v) {
            const uint32_t sh = 2u * (uint32_t)(v % 16);
            if (r.kind[v] == kRowsCore) {
                node_pos[v] = t.pos[v];
            } else if (r.kind[v] == kRowsLeaf) {
                node_pos[v] = t.pos[col[rp[v]]];
                node_flags[v / 16] |= 1u << sh;
            } else {
                node_flags[v / 16] |= 2u << sh;
            }
        }
    }
    std::vector<BfsJob> jobs;
    const int bw = r.plan.batch();
    // last batch first: the source order puts the farthest-reaching sources
    // (the longest searches) at the end
    for (int s0 = (n_core + bw - 1) / bw * bw - bw; s0 >= 0; s0 -= bw) jobs.push_back(BfsJob{0, s0, 0u, 0u});
    std::vector<NodeJob> rjobs;
    for (int i = 0; i < r.dev.n_rest; i += 32) rjobs.push_back(NodeJob{0, i, 0});
    // one buffer and few copies: on a small graph each allocation and each
    // copy cost as much as the search (a 10-node graph's first distances
    // 593 us with 26 of both)
    size_t bytes = 0;
    std::vector<HostSpan> spans;
    auto place = [&](const auto &v) {
        const size_t at = bytes, size = v.size() * sizeof(v[0]);
        spans.push_back(HostSpan{(void *)at, (const void *)v.data(), size});
        bytes += (std::max<size_t>(size, 1) + 255) & ~(size_t)255;
        return at;
    };
    const size_t at_src = place(src), at_col_pos = place(t.col_pos), at_codes = place(t.codes),
                 at_wave_row = place(t.wave_row), at_wave_unit = place(t.wave_unit), at_leaf = place(t.leaf),
                 at_rest = place(rest), at_jobs = place(jobs), at_rest_jobs = place(rjobs),
                 at_node_pos = place(node_pos), at_node_flags = place(node_flags), at_units = place(t.units),
                 at_ent = place(t.ent);
    QC_TRY(galloc(g, &r.d_base, bytes));
    for (HostSpan &x : spans) x.dst = r.d_base + (size_t)x.dst;
    const qc_status s = upload_group(g, spans, true);
    if (s != QC_OK) {
        free_rows(g, r);
        return s;
    }
    r.d_src = (uint32_t *)(r.d_base + at_src);
    r.d_jobs = (BfsJob *)(r.d_base + at_jobs);
    r.d_rest_jobs = (NodeJob *)(r.d_base + at_rest_jobs);
    r.dev.src = r.d_src;
    r.dev.col_pos = (const uint16_t *)(r.d_base + at_col_pos);
    r.dev.codes = (const uint32_t *)(r.d_base + at_codes);
    r.dev.wave_row = (const uint32_t *)(r.d_base + at_wave_row);
    r.dev.wave_unit = (const uint32_t *)(r.d_base + at_wave_unit);
    r.dev.ent = r.d_base + at_ent;
    r.dev.units = r.d_base + at_units;
    r.dev.leaf = r.d_base + at_leaf;
    r.dev.rest = (const uint32_t *)(r.d_base + at_rest);
    r.dev.node_pos = (const uint16_t *)(r.d_base + at_node_pos);
    r.dev.node_flags = (const uint32_t *)(r.d_base + at_node_flags);
    r.n_jobs = (int)jobs.size();
    r.n_rest_jobs = (int)rjobs.size();
    r.ready = true;
    return QC_OK;
}

qc_status ensure_rows(qc_graph g) { return g->rows.ready ? QC_OK : make_rows(g, g->rows, false); }

qc_status ensure_dist_rows(qc_graph g) { return g->drows.ready ? QC_OK : make_rows(g, g->drows, true); }

qc_status reorder_rows(qc_graph g)
{
    for (RowsState *r : {&g->rows, &g->drows})
        if (r->ready && r->d_src) QC_TRY(upload(r->d_src, source_table(g, *r)));
    return QC_OK;
}

// The descriptor with the tables of the search about to run.
static qc_status push_rows(qc_graph g, bool dist, hipStream_t st)
{
    g->dist_desc = dist;
    return push_desc(g, st);
}

qc_status run_counts(qc_graph g, hipStream_t st)
{
    QC_TRY(ensure_rows(g));
    const bool first = g->dmax < 0;
    // rows for the bound the host sweeps gave on every distance, or for the
    // largest one an int8 distance can hold
    if (first) g->K = bins_for(g->dist_bound >= 0 ? g->dist_bound : kMaxDist);
    if (!g->d_hist || first) {
        int32_t *hist = nullptr;
        QC_TRY(galloc(g, &hist, (size_t)g->n * g->K));
        gfree(g, g->d_hist);
        g->d_hist = hist;
    }
    // (later searches of the same graph find what the first one latched)
    if (first) QC_HIP(launch_fill_i32(g->d_status, 2, 0, st));
    for (;;) {
        QC_TRY(push_rows(g, false, st));
        {
            StageTimer t(QC_STAGE_BFS, st);
            QC_HIP(launch_count(g->rows.plan.nq, g->rows.plan.threads, g->rows.plan.per, g->d_desc, g->rows.d_jobs,
                                g->rows.n_jobs, st));
        }
        {
            StageTimer t(QC_STAGE_HIST, st);
            QC_HIP(launch_hist_rest(g->K, g->d_desc, g->rows.d_rest_jobs, g->rows.n_rest_jobs,
                                    hist_waves(g->K, 0), st));
        }
        if (g->dmax >= 0) break;
        int32_t status[2];
        QC_HIP(hipMemcpyAsync(status, g->d_status, sizeof status, hipMemcpyDeviceToHost, st));
        QC_HIP(hipStreamSynchronize(st));
        if (status[1] & 1) return QC_E_OVERFLOW;
        const int K = bins_for(status[0]);
        const bool again = K != g->K;
        if (again) {
            // rows of the exact length, and the search once more into them
            int32_t *h = nullptr;
            QC_TRY(galloc(g, &h, (size_t)g->n * K));
            gfree(g, g->d_hist);
            g->d_hist = h;
            g->K = K;
        }
        g->dmax = g->dmax_bfs = status[0];
        if (!again) {
            QC_TRY(push_desc(g, st));
            break;
        }
    }
    if (first && g->ecc_order) QC_TRY(exact_source_order(g, st));
    g->have_dist = true;
    return QC_OK;
}

qc_status run_dist_rows(qc_graph g, hipStream_t st)
{
    const RowsState &r = g->drows;
    QC_TRY(push_rows(g, true, st));
    {
        StageTimer t(QC_STAGE_BFS, st);
        if (r.n_jobs > 0)
            QC_HIP((r.planes == 4 ? launch_dist_4 : r.planes == 5 ? launch_dist_5 : launch_dist_7)(
                r.plan.nq, r.nqn, g->d_desc, r.d_jobs, r.n_jobs, st));
    }
    {
        StageTimer t(QC_STAGE_HIST, st);
        QC_HIP(launch_dist_rest(g->K, g->d_desc, r.dev.n_rest, st));
    }
    g->have_dist = true;
    return QC_OK;
}

}  // namespace qc
