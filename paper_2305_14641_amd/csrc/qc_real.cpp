// Real edge weights (include/qc.h: qc_distances_real, qc_cluster_real):
// shortest paths per source on the GPU, then Algorithm 1 on the dense
// lengths and the descent along the graph's own edges.
#include <float.h>
#include <hip/hip_runtime.h>
#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "qc_handle.h"

using namespace qc;

namespace {

// The CSR and its weights checked for qc_distances_real: a canonical CSR,
// every weight finite and normal (>= FLT_MIN), an undirected edge's two
// entries of equal weight.
qc_status validate_real(int32_t n, int64_t nnz, const int32_t *row_ptr, const int32_t *col_idx,
                        const float *weights, uint32_t flags, std::vector<int32_t> &rp,
                        std::vector<int32_t> &col)
{
    if (flags & ~(uint32_t)QC_GRAPH_DIRECTED) return QC_E_INVAL;
    if (n < 1 || n > kSsspMaxNodes) return QC_E_INVAL;
    if (nnz > 0 && !weights) return QC_E_INVAL;
    const bool directed = (flags & QC_GRAPH_DIRECTED) != 0;
    QC_TRY(validate_csr(n, nnz, row_ptr, col_idx, false, rp, col, directed));
    for (int64_t e = 0; e < nnz; ++e)
        if (!(weights[e] >= FLT_MIN) || !std::isfinite(weights[e])) return QC_E_INVAL;
    if (!directed) {
        for (int32_t v = 0; v < n; ++v)
            for (int32_t e = rp[v]; e < rp[v + 1]; ++e) {
                const int32_t u = col[e];
                const int32_t *b = col.data() + rp[u], *f = col.data() + rp[u + 1];
                const int32_t *it = std::lower_bound(b, f, v);
                if (it == f || *it != v || weights[it - col.data()] != weights[e])
                    return QC_E_NOT_SYMMETRIC;
            }
    }
    return QC_OK;
}

// Entries of a list that one lane of the sweep takes (longer lists are cut).
constexpr int kPart = 32;

// Tables of at most so many bytes (without the out-edges) go up in one copy:
// a copy costs about as much as moving that much on the host.
constexpr size_t kOneUpload = 256 << 10;

// The search's tables (see SsspDev) of a CSR and its weights: the two large
// ones, and one image of the others.
struct SsspTables {
    std::vector<uint32_t> edges, rows;
    std::vector<char> image;
    size_t off[4];
    int32_t n_cut = 0;
    template <class V>
    void add(int i, const std::vector<V> &v)
    {
        off[i] = (image.size() + 255) & ~(size_t)255;
        image.resize(off[i] + v.size() * sizeof(V));
        if (!v.empty()) memcpy(image.data() + off[i], v.data(), v.size() * sizeof(V));
    }
};

SsspTables build_sssp(int32_t n, const std::vector<int32_t> &rp, const std::vector<int32_t> &col,
                      const float *weights, bool directed)
{
    // in-edges: the CSR itself when undirected, else its transpose
    std::vector<int32_t> irp, icol;
    std::vector<float> iw;
    if (directed) {
        irp.assign((size_t)n + 1, 0);
        for (int32_t c : col) ++irp[c + 1];
        for (int32_t v = 0; v < n; ++v) irp[v + 1] += irp[v];
        icol.resize(col.size());
        iw.resize(col.size());
        std::vector<int32_t> at(irp.begin(), irp.end() - 1);
        for (int32_t v = 0; v < n; ++v)
            for (int32_t e = rp[v]; e < rp[v + 1]; ++e) {
                iw[at[col[e]]] = weights[e];
                icol[at[col[e]]++] = v;
            }
    }
    const std::vector<int32_t> &R = directed ? irp : rp, &C = directed ? icol : col;
    const float *const W = directed ? iw.data() : weights;
    // slots by decreasing number of in-edges (counting sort)
    int32_t most = 0;
    for (int32_t v = 0; v < n; ++v) most = std::max(most, R[v + 1] - R[v]);
    std::vector<int32_t> start((size_t)most + 2, 0), node(n);
    std::vector<uint16_t> slot(n);
    for (int32_t v = 0; v < n; ++v) ++start[most - (R[v + 1] - R[v]) + 1];
    for (int32_t k = 0; k <= most; ++k) start[k + 1] += start[k];
    for (int32_t v = 0; v < n; ++v) {
        const int32_t s = start[most - (R[v + 1] - R[v])]++;
        slot[v] = (uint16_t)s;
        node[s] = v;
    }
    auto in_degree = [&](int32_t s) { return R[node[s] + 1] - R[node[s]]; };
    SsspTables t;
    while (t.n_cut < n && in_degree(t.n_cut) > kPart) ++t.n_cut;
    t.n_cut = std::min((t.n_cut + 63) / 64 * 64, (n + 63) / 64 * 64);
    // out-edges in slot order
    std::vector<int32_t> orp((size_t)n + 1, 0);
    std::vector<uint32_t> &edges = t.edges;
    edges.reserve(2 * col.size());
    for (int32_t s = 0; s < n; ++s) {
        for (int32_t e = rp[node[s]]; e < rp[node[s] + 1]; ++e) {
            edges.push_back(slot[col[e]]);
            uint32_t bits;
            memcpy(&bits, &weights[e], sizeof bits);
            edges.push_back(bits);
        }
        orp[s + 1] = (int32_t)(edges.size() / 2);
    }
    // the lists that lanes take: parts of the cut ones, then the others
    struct List {
        int32_t slot, e0, e1;
    };
    std::vector<List> lists;
    for (int32_t s = 0; s < std::min(t.n_cut, n); ++s)
        for (int32_t e = R[node[s]]; e < R[node[s] + 1]; e += kPart)
            lists.push_back(List{s, e, std::min(e + kPart, R[node[s] + 1])});
    std::stable_sort(lists.begin(), lists.end(), [](const List &x, const List &y) { return x.e1 - x.e0 > y.e1 - y.e0; });
    const int32_t n_parts = (int32_t)lists.size();
    for (int32_t s = t.n_cut; s < n; ++s) lists.push_back(List{s, R[node[s]], R[node[s] + 1]});
    // slices of 64 lists, each of one kind, dealt to the wavefront with the
    // fewest rows so far
    const int waves = sssp_waves(n);
    struct Slice {
        int32_t first, count, rows;
        bool cut;
    };
    std::vector<std::vector<Slice>> of(waves);
    std::vector<int32_t> load(waves, 0);
    auto deal = [&](int32_t from, int32_t to, bool cut) {
        for (int32_t i = from; i < to; i += 64) {
            Slice x{i, std::min(64, to - i), 0, cut};
            for (int32_t k = i; k < i + x.count; ++k) x.rows = std::max(x.rows, (lists[k].e1 - lists[k].e0 + 1) / 2);
            if (cut) ++x.rows;
            if (x.rows == 0) break;   // (no in-edges from here on)
            const int w = (int)(std::min_element(load.begin(), load.end()) - load.begin());
            of[w].push_back(x);
            load[w] += x.rows;
        }
    };
    deal(0, n_parts, true);
    deal(n_parts, (int32_t)lists.size(), false);
    std::vector<int32_t> wave_block(1, 0);
    for (int w = 0; w < waves; ++w) wave_block.push_back(wave_block[w] + (load[w] + kSsspBlockRows - 1) / kSsspBlockRows);
    std::vector<uint64_t> codes((size_t)wave_block[waves] + 1, 0u);
    std::vector<uint32_t> &rows = t.rows;
    rows.assign(((size_t)wave_block[waves] * kSsspBlockRows + 1) * 192, 0u);
    const uint32_t none = (uint32_t)n << 16 | (uint32_t)n;
    for (size_t i = 0; i < rows.size(); i += 3) rows[i] = none;
    for (int w = 0; w < waves; ++w) {
        size_t row = (size_t)wave_block[w] * kSsspBlockRows;
        for (const Slice &x : of[w]) {
            const size_t last = row + x.rows - 1;
            for (int32_t l = 0; l < x.count; ++l) {
                const List &list = lists[x.first + l];
                uint32_t *to = &rows[row * 192 + 3 * l];
                for (int32_t e = list.e0; e < list.e1; e += 2, to += 192) {
                    const bool two = e + 1 < list.e1;
                    to[0] = (uint32_t)slot[C[e]] | (two ? (uint32_t)slot[C[e + 1]] : (uint32_t)n) << 16;
                    memcpy(&to[1], &W[e], 4);
                    if (two) memcpy(&to[2], &W[e + 1], 4);
                }
                if (x.cut) rows[last * 192 + 3 * l] = (uint32_t)list.slot | (uint32_t)n << 16;
            }
            const uint32_t code = x.cut ? kSsspCut << 14 : kSsspEnd << 14 | (uint32_t)lists[x.first].slot / 64;
            codes[last / kSsspBlockRows] |= (uint64_t)code << (16 * (last % kSsspBlockRows));
            row = last + 1;
        }
    }
    t.add(0, slot);
    t.add(1, orp);
    t.add(2, codes);
    t.add(3, wave_block);
    return t;
}

// The distances into dist (stride ld), on st, from tables of the CSR and
// weights made here; waits for st before freeing them.
qc_status real_distances(int32_t n, const std::vector<int32_t> &rp, const std::vector<int32_t> &col,
                         const float *weights, bool directed, float *dist, int64_t ld, hipStream_t st)
{
    // (all host memory is taken before any device work)
    SsspTables t;
    std::vector<char> all;
    size_t rows_at = 0, edges_at = 0;
    QC_TRY(guarded([&] {
        auto whole = [](size_t bytes) { return (bytes + 255) & ~(size_t)255; };
        t = build_sssp(n, rp, col, weights, directed);
        rows_at = whole(t.image.size());
        edges_at = rows_at + whole(t.rows.size() * 4);
        if (edges_at <= kOneUpload) {
            all.resize(edges_at + t.edges.size() * 4);
            memcpy(all.data(), t.image.data(), t.image.size());
            memcpy(all.data() + rows_at, t.rows.data(), t.rows.size() * 4);
            if (!t.edges.empty()) memcpy(all.data() + edges_at, t.edges.data(), t.edges.size() * 4);
        }
        return QC_OK;
    }));
    char *base = nullptr;
    qc_status s = dalloc(&base, edges_at + t.edges.size() * 4);
    if (s == QC_OK && !all.empty()) {
        s = upload(base, all);
    } else {
        if (s == QC_OK) s = upload(base, t.image);
        if (s == QC_OK) s = upload((uint32_t *)(base + rows_at), t.rows);
        if (s == QC_OK) s = upload((uint32_t *)(base + edges_at), t.edges);
    }
    if (s == QC_OK) {
        StageTimer timer(QC_STAGE_SSSP, st);
        auto at = [&](int i) { return (const void *)(base + t.off[i]); };
        const SsspDev dev{n,
                          t.n_cut,
                          (const uint16_t *)at(0),
                          (const int32_t *)at(1),
                          (const uint2 *)(base + edges_at),
                          (const uint32_t *)(base + rows_at),
                          (const uint64_t *)at(2),
                          (const int32_t *)at(3)};
        s = from_hip(launch_sssp(dev, dist, ld, 0, n, st));
    }
    if (s == QC_OK) s = from_hip(hipStreamSynchronize(st));
    dfree(base);
    return s;
}

}  // namespace

extern "C" {

qc_status qc_distances_real(int32_t n, int64_t nnz, const int32_t *row_ptr, const int32_t *col_idx,
                            const float *weights, uint32_t flags, float *dist_out, int64_t ld,
                            void *stream)
{
    if (!dist_out || ld < n) return QC_E_INVAL;
    std::vector<int32_t> rp, col;
    QC_TRY(validate_real(n, nnz, row_ptr, col_idx, weights, flags, rp, col));
    int dev = 0;
    QC_TRY(check_device(&dev));
    return real_distances(n, rp, col, weights, (flags & QC_GRAPH_DIRECTED) != 0, dist_out, ld, as_stream(stream));
}

qc_status qc_cluster_real(int32_t n, int64_t nnz, const int32_t *row_ptr, const int32_t *col_idx,
                          const float *weights, uint32_t flags, const double *sigmas,
                          int32_t n_sigmas, uint32_t tie_mode, float *dist_out, double *psi_out,
                          double *v_out, int32_t *labels_out, void *stream)
{
    if (!labels_out || tie_mode > QC_TIE_MERGE) return QC_E_INVAL;
    QC_TRY(validate_sigmas(sigmas, n_sigmas));
    for (int32_t s = 0; s < n_sigmas; ++s)
        if (sigmas[s] < 1e-100) return QC_E_INVAL;
    std::vector<int32_t> rp, col;
    QC_TRY(validate_real(n, nnz, row_ptr, col_idx, weights, flags, rp, col));
    hipStream_t st = as_stream(stream);

    // The handle carries the descent's neighbour lists and the resident
    // potentials; its hop distances are never computed.
    qc_graph g = nullptr;
    QC_TRY(create_graph(n, nnz, row_ptr, col_idx, flags, st, nullptr, 0, &g, nullptr, false));
    float *dist = dist_out;
    double *psi = psi_out;
    qc_status s = QC_OK;
    if (!dist) s = dalloc(&dist, (size_t)n * n);
    if (s == QC_OK && !psi) s = dalloc(&psi, (size_t)n_sigmas * n);
    if (s == QC_OK) s = real_distances(n, rp, col, weights, (flags & QC_GRAPH_DIRECTED) != 0, dist, n, st);
    // Algorithm 1 on the lengths: FP64 V straight into the handle's FP64 V
    // (the values the descent re-decides near ties on), its FP32 copy in the
    // resident layout
    if (s == QC_OK) s = ensure_sigma_buffers(g, n_sigmas);
    if (s == QC_OK) {
        g->n_sigmas = n_sigmas;
        g->pot_precision = QC_PREC_FP64ACC;
        g->sigmas_loaded.clear();   // the weight tables are not this sigma list's
        s = push_desc(g, st);
    }
    if (s == QC_OK) {
        StageTimer t(QC_STAGE_DENSE, st);
        s = from_hip(launch_dense(dist, n, n, n, sigmas, n_sigmas, psi, g->d_v64, st));
    }
    if (s == QC_OK) s = from_hip(launch_v_resident(g->d_v64, n, n_sigmas, g->d_v, st));
    if (s == QC_OK && v_out)
        s = from_hip(hipMemcpyAsync(v_out, g->d_v64, sizeof(double) * n_sigmas * n,
                                    hipMemcpyDeviceToDevice, st));
    if (s == QC_OK) {
        g->have_pot = true;
        s = all_labels(g, tie_mode, labels_out, st);
    }
    const qc_status sync = from_hip(hipStreamSynchronize(st));
    if (s == QC_OK) s = sync;
    if (!dist_out) dfree(dist);
    if (!psi_out) dfree(psi);
    destroy(g, false);
    return s;
}

}  // extern "C"
