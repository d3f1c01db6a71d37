// Algorithm 4 in one call (see qc_onecall.h): one host-to-device copy of all
// tables, three launches (search; potentials with the rows it leaves out; descent
// and pointer jumping of every width, two where descends_in_lds says no), one
// 8-byte copy back.
#include "qc_onecall.h"

#include <math.h>
#include <string.h>

#include <algorithm>
#include <memory>
#include <new>

namespace qc {

namespace {

size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

// Parts of the image, in order.
enum {
    kDesc, kStatus, kRecheck, kOrder, kSellCol, kSellOff, kSellDeg, kSrc, kColPos, kCodes, kWaveRow, kWaveUnit,
    kEnt, kUnits, kLeaf, kRest, kJobs, kNodeJobs, kW64, kInvA, kParts
};

const int32_t kZero[2] = {0, 0};

}  // namespace

OneCall::OneCall(int32_t n, const std::vector<int32_t> &rp, const std::vector<int32_t> &col, const double *sigmas,
                 int32_t n_sigmas, bool with_outputs, bool with_potentials)
    : n_(n), S_(n_sigmas), nnz_((int64_t)col.size()), sigmas_(sigmas), with_outputs_(with_outputs),
      with_potentials_(with_potentials)
{
    const std::vector<uint8_t> kind = rows_kinds(n, rp, col, true);
    const int32_t n_core = (int32_t)std::count(kind.begin(), kind.end(), (uint8_t)kRowsCore);
    std::vector<int32_t> comp;
    (void)count_components(n, rp, col, &comp);
    plan_ = plan_rows(n_core);
    t_ = build_rows(n, rp, col, false, comp, kind, plan_);
    rest_.assign(n, 0u);
    for (int32_t v = 0; v < n; ++v)
        if (kind[v] == kRowsLeaf) rest_[v] = kRestLeaf << 16 | (uint32_t)col[rp[v]];
        else if (kind[v] != kRowsCore) rest_[v] = (kind[v] == kRowsPair ? kRestPair : kRestAlone) << 16;
    // The sources in the order of their positions (by decreasing number of
    // entries, which puts far-reaching sources together at the end): one
    // search does not repay the host sweeps that bound eccentricities.
    src_.resize(4 * (size_t)n_core);
    for (int32_t v = 0; v < n; ++v) {
        if (kind[v] != kRowsCore) continue;
        uint32_t *const s = &src_[4 * (size_t)t_.pos[v]];
        s[0] = (uint32_t)v | (uint32_t)t_.pos[v] << 16;
        s[1] = t_.first[v];
        s[2] = (uint32_t)(rp[v + 1] - rp[v]) | (t_.first[v + 1] - t_.first[v]) << 16;
        s[3] = (uint32_t)comp[v];
    }
    descent_ = build_descent(n, rp, col);
    // Paths, cycles, ladders and the like: a sweep of the host from a node of
    // every component costs a microsecond, a search that finds its rows too
    // short as much as the one that follows it (a path of 120 nodes: 407 us
    // for the call, 250 with the rows right at once).
    if (n <= 512 && nnz_ <= 3 * (int64_t)n) {
        std::vector<int32_t> dist(n, -1), queue(n);
        int32_t tail = 0, far = 0;
        for (int32_t v = 0, head = 0; v < n; ++v) {
            if (dist[v] >= 0) continue;
            dist[v] = 0;
            queue[tail++] = v;
            while (head < tail) {
                const int32_t u = queue[head++];
                far = std::max(far, dist[u]);
                for (int32_t e = rp[u]; e < rp[u + 1]; ++e)
                    if (dist[col[e]] < 0) {
                        dist[col[e]] = dist[u] + 1;
                        queue[tail++] = col[e];
                    }
            }
        }
        first_bins_ = bins_for(std::min(far, kMaxDist));
    }
    const int bw = plan_.batch();
    for (int s0 = (n_core + bw - 1) / bw * bw - bw; s0 >= 0; s0 -= bw) jobs_.push_back(BfsJob{0, s0, 0u, 0u});
    for (int i = 0; i < n; i += kNodesPerJob) node_jobs_.push_back(NodeJob{0, i, 0});
}

size_t OneCall::results_bytes() const { return (size_t)S_ * n_ * (with_potentials_ ? 12 : 4); }

// Offsets of everything for `bins` histogram bins.
size_t OneCall::lay_out(int bins)
{
    if (bins_ == bins) return total_;
    bins_ = bins;
    w64_.resize((size_t)S_ * bins);
    inv_a_.resize(S_);
    parts_.assign(kParts, Part{nullptr, 0, 0});
    auto part = [&](int i, const auto &v) { parts_[i] = Part{v.data(), v.size() * sizeof(v[0]), 0}; };
    parts_[kDesc] = Part{nullptr, sizeof(GraphDev), 0};   // (its contents follow from the address)
    parts_[kStatus] = Part{kZero, 8, 0};
    parts_[kRecheck] = Part{kZero, 8, 0};
    part(kOrder, descent_.order);
    part(kSellCol, descent_.col);
    part(kSellOff, descent_.off);
    part(kSellDeg, descent_.deg);
    part(kSrc, src_);
    part(kColPos, t_.col_pos);
    part(kCodes, t_.codes);
    part(kWaveRow, t_.wave_row);
    part(kWaveUnit, t_.wave_unit);
    part(kEnt, t_.ent);
    part(kUnits, t_.units);
    part(kLeaf, t_.leaf);
    part(kRest, rest_);
    part(kJobs, jobs_);
    part(kNodeJobs, node_jobs_);
    part(kW64, w64_);
    part(kInvA, inv_a_);
    size_t off = 0;
    for (Part &p : parts_) {
        p.off = off;
        off += up256(p.bytes);
    }
    image_ = off;
    const size_t N = (size_t)n_, S = (size_t)S_;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += up256(bytes);
        return at;
    };
    hist_ = take(N * bins * 4);
    psi_ = take(N * S * 4);
    v_ = take((size_t)v_floats(n_, S_) * 4);
    v64_ = take(N * S * 8);
    parent_ = take(N * S * 4);
    if (with_outputs_) out_ = take(results_bytes());
    total_ = off;
    return total_;
}

// The weight tables of the current layout: exp(-k^2 / a) by the host C
// library, as weight_tables.
void OneCall::set_weights()
{
    for (int s = 0; s < S_; ++s) {
        const double a = (2.0 * sigmas_[s]) * sigmas_[s];
        inv_a_[s] = 1.0 / a;
        for (int k = 0; k < bins_; ++k) w64_[(size_t)s * bins_ + k] = exp(-(double)(k * k) / a);
    }
}

size_t OneCall::bytes(int bins) { return lay_out(bins); }

qc_status OneCall::run(char *base, size_t limit, uint32_t tie_mode, float *psi_out, float *v_out,
                       int32_t *labels_out, hipStream_t st, int32_t *dmax_out)
{
    std::unique_ptr<char[]> image;
    // Rows of 32 bins hold all but unusually long graphs, most of which
    // first_bins_ knows where they are small; the search reports
    // the largest distance, and a longer one repeats the call with rows that
    // hold it. (The outputs are written by the run whose rows do: an error
    // finds them as they were.)
    for (int bins = first_bins_;;) {
        if (lay_out(bins) > limit) return QC_E_TOO_LARGE;
        set_weights();
        // (this layout's addresses: longer rows move everything behind them)
        int32_t *labels = labels_out;
        float *psi = psi_out, *v = v_out;
        if (with_outputs_) {
            results_ = base + out_;
            if (!labels) labels = (int32_t *)results_;
            if (with_potentials_ && !psi) psi = (float *)(results_ + (size_t)S_ * n_ * 4);
            if (with_potentials_ && !v) v = (float *)(results_ + (size_t)S_ * n_ * 8);
        }
        auto at = [&](int i) { return (void *)(base + parts_[i].off); };
        GraphDev d;
        memset(&d, 0, sizeof d);
        d.n = d.n_bfs = n_;
        d.K = bins;
        d.dmax = bins - 1;   // (bins past the largest distance are zero)
        d.n_sigmas = d.n_labels = S_;
        d.nnz = d.nnz_bfs = nnz_;
        d.order = (const int32_t *)at(kOrder);
        d.sell_col = (const uint32_t *)at(kSellCol);
        d.sell_off = (const int32_t *)at(kSellOff);
        d.sell_deg = (const int32_t *)at(kSellDeg);
        d.hist = (int32_t *)(base + hist_);
        d.psi = (float *)(base + psi_);
        d.v = (float *)(base + v_);
        d.v64 = (double *)(base + v64_);
        d.parent = (int32_t *)(base + parent_);
        d.w64 = (const double *)at(kW64);
        d.inv_a = (const double *)at(kInvA);
        d.status = (int32_t *)at(kStatus);
        d.recheck = (unsigned long long *)at(kRecheck);
        d.rows.src = at(kSrc);
        d.rows.col_pos = (const uint16_t *)at(kColPos);
        d.rows.codes = (const uint32_t *)at(kCodes);
        d.rows.wave_row = (const uint32_t *)at(kWaveRow);
        d.rows.wave_unit = (const uint32_t *)at(kWaveUnit);
        d.rows.ent = at(kEnt);
        d.rows.units = at(kUnits);
        d.rows.leaf = at(kLeaf);
        d.rows.rest = (const uint32_t *)at(kRest);
        d.rows.ent_bytes = (uint32_t)parts_[kEnt].bytes;
        d.rows.n_hub = t_.n_hub;
        d.rows.n_pos = d.rows.n_search = t_.n_pos;
        d.rows.n_leaf = t_.n_leaf;
        parts_[kDesc].src = &d;
        // (unset between the parts, which nothing reads)
        image.reset(new (std::nothrow) char[image_]);
        if (!image) return QC_E_OOM;   // (the caller has a buffer to give back)
        for (const Part &p : parts_)
            if (p.bytes) memcpy(image.get() + p.off, p.src, p.bytes);
        parts_[kDesc].src = nullptr;
        QC_HIP(hipMemcpyAsync(base, image.get(), image_, hipMemcpyHostToDevice, st));
        const GraphDev *const desc = (const GraphDev *)at(kDesc);
        const NodeJob *const nodes = (const NodeJob *)at(kNodeJobs);
        // (whatever fails from here on, `image` and the caller's memory are
        // only given up once the stream has drained)
        hipError_t e = hipSuccess;
        auto stage = [&](int id, auto launch) {
            if (e != hipSuccess) return;
            StageTimer t(id, st);
            e = launch();
        };
        stage(QC_STAGE_BFS, [&] {
            return launch_count(plan_.nq, plan_.threads, plan_.per, desc, (const BfsJob *)at(kJobs), (int)jobs_.size(), st);
        });
        stage(QC_STAGE_POTENTIAL, [&] {
            return launch_potential(QC_PREC_FP64ACC, bins, desc, nodes, (int)node_jobs_.size(), psi, v, n_, st, true);
        });
        if (descends_in_lds(n_, nnz_, descent_.max_degree, S_)) {
            stage(QC_STAGE_GGD, [&] { return launch_descend((int)tie_mode, desc, nodes, 1, 0, S_, labels, n_, n_, st); });
        } else {
            stage(QC_STAGE_GGD, [&] {
                return launch_ggd_parent((int)tie_mode, desc, nodes, (int)node_jobs_.size(), 0, S_, st);
            });
            stage(QC_STAGE_JUMP, [&] { return launch_pointer_jump(desc, nodes, 1, 0, S_, labels, n_, st); });
        }
        int32_t status[2] = {0, 0};
        if (e == hipSuccess) e = hipMemcpyAsync(status, at(kStatus), sizeof status, hipMemcpyDeviceToHost, st);
        const hipError_t sync = hipStreamSynchronize(st);
        QC_HIP(e);
        QC_HIP(sync);
        if (status[1] & 1) return QC_E_OVERFLOW;
        if (dmax_out) *dmax_out = status[0];
        if (status[0] < bins) return QC_OK;
        bins = bins_for(status[0]);
    }
}

}  // namespace qc
