// Algorithm 4 in one call on a canonical undirected graph, without a handle
// and without a distance matrix (qc_onecall.cpp).
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

#include "qc_handle.h"

namespace qc {

// The host half: every table the kernels read, packed into one image with
// the descriptor, and the layout of the device memory behind it. Built
// without touching the device.
class OneCall {
  public:
    // n, rp, col: a canonical undirected CSR (validate_csr), kept by the caller
    // until run() returns; sigmas: validated. with_outputs: the labels, psi and
    // V live in this call's memory too, one after another (results()).
    OneCall(int32_t n, const std::vector<int32_t> &rp, const std::vector<int32_t> &col, const double *sigmas,
            int32_t n_sigmas, bool with_outputs, bool with_potentials);

    // Device bytes for histogram rows of `bins` (32, 64 or 128).
    size_t bytes(int bins);

    // Run on st in `base` (256-byte aligned, `limit` bytes of device memory);
    // waits for st. Outputs [n_sigmas][n], each device or null (then, with
    // `with_outputs`, in this call's memory). dmax_out (host, may be null)
    // receives the largest distance. QC_E_TOO_LARGE: the graph's largest
    // distance asks for more than `limit` (nothing usable was written).
    qc_status run(char *base, size_t limit, uint32_t tie_mode, float *psi_out, float *v_out, int32_t *labels_out,
                  hipStream_t st, int32_t *dmax_out);

    // Buffers the call carves from its memory.
    int buffers() const { return (int)parts_.size() + 5 + (with_outputs_ ? 1 : 0); }

    // Device address of the labels, followed by psi and V (with_potentials).
    char *results() const { return results_; }
    size_t results_bytes() const;

  private:
    struct Part {
        const void *src;
        size_t bytes, off;
    };
    size_t lay_out(int bins);
    void set_weights();

    int32_t n_, S_;
    int64_t nnz_;
    const double *sigmas_;
    bool with_outputs_, with_potentials_;
    RowsPlan plan_;
    RowsTables t_;
    std::vector<uint32_t> src_, rest_;
    Descent descent_;
    std::vector<BfsJob> jobs_;
    std::vector<NodeJob> node_jobs_;
    std::vector<double> w64_, inv_a_;
    std::vector<Part> parts_;
    size_t image_ = 0, total_ = 0;
    size_t hist_ = 0, psi_ = 0, v_ = 0, v64_ = 0, parent_ = 0, out_ = 0;
    int bins_ = 0, first_bins_ = 32;
    char *results_ = nullptr;
};

}  // namespace qc
