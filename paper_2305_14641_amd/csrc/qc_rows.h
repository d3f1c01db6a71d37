// Host side of the counting search (qc_count.h): its launch plan and tables.
#pragma once

#include <stdint.h>

#include <vector>

namespace qc {

// Launch shape: `nq` quads of positions per thread, `threads` per workgroup,
// 1 or 2 positions per 32-bit word (batches of 32 or 16 sources).
struct RowsPlan {
    int nq = 0, threads = 0, per = 1;
    int batch() const { return 32 / per; }
    int capacity() const { return nq * threads * 4; }
};

// The shape for n_pos positions.
RowsPlan plan_rows(int32_t n_pos);

// The shape of the search that also writes the distance rows of a graph of
// n nodes, n_pos positions and largest level dmax: `planes` bit-planes of the
// level (levels up to 2^planes - 2), `nqn` quads of consecutive nodes per
// thread. rows.nq = 0: no shape holds it.
struct RowsDistPlan {
    RowsPlan rows;
    int planes = 0, nqn = 0;
};
RowsDistPlan plan_rows_dist(int32_t n, int32_t n_pos, int32_t dmax);

// What the counting search does with a node: searched from and held in LDS
// (core), or neither, its histogram following from its neighbour's (leaf:
// one neighbour, undirected) or from nothing (pair: both ends of an isolated
// edge; alone: no edges).
enum RowsKind : uint8_t { kRowsCore = 0, kRowsLeaf = 1, kRowsPair = 2, kRowsAlone = 3 };

// One kind per node of a canonical CSR. With `leaves` false (directed graphs)
// every node with an edge is a core node.
std::vector<uint8_t> rows_kinds(int32_t n, const std::vector<int32_t> &rp,
                                const std::vector<int32_t> &col, bool leaves);

struct RowsTables {
    RowsPlan plan;
    int32_t n_pos = 0, n_hub = 0, n_leaf = 0;
    std::vector<uint16_t> pos;         // [n] position of every core node (not uploaded)
    std::vector<uint32_t> first;       // [n + 1] its entries in col_pos (not uploaded)
    std::vector<uint16_t> col_pos;
    std::vector<uint32_t> codes;       // [waves * quads]
    std::vector<uint32_t> wave_row;    // [waves]
    std::vector<uint32_t> wave_unit;   // [waves + 1]
    std::vector<uint16_t> ent;         // 512 per row
    std::vector<uint32_t> units;       // 320 words per unit slice
    std::vector<uint16_t> leaf;        // n_leaf
};

// Tables of a canonical CSR (rows = out-neighbours) for the shape of its core
// nodes: positions by decreasing number of entries (the nodes of the largest
// component first), so that the 256 rows of a wavefront's quad have nearly
// equal lengths and finish together; quads dealt to the wavefronts in turn,
// hub units to the least loaded ones.
RowsTables build_rows(int32_t n, const std::vector<int32_t> &rp, const std::vector<int32_t> &col,
                      bool directed, const std::vector<int32_t> &comp_size,
                      const std::vector<uint8_t> &kind, const RowsPlan &plan);

// The nodes that are not searched: node | neighbour << 16 (0 for none),
// leaves first, then the ends of isolated edges, then the nodes without
// edges; n_leaf and n_pair receive the first two counts.
std::vector<uint32_t> rest_table(int32_t n, const std::vector<int32_t> &rp, const std::vector<int32_t> &col,
                                 const std::vector<uint8_t> &kind, int32_t &n_leaf, int32_t &n_pair);

}  // namespace qc
