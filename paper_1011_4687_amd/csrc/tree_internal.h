// Multipole tree of an environment (not part of the C ABI).
//
// Every fragment group's items (its primitive pairs and its nuclei) sit in a
// tree of cells.  A pair belongs to the smallest cell whose edge is not
// below kTreeKappa times the pair's far-field radius, so a cell's own pairs
// have radii in step with its size and a node's whole subtree is in the far
// field a few cell edges away.  A node holds the multipole moments of its
// subtree (electrons minus nuclei, FP64) about the middle of its items; a
// block of points farther from that centre than the node's accepted radius
// evaluates the node once, any other block evaluates the node's own items
// and looks at its children.
#pragma once

#include <cstdint>
#include <vector>

#include "envpot_internal.h"

namespace envpot {

// Highest order of the moments.  Pairs: with cells in step with the pairs'
// radii an accepted node lies at least about 4 of its radii away, where
// these orders reach the tolerances (mean order used 6.5 and 14.3 on the
// 200-atom ensemble; higher maxima save nothing).  Point charges have no
// radius of their own, so a higher order accepts nodes nearer by and the
// points meet fewer of them (268,398 cells, 131,072 points, FP32C: 630 nodes
// a block with 12, 310 with 16; FP64 1660 with 20, 610 with 28).
constexpr int kTreeOrd32 = 12;
constexpr int kTreeOrd64 = 20;
constexpr int kTreeOrdCells32 = 16;
constexpr int kTreeOrdCells64 = 28;
// Truncation tolerance of one node, relative to the sum of its items'
// absolute charges over the distance: a quarter of (FP32C) and half of
// (FP64) the tolerance of the Boys function's far form (2^-28, 2^-56).
// Cells (V measured against 64 bits, without / with the tree): FP32C
// 1.4e-7 / 1e-8, FP64 3.3e-14 / 3.2e-14.
constexpr double kTreeEps32 = 9.313225746154785e-10;       // 2^-30
constexpr double kTreeEps64 = 6.938893903907228e-18;       // 2^-57
constexpr double kTreeEpsCells32 = 3.725290298461914e-09;  // 2^-28
constexpr double kTreeEpsCells64 = 5.551115123125783e-17;  // 2^-54
constexpr double kTreeKappa = 0.2;
constexpr int kTreeLevels = 10;            // 3 bits of the cell code per level
// Classes of far-field radius per cell: with two, the items of the smaller
// radii are a node of their own, accepted nearer by.  200 atoms, 131,072 /
// 16,384 points: FP32C 1.43 / 0.49 ms with two, 1.69 / 0.51 with one (5000
// atoms, 200,003 points: 1.68 / 1.95); FP64, where fewer items are evaluated
// in their far form, 4.7 / 1.45 and 5.1 / 1.36, and the twice as many depths
// cost a density update 0.2 ms.
constexpr int tree_steps(bool fp64) { return fp64 ? 1 : 2; }
constexpr int kTreeTypes = kLMax + 2;      // items of a node: pairs by L, then nuclei
// Cost of one own item by type (an L = 0 pair is 4), for the shares of waves.
constexpr int kTreeW[kTreeTypes] = {4, 6, 10, 18, 30, 3};
// A subtree cheaper than this is one node; a child cheaper than a quarter of
// it joins its parent's own items (a node's evaluation costs as much as about
// 20 pairs).  Pairs: 131,072 points FP32C 1.69 ms with 600, 1.70 with 300, 1.71
// with 1500; FP64 5.06, 5.30, 5.17.  Cells: FP32C 1.04 ms with 600, 1.05 with
// 300, 1.09 with 1200; FP64, whose order 28 costs more, 3.69 ms with 600, 5.01
// with 300, 3.22 with 1200, 3.54 with 2400.
constexpr int64_t tree_min_cost(int P) { return P >= kTreeOrdCells64 ? 1200 : 600; }
// Fewer items than this are evaluated without a tree, one after the other
// (1,830 pairs: 1024 points 46 us without, 78 with).
constexpr int64_t kTreeMinItems = 8192;
constexpr int64_t kTreeMaxItems = int64_t(1) << 26;   // run costs stay below 2^31

constexpr int tree_ncoef(int P) { return (P + 1) * (P + 2) / 2; }        // (n, m >= 0)
constexpr int tree_index(int P, int n, int m) { return m * (P + 1) - m * (m - 1) / 2 + (n - m); }
constexpr int tree_thr_row(int P) { return (P + 1 + 3) & ~3; }           // floats per node
constexpr int kTreeHead = 4;                                             // doubles before the coefficients
constexpr int tree_words(int P) { return kTreeHead + 2 * tree_ncoef(P); }// doubles per node

// Points per lane of a tree evaluation of n points: two, or one where that
// leaves too few blocks (200 atoms, with one class of radius: FP32C 1.66 ms for 131,072 points with two,
// 1.78 with four, 1.82 with one; 32 points 53 us with one, 61 with two; FP64
// 1000 points 0.25 / 0.28 ms with one / two, 131,072 points 5.5 / 5.0).
constexpr int tree_np(int64_t n, bool fp64) { return n <= (fp64 ? 2048 : 512) ? 1 : 2; }
// Split factor 2^k of a tree evaluation of that many blocks: each of a
// block's workgroups tests the tree's nodes again, so the fewest that fill
// the chip and even out the blocks' different work.  Few blocks differ
// little: 4 workgroups per compute unit (1000 points FP32C: 0.14 ms with 4,
// 0.20 with 16); more blocks up to 16 (200 / 5000 atoms, 12,000 points: 0.38 /
// 0.31 ms with 32 splits, 0.38 / 0.37 with 64; 30,000: 0.61 / 0.56 with 16,
// 0.60 / 0.59 with 32), and four splits where the blocks alone fill the chip:
// their near work differs, and the last ones run alone (5000 atoms: 200,003
// points 1.63 ms with four, 1.92 with two; 400,000 2.90 / 3.30; 1,048,576 6.7 /
// 7.6, with eight 8.5).
constexpr int tree_klog(int64_t blocks, int64_t cu_count, int kmax) {
    int k = 0;
    if (blocks <= 64) {
        while (k < kmax && (blocks << k) < 4 * cu_count) ++k;
        return k;
    }
    while (k < kmax && (blocks << (k + 1)) <= 16 * cu_count) ++k;
    constexpr int least = 2;
    return k > least ? k : (least < kmax ? least : kmax);
}

// Points of one launch of a tree evaluation; more are taken piece by piece.  A
// workgroup's 256 threads stand for 64 or 128 points, so that 2^30 points would
// pass the 2^32 threads of a launch, and the partials of four splits stay
// within 1 GiB (`values` doubles per point).
constexpr int64_t tree_call_max(int values) { return (int64_t(1) << 25) / values; }

// Acceptance test of a node: centre and squared accepted radius, its own and
// its parent's (a root's parent is never accepted: +inf); cost of its own
// items.
struct TreeTest {
    double c[3], pc[3];
    float r2, pr2;
    int32_t cost, pad;
};

// A node's own items.
struct TreeNode {
    int64_t rec_off;        // first own pair record (4-byte words), pairs by L
    int32_t cnt[kLMax + 1]; // own pairs per L
    int32_t nuc_begin, nuc_end;
    int32_t cost;           // sum of kTreeW over the own items
};

// Device side of one handle's tree.
struct Tree {
    int P = 0;
    double eps = 0.0;
    bool fp64 = false;
    int32_t n_trees = 0;
    int64_t n_nodes = 0, n_pairs = 0, n_nuc = 0, rec_words = 0;
    std::vector<int32_t> level_begin;   // nodes by depth: ranges of d_by_depth
    TreeTest* d_test = nullptr;
    TreeTest* d_test_field = nullptr;   // the same for V and E (pairs only): larger radii
    float* d_thr_field = nullptr;
    TreeNode* d_node = nullptr;
    float* d_thr = nullptr;
    double* d_coef = nullptr;
    double* d_tab = nullptr;            // beta, conversion and moment tables
    int32_t* d_first = nullptr;
    uint32_t* d_rec = nullptr;
    double* d_nuc = nullptr;
    int64_t* d_word = nullptr;          // per pair (pair-list order): word of its record in d_rec
    int32_t* d_parent = nullptr;        // per node
    int32_t* d_child = nullptr;         // children lists
    int32_t* d_child_begin = nullptr;   // per node + 1
    int32_t* d_by_depth = nullptr;
    double* d_geo = nullptr;            // per node: centre, item radius, far radius, field's far radius
    void* d_chunk = nullptr;            // shares of the nodes' own items
    int32_t* d_chunk_begin = nullptr;   // per node + 1
    int64_t n_chunks = 0;
    int32_t* d_chunk_end = nullptr;     // per node: one past its subtree's chunks
    int32_t* d_depth = nullptr;         // per node
    int64_t* d_tail_begin = nullptr;    // per chunk + 1: its shares of its ancestors' bounds
    int32_t* d_tail_node = nullptr;     // per share: the ancestor
    double* d_work = nullptr;           // of a refresh: moments of chunks and nodes, radii, bounds
    uint32_t* d_sph = nullptr;          // of a refresh: the pairs' spherical moments (rec_words)
    int64_t device_bytes = 0;
    int64_t room = INT64_MAX;           // device bytes that the tree may still take
    void* owned = nullptr;              // the one allocation behind all of these
};

struct UpdPair;

// What a tree is built over, on the current device: pairs grouped by
// fragment, with their records, and nuclei (point charges), grouped alike.
struct TreeSource {
    const UpdPair* pairs = nullptr;     // n_pairs: L, group and record word of each
    int64_t n_pairs = 0;
    const int64_t* group_pairs = nullptr;  // n_groups + 1: first pair of each group
    const uint32_t* rec = nullptr;
    int32_t n_groups = 0;
    const double* cells = nullptr;      // host, n_cells x 4: x, y, z, electrons; items of group 0 after the nuclei
    int64_t n_cells = 0;
    int order = 0;                      // highest order (one of the four above) and tolerance
    double eps = 0.0;
    double nuc_eps = 0.0;               // tolerance against the nuclei's charges (FP64 in both precisions)
    bool field = false;                 // radii for the field too, from ...
    double field_ratio[kLMax + 1] = {}; // ... squared far-field radius of the field over the record's, per L
};

// Build the tree (synchronous).  nullptr with *st == ENV_OK when the input
// does not fit the tree's index widths, or the memory (ENVPOT_TREE_MAX_MB or the
// device's) the tree: the handle then evaluates every item.
// nuc: n x 4 (position, charge); nuc_begin, nuc_end: range of each group.
Tree* build_tree(const TreeSource& src, const std::vector<double>& nuc, const std::vector<int32_t>& nuc_begin,
                 const std::vector<int32_t>& nuc_end, bool fp64, env_status* st);
void free_tree(Tree* t);

// Copy the records into the tree's order and recompute every node's moments,
// coefficients and accepted radii (after the build and after each density
// fold), asynchronous on the stream.
int refresh_tree(const Tree& t, const TreeSource& src, void* stream);

TreeView tree_view(const Tree& t);
TreeView tree_view_field(const Tree& t);

struct UpdateState;
struct FieldParams;
TreeSource tree_source(const UpdateState& u, const uint32_t* d_rec, const FieldParams& fp, bool fp64);  // update.cpp

}  // namespace envpot
