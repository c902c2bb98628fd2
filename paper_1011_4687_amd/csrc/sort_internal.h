// Spatial ordering of evaluation points (sortpts.hip).  Not part of the C ABI.
#pragma once

#include <cstdint>

namespace envpot {

// Points with at least this many entries are evaluated in Morton order
// (not while the stream is being captured into a graph: the sort library
// may record memory-set nodes).
constexpr int64_t kSortMinPoints = 32768;

// With a multipole tree every call of more than one block of points is
// evaluated in a spatial order.  Where the sort above is not taken, a kernel
// that is part of a captured graph like any other orders up to kOrderSmallMax
// points (15 bits of index) by a coarser grid, and more of them in slices of
// whole blocks, each by itself (131,072 points, 200 atoms, FP32C / FP64: without
// an order 6.1 / 16.8 ms, by slices 1.64 / 5.93, sorted 1.41 / 5.11).
constexpr int64_t kOrderMin = 129;
constexpr int64_t kOrderSmallMax = 32768;
constexpr int64_t kOrderSlice = 255 * 128;
static_assert(kSortMinPoints <= kOrderSmallMax && kOrderSlice < kOrderSmallMax, "a slice fits the kernel");
// Points per slice: all of a small call, else equal slices of whole blocks.
constexpr int64_t order_slice(int64_t n) {
    if (n < kSortMinPoints) return n;
    const int64_t slices = (n + kOrderSlice - 1) / kOrderSlice;
    return ((n + slices - 1) / slices + 127) / 128 * 128;
}

// order: the spatial order of the points by that kernel, for kOrderMin <= count;
// the count is *n_dev (n_dev not null; none above n) or n.  One launch, nothing else.
int order_points(const double* points, int64_t n, const int64_t* n_dev, uint32_t* order, void* stream);

// The same for several instances (or slices of them) in one launch.
struct OrderDesc {
    const double* pts;
    uint32_t* order;
    int64_t n;      // at most kOrderSmallMax
    int64_t base;   // index of the first of them in their call
};
int order_points_multi(const OrderDesc* d, int n_desc, void* stream);

// Whether a tree evaluation that allocates orders its n points (not with
// ENVPOT_NO_SORT=1, and not from kSortMinPoints on while the stream is being
// captured), and their order: the sort from kSortMinPoints on, else the kernel.
bool sort_disabled();
bool tree_orders(int64_t n, void* stream);
int tree_order(const double* points, int64_t n, uint32_t* order, void* stream);

// True when `stream` is capturing (or its state cannot be read).
bool stream_capturing(void* stream);

// sorted[i] = points[order[i]] with order by Morton key (0.25-bohr grid);
// stream-ordered, temporary buffers from the stream's pool.  n < 2^31.
int sort_points(const double* points, int64_t n, double* sorted, uint32_t* order, void* stream);

// order alone (the evaluation reads the points through it).
int sort_order(const double* points, int64_t n, uint32_t* order, void* stream);

// out[order[i]] = v[i].
int scatter_values(const double* v, const uint32_t* order, int64_t n, double* out, void* stream);

// One instance of a multi-instance scatter: out[order[i]] = v[i], i < n.
struct ScatterDesc {
    const double* v;
    const uint32_t* order;
    double* out;
    int64_t n;
};

// The scatters of n_desc instances in one launch (grid.y = instance).
int scatter_values_multi(const ScatterDesc* d, int n_desc, int64_t max_n, void* stream);

// Rows of 4: out[4 order[i] + c] = v[4 i + c].
int scatter_rows4(const double* v, const uint32_t* order, int64_t n, double* out, void* stream);

}  // namespace envpot
