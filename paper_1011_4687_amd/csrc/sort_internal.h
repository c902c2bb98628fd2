// Spatial ordering of evaluation points (sortpts.hip).  Not part of the C ABI.
#pragma once

#include <cstdint>

namespace envpot {

// Points with at least this many entries are evaluated in Morton order
// (not while the stream is being captured into a graph: the sort library
// may record memory-set nodes).
constexpr int64_t kSortMinPoints = 32768;

// With a multipole tree, fewer points (the kernel that orders them is part
// of a captured graph like any other) are evaluated in the order of a coarser
// grid.  One block of points needs no order.
constexpr int64_t kOrderSmallMin = 129;
constexpr int64_t kOrderSmallMax = 32768;  // 15 bits of index
static_assert(kSortMinPoints <= kOrderSmallMax, "every count has one of the two orders");
constexpr bool order_small(int64_t n) { return n >= kOrderSmallMin && n < kSortMinPoints; }

// order: a spatial order of the points where order_small(count); the count is
// *n_dev (n_dev not null) or n.  One launch, nothing else.
int order_points(const double* points, int64_t n, const int64_t* n_dev, uint32_t* order, void* stream);

// The same for several instances in one launch.
struct OrderDesc {
    const double* pts;
    uint32_t* order;
    int64_t n;
};
int order_points_multi(const OrderDesc* d, int n_desc, void* stream);

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
