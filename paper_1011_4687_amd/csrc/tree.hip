// Build and refresh of the multipole tree (tree_internal.h).
//
// Build, once per handle: the cell and level of every item from its group's
// cube and its far-field radius (one thread per item); a radix sort of
// (group, cell code, level, type); the host turns the unique runs into nodes
// (a few words per run); a second, stable sort by (node, type) places every
// record.  Refresh, after each density fold: a copy of the records into the
// tree's order and the spherical form of every pair, the moments of every
// node's own items (a workgroup per 128 items), then one launch per depth from
// the leaves up, a workgroup per node (the sum with its children's moments,
// the evaluation coefficients, the shift to its parent's centre), and for all
// nodes at once the bound of the degrees beyond the order, the radii, raised
// along the ancestors, and the tests.
//
// Harmonics: R_n^m(x) = r^n P_n^m(cos) e^{i m phi} / (n+m)! without the
// Condon-Shortley phase, R_m^m = (x+iy)^m / (2^m m!),
//   R_{n+1}^m = ((2n+1) z R_n^m - r^2 R_{n-1}^m) / ((n+1)^2 - m^2),
// R_n^{-m} = (-1)^m conj R_n^m, and
//   d/dz R_n^m = R_{n-1}^m, (d/dx - i d/dy) R_n^m = R_{n-1}^{m-1},
//   (d/dx + i d/dy) R_n^m = -R_{n-1}^{m+1}.
// A pair's Hermite density acts as derivatives on 1/|r - P|, so its moments
// about c are M_n^m = sum_{k<=L} sum_j Q_k^j R_{n-k}^{m-j}(P - c) with Q the
// densities D_tuv folded through those rules; a child's moments shift by the
// same sum with k up to n.  The potential of a node at X = r - c is
//   (1/R) sum_{n,m>=0} (2 - d_m0) (n-m)! (n+m)! Re[conj(M_n^m) R_n^m(X/R^2)].
#include <hip/hip_runtime.h>

#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <new>

#include "device_math.h"
#include "tree_internal.h"
#include "update_internal.h"

namespace envpot {
namespace {

constexpr int kB = 256;

// Doubles of Tree::d_tab: recursion coefficients of the evaluation, factor
// from moment to evaluation coefficient, weight of |M|^2 in a degree's norm,
// fold of D_tuv into Q_k^j (35 components x 5 values of j, complex), factor
// of the step to R_n^m in its recursion, factor of d Q_n / dz.
constexpr int tab_beta() { return 0; }
constexpr int tab_fac(int P) { return tree_ncoef(P); }
constexpr int tab_norm(int P) { return 2 * tree_ncoef(P); }
constexpr int tab_fold(int P) { return 3 * tree_ncoef(P); }
constexpr int tab_den(int P) { return tab_fold(P) + 35 * 5 * 2; }
constexpr int tab_gamma(int P) { return tab_den(P) + tree_ncoef(P); }
constexpr int tab_words(int P) { return tab_gamma(P) + tree_ncoef(P); }
constexpr int kGeo = 6;   // doubles per node in d_geo: centre, item radius, far radius, field's far radius

__host__ __device__ inline int rec_words_of(int L, bool fp64) { return fp64 ? rec64_words(L) : rec32_words(L); }
__device__ inline int64_t gid() { return int64_t(blockIdx.x) * kB + threadIdx.x; }
unsigned grid_of(int64_t n) { return unsigned((n + kB - 1) / kB); }

// Centre and far-field radius of item i (pairs, then nuclei).
__device__ inline void item_geo(const UpdPair* pairs, const uint32_t* rec, const double* nuc, int64_t n_pairs,
                                int fp64, int64_t i, double* c, double* rf) {
    if (i < n_pairs) {
        const uint32_t* r = rec + pairs[i].word;
        const double* d = reinterpret_cast<const double*>(r);
        c[0] = d[0];
        c[1] = d[1];
        c[2] = d[2];
        *rf = sqrt(fp64 ? d[3] : double(reinterpret_cast<const float*>(r)[6])) * (1.0 + 1e-6);
    } else {
        const double* d = nuc + 4 * (i - n_pairs);
        c[0] = d[0];
        c[1] = d[1];
        c[2] = d[2];
        *rf = 0.0;
    }
}

// Doubles as unsigned integers of the same order (for atomic min and max).
__device__ inline unsigned long long ordered(double x) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__host__ __device__ inline double unordered(unsigned long long u) {
    const unsigned long long b = (u >> 63) ? (u & 0x7fffffffffffffffull) : ~u;
    double d;
    __builtin_memcpy(&d, &b, 8);
    return d;
}

// Box of each group's items (a group's by blockIdx.x, its parts by blockIdx.y).
__global__ __launch_bounds__(kB) void k_tree_boxes(const UpdPair* pairs, const uint32_t* rec, const double* nuc,
                                                   int64_t n_pairs, int fp64, const int64_t* gpb,
                                                   const int32_t* gnb, const int32_t* gne, unsigned long long* box) {
    __shared__ double red[6][kB];
    const int g = blockIdx.x, t = threadIdx.x;
    double v[6] = {HUGE_VAL, HUGE_VAL, HUGE_VAL, -HUGE_VAL, -HUGE_VAL, -HUGE_VAL};
    const int64_t np = gpb[g + 1] - gpb[g], nn = gne[g] - gnb[g];
    if (int64_t(blockIdx.y) * kB >= np + nn) return;
    for (int64_t k = int64_t(blockIdx.y) * kB + t; k < np + nn; k += int64_t(gridDim.y) * kB) {
        double c[3], rf;
        item_geo(pairs, rec, nuc, n_pairs, fp64, k < np ? gpb[g] + k : n_pairs + gnb[g] + (k - np), c, &rf);
        for (int d = 0; d < 3; ++d) {
            v[d] = fmin(v[d], c[d]);
            v[3 + d] = fmax(v[3 + d], c[d]);
        }
    }
    for (int d = 0; d < 6; ++d) red[d][t] = v[d];
    __syncthreads();
    for (int w = kB / 2; w > 0; w >>= 1) {
        if (t < w)
            for (int d = 0; d < 3; ++d) {
                red[d][t] = fmin(red[d][t], red[d][t + w]);
                red[3 + d][t] = fmax(red[3 + d][t], red[3 + d][t + w]);
            }
        __syncthreads();
    }
    if (t < 3) atomicMin(&box[6 * int64_t(g) + t], ordered(red[t][0]));
    else if (t < 6) atomicMax(&box[6 * int64_t(g) + t], ordered(red[t][0]));
}

// Cube of each group: smallest corner and edge.
__global__ __launch_bounds__(kB) void k_tree_cubes(const unsigned long long* box, int64_t n_groups, double* cube) {
    const int64_t g = gid();
    if (g >= n_groups) return;
    double e = 0.0;
    for (int d = 0; d < 3; ++d) {
        cube[4 * g + d] = unordered(box[6 * g + d]);
        e = fmax(e, unordered(box[6 * g + 3 + d]) - unordered(box[6 * g + d]));
    }
    cube[4 * g + 3] = e > 0.0 ? e * (1.0 + 1e-9) : 0.0;
}

// Boxes of n nodes or groups, empty.
__global__ __launch_bounds__(kB) void k_tree_no_boxes(int64_t n, unsigned long long* box) {
    const int64_t i = gid();
    if (i < 6 * n) box[i] = i % 6 < 3 ? ~0ull : 0ull;
}

// Sort key of every item: group (26 bits), cell code of its level left
// aligned (30), step (5), type (3): cells come out in preorder, and within a
// cell the items of larger far-field radius first.
__global__ __launch_bounds__(kB) void k_tree_keys(const UpdPair* pairs, const uint32_t* rec, const double* nuc,
                                                  const int32_t* nuc_group, int64_t n_pairs, int64_t n_items,
                                                  int fp64, const double* cube, unsigned long long* key,
                                                  uint32_t* val) {
    const int64_t i = gid();
    if (i >= n_items) return;
    double c[3], rf;
    item_geo(pairs, rec, nuc, n_pairs, fp64, i, c, &rf);
    const int g = i < n_pairs ? pairs[i].group : nuc_group[i - n_pairs];
    const int type = i < n_pairs ? pairs[i].L : kLMax + 1;
    const double* q = cube + 4 * g;
    double h = q[3];
    int level = 0;
    while (level < kTreeLevels && h > 0.0 && rf * kTreeKappa <= 0.5 * h) {
        h *= 0.5;
        ++level;
    }
    unsigned long long code = 0;
    if (level > 0) {
        const double inv = double(1 << kTreeLevels) / q[3];
        uint32_t s[3];
        for (int d = 0; d < 3; ++d) {
            const double x = (c[d] - q[d]) * inv;
            const int top = (1 << kTreeLevels) - 1;
            s[d] = x <= 0.0 ? 0u : (x >= double(top) ? uint32_t(top) : uint32_t(x));
        }
        for (int l = 0; l < level; ++l) {
            const int b = kTreeLevels - 1 - l;
            code |= (unsigned long long)((((s[0] >> b) & 1u) << 2) | (((s[1] >> b) & 1u) << 1) | ((s[2] >> b) & 1u))
                    << (3 * b);
        }
    }
    const int steps = tree_steps(fp64 != 0);
    int step = level * steps;
    if (level < kTreeLevels)
        for (int k = 1; k < steps && rf * kTreeKappa <= h * exp2(-double(k) / steps); ++k) ++step;
    key[i] = ((unsigned long long)g << 38) | (code << 8) | ((unsigned long long)step << 3) |
             (unsigned long long)type;
    val[i] = uint32_t(i);
}

// A tree of point charges alone: every key stands at the last level, finer than
// any leaf.  Its code cut to the cells that the host can meet: the children of a
// cell of `least` items or more (a cell of fewer is one node).  keys: sorted.
__global__ __launch_bounds__(kB) void k_tree_cut(const unsigned long long* __restrict__ keys, int64_t n, int steps,
                                                 int64_t least, unsigned long long* __restrict__ cut) {
    const int64_t i = gid();
    if (i >= n) return;
    const unsigned long long k = keys[i];
    int level = kTreeLevels;
    for (; level > 0; --level) {  // the parent of the cell at `level`
        const int shift = 8 + 3 * (kTreeLevels - level + 1);
        const unsigned long long lo = k >> shift << shift, hi = lo + (1ull << shift);
        int64_t a = 0, b = i;     // first key of the cell
        while (a < b) {
            const int64_t m = (a + b) >> 1;
            if (keys[m] < lo) a = m + 1;
            else b = m;
        }
        int64_t c = i, d = n;     // one past its last
        while (c < d) {
            const int64_t m = (c + d) >> 1;
            if (keys[m] < hi) c = m + 1;
            else d = m;
        }
        if (c - a >= least) break;
    }
    const int shift = 8 + 3 * (kTreeLevels - level);
    cut[i] = (k >> shift << shift) | ((unsigned long long)(level * steps) << 3) | (k & 7ull);
}

__global__ __launch_bounds__(kB) void k_tree_negate(double* nuc, int64_t n) {
    const int64_t i = gid();
    if (i < n) nuc[4 * i + 3] = -nuc[4 * i + 3];
}

__global__ __launch_bounds__(kB) void k_tree_heads(const unsigned long long* key, int64_t n, int32_t* head) {
    const int64_t i = gid();
    if (i >= n) return;
    head[i] = (i == 0 || key[i] != key[i - 1]) ? 1 : 0;
}

// runid: inclusive scan of the heads; the first item of every run.
__global__ __launch_bounds__(kB) void k_tree_runs(const unsigned long long* key, const int32_t* runid, int64_t n,
                                                  unsigned long long* rkey, uint32_t* rstart) {
    const int64_t i = gid();
    if (i >= n) return;
    if (i == 0 || key[i] != key[i - 1]) {
        rkey[runid[i] - 1] = key[i];
        rstart[runid[i] - 1] = uint32_t(i);
    }
}

__global__ __launch_bounds__(kB) void k_tree_nodekeys(const unsigned long long* key, const int32_t* runid,
                                                      const int32_t* run_node, int64_t n, uint32_t* nkey) {
    const int64_t i = gid();
    if (i >= n) return;
    nkey[i] = uint32_t(run_node[runid[i] - 1]) * kTreeTypes + uint32_t(key[i] & 7ull);
}

// Place every item: word of a pair's record, copy of a nucleus.
__global__ __launch_bounds__(kB) void k_tree_place(const uint32_t* nkey, const uint32_t* val, const uint32_t* start,
                                                   const TreeNode* node, int64_t n_pairs, int64_t n_items, int fp64,
                                                   const double* nuc, int64_t* word, double* tnuc,
                                                   int32_t* item_node) {
    const int64_t i = gid();
    if (i >= n_items) return;
    const uint32_t k = nkey[i];
    const int nd = int(k / kTreeTypes), type = int(k % kTreeTypes);
    const int64_t rank = i - int64_t(start[k]);
    const int64_t it = val[i];
    item_node[it] = nd;
    if (type <= kLMax) {
        int64_t w = node[nd].rec_off;
        for (int L = 0; L < type; ++L) w += int64_t(node[nd].cnt[L]) * rec_words_of(L, fp64 != 0);
        word[it] = w + rank * rec_words_of(type, fp64 != 0);
    } else {
        const int64_t o = node[nd].nuc_begin + rank;
        for (int d = 0; d < 4; ++d) tnuc[4 * o + d] = nuc[4 * (it - n_pairs) + d];
    }
}

// Bounding box of every node's subtree: each item climbs its ancestors to the
// root (minimum and maximum do not depend on the order).
__global__ __launch_bounds__(kB) void k_tree_bounds(const UpdPair* pairs, const uint32_t* rec, const double* nuc,
                                                    int64_t n_pairs, int64_t n_items, int fp64,
                                                    const int32_t* item_node, const int32_t* parent,
                                                    unsigned long long* box) {
    const int64_t i = gid();
    if (i >= n_items) return;
    double c[3], rf;
    item_geo(pairs, rec, nuc, n_pairs, fp64, i, c, &rf);
    for (int nd = item_node[i]; nd >= 0; nd = parent[nd])
        for (int d = 0; d < 3; ++d) {
            const unsigned long long u = ordered(c[d]);
            if (box[6 * int64_t(nd) + d] > u) atomicMin(&box[6 * int64_t(nd) + d], u);
            if (box[6 * int64_t(nd) + 3 + d] < u) atomicMax(&box[6 * int64_t(nd) + 3 + d], u);
        }
}

__global__ __launch_bounds__(kB) void k_tree_centres(const unsigned long long* box, int64_t n_nodes, double* geo,
                                                     unsigned long long* rad) {
    const int64_t i = gid();
    if (i >= n_nodes) return;
    for (int d = 0; d < 3; ++d)
        geo[kGeo * i + d] = 0.5 * (unordered(box[6 * i + d]) + unordered(box[6 * i + 3 + d]));
    rad[3 * i] = rad[3 * i + 1] = rad[3 * i + 2] = 0ull;
}

struct Ratios {
    double r[kLMax + 2];  // square roots, per type
};

// Largest |item - centre| and largest |item - centre| + far-field radius (the
// potential's and the field's).
__global__ __launch_bounds__(kB) void k_tree_radii(const UpdPair* pairs, const uint32_t* rec, const double* nuc,
                                                   int64_t n_pairs, int64_t n_items, int fp64,
                                                   const int32_t* item_node, const int32_t* parent, const double* geo,
                                                   Ratios ratios, unsigned long long* rad) {
    const int64_t i = gid();
    if (i >= n_items) return;
    double c[3], rf;
    item_geo(pairs, rec, nuc, n_pairs, fp64, i, c, &rf);
    const double rff = rf * ratios.r[i < n_pairs ? pairs[i].L : kLMax + 1];
    for (int nd = item_node[i]; nd >= 0; nd = parent[nd]) {
        const double* q = geo + kGeo * int64_t(nd);
        const double dx = c[0] - q[0], dy = c[1] - q[1], dz = c[2] - q[2];
        const double d = sqrt(dx * dx + dy * dy + dz * dz) * (1.0 + 1e-12);
        // non-negative doubles order like their bits
        const double v[3] = {d, d + rf, d + rff};
        for (int k = 0; k < 3; ++k) {
            const unsigned long long b = (unsigned long long)__double_as_longlong(v[k]);
            if (rad[3 * int64_t(nd) + k] < b) atomicMax(&rad[3 * int64_t(nd) + k], b);
        }
    }
}

__global__ __launch_bounds__(kB) void k_tree_radii_out(const unsigned long long* rad, int64_t n_nodes, double* geo) {
    const int64_t i = gid();
    if (i >= n_nodes) return;
    for (int k = 0; k < 3; ++k) geo[kGeo * i + 3 + k] = __longlong_as_double((long long)rad[3 * i + k]);
}

// ---------------------------------------------------------------- refresh

// One thread per pair and 8-byte word of the largest record would leave most
// idle; a quarter wave per pair copies its record.
__global__ __launch_bounds__(kB) void k_tree_copy(const UpdPair* pairs, const int64_t* word, int64_t n_pairs,
                                                  int fp64, const uint32_t* rec, uint32_t* trec) {
    const int64_t i = int64_t(blockIdx.x) * (kB / 16) + (threadIdx.x >> 4);
    if (i >= n_pairs) return;
    const int lane = threadIdx.x & 15;
    const UpdPair q = pairs[i];
    const int nw = rec_words_of(q.L, fp64 != 0) / 2;
    const uint64_t* s = reinterpret_cast<const uint64_t*>(rec + q.word);
    uint64_t* d = reinterpret_cast<uint64_t*>(trec + word[i]);
    for (int k = lane; k < nw; k += 16) d[k] = s[k];
}

// A share of one node's own items (in their order: pairs by L, then nuclei).
struct Chunk {
    int32_t node, begin, end;
};

struct MomentArgs {
    const Chunk* chunk;          // chunks in node order
    const int32_t* chunk_begin;  // per node + 1
    const int32_t* chunk_end;    // per node: one past its subtree's chunks (preorder: they follow one another)
    const int32_t* depth;        // per node
    const int64_t* tail_begin;   // per chunk + 1: its entries in tail, one per ancestor from the root on
    const int32_t* tail_node;    // per entry: the ancestor
    const int32_t* by_depth;     // the nodes of this launch
    const TreeNode* node;
    const uint32_t* rec;
    const uint32_t* sph;         // spherical form of every pair, at its record's place
    const double* nuc;
    const int32_t* child;
    const int32_t* child_begin;
    const int32_t* parent;
    const double* geo;
    const double* tab;
    double* part;                // per chunk: moments about the node's centre, absolute charge
    double* up;                  // per node: its moments about its parent's centre, absolute charge
    double* mom;                 // per node: its moments, absolute charge
    double* tail;                // per entry: the chunk's share of the ancestor's A_k (k_tree_tails)
    unsigned long long* own;     // per node, potential and field: bits of the radius its moments ask for
    unsigned long long* radius;  // the same, with its descendants'
    double* coef;
    float* thr;
    float* thr_field;            // or nullptr
    double eps;
    double nuc_size;             // what a unit of nuclear charge adds to the absolute charge
};

struct alignas(16) Cplx {
    double r, i;
};

constexpr int kChunk = 128;      // items per chunk
constexpr int part_words(int P) { return 2 * tree_ncoef(P) + 2; }

// Scale of a node's moments (by s^-n): no power of a coordinate overflows.
__device__ __forceinline__ double node_scale(const double* geo) {
    const double s = fmax(geo[3], 0.1 * geo[4]);
    return s > 0.0 ? s : 1.0;
}

constexpr int full_index(int n, int m) { return n * n + n + m; }

// R_n^m(x) of one x, by the thread of order m >= 0, to put(n, R).
template <int P, typename Put>
__device__ __forceinline__ void harmonics(double x, double y, double z, int m, const double* den, Put put) {
    double cr = 1.0, ci = 0.0;
    for (int k = 1; k <= m; ++k) {
        const double f = den[tree_index(P, k, k)], nr = (cr * x - ci * y) * f;
        ci = (cr * y + ci * x) * f;
        cr = nr;
    }
    const double r2 = x * x + y * y + z * z;
    Cplx a{0.0, 0.0}, b{cr, ci};  // R_{n-1}, R_n
    const int at = tree_index(P, m, m);
    for (int n = m;; ++n) {
        put(n, b);
        if (n == P) break;
        const double f = den[at + n + 1 - m], u = (2 * n + 1) * z;
        const Cplx c{(u * b.r - r2 * a.r) * f, (u * b.i - r2 * a.i) * f};
        a = b;
        b = c;
    }
}
// R_n^{-m} = (-1)^m conj R_n^m.
__device__ __forceinline__ Cplx mirrored(int m, const Cplx& v) {
    return (m & 1) ? Cplx{-v.r, v.i} : Cplx{v.r, -v.i};
}

// Index of Hermite component (a, b, c) among those of order up to L.
__host__ __device__ constexpr int comp_index(int L, int a, int b, int c) {
    const int m = L - a;
    // components with a smaller first exponent, then with a smaller second
    const int first = (L + 1) * (L + 2) * (L + 3) / 6 - (m + 1) * (m + 2) * (m + 3) / 6;
    return first + b * (m + 1) - b * (b - 1) / 2 + c;
}

// (n, m) of coefficient t.
template <int P>
__device__ __forceinline__ void coef_nm(int t, int& n, int& m) {
    m = 0;
    while (m <= P && t >= P + 1 - m) {
        t -= P + 1 - m;
        ++m;
    }
    n = m + t;
}

// Spherical form of a pair: Q_k^j (k <= L, 0 <= j <= k) from its Hermite
// components, the sum of their sizes against 1/R where its far field begins,
// and the norms of its orders 1 .. L (order 0 has one component), at the
// pair's own place in q (a record holds as many words).
constexpr int q_index(int k, int j) { return k * (k + 1) / 2 + j; }
constexpr int q_size(int L) { return 2 * q_index(L, L) + 2; }
constexpr int q_norm(int L, int k) { return q_size(L) + k; }

// Weight of |Q_k^j|^2 (j and -j together) in the squared norm of order k.
constexpr double norm_weight(int k, int j) {
    double f = j ? 2.0 : 1.0;
    for (int i = 2; i <= k - j; ++i) f *= i;
    for (int i = 2; i <= k + j; ++i) f *= i;
    return f;
}

template <int L, bool F64>
__device__ __forceinline__ void pair_moments(const uint32_t* r, const double* __restrict__ fold, double* q) {
    constexpr int nc = kNComp[L];
    static_assert(q_norm(L, L) < (F64 ? rec64_words(L) : rec32_words(L)) / 2, "fits a record");
    const double* d = reinterpret_cast<const double*>(r);
    const float* f = reinterpret_cast<const float*>(r);
    const double ir = rsqrt(F64 ? d[3] : double(f[6]));
    double size = 0.0, scale = 1.0;
#pragma unroll
    for (int k = 0; k <= L; ++k) {
        Cplx o[kLMax + 1] = {};
        double part = 0.0;
#pragma unroll
        for (int a = 0; a <= k; ++a)
#pragma unroll
            for (int b = 0; b <= k - a; ++b) {
                const int c = k - a - b, at = comp_index(L, a, b, c), row = 10 * comp_index(kLMax, a, b, c);
                const double D = F64 ? d[kRec64Head + nc + at] : double(f[kRec32Head + nc + at]);
                part += fabs(D);
#pragma unroll
                for (int j = 0; j <= k; ++j) {
                    o[j].r = fma(D, fold[row + 2 * j], o[j].r);
                    o[j].i = fma(D, fold[row + 2 * j + 1], o[j].i);
                }
            }
        double norm = 0.0;
#pragma unroll
        for (int j = 0; j <= k; ++j) {
            q[2 * q_index(k, j)] = o[j].r;
            q[2 * q_index(k, j) + 1] = o[j].i;
            norm = fma(norm_weight(k, j), fma(o[j].r, o[j].r, o[j].i * o[j].i), norm);
        }
        if (k > 0) q[q_norm(L, k)] = sqrt(norm);
        size = fma(part, scale, size);
        scale *= ir;
    }
    q[q_size(L)] = size;
}

template <bool F64>
__global__ __launch_bounds__(kB) void k_tree_spherical(const UpdPair* pairs, const int64_t* word, int64_t n_pairs,
                                                       const uint32_t* __restrict__ rec,
                                                       const double* __restrict__ fold, uint32_t* __restrict__ out) {
    const int64_t i = gid();
    if (i >= n_pairs) return;
    const UpdPair p = pairs[i];
    const uint32_t* r = rec + p.word;
    double* q = reinterpret_cast<double*>(out + word[i]);
    switch (p.L) {
        case 0: pair_moments<0, F64>(r, fold, q); break;
        case 1: pair_moments<1, F64>(r, fold, q); break;
        case 2: pair_moments<2, F64>(r, fold, q); break;
        case 3: pair_moments<3, F64>(r, fold, q); break;
        default: pair_moments<4, F64>(r, fold, q); break;
    }
}

// Harmonics of one item in LDS: rows n = -4 .. P, columns m = -4 .. P + 4,
// zero where |m| > n, so that a shift by any (k, j) reads without a test.
constexpr int kPad = kLMax;
constexpr int pad_cols(int P) { return P + 1 + 2 * kPad; }
constexpr int pad_size(int P) { return (P + 1 + kPad) * pad_cols(P); }
constexpr int pad_index(int P, int n, int m) { return (n + kPad) * pad_cols(P) + m + kPad; }
// Items a wave takes at once: a lane per item and order, as LDS allows two
// waves per SIMD or more.
constexpr int p2m_items(int P) { return P <= 16 ? 2 : 1; }

__device__ __forceinline__ double lane_value(double v, int lane) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), lane);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// acc(n, m) += sum_j Q_K^j R_{n-K}^{m-j} of one item, whose Q_k^j lane
// q0 + q_index(k, j) holds; at[c] is where (n, m) of the lane's coefficient c
// stands in R.
template <int P, int K, int NT>
__device__ __forceinline__ void shift_order(const Cplx& q, int q0, const Cplx* R, const int (&at)[NT], Cplx (&acc)[NT]) {
#pragma unroll
    for (int j = -K; j <= K; ++j) {
        Cplx v{lane_value(q.r, q0 + q_index(K, j < 0 ? -j : j)), lane_value(q.i, q0 + q_index(K, j < 0 ? -j : j))};
        if (j < 0) v = mirrored(-j, v);
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            const Cplx r = R[at[c] - K * pad_cols(P) - j];
            acc[c].r = fma(v.r, r.r, fma(-v.i, r.i, acc[c].r));
            acc[c].i = fma(v.r, r.i, fma(v.i, r.r, acc[c].i));
        }
    }
}

// Moments of one chunk of own items about their node's centre, a workgroup
// per chunk.  Every wave takes some items at once: a lane per item and order
// forms the harmonics in LDS, then every lane adds each item's shifts to its
// coefficients, the harmonics from LDS and the item's Q from the lanes that
// loaded it.  Bound by the FP64 instructions (770 per item and wave at order
// 20, half of them the harmonics with two thirds of the lanes idle) and their
// chain; the loads of the next items are under way meanwhile.  375,461 pairs:
// FP64 1.14 -> 0.94 ms, FP32C 0.56 -> 0.33 (9 million 9.6 -> 7.1); as many
// items at once as there are lanes left one wave per SIMD: 1.11 and 0.70.
template <int P>
__global__ __launch_bounds__(kB) void k_tree_p2m(MomentArgs A, int fp64) {
    constexpr int NC = tree_ncoef(P);
    constexpr int NT = (NC + 63) / 64;  // coefficients of a lane: lane, lane + 64, ...
    constexpr int G = p2m_items(P);
    constexpr int kQ = q_index(kLMax, kLMax) + 1;
    static_assert(G >= 1 && G * kQ <= 64, "a lane per item and Q");
    static_assert(4 * NC <= 4 * G * pad_size(P), "the waves' sums fit the harmonics");
    __shared__ Cplx R[4 * G * pad_size(P)];
    __shared__ double qabs[4];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    for (int k = t; k < 4 * G * pad_size(P); k += kB) R[k] = Cplx{0.0, 0.0};
    const Chunk ck = A.chunk[blockIdx.x];
    const double* geo = A.geo + kGeo * int64_t(ck.node);
    const double g0 = geo[0], g1 = geo[1], g2 = geo[2], inv = 1.0 / node_scale(geo);
    const TreeNode& node = A.node[ck.node];
    // this lane's Q (item lane / 15 of the wave's) and harmonic order
    const int qi = lane / kQ, hi = lane / (P + 1), hm = lane % (P + 1);
    int qk = 0, qj = lane % kQ;
    while (qj > qk) qj -= ++qk;
    double qs = 1.0;  // s^-k
    for (int k = 0; k < qk; ++k) qs *= inv;
    struct Items {          // as loaded: nothing waits for them here
        int L;              // of item `lane`; -1: none
        Cplx q;
        double x, y, z, size;
    };
    auto load = [&](int first) -> Items {
        Items v;
        int i = first + lane, L = 0;
        int64_t w = node.rec_off;
#pragma unroll
        for (int l = 0; l <= kLMax; ++l) {
            const int c = node.cnt[l];
            if (L == l && i >= c) {
                i -= c;
                w += int64_t(c) * rec_words_of(l, fp64 != 0);
                ++L;
            }
        }
        v.L = lane < G && first + lane < ck.end ? L : -1;
        w = L <= kLMax ? w + int64_t(i) * rec_words_of(L, fp64 != 0) : int64_t(node.nuc_begin + i);
        const int qL = __shfl(v.L, qi < G ? qi : 0), hL = __shfl(v.L, hi < G ? hi : 0);
        const int64_t qw = __shfl(w, qi < G ? qi : 0), hw = __shfl(w, hi < G ? hi : 0);
        v.q = Cplx{0.0, 0.0};
        v.size = 0.0;
        if (qi < G && qL >= 0) {
            if (qL > kLMax) {
                if (qk == 0) v.q.r = -A.nuc[4 * qw + 3];
            } else if (qk <= qL) {
                const double* q = reinterpret_cast<const double*>(A.sph + qw);
                v.q.r = q[2 * q_index(qk, qj)];
                v.q.i = q[2 * q_index(qk, qj) + 1];
                if (qk == 0) v.size = q[q_size(qL)];
            }
        }
        v.x = v.y = v.z = 0.0;
        if (hi < G && hL >= 0) {
            const double* d = hL <= kLMax ? reinterpret_cast<const double*>(A.rec + hw) : A.nuc + 4 * hw;
            v.x = d[0];
            v.y = d[1];
            v.z = d[2];
        }
        return v;
    };
    // the factor of each step for the lane's order
    double step[P];
#pragma unroll
    for (int n = 0; n < P; ++n)
        step[n] = A.tab[tab_den(P) + (n < hm ? tree_index(P, n + 1, n + 1) : tree_index(P, n + 1, min(hm, n)))];
    int at[NT];
    Cplx acc[NT];
#pragma unroll
    for (int c = 0; c < NT; ++c) {
        int n = 0, m = 0;
        if (lane + 64 * c < NC) coef_nm<P>(lane + 64 * c, n, m);
        at[c] = pad_index(P, n, m);
        acc[c] = Cplx{0.0, 0.0};
    }
    double qa = 0.0;
    Cplx* mine = R + wave * (G * pad_size(P));
    Items v{};
    int first = ck.begin + wave * G;
    if (first < ck.end) v = load(first);
    __syncthreads();
    for (; first < ck.end; first += 4 * G) {
        Items next{};
        if (first + 4 * G < ck.end) next = load(first + 4 * G);
        if (hi < G) {
            // R_n^m by steps of n alike in all lanes: the power of x + iy up to
            // n = m, then the recurrence in n
            const double x = (v.x - g0) * inv, y = (v.y - g1) * inv, z = (v.z - g2) * inv;
            const double r2 = x * x + y * y + z * z;
            Cplx* T = mine + hi * pad_size(P) + pad_index(P, 0, hm);
            Cplx a{0.0, 0.0}, b{1.0, 0.0};
#pragma unroll
            for (int n = 0; n <= P; ++n) {
                if (n >= hm) {
                    T[n * pad_cols(P)] = b;
                    if (hm > 0 && hm <= kPad) T[n * pad_cols(P) - 2 * hm] = mirrored(hm, b);
                }
                if (n == P) break;
                const bool up = n < hm;
                const double u = up ? x : (2 * n + 1) * z;
                const double w = up ? y : r2;
                // up: (x + iy) b; else (2n + 1) z b - r^2 a
                const Cplx c{u * b.r - w * (up ? b.i : a.r), u * b.i + w * (up ? b.r : -a.i)};
                if (!up) a = b;
                b.r = c.r * step[n];
                b.i = c.i * step[n];
            }
        }
        // (a nucleus's size comes from its charge)
        const int own = __shfl(v.L, qi < G ? qi : 0);
        qa += own > kLMax ? fabs(v.q.r) * A.nuc_size : v.size;
        v.q.r *= qs;
        v.q.i *= qs;
        wave_sync();
#pragma unroll 1
        for (int it = 0; it < G; ++it) {
            const int L = __builtin_amdgcn_readlane(v.L, it), q0 = it * kQ;
            if (L < 0) break;
            const Cplx* T = mine + it * pad_size(P);
            shift_order<P, 0>(v.q, q0, T, at, acc);
            if (L > kLMax) continue;  // a nucleus
            if (L >= 1) shift_order<P, 1>(v.q, q0, T, at, acc);
            if (L >= 2) shift_order<P, 2>(v.q, q0, T, at, acc);
            if (L >= 3) shift_order<P, 3>(v.q, q0, T, at, acc);
            if (L >= 4) shift_order<P, 4>(v.q, q0, T, at, acc);
        }
        wave_sync();
        v = next;
    }
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) qa += __shfl_xor(qa, w);
    // the waves' sums in wave order
    __syncthreads();
#pragma unroll
    for (int c = 0; c < NT; ++c)
        if (lane + 64 * c < NC) R[wave * NC + lane + 64 * c] = acc[c];
    if (lane == 0) qabs[wave] = qa;
    __syncthreads();
    double* o = A.part + int64_t(part_words(P)) * blockIdx.x;
    for (int k = t; k < NC; k += kB) {
        const Cplx a = R[k], b = R[NC + k], c = R[2 * NC + k], d = R[3 * NC + k];
        o[2 * k] = (a.r + b.r) + (c.r + d.r);
        o[2 * k + 1] = (a.i + b.i) + (c.i + d.i);
    }
    if (t == 0) o[2 * NC] = (qabs[0] + qabs[1]) + (qabs[2] + qabs[3]);
}

constexpr int node_threads(int P) { return tree_ncoef(P) < kB ? kB : 2 * kB; }

// One node of a depth: the sum of its chunks' moments and of its children's
// shifted ones (fixed order), kept for the radii, its evaluation
// coefficients, and its moments shifted to its parent's centre.  A workgroup
// per node; a depth has few, so this is bound by the latency of one shift
// (up to 231 terms in a thread): only what the next depth waits for is here
// (200 atoms, per depth: FP64 70 -> 28 us, FP32C 50 -> 14, the radii after it
// 45 us for all nodes at once).
template <int P>
__global__ __launch_bounds__(node_threads(P)) void k_tree_nodes(MomentArgs A) {
    constexpr int NC = tree_ncoef(P), NF = (P + 1) * (P + 1);
    static_assert(NC < node_threads(P), "one thread per coefficient and one for the charge");
    __shared__ Cplx Q[NF];
    __shared__ Cplx R[NF];
    __shared__ double den[NC];
    const int t = threadIdx.x;
    const int nd = A.by_depth[blockIdx.x], par = A.parent[nd];
    const double* geo = A.geo + kGeo * int64_t(nd);
    const double s = node_scale(geo);
    const int w = t < NC ? 2 * t : 2 * NC;  // every thread past the coefficients adds up the charge
    if (t < NC) den[t] = A.tab[tab_den(P) + t];
    int n, m;
    coef_nm<P>(t, n, m);
    double inv = 0.0, x[3] = {0.0, 0.0, 0.0};
    if (par >= 0) {
        const double* pg = A.geo + kGeo * int64_t(par);
        inv = 1.0 / node_scale(pg);
        for (int d = 0; d < 3; ++d) x[d] = (geo[d] - pg[d]) * inv;
    }
    Cplx acc{0.0, 0.0};
#pragma unroll 4
    for (int c = A.chunk_begin[nd]; c < A.chunk_begin[nd + 1]; ++c) {
        const double* q = A.part + int64_t(part_words(P)) * c + w;
        acc.r += q[0];
        acc.i += q[1];
    }
#pragma unroll 4
    for (int c = A.child_begin[nd]; c < A.child_begin[nd + 1]; ++c) {
        const double* q = A.up + int64_t(part_words(P)) * A.child[c] + w;
        acc.r += q[0];
        acc.i += q[1];
    }
    double* mo = A.mom + int64_t(part_words(P)) * nd;
    if (t < NC) {
        mo[2 * t] = acc.r;
        mo[2 * t + 1] = acc.i;
        double* co = A.coef + int64_t(tree_words(P)) * nd + kTreeHead;
        const double f = A.tab[tab_fac(P) + t];
        co[2 * t] = acc.r * f;
        co[2 * t + 1] = acc.i * f;
    }
    if (t == NC) {
        mo[2 * NC] = acc.r;
        double* co = A.coef + int64_t(tree_words(P)) * nd;
        for (int d = 0; d < 3; ++d) co[d] = geo[d];
        co[3] = s;
    }
    if (par < 0) return;
    if (t < NC) {
        const double ratio = s * inv;
        double f = 1.0;
        for (int k = 0; k < n; ++k) f *= ratio;
        const Cplx q{acc.r * f, acc.i * f};
        Q[full_index(n, m)] = q;
        if (m > 0) Q[full_index(n, -m)] = mirrored(m, q);
    }
    __syncthreads();
    if (t <= P)
        harmonics<P>(x[0], x[1], x[2], t, den, [&](int k, const Cplx& v) {
            R[full_index(k, t)] = v;
            if (t > 0) R[full_index(k, -t)] = mirrored(t, v);
        });
    __syncthreads();
    double* o = A.up + int64_t(part_words(P)) * nd;
    if (t < NC) {
        Cplx u{0.0, 0.0};
        for (int k = 0; k <= n; ++k) {
            const int nn = n - k, j0 = max(-k, m - nn), j1 = min(k, m + nn);  // |m - j| <= n - k
            const Cplx* q = Q + full_index(k, j0);
            const Cplx* r = R + full_index(nn, m - j0);
#pragma unroll 4
            for (int j = j0; j <= j1; ++j, ++q, --r) {
                u.r = fma(q->r, r->r, fma(-q->i, r->i, u.r));
                u.i = fma(q->r, r->i, fma(q->i, r->r, u.i));
            }
        }
        o[2 * t] = u.r;
        o[2 * t + 1] = u.i;
    }
    if (t == NC) o[2 * NC] = acc.r;
}

// Sums that bound a node's degrees beyond P.  A source of order k and norm q
// at distance rho from the centre has, in degree n, a norm of at most
// C(n, k) q rho^(n-k) (attained along its axis), so with s the node's scale,
// a s the radius of its items and
//   A_k = sum q_k s^-k (rho / s)^(P+1-k)
// over all items of the subtree, B_n <= sum_k A_k C(n, k) a^(n-P-1) for n > P,
// whatever cancels in the degrees up to P (charges on the points of a
// quadrature of the sphere have none between 0 and its own).  Formed from the
// items of the subtree themselves: from the children's sums, by the distance of
// the centres, the radii would grow by up to a half.  A workgroup per chunk
// loads its items once; eight lanes per ancestor add up an eighth of them each
// (375,461 pairs, FP32C / FP64, 18 / 9 depths: 23 / 24 us; an item per thread and
// a sum over the workgroup per ancestor 97 / 54).
template <int P>
__global__ __launch_bounds__(kChunk) void k_tree_tails(MomentArgs A, int fp64) {
    __shared__ double item[3 + kLMax + 1][kChunk];  // position, norms
    const Chunk ck = A.chunk[blockIdx.x];
    const TreeNode& node = A.node[ck.node];
    const int n_items = ck.end - ck.begin;
    if (int(threadIdx.x) < n_items) {
        int i = ck.begin + threadIdx.x, L = 0;
        int64_t w = node.rec_off;
        while (L <= kLMax && i >= node.cnt[L]) {
            i -= node.cnt[L];
            w += int64_t(node.cnt[L]) * rec_words_of(L, fp64 != 0);
            ++L;
        }
        const double *d, *q;
        if (L <= kLMax) {
            w += int64_t(i) * rec_words_of(L, fp64 != 0);
            d = reinterpret_cast<const double*>(A.rec + w);
            q = reinterpret_cast<const double*>(A.sph + w);
        } else {
            d = A.nuc + 4 * int64_t(node.nuc_begin + i);
            q = d + 3;
            L = 0;
        }
        for (int c = 0; c < 3; ++c) item[c][threadIdx.x] = d[c];
        item[3][threadIdx.x] = fabs(q[0]);
#pragma unroll
        for (int k = 1; k <= kLMax; ++k) item[3 + k][threadIdx.x] = k <= L ? q[q_norm(L, k)] : 0.0;
    }
    __syncthreads();
    const int g = threadIdx.x & 7;
    for (int64_t e = A.tail_begin[blockIdx.x] + (threadIdx.x >> 3); e < A.tail_begin[blockIdx.x + 1]; e += kChunk / 8) {
        const double* geo = A.geo + kGeo * int64_t(A.tail_node[e]);
        const double g0 = geo[0], g1 = geo[1], g2 = geo[2], inv = 1.0 / node_scale(geo);
        double acc[kLMax + 1] = {};
        for (int i = g; i < n_items; i += 8) {
            const double x = (item[0][i] - g0) * inv, y = (item[1][i] - g1) * inv, z = (item[2][i] - g2) * inv;
            // (from above: the instruction's relative error is below 2^-22)
            const double rho2 = fma(x, x, fma(y, y, z * z)),
                         rho = rho2 > 0.0 ? rho2 * __builtin_amdgcn_rsq(rho2) * (1.0 + 1e-6) : 0.0;
            double pw = (P + 1 - kLMax) % 2 ? rho : 1.0;  // rho^(P+1-k)
#pragma unroll
            for (int n = 0; n < (P + 1 - kLMax) / 2; ++n) pw *= rho2;
#pragma unroll
            for (int k = kLMax; k >= 0; --k) {
                acc[k] = fma(item[3 + k][i], pw, acc[k]);
                pw *= rho;
            }
        }
        double sk = 1.0;  // s^-k
#pragma unroll
        for (int k = 0; k <= kLMax; ++k) {
            acc[k] *= sk;
            sk *= inv;
#pragma unroll
            for (int o = 1; o < 8; o <<= 1) acc[k] += __shfl_xor(acc[k], o);
            if (g == 0) A.tail[(kLMax + 1) * e + k] = acc[k];
        }
    }
}

constexpr double binomial(int n, int k) {
    double c = 1.0;
    for (int i = 1; i <= k; ++i) c = c * (n - k + i) / i;
    return c;
}

// Radii of every node from its moments, one wave per node: row[p] is
// the smallest radius (at least the far-field radius and outside the items)
// from which the degrees above p stay below eps |charge|/R,
//   sum_{P>=n>p} w_n B_n x^n + sum_{n>P} w_n x^n sum_k A_k C(n, k) a^(n-P-1)
//     <= eps |charge|, x = s/R,
// with B_n the norm of degree n (no value of its potential times R^(n+1)
// is larger), w_n = 1, for the gradient (against |charge|/R^2) n + 1 (along a
// great circle a degree is a trigonometric polynomial f of degree n, so
// f'^2 + n^2 f^2 <= n^2 B_n^2, and the radial derivative is (n+1) f), and A_k of
// k_tree_tails.  The sum
// beyond P in closed form, with y = a x and t = y/(1-y):
//   sum_m C(N+m, k) y^m = 1/(1-y) sum_{j<=k} C(N, k-j) t^j.
// radius: the largest order's.
template <int P>
__global__ __launch_bounds__(kB) void k_tree_radius(MomentArgs A, int64_t n_nodes) {
    constexpr int NC = tree_ncoef(P), TR = tree_thr_row(P);
    static_assert(2 * TR <= 64, "a lane per order of the potential and of the field");
    __shared__ double bn[kB / 64][P + 1];
    __shared__ double an[kB / 64][kLMax + 1];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t nd = int64_t(blockIdx.x) * (kB / 64) + wave;
    const bool live = nd < n_nodes;
    const double* mo = A.mom + int64_t(part_words(P)) * (live ? nd : 0);
    if (lane <= P) {
        double b = 0.0;
        for (int m = 0; m <= lane; ++m) {
            const int i = tree_index(P, lane, m);
            b += A.tab[tab_norm(P) + i] * (mo[2 * i] * mo[2 * i] + mo[2 * i + 1] * mo[2 * i + 1]);
        }
        bn[wave][lane] = sqrt(b);
    }
    {
        // eight lanes per chunk of the subtree, eight chunks at a time
        double v = 0.0;
        if (live && (lane & 7) <= kLMax) {
            const int depth = A.depth[nd];
#pragma unroll 4
            for (int c = A.chunk_begin[nd] + (lane >> 3); c < A.chunk_end[nd]; c += 8)
                v += A.tail[(kLMax + 1) * (A.tail_begin[c] + depth) + (lane & 7)];
        }
        for (int o = 8; o < 64; o <<= 1) v += __shfl_xor(v, o);
        if (lane <= kLMax) an[wave][lane] = v * (1.0 + 1e-9);
    }
    __syncthreads();
    if (!live) return;
    const int fld = lane / TR, row = lane % TR;
    if (fld > 1 || (fld == 1 && !A.thr_field)) return;
    const double *b = bn[wave], *ak = an[wave];
    const double* geo = A.geo + kGeo * nd;
    const double s = node_scale(geo), tol = A.eps * mo[2 * NC];
    const double rmin = fmax(geo[4 + fld], 1.02 * geo[3]);
    const double xmax = rmin > 0.0 ? s / rmin : 0.98;
    const double a = geo[3] / s;
    auto over = [&](double x) {
        const double y = a * x, g = 1.0 / (1.0 - y), t = y * g;
        double v = 0.0;
#pragma unroll
        for (int k = 0; k <= kLMax; ++k) {
            double c = 0.0;
            if (fld) {
                // (n + 1) C(n, k) = (k + 1) C(n + 1, k + 1)
#pragma unroll
                for (int j = k + 1; j >= 0; --j) c = fma(c, t, (k + 1) * binomial(P + 2, k + 1 - j));
            } else {
#pragma unroll
                for (int j = k; j >= 0; --j) c = fma(c, t, binomial(P + 1, k - j));
            }
            v = fma(ak[k], c, v);
        }
        v *= x * g;
        for (int k = P; k > row; --k) v = (v + (fld ? double(k + 1) : 1.0) * b[k]) * x;
        for (int k = 0; k < row; ++k) v *= x;
        return !(v <= tol);
    };
    double r = HUGE_VAL;
    if (row <= P) {
        if (!over(xmax)) {
            r = s / xmax;
        } else {
            double lo = 0.0, hi = 40.0;  // x = xmax 2^-lo is too large, 2^-hi small enough
            if (!over(xmax * exp2(-hi))) {
                for (int it = 0; it < 12; ++it) {
                    const double mid = 0.5 * (lo + hi);
                    if (over(xmax * exp2(-mid))) lo = mid;
                    else hi = mid;
                }
                r = s / (xmax * exp2(-hi));
            }
        }
    }
    float* thr = (fld ? A.thr_field : A.thr) + int64_t(TR) * nd;
    thr[row] = row <= P ? float(r * (1.0 + 1e-6)) : 0.0f;  // a radius still
    if (row == P) {
        const unsigned long long u = (unsigned long long)__double_as_longlong(double(thr[row]));
        A.own[2 * nd + fld] = u;
        A.radius[2 * nd + fld] = u;
    }
}

// A node is accepted only where its children would be: its radius is at least
// each child's plus the distance of their centres.  Every node carries its
// own up to the root (a maximum, so the order does not matter; positive
// doubles order like their bits).
__global__ __launch_bounds__(kB) void k_tree_raise(const int32_t* parent, const double* geo, int64_t n_nodes,
                                                   int fields, const unsigned long long* own,
                                                   unsigned long long* radius) {
    const int64_t i = gid();
    if (i >= n_nodes) return;
    double r[2] = {0.0, 0.0};
    for (int f = 0; f < fields; ++f) r[f] = __longlong_as_double((long long)own[2 * i + f]);
    const double* c = geo + kGeo * i;
    for (int nd = parent[i]; nd >= 0; nd = parent[nd]) {
        const double* q = geo + kGeo * int64_t(nd);
        const double dx = c[0] - q[0], dy = c[1] - q[1], dz = c[2] - q[2];
        const double d = sqrt(dx * dx + dy * dy + dz * dz);
        c = q;
        for (int f = 0; f < fields; ++f) {
            r[f] = (r[f] + d) * (1.0 + 1e-6);
            const unsigned long long u = (unsigned long long)__double_as_longlong(r[f]);
            if (radius[2 * int64_t(nd) + f] < u) atomicMax(&radius[2 * int64_t(nd) + f], u);
        }
    }
}

// Squared radii by order, not growing with the order and none below the
// node's raised radius, and the node's test (its parent's radius included).
__global__ __launch_bounds__(kB) void k_tree_tests(const int32_t* parent, const double* geo, const TreeNode* node,
                                                   int64_t n_nodes, int P, const unsigned long long* radius, float* thr,
                                                   TreeTest* test, int fld) {
    const int64_t i = gid();
    if (i >= n_nodes) return;
    auto squared = [&](int64_t nd) {
        const double r = __longlong_as_double((long long)radius[2 * nd + fld]);
        return float(r * r * (1.0 + 1e-6));
    };
    const float least = squared(i);
    float* row = thr + int64_t(tree_thr_row(P)) * i;
    float v = HUGE_VALF;
    for (int p = 0; p <= P; ++p) {
        const double r = row[p];
        v = fminf(v, fmaxf(float(r * r * (1.0 + 1e-6)), least));
        row[p] = v;
    }
    const int par = parent[i];
    TreeTest q;
    for (int d = 0; d < 3; ++d) {
        q.c[d] = geo[kGeo * i + d];
        q.pc[d] = par >= 0 ? geo[kGeo * int64_t(par) + d] : 0.0;
    }
    q.r2 = v;
    q.pr2 = par >= 0 ? squared(par) : HUGE_VALF;
    q.cost = node[i].cost;
    q.pad = 0;
    test[i] = q;
}

// ------------------------------------------------------------------- host

struct Run {
    uint32_t code;
    int32_t step, type;
    int64_t count;
};

struct HostNode {
    int32_t parent;
    int32_t depth;
    int64_t cnt[kTreeTypes];
};

struct Builder {
    const std::vector<Run>& runs;
    const int steps;
    const int64_t min_cost;
    std::vector<int64_t> cost;        // prefix
    std::vector<HostNode> nodes;
    std::vector<int32_t> run_node;

    Builder(const std::vector<Run>& r, bool fp64, int P)
        : runs(r), steps(tree_steps(fp64)), min_cost(tree_min_cost(P)), cost(r.size() + 1, 0),
          run_node(r.size(), -1) {
        for (size_t i = 0; i < r.size(); ++i) cost[i + 1] = cost[i] + r[i].count * kTreeW[r[i].type];
    }
    static int digit(uint32_t code, int level) { return int((code >> (3 * (kTreeLevels - 1 - level))) & 7u); }
    void own(int32_t nd, size_t a, size_t b) {
        for (size_t i = a; i < b; ++i) {
            run_node[i] = nd;
            nodes[size_t(nd)].cnt[runs[i].type] += runs[i].count;
        }
    }
    void build(size_t a, size_t b, int step, int32_t parent, int depth) {
        const int32_t nd = int32_t(nodes.size());
        nodes.push_back(HostNode{parent, depth, {}});
        if (cost[b] - cost[a] < min_cost) {
            own(nd, a, b);
            return;
        }
        for (; step < kTreeLevels * steps; ++step) {
            // the next step halves the cell's edge, or keeps the cell and
            // lowers the radii
            const int level = step % steps == steps - 1 ? step / steps : -1;
            auto part = [&](size_t i) { return level < 0 ? 0 : digit(runs[i].code, level); };
            size_t i = a;  // this step's own runs come first
            while (i < b && runs[i].step == step) ++i;
            if (i == b) break;
            // a step with nothing of its own and one child is that child
            if (i == a && part(a) == part(b - 1)) continue;
            own(nd, a, i);
            while (i < b) {
                size_t j = i;
                const int d = part(i);
                while (j < b && part(j) == d) ++j;
                if (cost[j] - cost[i] < min_cost / 4) own(nd, i, j);
                else build(i, j, step + 1, nd, depth + 1);
                i = j;
            }
            return;
        }
        own(nd, a, b);
    }
};

std::vector<double> tables(int P) {
    std::vector<double> t(size_t(tab_words(P)), 0.0);
    auto fact = [](int k) {
        double f = 1.0;
        for (int i = 2; i <= k; ++i) f *= i;
        return f;
    };
    for (int m = 0; m <= P; ++m) {
        double lead = 1.0;  // coefficient of z^(n-m) (x+iy)^m in R_n^m
        for (int k = 1; k <= m; ++k) lead *= 0.5 / k;
        for (int n = m; n <= P; ++n) {
            const int i = tree_index(P, n, m);
            const double w = (m ? 2.0 : 1.0) * fact(n - m) * fact(n + m);
            t[size_t(tab_beta() + i)] =
                (double(n + 1) * (n + 1) - double(m) * m) / (4.0 * double(n + 1) * (n + 1) - 1.0);
            t[size_t(tab_fac(P) + i)] = w * lead;
            t[size_t(tab_norm(P) + i)] = w;
            t[size_t(tab_den(P) + i)] = n == m ? (m ? 0.5 / m : 1.0) : 1.0 / (double(n - m) * double(n + m));
            t[size_t(tab_gamma(P) + i)] = n > m ? (double(n) * n - double(m) * m) / (2.0 * n - 1.0) : 0.0;
            lead *= (2 * n + 1) / (double(n + 1 - m) * double(n + 1 + m));
        }
    }
    // d/dx = (a - b)/2, d/dy = (i/2)(a + b), d/dz = c, where a, b, c lower n by
    // one and move m by -1, +1, 0: the (t, u, v) derivative is a polynomial in
    // them, its a^alpha b^beta term one of Q_k^j with j = alpha - beta
    for (int a = 0; a <= kLMax; ++a)
        for (int b = 0; b <= kLMax - a; ++b)
            for (int c = 0; c <= kLMax - a - b; ++c) {
                double re[9] = {0}, im[9] = {0};  // by j + 4
                re[4] = 1.0;
                auto step = [&](double ar, double ai, double br, double bi) {  // times (a's factor, b's factor)
                    double nr[9] = {0}, ni[9] = {0};
                    for (int j = 0; j < 9; ++j) {
                        if (j + 1 < 9) {
                            nr[j + 1] += re[j] * ar - im[j] * ai;
                            ni[j + 1] += re[j] * ai + im[j] * ar;
                        }
                        if (j > 0) {
                            nr[j - 1] += re[j] * br - im[j] * bi;
                            ni[j - 1] += re[j] * bi + im[j] * br;
                        }
                    }
                    std::copy(nr, nr + 9, re);
                    std::copy(ni, ni + 9, im);
                };
                for (int k = 0; k < a; ++k) step(0.5, 0.0, -0.5, 0.0);
                for (int k = 0; k < b; ++k) step(0.0, 0.5, 0.0, 0.5);
                double* f = &t[size_t(tab_fold(P) + 10 * hermite_index(kLMax, a, b, c))];
                for (int j = 0; j <= 4; ++j) {
                    f[2 * j] = re[4 + j];
                    f[2 * j + 1] = im[4 + j];
                }
            }
    return t;
}

// Device memory of the build, nullptr when there is not as much or `room`
// (bytes that are left to the tree) is used up.
void* device_memory(int64_t& room, size_t nb) {
    void* q = nullptr;
    if (int64_t(nb) > room || hipMalloc(&q, nb) != hipSuccess) return nullptr;
    room -= int64_t(nb);
    return q;
}

size_t aligned(size_t nb) { return (std::max<size_t>(nb, 1) + 255) & ~size_t(255); }

// Temporary memory of the build, cut from few allocations (each takes 30 to 60 us,
// and as much to free).
struct Temp {
    int64_t& room;
    std::vector<void*> p;
    char* at = nullptr;
    size_t left = 0;
    explicit Temp(int64_t& r) : room(r) {}
    bool reserve(size_t nb) {
        void* q = device_memory(room, nb);
        if (!q) return false;
        p.push_back(q);
        at = static_cast<char*>(q);
        left = nb;
        return true;
    }
    template <class T>
    T* get(int64_t n) {
        const size_t nb = aligned(size_t(std::max<int64_t>(n, 0)) * sizeof(T));
        if (nb > left && !reserve(std::max(nb, size_t(1) << 20))) return nullptr;
        T* q = reinterpret_cast<T*>(at);
        at += nb;
        left -= nb;
        return q;
    }
    ~Temp() {
        for (void* q : p) (void)hipFree(q);
    }
};

// The arrays that stay with the tree, one allocation.
struct Keep {
    struct Part {
        void** p;
        size_t nb;
    };
    std::vector<Part> parts;
    template <class T>
    void add(T** p, int64_t n) {
        parts.push_back({reinterpret_cast<void**>(p), aligned(size_t(std::max<int64_t>(n, 0)) * sizeof(T))});
    }
    bool allocate(Tree* t) const {
        size_t all = 0;
        for (const Part& q : parts) all += q.nb;
        char* at = static_cast<char*>(device_memory(t->room, all));
        if (!at) return false;
        t->owned = at;
        t->device_bytes += int64_t(all);
        for (const Part& q : parts) {
            *q.p = at;
            at += q.nb;
        }
        return true;
    }
};

template <class T>
bool put(T* d, const std::vector<T>& v, hipStream_t st) {
    return v.empty() || hipMemcpyAsync(d, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, st) == hipSuccess;
}

int bits_for(uint64_t top) {  // smallest b with 2^b > top
    int b = 1;
    while (b < 64 && (uint64_t(1) << b) <= top) ++b;
    return b;
}

#define TREE_LAUNCH(n, kern, ...)                                                              \
    do {                                                                                       \
        if ((n) > 0) {                                                                         \
            hipLaunchKernelGGL(kern, dim3(grid_of(n)), dim3(kB), 0, st, __VA_ARGS__);             \
            if (hipGetLastError() != hipSuccess) return ENV_E_DEVICE;                          \
        }                                                                                      \
    } while (0)
#define TREE_CHECK(x)                        \
    do {                                     \
        if (!(x)) return ENV_E_DEVICE;       \
    } while (0)

env_status build(Tree* t, const TreeSource& u, const std::vector<double>& nuc, const std::vector<int32_t>& nuc_begin,
                 const std::vector<int32_t>& nuc_end) {
    hipStream_t st = nullptr;
    if (hipStreamCreateWithFlags(&st, hipStreamNonBlocking) != hipSuccess) return ENV_E_DEVICE;
    struct Guard {
        hipStream_t s;
        ~Guard() {
            (void)hipStreamSynchronize(s);
            (void)hipStreamDestroy(s);
        }
    };
    Temp tmp(t->room);  // freed after the stream has drained (declared before the guard)
    Guard guard{st};
    const int fp64 = t->fp64 ? 1 : 0, P = t->P;
    const int64_t n_pairs = t->n_pairs, n_nuc = t->n_nuc, n = n_pairs + n_nuc;
    const int ng = u.n_groups;
    std::vector<int32_t> nuc_group(nuc.size() / 4, 0);
    for (int g = 0; g < ng; ++g)
        for (int32_t k = nuc_begin[g]; k < nuc_end[g] && size_t(k) < nuc_group.size(); ++k) nuc_group[size_t(k)] = g;
    // the arrays of all items, and about what the sort takes
    if (!tmp.reserve(size_t(n) * 80 + size_t(n_nuc) * 40 + size_t(ng) * 128 + (size_t(1) << 20))) return ENV_E_NOMEM;
    double* d_nuc0 = tmp.get<double>(4 * n_nuc);
    int32_t* d_ng = tmp.get<int32_t>(n_nuc);
    int32_t* d_gnb = tmp.get<int32_t>(ng);
    int32_t* d_gne = tmp.get<int32_t>(ng);
    double* d_cube = tmp.get<double>(4 * int64_t(ng));
    unsigned long long* d_gbox = tmp.get<unsigned long long>(6 * int64_t(ng));
    unsigned long long* key = tmp.get<unsigned long long>(n);
    unsigned long long* key_s = tmp.get<unsigned long long>(n);
    uint32_t* val = tmp.get<uint32_t>(n);
    uint32_t* val_s = tmp.get<uint32_t>(n);
    int32_t* head = tmp.get<int32_t>(n);
    int32_t* runid = tmp.get<int32_t>(n);
    uint32_t* nkey = tmp.get<uint32_t>(n);
    uint32_t* nkey_s = tmp.get<uint32_t>(n);
    int32_t* item_node = tmp.get<int32_t>(n);
    if (!d_nuc0 || !d_ng || !d_gnb || !d_gne || !d_cube || !d_gbox || !key || !key_s || !val || !val_s || !head || !runid ||
        !nkey || !nkey_s || !item_node)
        return ENV_E_NOMEM;
    if (u.n_cells > 0) {
        const int64_t at = n_nuc - u.n_cells;
        TREE_CHECK(hipMemcpyAsync(d_nuc0 + 4 * at, u.cells, size_t(u.n_cells) * 4 * sizeof(double), hipMemcpyHostToDevice,
                                  st) == hipSuccess &&
                   hipMemsetAsync(d_ng + at, 0, size_t(u.n_cells) * sizeof(int32_t), st) == hipSuccess);
        TREE_LAUNCH(u.n_cells, k_tree_negate, d_nuc0 + 4 * at, u.n_cells);
    }
    TREE_CHECK(put(d_nuc0, nuc, st) && put(d_ng, nuc_group, st) && put(d_gnb, nuc_begin, st) &&
               put(d_gne, nuc_end, st));
    TREE_LAUNCH(6 * int64_t(ng), k_tree_no_boxes, int64_t(ng), d_gbox);
    // (parts of 4096 items, as many as a group of all items would have)
    hipLaunchKernelGGL(k_tree_boxes, dim3(unsigned(ng), unsigned(std::min<int64_t>((n + 4095) / 4096, 256))), dim3(kB), 0, st,
                       u.pairs, u.rec, d_nuc0, n_pairs, fp64, u.group_pairs, d_gnb, d_gne, d_gbox);
    TREE_CHECK(hipGetLastError() == hipSuccess);
    TREE_LAUNCH(int64_t(ng), k_tree_cubes, d_gbox, int64_t(ng), d_cube);
    TREE_LAUNCH(n, k_tree_keys, u.pairs, u.rec, d_nuc0, d_ng, n_pairs, n, fp64, d_cube, key, val);
    size_t tb = 0;
    const int kb = 38 + bits_for(uint64_t(std::max(ng - 1, 0)));
    TREE_CHECK(hipcub::DeviceRadixSort::SortPairs(nullptr, tb, key, key_s, val, val_s, int(n), 0, kb, st) ==
               hipSuccess);
    void* work = tmp.get<char>(int64_t(tb));
    if (!work) return ENV_E_NOMEM;
    TREE_CHECK(hipcub::DeviceRadixSort::SortPairs(work, tb, key, key_s, val, val_s, int(n), 0, kb, st) ==
               hipSuccess);
    if (n_pairs == 0) {
        const int64_t w = kTreeW[kTreeTypes - 1];
        TREE_LAUNCH(n, k_tree_cut, key_s, n, tree_steps(t->fp64), (tree_min_cost(P) + w - 1) / w, key);
        std::swap(key, key_s);
    }
    TREE_LAUNCH(n, k_tree_heads, key_s, n, head);
    size_t ts = 0;
    TREE_CHECK(hipcub::DeviceScan::InclusiveSum(nullptr, ts, head, runid, int(n), st) == hipSuccess);
    void* work2 = tmp.get<char>(int64_t(ts));
    if (!work2) return ENV_E_NOMEM;
    TREE_CHECK(hipcub::DeviceScan::InclusiveSum(work2, ts, head, runid, int(n), st) == hipSuccess);
    int32_t n_runs = 0;
    TREE_CHECK(hipMemcpyAsync(&n_runs, runid + (n - 1), sizeof(int32_t), hipMemcpyDeviceToHost, st) == hipSuccess &&
               hipStreamSynchronize(st) == hipSuccess);
    unsigned long long* d_rkey = tmp.get<unsigned long long>(n_runs);
    uint32_t* d_rstart = tmp.get<uint32_t>(n_runs);
    int32_t* d_run_node = tmp.get<int32_t>(n_runs);
    if (!d_rkey || !d_rstart || !d_run_node) return ENV_E_NOMEM;
    TREE_LAUNCH(n, k_tree_runs, key_s, runid, n, d_rkey, d_rstart);
    std::vector<unsigned long long> rkey(static_cast<size_t>(n_runs));
    std::vector<uint32_t> rstart(static_cast<size_t>(n_runs));
    TREE_CHECK(hipMemcpyAsync(rkey.data(), d_rkey, rkey.size() * 8, hipMemcpyDeviceToHost, st) == hipSuccess &&
               hipMemcpyAsync(rstart.data(), d_rstart, rstart.size() * 4, hipMemcpyDeviceToHost, st) == hipSuccess &&
               hipStreamSynchronize(st) == hipSuccess);

    // nodes
    std::vector<Run> runs(static_cast<size_t>(n_runs));
    std::vector<size_t> group_at;  // first run of every tree
    for (size_t i = 0; i < runs.size(); ++i) {
        runs[i].type = int32_t(rkey[i] & 7ull);
        runs[i].step = int32_t((rkey[i] >> 3) & 31ull);
        runs[i].code = uint32_t((rkey[i] >> 8) & 0x3fffffffull);
        runs[i].count = (i + 1 < runs.size() ? int64_t(rstart[i + 1]) : n) - int64_t(rstart[i]);
        if (i == 0 || (rkey[i] >> 38) != (rkey[i - 1] >> 38)) group_at.push_back(i);
    }
    group_at.push_back(runs.size());
    Builder b(runs, t->fp64, t->P);
    std::vector<int32_t> first;
    for (size_t g = 0; g + 1 < group_at.size(); ++g) {
        first.push_back(int32_t(b.nodes.size()));
        b.build(group_at[g], group_at[g + 1], 0, -1, 0);
    }
    first.push_back(int32_t(b.nodes.size()));
    const int64_t nn = int64_t(b.nodes.size());
    t->n_nodes = nn;
    t->n_trees = int32_t(first.size()) - 1;
    std::vector<TreeNode> node(static_cast<size_t>(nn));
    std::vector<uint32_t> start(size_t(nn) * kTreeTypes);
    std::vector<int32_t> parent(static_cast<size_t>(nn)), by_depth(static_cast<size_t>(nn)), child,
        child_begin(size_t(nn) + 1, 0);
    std::vector<Chunk> chunk;
    std::vector<int32_t> chunk_begin(size_t(nn) + 1, 0);
    std::vector<int32_t> chunk_end(static_cast<size_t>(nn)), depth(static_cast<size_t>(nn));
    std::vector<int64_t> tail_begin(1, 0);
    std::vector<int32_t> tail_node;
    int64_t words = 0, item = 0, nucs = 0;
    int max_depth = 0;
    for (int64_t k = 0; k < nn; ++k) {
        const HostNode& h = b.nodes[size_t(k)];
        TreeNode& o = node[size_t(k)];
        int64_t cost = 0;
        o.rec_off = words;
        for (int ty = 0; ty < kTreeTypes; ++ty) {
            start[size_t(k) * kTreeTypes + ty] = uint32_t(item);
            item += h.cnt[ty];
            cost += h.cnt[ty] * kTreeW[ty];
            if (ty <= kLMax) {
                o.cnt[ty] = int32_t(h.cnt[ty]);
                words += h.cnt[ty] * rec_words_of(ty, t->fp64);
            }
        }
        o.nuc_begin = int32_t(nucs);
        nucs += h.cnt[kTreeTypes - 1];
        o.nuc_end = int32_t(nucs);
        o.cost = int32_t(cost);
        const int64_t items = h.cnt[0] + h.cnt[1] + h.cnt[2] + h.cnt[3] + h.cnt[4] + h.cnt[5];
        for (int64_t a = 0; a < items; a += kChunk)
            chunk.push_back(Chunk{int32_t(k), int32_t(a), int32_t(std::min<int64_t>(items, a + kChunk))});
        chunk_begin[size_t(k) + 1] = int32_t(chunk.size());
        parent[size_t(k)] = h.parent;
        max_depth = std::max(max_depth, int(h.depth));
        if (h.parent >= 0) ++child_begin[size_t(h.parent) + 1];
    }
    for (int64_t k = 0; k < nn; ++k) child_begin[size_t(k) + 1] += child_begin[size_t(k)];
    child.resize(size_t(child_begin[size_t(nn)]));
    {
        std::vector<int32_t> at(child_begin.begin(), child_begin.end() - 1);
        for (int64_t k = 0; k < nn; ++k)
            if (parent[size_t(k)] >= 0) child[size_t(at[size_t(parent[size_t(k)])]++)] = int32_t(k);
        t->level_begin.assign(size_t(max_depth) + 2, 0);
        for (int64_t k = 0; k < nn; ++k) ++t->level_begin[size_t(b.nodes[size_t(k)].depth) + 1];
        for (int d = 0; d <= max_depth; ++d) t->level_begin[size_t(d) + 1] += t->level_begin[size_t(d)];
        std::vector<int32_t> lv(t->level_begin.begin(), t->level_begin.end() - 1);
        for (int64_t k = 0; k < nn; ++k) by_depth[size_t(lv[size_t(b.nodes[size_t(k)].depth)]++)] = int32_t(k);
    }
    for (int64_t k = nn - 1; k >= 0; --k) {
        int32_t& e = chunk_end[size_t(k)];
        e = std::max(e, chunk_begin[size_t(k) + 1]);
        if (parent[size_t(k)] >= 0) chunk_end[size_t(parent[size_t(k)])] = std::max(chunk_end[size_t(parent[size_t(k)])], e);
    }
    std::vector<int32_t> path;  // the ancestors of node k, from the root to k
    for (int64_t k = 0; k < nn; ++k) {
        depth[size_t(k)] = b.nodes[size_t(k)].depth;
        path.resize(size_t(depth[size_t(k)]));
        path.push_back(int32_t(k));
        for (int32_t c = chunk_begin[size_t(k)]; c < chunk_begin[size_t(k) + 1]; ++c) {
            tail_node.insert(tail_node.end(), path.begin(), path.end());
            tail_begin.push_back(int64_t(tail_node.size()));
        }
    }
    t->rec_words = words;
    const std::vector<double> tab = tables(P);
    t->n_chunks = int64_t(chunk.size());
    Chunk* d_chunk = nullptr;
    Keep keep;
    keep.add(&t->d_test, nn);
    keep.add(&t->d_node, nn);
    keep.add(&t->d_thr, nn * tree_thr_row(P));
    if (u.field) {
        keep.add(&t->d_test_field, nn);
        keep.add(&t->d_thr_field, nn * tree_thr_row(P));
    }
    keep.add(&t->d_coef, nn * tree_words(P));
    keep.add(&t->d_tab, tab_words(P));
    keep.add(&t->d_first, int64_t(first.size()));
    keep.add(&t->d_rec, words);
    keep.add(&t->d_nuc, 4 * n_nuc);
    keep.add(&t->d_word, n_pairs);
    keep.add(&t->d_parent, nn);
    keep.add(&t->d_child, int64_t(child.size()));
    keep.add(&t->d_child_begin, nn + 1);
    keep.add(&t->d_by_depth, nn);
    keep.add(&t->d_geo, nn * kGeo);
    keep.add(&d_chunk, t->n_chunks);
    keep.add(&t->d_chunk_begin, nn + 1);
    keep.add(&t->d_chunk_end, nn);
    keep.add(&t->d_depth, nn);
    keep.add(&t->d_tail_begin, t->n_chunks + 1);
    keep.add(&t->d_tail_node, int64_t(tail_node.size()));
    // chunks' moments, nodes' shifted and own moments, radii, chunks' shares of the bounds
    keep.add(&t->d_work, t->n_chunks * part_words(P) + nn * (2 * part_words(P) + 4) + int64_t(tail_node.size()) * (kLMax + 1));
    keep.add(&t->d_sph, t->rec_words);
    uint32_t* d_start = tmp.get<uint32_t>(int64_t(start.size()));
    unsigned long long* d_box = tmp.get<unsigned long long>(6 * nn);
    unsigned long long* d_rad = tmp.get<unsigned long long>(3 * nn);
    if (!keep.allocate(t) || !d_start || !d_box || !d_rad) return ENV_E_NOMEM;
    t->d_chunk = d_chunk;
    TREE_CHECK(put(t->d_node, node, st) && put(t->d_tab, tab, st) && put(t->d_first, first, st) &&
               put(t->d_parent, parent, st) && put(t->d_child, child, st) && put(t->d_child_begin, child_begin, st) &&
               put(t->d_by_depth, by_depth, st) && put(d_start, start, st) && put(d_run_node, b.run_node, st) && put(d_chunk, chunk, st) &&
               put(t->d_chunk_begin, chunk_begin, st) && put(t->d_chunk_end, chunk_end, st) &&
               put(t->d_depth, depth, st) && put(t->d_tail_begin, tail_begin, st) &&
               put(t->d_tail_node, tail_node, st));
    // records by (node, type), in pair order within
    TREE_LAUNCH(n, k_tree_nodekeys, key_s, runid, d_run_node, n, nkey);
    const int nb = bits_for(uint64_t(nn) * kTreeTypes);
    size_t tb2 = 0;
    TREE_CHECK(hipcub::DeviceRadixSort::SortPairs(nullptr, tb2, nkey, nkey_s, val_s, val, int(n), 0, nb, st) ==
               hipSuccess);
    void* work3 = tmp.get<char>(int64_t(tb2));
    if (!work3) return ENV_E_NOMEM;
    TREE_CHECK(hipcub::DeviceRadixSort::SortPairs(work3, tb2, nkey, nkey_s, val_s, val, int(n), 0, nb, st) ==
               hipSuccess);
    TREE_LAUNCH(n, k_tree_place, nkey_s, val, d_start, t->d_node, n_pairs, n, fp64, d_nuc0, t->d_word, t->d_nuc,
                item_node);
    // geometry
    Ratios ratios{};
    for (int L = 0; L <= kLMax; ++L) ratios.r[L] = u.field ? std::sqrt(u.field_ratio[L]) * (1.0 + 1e-6) : 1.0;
    ratios.r[kLMax + 1] = 1.0;
    TREE_LAUNCH(6 * nn, k_tree_no_boxes, nn, d_box);
    TREE_LAUNCH(n, k_tree_bounds, u.pairs, u.rec, d_nuc0, n_pairs, n, fp64, item_node, t->d_parent, d_box);
    TREE_LAUNCH(nn, k_tree_centres, d_box, nn, t->d_geo, d_rad);
    TREE_LAUNCH(n, k_tree_radii, u.pairs, u.rec, d_nuc0, n_pairs, n, fp64, item_node, t->d_parent, t->d_geo,
                ratios, d_rad);
    TREE_LAUNCH(nn, k_tree_radii_out, d_rad, nn, t->d_geo);
    TREE_CHECK(hipStreamSynchronize(st) == hipSuccess);
    return ENV_OK;
}

}  // namespace

Tree* build_tree(const TreeSource& u, const std::vector<double>& nuc, const std::vector<int32_t>& nuc_begin,
                 const std::vector<int32_t>& nuc_end, bool fp64, env_status* st) {
    *st = ENV_OK;
    const int64_t n_nuc = int64_t(nuc.size() / 4) + u.n_cells, n = u.n_pairs + n_nuc;
    if (n < kTreeMinItems || n > kTreeMaxItems || u.n_groups <= 0 || u.n_groups >= (1 << 26) ||
        int64_t(nuc_begin.size()) != u.n_groups || int64_t(nuc_end.size()) != u.n_groups)
        return nullptr;
    Tree* t = new (std::nothrow) Tree;
    if (!t) return nullptr;
    t->fp64 = fp64;
    t->P = u.order;
    t->eps = u.eps;
    t->n_pairs = u.n_pairs;
    t->n_nuc = n_nuc;
    if (const char* e = std::getenv("ENVPOT_TREE_MAX_MB"))
        if (*e) t->room = std::max<int64_t>(std::atoll(e), 0) << 20;
    try {
        *st = build(t, u, nuc, nuc_begin, nuc_end);
    } catch (const std::bad_alloc&) {
        *st = ENV_E_NOMEM;
    }
    if (*st != ENV_OK) {
        free_tree(t);
        if (*st == ENV_E_NOMEM) {
            *st = ENV_OK;              // every item can be evaluated without one
            (void)hipGetLastError();   // the allocation's
        }
        return nullptr;
    }
    return t;
}

void free_tree(Tree* t) {
    if (!t) return;
    (void)hipFree(t->owned);
    delete t;
}

int refresh_tree(const Tree& t, const TreeSource& u, void* stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (t.n_pairs > 0) {
        const int per = kB / 16;
        hipLaunchKernelGGL(k_tree_copy, dim3(unsigned((t.n_pairs + per - 1) / per)), dim3(kB), 0, st, u.pairs,
                           t.d_word, t.n_pairs, t.fp64 ? 1 : 0, u.rec, t.d_rec);
        if (hipGetLastError() != hipSuccess) return -1;
    }
    MomentArgs a{};
    a.chunk = static_cast<const Chunk*>(t.d_chunk);
    a.chunk_begin = t.d_chunk_begin;
    a.node = t.d_node;
    a.rec = t.d_rec;
    a.nuc = t.d_nuc;
    a.child = t.d_child;
    a.child_begin = t.d_child_begin;
    a.parent = t.d_parent;
    a.geo = t.d_geo;
    a.tab = t.d_tab;
    a.coef = t.d_coef;
    a.thr = t.d_thr;
    a.thr_field = t.d_thr_field;
    a.eps = t.eps;
    a.nuc_size = u.nuc_eps / u.eps;
    const size_t pw = size_t(part_words(t.P)), nn = size_t(t.n_nodes);
    double* work = t.d_work;
    a.part = work;
    a.up = a.part + size_t(t.n_chunks) * pw;
    a.mom = a.up + nn * pw;
    a.own = reinterpret_cast<unsigned long long*>(a.mom + nn * pw);
    a.radius = a.own + 2 * nn;
    a.tail = reinterpret_cast<double*>(a.radius + 2 * nn);
    a.chunk_end = t.d_chunk_end;
    a.depth = t.d_depth;
    a.tail_begin = t.d_tail_begin;
    a.tail_node = t.d_tail_node;
    bool ok = true;
    uint32_t* sph = t.d_sph;
    if (t.n_pairs > 0) {
        if (t.fp64)
            hipLaunchKernelGGL(k_tree_spherical<true>, dim3(grid_of(t.n_pairs)), dim3(kB), 0, st, u.pairs, t.d_word,
                               t.n_pairs, u.rec, t.d_tab + tab_fold(t.P), sph);
        else
            hipLaunchKernelGGL(k_tree_spherical<false>, dim3(grid_of(t.n_pairs)), dim3(kB), 0, st, u.pairs, t.d_word,
                               t.n_pairs, u.rec, t.d_tab + tab_fold(t.P), sph);
        ok = hipGetLastError() == hipSuccess;
    }
    a.sph = sph;
    ok = ok && (t.P == kTreeOrd32 || t.P == kTreeOrd64 || t.P == kTreeOrdCells32 || t.P == kTreeOrdCells64);
    const dim3 chunks(unsigned(t.n_chunks));
    if (t.P == kTreeOrd32) hipLaunchKernelGGL((k_tree_p2m<kTreeOrd32>), chunks, dim3(kB), 0, st, a, t.fp64 ? 1 : 0);
    else if (t.P == kTreeOrd64) hipLaunchKernelGGL((k_tree_p2m<kTreeOrd64>), chunks, dim3(kB), 0, st, a, t.fp64 ? 1 : 0);
    else if (t.P == kTreeOrdCells32) hipLaunchKernelGGL((k_tree_p2m<kTreeOrdCells32>), chunks, dim3(kB), 0, st, a, t.fp64 ? 1 : 0);
    else if (t.P == kTreeOrdCells64) hipLaunchKernelGGL((k_tree_p2m<kTreeOrdCells64>), chunks, dim3(kB), 0, st, a, t.fp64 ? 1 : 0);
    ok = ok && hipGetLastError() == hipSuccess;
    for (int d = int(t.level_begin.size()) - 2; d >= 0 && ok; --d) {
        const int n = t.level_begin[size_t(d) + 1] - t.level_begin[size_t(d)];
        if (n <= 0) continue;
        a.by_depth = t.d_by_depth + t.level_begin[size_t(d)];
        const dim3 nodes = dim3(unsigned(n)), threads = dim3(unsigned(node_threads(t.P)));
        if (t.P == kTreeOrd32) hipLaunchKernelGGL((k_tree_nodes<kTreeOrd32>), nodes, threads, 0, st, a);
        else if (t.P == kTreeOrd64) hipLaunchKernelGGL((k_tree_nodes<kTreeOrd64>), nodes, threads, 0, st, a);
        else if (t.P == kTreeOrdCells32) hipLaunchKernelGGL((k_tree_nodes<kTreeOrdCells32>), nodes, threads, 0, st, a);
        else hipLaunchKernelGGL((k_tree_nodes<kTreeOrdCells64>), nodes, threads, 0, st, a);
        ok = hipGetLastError() == hipSuccess;
    }
    if (ok) {
        const dim3 block(kChunk);
        const int fp64 = t.fp64 ? 1 : 0;
        if (t.P == kTreeOrd32) hipLaunchKernelGGL((k_tree_tails<kTreeOrd32>), chunks, block, 0, st, a, fp64);
        else if (t.P == kTreeOrd64) hipLaunchKernelGGL((k_tree_tails<kTreeOrd64>), chunks, block, 0, st, a, fp64);
        else if (t.P == kTreeOrdCells32) hipLaunchKernelGGL((k_tree_tails<kTreeOrdCells32>), chunks, block, 0, st, a, fp64);
        else hipLaunchKernelGGL((k_tree_tails<kTreeOrdCells64>), chunks, block, 0, st, a, fp64);
        ok = hipGetLastError() == hipSuccess;
    }
    if (ok) {
        const dim3 waves(unsigned((t.n_nodes + kB / 64 - 1) / (kB / 64)));
        if (t.P == kTreeOrd32) hipLaunchKernelGGL((k_tree_radius<kTreeOrd32>), waves, dim3(kB), 0, st, a, t.n_nodes);
        else if (t.P == kTreeOrd64) hipLaunchKernelGGL((k_tree_radius<kTreeOrd64>), waves, dim3(kB), 0, st, a, t.n_nodes);
        else if (t.P == kTreeOrdCells32) hipLaunchKernelGGL((k_tree_radius<kTreeOrdCells32>), waves, dim3(kB), 0, st, a, t.n_nodes);
        else hipLaunchKernelGGL((k_tree_radius<kTreeOrdCells64>), waves, dim3(kB), 0, st, a, t.n_nodes);
        const dim3 grid = grid_of(t.n_nodes);
        hipLaunchKernelGGL(k_tree_raise, grid, dim3(kB), 0, st, t.d_parent, t.d_geo, t.n_nodes, t.d_test_field ? 2 : 1,
                           a.own, a.radius);
        hipLaunchKernelGGL(k_tree_tests, grid, dim3(kB), 0, st, t.d_parent, t.d_geo, t.d_node, t.n_nodes, t.P,
                           a.radius, t.d_thr, t.d_test, 0);
        if (t.d_test_field)
            hipLaunchKernelGGL(k_tree_tests, grid, dim3(kB), 0, st, t.d_parent, t.d_geo, t.d_node, t.n_nodes, t.P,
                               a.radius, t.d_thr_field, t.d_test_field, 1);
        ok = hipGetLastError() == hipSuccess;
    }
    return ok ? 0 : -1;
}

TreeView tree_view(const Tree& t) {
    TreeView v{};
    v.test = t.d_test;
    v.node = t.d_node;
    v.thr = t.d_thr;
    v.coef = t.d_coef;
    v.beta = t.d_tab + tab_beta();
    v.first = t.d_first;
    v.rec = t.d_rec;
    v.nuc = t.d_nuc;
    v.n_trees = t.n_trees;
    v.P = t.P;
    v.gamma = t.d_tab + tab_gamma(t.P);
    return v;
}

TreeView tree_view_field(const Tree& t) {
    TreeView v = tree_view(t);
    v.test = t.d_test_field;
    v.thr = t.d_thr_field;
    return v;
}

}  // namespace envpot
