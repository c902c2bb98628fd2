// Evaluation of a multipole tree (tree_internal.h) for one block of points:
// the walk shared by the potential, field and cell-sum kernels.  A workgroup
// holds one block of points in every one of its four waves, tests the nodes
// against the block's bounding box, one node per thread, and collects the
// accepted ones and the nodes whose own items are to be evaluated.
#pragma once

#include <hip/hip_runtime.h>

#include "device_math.h"
#include "envpot_internal.h"
#include "tree_internal.h"

namespace envpot {

// Lists of one workgroup: every wave appends to its own part.
constexpr int kNearWave = 128;  // nodes whose own items are to be evaluated
constexpr int kFarWave = 128;   // accepted nodes
constexpr int kChunkCap = 256;  // runs of up to 64 nodes of open trees, one per wave step

struct TreeLists {
    int32_t near_node[4][kNearWave];
    int32_t near_cost[4][kNearWave];
    int32_t far_node[4][kFarWave];
    int32_t list_node[4 * kNearWave];   // the waves' parts one after the other
    int64_t list_cost[4 * kNearWave];   // ... and the exclusive prefix of their cost
    int32_t list_far[4 * kFarWave];
    int32_t list_order[4 * kFarWave];
    int32_t chunk_begin[kChunkCap];
    int32_t chunk_end[kChunkCap];
    uint64_t scan[4];
    int32_t count[4];                   // near | far << 16, per wave
    int32_t more[4];
};

// LDS of a tree kernel besides its Boys table: the lists, then the waves' sums.
template <int WORDS>
union TreeShared {
    TreeLists lists;
    double acc[4][WORDS];
};

// The value of v in the first active lane, as a wave-uniform (scalar) value.
__device__ __forceinline__ double wave_uniform(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ double wave_min(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o));
    return wave_uniform(v);
}

// Squared distance of the block's box from a node's centre.
__device__ __forceinline__ double box_r2(const double* c, const double* lo, const double* hi) {
    double r2 = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double g = fmax(0.0, fmax(lo[d] - c[d], c[d] - hi[d]));
        r2 = __builtin_fma(g, g, r2);
    }
    return r2;
}

// Exclusive prefix sum over the workgroup in thread order; total in *sum.
__device__ __forceinline__ uint64_t block_scan(uint64_t v, uint64_t* tmp, uint64_t* sum) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint64_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    __syncthreads();
    if (lane == 63) tmp[wave] = x;
    __syncthreads();
    uint64_t base = 0, all = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if (w < wave) base += tmp[w];
        all += tmp[w];
    }
    *sum = all;
    return base + x - v;
}

// Items [a, b) of a run of cnt items of weight W that starts at cost c,
// within the cost range [lo, hi): an item belongs to the range its first
// cost unit lies in.
template <int W>
__device__ __forceinline__ void run_share(int64_t c, int cnt, int64_t lo, int64_t hi, int& a, int& b) {
    const int64_t top = int64_t(cnt) * W;
    const int64_t l = lo - c, h = hi - c;
    const uint32_t lc = uint32_t(l < 0 ? 0 : (l > top ? top : l)), hc = uint32_t(h < 0 ? 0 : (h > top ? top : h));
    a = int((lc + W - 1) / W);
    b = int((hc + W - 1) / W);
}

// The part of a run of pairs of one L that lies in the cost range.
template <int L, bool F64, class Eval>
__device__ __forceinline__ void tree_run(const GLB uint32_t* __restrict__ rec, int64_t& word, int64_t& c, int cnt,
                                         int64_t lo, int64_t hi, Eval& ev) {
    constexpr int RW = F64 ? rec64_words(L) : rec32_words(L);
    int a, b;
    run_share<kTreeW[L]>(c, cnt, lo, hi, a, b);
    if (b > a) ev.template run<L>(rec + word + int64_t(a) * RW, b - a);
    c += int64_t(cnt) * kTreeW[L];
    word += int64_t(cnt) * RW;
}

// Smallest and largest coordinates of the wave's points.
template <int NP>
__device__ __forceinline__ void block_box(const double* cx, const double* cy, const double* cz, double* lo,
                                          double* hi) {
    const double* c[3] = {cx, cy, cz};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        double a = c[d][0], b = c[d][0];
#pragma unroll
        for (int k = 1; k < NP; ++k) {
            a = fmin(a, c[d][k]);
            b = fmax(b, c[d][k]);
        }
        lo[d] = wave_min(a);
        hi[d] = -wave_min(-b);
    }
}

// Split s of tv.S of the block with the box [lo, hi]: all waves call this
// together.  The own items' cost is cut into 4 S equal parts and part
// 4 s + w is wave w's: all S workgroups of a block collect the same own
// items, so the cut is exact however the near work is spread over the tree.
// An accepted node belongs to the split its index gives, and goes round that
// workgroup's waves.  The sums have a fixed order.
// Eval: run<L>(records, n), nucleus(x, y, z, Z), far(coefficients, beta, order).
template <bool F64, class Eval>
__device__ __forceinline__ void tree_walk(const TreeView& tv, int s, const double* lo, const double* hi, TreeLists& sh,
                                          Eval& ev) {
    const int P = tv.P, TR = tree_thr_row(P);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int parts = 4 * tv.S, part = 4 * s + wave;
    const GLB TreeNode* nodes = glb(tv.node);
    const GLB uint32_t* rec = glb(tv.rec);
    const GLB double* nuc = glb(tv.nuc);
    const GLB double* coef = glb(tv.coef);
    const GLB double* beta = glb(tv.beta);
    int nn = 0, nf = 0;  // entries of this wave's part of the lists

    // The order an accepted node needs.
    auto order_of = [&](int nd) -> int {
        const float4* th = reinterpret_cast<const float4*>(tv.thr + int64_t(nd) * TR);
        const double cc[3] = {tv.test[nd].c[0], tv.test[nd].c[1], tv.test[nd].c[2]};
        const float rf = float(box_r2(cc, lo, hi) * (1.0 - 1e-6));
        int o = 0;
#pragma unroll 4
        for (int q = 0; q < TR / 4; ++q) {
            const float4 v = th[q];
            o += (v.x > rf) + (v.y > rf) + (v.z > rf) + (v.w > rf);
        }
        return o < P ? o : P;
    };
    // A full list of accepted nodes is evaluated by its wave alone: nothing
    // that depends on the split may move the meeting points of the waves,
    // which cut the own items (the same in every split) into parts.
    auto far_alone = [&]() {
        wave_sync();
        for (int e0 = 0; e0 < nf; e0 += 64) {
            const int k = min(64, nf - e0);
            int nd = 0, o = 0;
            if (lane < k) {
                nd = sh.far_node[wave][e0 + lane];
                o = order_of(nd);
            }
            for (int q = 0; q < k; ++q)
                ev.far(coef + int64_t(__builtin_amdgcn_readlane(nd, q)) * tree_words(P), beta,
                       __builtin_amdgcn_readlane(o, q));
        }
        nf = 0;
        wave_sync();
    };
    // Evaluate the collected lists: they are put together in wave order, cut
    // by cost, and every wave evaluates its share.
    auto evaluate = [&]() {
        int nw[4], fw[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int c = __builtin_amdgcn_readfirstlane(sh.count[w]);
            nw[w] = c & 0xffff;
            fw[w] = c >> 16;
        }
        const int n_near = nw[0] + nw[1] + nw[2] + nw[3], n_far = fw[0] + fw[1] + fw[2] + fw[3];
        auto part_of = [](const int* c, int e, int& w) {  // entry e of the concatenation: its part and place
            w = 0;
            while (w < 3 && e >= c[w]) e -= c[w++];
            return e;
        };
        uint64_t own = 0, cost;
        constexpr int kEach = 4 * kNearWave / kBlock;
        int32_t node[kEach], pc[kEach];
#pragma unroll
        for (int q = 0; q < kEach; ++q) {
            const int e = kEach * tid + q;
            node[q] = pc[q] = 0;
            if (e < n_near) {
                int w;
                const int f = part_of(nw, e, w);
                node[q] = sh.near_node[w][f];
                pc[q] = sh.near_cost[w][f];
            }
            own += uint64_t(pc[q]);
        }
        uint64_t at = block_scan(own, sh.scan, &cost);
#pragma unroll
        for (int q = 0; q < kEach; ++q) {
            const int e = kEach * tid + q;
            if (e < n_near) {
                sh.list_node[e] = node[q];
                sh.list_cost[e] = int64_t(at);
            }
            at += uint64_t(pc[q]);
        }
        for (int f = tid; f < n_far; f += kBlock) {
            int w;
            const int at_w = part_of(fw, f, w);
            const int nd = sh.far_node[w][at_w];
            sh.list_far[f] = nd;
            sh.list_order[f] = order_of(nd);
        }
        __syncthreads();
        const int64_t total = int64_t((uint64_t(__builtin_amdgcn_readfirstlane(uint32_t(cost >> 32))) << 32) |
                                      __builtin_amdgcn_readfirstlane(uint32_t(cost)));
        const int64_t clo = total / parts * part + total % parts * part / parts;
        const int64_t chi = total / parts * (part + 1) + total % parts * (part + 1) / parts;
        if (chi > clo) {
            int a = 0, b = n_near;  // the last node whose cost begins at clo or before
            while (b - a > 1) {
                const int mid = (a + b) >> 1;
                if (sh.list_cost[mid] <= clo) a = mid;
                else b = mid;
            }
            for (int e = __builtin_amdgcn_readfirstlane(a); e < n_near; ++e) {
                const uint64_t cv = uint64_t(sh.list_cost[e]);
                int64_t c = int64_t((uint64_t(__builtin_amdgcn_readfirstlane(uint32_t(cv >> 32))) << 32) |
                                    __builtin_amdgcn_readfirstlane(uint32_t(cv)));
                if (c >= chi) break;
                const GLB TreeNode* nd = nodes + __builtin_amdgcn_readfirstlane(sh.list_node[e]);
                int64_t word = nd->rec_off;
                tree_run<0, F64>(rec, word, c, nd->cnt[0], clo, chi, ev);
                tree_run<1, F64>(rec, word, c, nd->cnt[1], clo, chi, ev);
                tree_run<2, F64>(rec, word, c, nd->cnt[2], clo, chi, ev);
                tree_run<3, F64>(rec, word, c, nd->cnt[3], clo, chi, ev);
                tree_run<4, F64>(rec, word, c, nd->cnt[4], clo, chi, ev);
                const int nb = nd->nuc_begin;
                int qa, qb;
                run_share<kTreeW[kLMax + 1]>(c, nd->nuc_end - nb, clo, chi, qa, qb);
                for (int q = nb + qa; q < nb + qb; ++q) ev.nucleus(nuc[4 * q], nuc[4 * q + 1], nuc[4 * q + 2], nuc[4 * q + 3]);
            }
        }
        for (int e = wave; e < n_far; e += 4) {
            const int nd = __builtin_amdgcn_readfirstlane(sh.list_far[e]);
            ev.far(coef + int64_t(nd) * tree_words(P), beta, __builtin_amdgcn_readfirstlane(sh.list_order[e]));
        }
    };
    // Class of a node: 2 accepted, 1 its own items are evaluated, 0 neither
    // (its parent is accepted, or it has none of its own).
    auto classify = [&](const TreeTest& t) -> int {
        const double rp = box_r2(t.pc, lo, hi), r2 = box_r2(t.c, lo, hi);
        if (rp >= double(t.pr2) && rp < 1e300) return 0;
        if (r2 >= double(t.r2) && r2 < 1e300) return 2;
        return t.cost > 0 ? 1 : 0;
    };
    auto append = [&](int cls, int nd, int cost) {
        if (cls == 2 && (nd & (tv.S - 1)) != s) cls = 0;  // another split's (S is a power of two)
        if (nf > kFarWave - 64) far_alone();
        const uint64_t mf = __builtin_amdgcn_ballot_w64(cls == 2), mn = __builtin_amdgcn_ballot_w64(cls == 1);
        auto below = [](uint64_t m) {
            return __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0));
        };
        if (cls == 2) sh.far_node[wave][nf + below(mf)] = nd;
        if (cls == 1) {
            const int f = nn + below(mn);
            sh.near_node[wave][f] = nd;
            sh.near_cost[wave][f] = cost;
        }
        nf += __popcll(mf);
        nn += __popcll(mn);
    };
    auto room = [&]() { return nn <= kNearWave - 64; };
    // Meeting point of the waves: the lists are evaluated when some wave has
    // no room for another step or `last` is set; false when some wave has
    // steps left (`left`).
    auto meet = [&](bool left, bool last) -> bool {
        if (lane == 0) {
            sh.count[wave] = nn | nf << 16;
            sh.more[wave] = (left ? 1 : 0) | (room() ? 0 : 2);
        }
        __syncthreads();
        const int m = __builtin_amdgcn_readfirstlane(sh.more[0] | sh.more[1] | sh.more[2] | sh.more[3]);
        if ((m & 2) || (last && !(m & 1))) {
            evaluate();
            nn = nf = 0;
        }
        __syncthreads();
        return !(m & 1);
    };

    for (int t0 = 0; t0 < tv.n_trees; t0 += kBlock) {
        // roots: accepted, or the tree is open and its nodes are tested in
        // runs of 64
        int cls = 0, root = 0, count = 0, cost = 0;
        if (t0 + tid < tv.n_trees) {
            root = tv.first[t0 + tid];
            const TreeTest t = tv.test[root];
            cls = classify(t);
            cost = t.cost;
            if (cls != 2) count = tv.first[t0 + tid + 1] - root - 1;
        }
        append(cls, root, cost);
        uint64_t sum;
        const int runs = (count + 63) >> 6;
        const int at = int(block_scan(uint64_t(runs), sh.scan, &sum));
        const int total = __builtin_amdgcn_readfirstlane(int(sum));
        for (int w0 = 0; w0 == 0 || w0 < total; w0 += kChunkCap) {
            for (int r = max(0, w0 - at); r < runs && at + r < w0 + kChunkCap; ++r) {
                sh.chunk_begin[at + r - w0] = root + 1 + 64 * r;
                sh.chunk_end[at + r - w0] = root + 1 + min(count, 64 * r + 64);
            }
            __syncthreads();
            const int here = min(kChunkCap, total - w0);
            const bool final = t0 + kBlock >= tv.n_trees && w0 + kChunkCap >= total;
            int c = wave;
            do {
                if (c < here && room()) {
                    int nd = sh.chunk_begin[c] + lane, end = sh.chunk_end[c];
                    TreeTest t;
                    if (nd < end) t = tv.test[nd];
                    for (;;) {
                        // the next run's tests are loaded while this one's are made
                        const int cn = c + 4;
                        int ndn = 0, endn = 0;
                        TreeTest tn;
                        if (cn < here) {
                            ndn = sh.chunk_begin[cn] + lane;
                            endn = sh.chunk_end[cn];
                            if (ndn < endn) tn = tv.test[ndn];
                        }
                        append(nd < end ? classify(t) : 0, nd, t.cost);
                        c = cn;
                        if (c >= here || !room()) break;
                        nd = ndn;
                        end = endn;
                        t = tn;
                    }
                }
            } while (!meet(c < here, final));
        }
    }
}

}  // namespace envpot
