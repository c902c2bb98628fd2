// gfx950 kernels of the incremental density update: every pair's Hermite
// density D (McMurchie-Davidson fold of the density block with the
// primitives' normalised coefficients and the Hermite expansion
// coefficients E^{ij}_t of the Gaussian product), its far-field
// coefficients h = M_L D, and the same-centre clusters' merged h, written
// into the handle's records in place.  One thread per pair, a wave per
// cluster.
#include <hip/hip_runtime.h>

#include "envpot_internal.h"
#include "update_internal.h"

namespace envpot {
namespace {

constexpr int kUpdBlock = 256;

// Index of Hermite component (t, u, v) among t + u + v <= L (t, then u, then v ascending).
__host__ __device__ constexpr int hidx(int L, int t, int u, int v) {
    const int m = L - t;
    return (L + 1) * (L + 2) * (L + 3) / 6 - (m + 1) * (m + 2) * (m + 3) / 6 + u * (m + 1) - u * (u - 1) / 2 + v;
}

// Cartesian exponents of the components of a shell (x-major: p = x, y, z;
// d = xx, xy, xz, yy, yz, zz), and of the Hermite components of order up to L.
template <int L>
struct Cart {
    int e[(L + 1) * (L + 2) / 2][3] = {};
    constexpr Cart() {
        int k = 0;
        for (int x = L; x >= 0; --x)
            for (int y = L - x; y >= 0; --y, ++k) {
                e[k][0] = x;
                e[k][1] = y;
                e[k][2] = L - x - y;
            }
    }
};
template <int L>
struct Herm {
    int e[kNComp[L]][3] = {};
    constexpr Herm() {
        int k = 0;
        for (int t = 0; t <= L; ++t)
            for (int u = 0; u <= L - t; ++u)
                for (int v = 0; v <= L - t - u; ++v, ++k) {
                    e[k][0] = t;
                    e[k][1] = u;
                    e[k][2] = v;
                }
    }
};

// Hermite expansion coefficients of one direction,
//   x_A^i x_B^j exp(-a x_A^2 - b x_B^2) = sum_t E[i][j][t] Lambda_t(x; p, P),
// raised first in j along i = 0, then in i:
//   E^{i,j+1}_t = E^{ij}_{t-1}/(2p) + X_PB E^{ij}_t + (t+1) E^{ij}_{t+1}   (likewise i with X_PA)
// The angular momenta are template arguments, so every array index is a
// constant and the coefficients live in registers (with run-time indexes
// they lived in scratch memory: 375,461 pairs folded in 0.69 ms, their
// charges in 0.28 ms).
template <int LI, int LJ>
struct Edir {
    double v[LI + 1][LJ + 1][LI + LJ + 1];

    __device__ __forceinline__ double get(int i, int j, int t) const { return (t < 0 || t > i + j) ? 0.0 : v[i][j][t]; }
    __device__ __forceinline__ Edir(double a, double b, double A, double B) {
        const double p = a + b, P = (a * A + b * B) / p;
        const double xpa = P - A, xpb = P - B, h = 0.5 / p, dab = A - B;
        v[0][0][0] = exp(-(a * b / p) * dab * dab);
#pragma unroll
        for (int j = 0; j < LJ; ++j)
#pragma unroll
            for (int t = 0; t <= j + 1; ++t) v[0][j + 1][t] = h * get(0, j, t - 1) + xpb * get(0, j, t) + (t + 1) * get(0, j, t + 1);
#pragma unroll
        for (int i = 0; i < LI; ++i)
#pragma unroll
            for (int j = 0; j <= LJ; ++j)
#pragma unroll
                for (int t = 0; t <= i + j + 1; ++t)
                    v[i + 1][j][t] = h * get(i, j, t - 1) + xpa * get(i, j, t) + (t + 1) * get(i, j, t + 1);
    }
};

struct PairPrim {
    double a, b, p, w2;
    const double* na;  // c N per component of primitive ia
    const double* nb;
    const double* W;   // the block's nI x nJ weights
    const double* A;   // centres
    const double* B;
};

__device__ __forceinline__ PairPrim pair_prim(const UpdateArgs& A, const UpdPair& q, int& lI, int& lJ) {
    const int I = A.blk[2 * q.blk], J = A.blk[2 * q.blk + 1];
    const UpdShell& SI = A.shells[I];
    const UpdShell& SJ = A.shells[J];
    lI = SI.l;
    lJ = SJ.l;
    PairPrim g;
    g.a = A.exps[SI.poff + q.ia];
    g.b = A.exps[SJ.poff + q.ib];
    g.p = g.a + g.b;
    g.w2 = (I == J && q.ia != q.ib) ? 2.0 : 1.0;
    g.na = A.cnorm + SI.noff + int64_t(q.ia) * ((lI + 1) * (lI + 2) / 2);
    g.nb = A.cnorm + SJ.noff + int64_t(q.ib) * ((lJ + 1) * (lJ + 2) / 2);
    g.W = A.W + A.woff[q.blk];
    g.A = SI.A;
    g.B = SJ.A;
    return g;
}

__device__ __forceinline__ double pp32(double p) {
    const double pp = 3.14159265358979323846 / p;
    return pp * sqrt(pp);
}

// The pair's code for its angular momenta (0..2 each).
template <class F>
__device__ __forceinline__ void by_momenta(int lI, int lJ, F f) {
    switch (3 * lI + lJ) {
        case 0: f.template operator()<0, 0>(); break;
        case 1: f.template operator()<0, 1>(); break;
        case 2: f.template operator()<0, 2>(); break;
        case 3: f.template operator()<1, 0>(); break;
        case 4: f.template operator()<1, 1>(); break;
        case 5: f.template operator()<1, 2>(); break;
        case 6: f.template operator()<2, 0>(); break;
        case 7: f.template operator()<2, 1>(); break;
        default: f.template operator()<2, 2>(); break;
    }
}

// Electron count of a pair: the t = u = v = 0 part of the fold.
struct Charge {
    const PairPrim& g;
    double& q;
    template <int LI, int LJ>
    __device__ __forceinline__ void operator()() {
        constexpr Cart<LI> CI{};
        constexpr Cart<LJ> CJ{};
        constexpr int nI = (LI + 1) * (LI + 2) / 2, nJ = (LJ + 1) * (LJ + 2) / 2;
        const Edir<LI, LJ> Ex(g.a, g.b, g.A[0], g.B[0]), Ey(g.a, g.b, g.A[1], g.B[1]), Ez(g.a, g.b, g.A[2], g.B[2]);
#pragma unroll
        for (int x = 0; x < nI; ++x)
#pragma unroll
            for (int y = 0; y < nJ; ++y)
                q += g.w2 * g.W[x * nJ + y] * g.na[x] * g.nb[y] * Ex.v[CI.e[x][0]][CJ.e[y][0]][0] *
                     Ey.v[CI.e[x][1]][CJ.e[y][1]][0] * Ez.v[CI.e[x][2]][CJ.e[y][2]][0];
    }
};

__global__ __launch_bounds__(kUpdBlock) void k_upd_charges(UpdateArgs A) {
    const int64_t i = int64_t(blockIdx.x) * kUpdBlock + threadIdx.x;
    if (i >= A.n_pairs + A.n_drop) return;
    int lI, lJ;
    const PairPrim g = pair_prim(A, A.pairs[i], lI, lJ);
    double q = 0.0;
    by_momenta(lI, lJ, Charge{g, q});
    A.charge[i] = q * pp32(g.p);
}

// D and h of a pair, scaled by (pi/p)^{3/2} and its group's factor, into its
// record, and h in FP64 into the clusters' member list where the pair is one.
struct Fold {
    const UpdateArgs& A;
    const UpdPair& q;
    const PairPrim& g;
    int64_t member;

    template <int LI, int LJ>
    __device__ __forceinline__ void operator()() {
        constexpr int L = LI + LJ, nc = kNComp[L];
        constexpr Cart<LI> CI{};
        constexpr Cart<LJ> CJ{};
        constexpr Herm<L> H{};
        constexpr int nI = (LI + 1) * (LI + 2) / 2, nJ = (LJ + 1) * (LJ + 2) / 2;
        double D[nc];
#pragma unroll
        for (int k = 0; k < nc; ++k) D[k] = 0.0;
        {
            const Edir<LI, LJ> Ex(g.a, g.b, g.A[0], g.B[0]), Ey(g.a, g.b, g.A[1], g.B[1]), Ez(g.a, g.b, g.A[2], g.B[2]);
#pragma unroll
            for (int x = 0; x < nI; ++x)
#pragma unroll
                for (int y = 0; y < nJ; ++y) {
                    const double f = g.w2 * g.W[x * nJ + y] * g.na[x] * g.nb[y];
#pragma unroll
                    for (int t = 0; t <= CI.e[x][0] + CJ.e[y][0]; ++t) {
                        const double ft = f * Ex.v[CI.e[x][0]][CJ.e[y][0]][t];
#pragma unroll
                        for (int u = 0; u <= CI.e[x][1] + CJ.e[y][1]; ++u) {
                            const double fu = ft * Ey.v[CI.e[x][1]][CJ.e[y][1]][u];
#pragma unroll
                            for (int v = 0; v <= CI.e[x][2] + CJ.e[y][2]; ++v)
                                D[hidx(L, t, u, v)] += fu * Ez.v[CI.e[x][2]][CJ.e[y][2]][v];
                        }
                    }
                }
        }
        const double sc = pp32(g.p), s = A.scale[q.group];
#pragma unroll
        for (int k = 0; k < nc; ++k) D[k] = (D[k] * sc) * s;
        const double* M = A.M + kFarMatOff[L];
        uint32_t* r = A.rec + q.word;
        double* rd = reinterpret_cast<double*>(r) + kRec64Head;
        float* rf = reinterpret_cast<float*>(r) + kRec32Head;
        double* hm = member >= 0 ? A.hm + A.moff[member] : nullptr;
#pragma unroll
        for (int i = 0; i < nc; ++i) {
            // the derivative (t, u, v) of 1/R holds monomials of its own
            // degree and parities only: the other entries of M are zero
            double h = 0.0;
#pragma unroll
            for (int j = 0; j < nc; ++j)
                if (H.e[i][0] + H.e[i][1] + H.e[i][2] == H.e[j][0] + H.e[j][1] + H.e[j][2] &&
                    ((H.e[i][0] ^ H.e[j][0]) & 1) == 0 && ((H.e[i][1] ^ H.e[j][1]) & 1) == 0 &&
                    ((H.e[i][2] ^ H.e[j][2]) & 1) == 0)
                    h += M[i * nc + j] * D[j];
            if (A.fp64) rd[i] = h;
            else rf[i] = float(h);
            if (hm) hm[i] = h;
        }
#pragma unroll
        for (int i = 0; i < nc; ++i) {
            if (A.fp64) rd[nc + i] = D[i];
            else rf[nc + i] = float(D[i]);
        }
    }
};

__global__ __launch_bounds__(kUpdBlock) void k_upd_pairs(UpdateArgs A) {
    const int64_t i = int64_t(blockIdx.x) * kUpdBlock + threadIdx.x;
    if (i >= A.n_pairs) return;
    const UpdPair q = A.pairs[i];
    int lI, lJ;
    const PairPrim g = pair_prim(A, q, lI, lJ);
    by_momenta(lI, lJ, Fold{A, q, g, int64_t(A.member_of[i])});
}

// member_of[pair] = its place in the clusters' member list (-1 elsewhere, set before).
__global__ __launch_bounds__(kUpdBlock) void k_member_of(const int64_t* members, int64_t n, int32_t* member_of) {
    const int64_t m = int64_t(blockIdx.x) * kUpdBlock + threadIdx.x;
    if (m < n) member_of[members[m]] = int32_t(m);
}

// Merged far-field coefficients of a cluster: the members' h summed in FP64
// in member order at the cluster's L (same exponents (a, b, c), re-indexed).
// A wave per cluster, a lane per coefficient; the members' L and places are
// read 64 at a time, so the loads of h do not wait for one another (a thread
// per cluster walked its members one dependent load after the other: 2.3 ms
// for 792 clusters of 63,672 members).
constexpr int kClWaves = kUpdBlock / 64;
__global__ __launch_bounds__(kUpdBlock) void k_upd_clusters(UpdateArgs A) {
    const int64_t c = int64_t(blockIdx.x) * kClWaves + (threadIdx.x >> 6);
    if (c >= A.n_clusters) return;
    const int lane = threadIdx.x & 63;
    const UpdCluster cl = A.clusters[c];
    const int Lc = cl.L, ncc = (Lc + 1) * (Lc + 2) * (Lc + 3) / 6;
    int ea = 0, eb = 0, ec = 0;  // this lane's exponents
    if (lane < ncc) {
        int k = lane;
        while (k >= (Lc - ea + 1) * (Lc - ea + 2) / 2) {
            k -= (Lc - ea + 1) * (Lc - ea + 2) / 2;
            ++ea;
        }
        while (k >= Lc - ea - eb + 1) {
            k -= Lc - ea - eb + 1;
            ++eb;
        }
        ec = k;
    }
    double hsum = 0.0;
    for (int64_t m0 = cl.begin; m0 < cl.end; m0 += 64) {
        const int n = int(cl.end - m0 < 64 ? cl.end - m0 : 64);
        int Lv = 0;
        int64_t ov = 0;
        if (lane < n) {
            Lv = A.pairs[A.members[m0 + lane]].L;
            ov = A.moff[m0 + lane];
        }
#pragma unroll 8
        for (int k = 0; k < n; ++k) {
            const int Lm = __shfl(Lv, k);
            const int64_t o = __shfl(ov, k);
            if (lane < ncc && ea + eb + ec <= Lm) hsum += A.hm[o + hidx(Lm, ea, eb, ec)];
        }
    }
    if (lane >= ncc) return;
    uint32_t* r = A.rec + cl.word;
    if (A.fp64) reinterpret_cast<double*>(r)[kClHead64 + lane] = hsum;
    else reinterpret_cast<float*>(r + kClHead32)[lane] = float(hsum);
}

unsigned blocks_for(int64_t n) { return unsigned((n + kUpdBlock - 1) / kUpdBlock); }

// One thread per stored element of a CSR density (ParseArgs).
__global__ __launch_bounds__(kUpdBlock) void k_parse_csr(ParseArgs a) {
    const int64_t k = (int64_t)blockIdx.x * kUpdBlock + threadIdx.x;
    if (k >= a.nnz) return;
    int lo = 0, hi = a.nbf;  // the row: row_ptr[lo] <= k < row_ptr[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (a.row_ptr[mid] <= k) lo = mid;
        else hi = mid;
    }
    const int mu = lo, nu = a.col[k];
    const double v = a.val[k];
    if (nu < 0 || nu >= a.nbf || !isfinite(v)) {
        atomicOr(a.err, 1);
        return;
    }
    if (v == 0.0) return;
    const int I = a.shell_of_bf[mu], J = a.shell_of_bf[nu];
    const int x = mu - a.bf0[I], y = nu - a.bf0[J];
    int64_t b0 = a.adj_begin[I], b1 = a.adj_begin[I + 1];  // first partner >= J
    const int64_t end = b1;
    while (b0 < b1) {
        const int64_t mid = (b0 + b1) >> 1;
        if (a.adj_J[mid] < J) b0 = mid + 1;
        else b1 = mid;
    }
    if (b0 == end || a.adj_J[b0] != J) {
        atomicOr(a.err, 2);
        return;
    }
    const int b = a.adj_blk[b0];
    const int lJ = a.shell_l[a.blk[2 * b + 1]];
    const int nJb = (lJ + 1) * (lJ + 2) / 2;
    if (a.adj_tr[b0]) atomicAdd(&a.Wt[a.woff[b] + y * nJb + x], v);  // element (J, I) of block (I, J)
    else atomicAdd(&a.Wd[a.woff[b] + x * nJb + y], v);
}

// One thread per block weight: symmetry against the transposed element,
// then W = f P s_x s_y (f = 2 off the diagonal blocks).
__global__ __launch_bounds__(kUpdBlock) void k_block_weights(ParseArgs a) {
    const int64_t total = a.woff[a.n_blocks];
    const int64_t e = (int64_t)blockIdx.x * kUpdBlock + threadIdx.x;
    if (e >= total) return;
    int64_t lo = 0, hi = a.n_blocks;  // the block: woff[lo] <= e < woff[hi]
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (a.woff[mid] <= e) lo = mid;
        else hi = mid;
    }
    const int b = (int)lo;
    const int I = a.blk[2 * b], J = a.blk[2 * b + 1];
    const int lJ = a.shell_l[J];
    const int nJ = (lJ + 1) * (lJ + 2) / 2;
    const int64_t r = e - a.woff[b];
    const int x = (int)(r / nJ), y = (int)(r % nJ);
    const double p = a.Wd[e];
    const double q = (I == J) ? a.Wd[a.woff[b] + y * nJ + x] : a.Wt[e];
    if (fabs(p - q) > 1e-10 * (fabs(p) + fabs(q))) atomicOr(a.err, 4);
    const double f = (I == J) ? 1.0 : 2.0;
    a.W[e] = f * p * a.cscale[a.bf0[I] + x] * a.cscale[a.bf0[J] + y];
}

// One workgroup per fragment group: its kept and its dropped pairs'
// charges, each summed by strided threads and then a fixed LDS tree.
__global__ __launch_bounds__(kUpdBlock) void k_group_charges(const double* __restrict__ charge,
                                                             const int64_t* __restrict__ gpb,
                                                             const int64_t* __restrict__ dropb, int64_t n_pairs,
                                                             double* __restrict__ gq) {
    __shared__ double sk[kUpdBlock], sd[kUpdBlock];
    const int g = blockIdx.x, t = threadIdx.x;
    double a = 0.0, d = 0.0;
    for (int64_t k = gpb[g] + t; k < gpb[g + 1]; k += kUpdBlock) a += charge[k];
    for (int64_t j = dropb[g] + t; j < dropb[g + 1]; j += kUpdBlock) d += charge[n_pairs + j];
    sk[t] = a;
    sd[t] = d;
    __syncthreads();
    for (int s = kUpdBlock / 2; s > 0; s >>= 1) {
        if (t < s) {
            sk[t] += sk[t + s];
            sd[t] += sd[t + s];
        }
        __syncthreads();
    }
    if (t == 0) {
        gq[2 * g] = sk[0];
        gq[2 * g + 1] = sd[0];
    }
}

}  // namespace

int launch_group_charges(const double* charge, const int64_t* gpb, const int64_t* dropb, int64_t n_pairs,
                         int n_groups, double* gq, void* stream) {
    if (n_groups <= 0) return 0;
    hipLaunchKernelGGL(k_group_charges, dim3(n_groups), dim3(kUpdBlock), 0, static_cast<hipStream_t>(stream), charge,
                       gpb, dropb, n_pairs, gq);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_parse_csr(const ParseArgs& a, void* stream) {
    if (a.nnz <= 0) return 0;
    hipLaunchKernelGGL(k_parse_csr, dim3(blocks_for(a.nnz)), dim3(kUpdBlock), 0, static_cast<hipStream_t>(stream), a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_block_weights(const ParseArgs& a, int64_t total, void* stream) {
    if (total <= 0) return 0;
    hipLaunchKernelGGL(k_block_weights, dim3(blocks_for(total)), dim3(kUpdBlock), 0,
                       static_cast<hipStream_t>(stream), a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_update_charges(const UpdateArgs& a, void* stream) {
    const int64_t n = a.n_pairs + a.n_drop;
    if (n <= 0) return 0;
    hipLaunchKernelGGL(k_upd_charges, dim3(blocks_for(n)), dim3(kUpdBlock), 0, static_cast<hipStream_t>(stream), a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_update_pairs(const UpdateArgs& a, void* stream) {
    if (a.n_pairs <= 0) return 0;
    hipLaunchKernelGGL(k_upd_pairs, dim3(blocks_for(a.n_pairs)), dim3(kUpdBlock), 0,
                       static_cast<hipStream_t>(stream), a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_member_of(const int64_t* members, int64_t n, int32_t* member_of, void* stream) {
    if (n <= 0) return 0;
    hipLaunchKernelGGL(k_member_of, dim3(blocks_for(n)), dim3(kUpdBlock), 0, static_cast<hipStream_t>(stream), members,
                       n, member_of);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_update_clusters(const UpdateArgs& a, void* stream) {
    if (a.n_clusters <= 0) return 0;
    hipLaunchKernelGGL(k_upd_clusters, dim3(unsigned((a.n_clusters + kClWaves - 1) / kClWaves)), dim3(kUpdBlock), 0,
                       static_cast<hipStream_t>(stream), a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace envpot
