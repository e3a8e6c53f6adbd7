// ccd_dense.hip -- CCD for small model spaces given by dense matrix elements
// (the pairing model of sec. "Developing a CCD code for infinite matter",
// eqs. sppairing / intpairing, or any Hamiltonian in a canonical Hartree-Fock
// basis): the Fock energies of eq. pairingsp, the MBPT2 start of eq. ccdGuess
// and Jacobi sweeps of eq. ccd3 with all eight terms, every sum in a fixed order.
// The quadratic terms go through four intermediates (O(n_h^2 n_p^2 (n_h + n_p)^2)
// a sweep); no symmetry of the elements beyond what eq. ccd3 writes is used.  It is
// a validation path: the plane-wave problems run on the channel-blocked kernels.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "ccd_internal.h"

namespace {

constexpr int kDenseMaxN = 48;

struct Dense {
    const double* v;    // <pq||rs> at (p n + q) vs + r n + s
    const double* eps;  // Fock energies
    int n, nh, np;
    int vs;             // n^2, or n^2 + 1 in LDS (consecutive q in different banks)
};

__device__ __forceinline__ double dv(const Dense& q, int p, int r, int s, int u) {
    return q.v[(p * q.n + r) * q.vs + s * q.n + u];  // (below 48^4: int is enough)
}
// t_ij^ab at ((i nh + j) np + a - nh) np + b - nh
__device__ __forceinline__ int tix(const Dense& q, int i, int j, int a, int b) {
    return ((i * q.nh + j) * q.np + (a - q.nh)) * q.np + (b - q.nh);
}

// ---- a sweep through intermediates --------------------------------------------
// with w = <kl||cd>:
//   W[ij][kl] = 1/2 <kl||ij> + 1/4 sum_cd w t_ij^cd      (HH, QHH: W t_kl^ab)
//   Y[jb][kc] = sum_ld w t_jl^bd                         (QRING: t_ik^ac Y)
//   H[i][l]   = sum_kcd w t_ik^dc, Hk its terms by k     (QHOLE)
//   P[a][d]   = sum_klc w t_lk^ac, Pk its terms by k     (QPART)
struct Mid {
    double *W, *Y, *Hk, *H, *Pk, *P;
};
__host__ __device__ inline size_t mid_doubles(int nh, int np) {
    const size_t o = nh, v = np;
    return o * o * o * o + o * o * v * v + o * o * o + o * o + v * v * o + v * v;
}
__host__ __device__ inline Mid mid_carve(double* p, int nh, int np) {
    const size_t o = nh, v = np;
    Mid m;
    m.W = p;
    m.Y = m.W + o * o * o * o;
    m.Hk = m.Y + o * o * v * v;
    m.H = m.Hk + o * o * o;
    m.Pk = m.H + o * o;
    m.P = m.Pk + v * v * o;
    return m;
}

// Sums over two indices x = 0 .. n1, y = 0 .. n2 by G lanes, lane g taking every
// G-th pair; every lane of the group gets the sum (fixed order).
template <int G, typename F>
__device__ __forceinline__ double dense_sum2(int n1, int n2, int g, F f) {
    double s = 0.0;
    int x = g / n2, y = g - x * n2;
    while (x < n1) {
        s += f(x, y);
        y += G;
        while (y >= n2) { y -= n2; x++; }
    }
#pragma unroll
    for (int o = 1; o < G; o <<= 1) s += __shfl_xor(s, o);
    return s;
}

// the intermediates' sums over two or three indices, shared by nthr threads, G to
// an entry
template <int G>
__device__ void dense_mid(const Dense& q, const double* t, const Mid& M, uint32_t m, unsigned tid, unsigned nthr) {
    const unsigned nh = q.nh, np = q.np;
    const int g = (int)(tid % G);
    const unsigned o2 = nh * nh, v2 = np * np, nW = o2 * o2, nY = o2 * v2, nH = o2 * nh, nP = v2 * nh;
    for (unsigned e = tid / G; e < nW + nY + nH + nP; e += nthr / G) {
        double x = 0.0;
        double* out;
        if (e < nW) {
            const int l = (int)(e % nh), k = (int)(e / nh % nh), j = (int)(e / o2 % nh), i = (int)(e / (o2 * nh));
            if (m & CCD_T_QHH)
                x = dense_sum2<G>(np, np, g, [&](int c, int d) {
                    return dv(q, k, l, nh + c, nh + d) * t[tix(q, i, j, nh + c, nh + d)];
                });
            x = ((m & CCD_T_HH) ? 0.5 * dv(q, k, l, i, j) : 0.0) + 0.25 * x;
            out = M.W + e;
        } else if (e < nW + nY) {
            if (!(m & CCD_T_QRING)) continue;
            const unsigned f = e - nW;
            const int c = nh + (int)(f % np), k = (int)(f / np % nh), b = nh + (int)(f / (np * nh) % np),
                      j = (int)(f / (v2 * nh));
            x = dense_sum2<G>(nh, np, g, [&](int l, int d) { return dv(q, k, l, c, nh + d) * t[tix(q, j, l, b, nh + d)]; });
            out = M.Y + f;
        } else if (e < nW + nY + nH) {
            if (!(m & CCD_T_QHOLE)) continue;
            const unsigned f = e - nW - nY;
            const int k = (int)(f % nh), l = (int)(f / nh % nh), i = (int)(f / o2);
            x = dense_sum2<G>(np, np, g, [&](int c, int d) {
                return dv(q, k, l, nh + c, nh + d) * t[tix(q, i, k, nh + d, nh + c)];
            });
            out = M.Hk + f;
        } else {
            if (!(m & CCD_T_QPART)) continue;
            const unsigned f = e - nW - nY - nH;
            const int k = (int)(f % nh), d = nh + (int)(f / nh % np), a = nh + (int)(f / (nh * np));
            x = dense_sum2<G>(nh, np, g, [&](int l, int c) { return dv(q, k, l, nh + c, d) * t[tix(q, l, k, a, nh + c)]; });
            out = M.Pk + f;
        }
        if (g == 0) *out = x;
    }
}
// H and P from their terms, in order of k
__device__ void dense_fold(const Dense& q, const Mid& M, uint32_t m, unsigned tid, unsigned nthr) {
    const int nh = q.nh;
    const unsigned o2 = nh * nh, v2 = q.np * q.np;
    for (unsigned e = tid; e < o2 + v2; e += nthr) {
        const bool hole = e < o2;
        if (!(m & (hole ? CCD_T_QHOLE : CCD_T_QPART))) continue;
        const double* x = hole ? M.Hk + e * nh : M.Pk + (e - o2) * nh;
        double s = 0.0;
        for (int k = 0; k < nh; k++) s += x[k];
        (hole ? M.H[e] : M.P[e - o2]) = s;
    }
}
// the new amplitude (i, j, a, b), unmixed, by G lanes
template <int G>
__device__ double dense_new(const Dense& q, const double* t, const Mid& M, uint32_t m, int i, int j, int a, int b, int g) {
    if (i == j || a == b) return 0.0;
    const int nh = q.nh, np = q.np;
    double r = dv(q, a, b, i, j);
    if (m & CCD_T_PP)
        r += 0.5 * dense_sum2<G>(np, np, g, [&](int c, int d) {
            return dv(q, a, b, nh + c, nh + d) * t[tix(q, i, j, nh + c, nh + d)];
        });
    if (m & (CCD_T_HH | CCD_T_QHH)) {
        const double* W = M.W + (i * nh + j) * nh * nh;
        r += dense_sum2<G>(nh, nh, g, [&](int k, int l) { return W[k * nh + l] * t[tix(q, k, l, a, b)]; });
    }
    if (m & (CCD_T_RING | CCD_T_QRING)) {
        // P(ij|ab) sum_kc <kb||cj> t_ik^ac and P(ij) sum_kc t_ik^ac Y_kc^jb
        const double* Yj = M.Y + (j * np + b - nh) * nh * np;
        const double* Yi = M.Y + (i * np + b - nh) * nh * np;
        const bool lin = (m & CCD_T_RING) != 0, quad = (m & CCD_T_QRING) != 0;
        r += dense_sum2<G>(nh, np, g, [&](int k, int x) {
            const int c = nh + x;
            const double ta = t[tix(q, i, k, a, c)], tb = t[tix(q, j, k, a, c)];
            double f = 0.0;
            if (lin)
                f = (dv(q, k, b, c, j) * ta - dv(q, k, b, c, i) * tb) -
                    (dv(q, k, a, c, j) * t[tix(q, i, k, b, c)] - dv(q, k, a, c, i) * t[tix(q, j, k, b, c)]);
            if (quad) f += ta * Yj[k * np + x] - tb * Yi[k * np + x];
            return f;
        });
    }
    if (m & CCD_T_QHOLE)
        r -= 0.5 * dense_sum2<G>(1, nh, g, [&](int, int l) {
            return M.H[i * nh + l] * t[tix(q, l, j, a, b)] - M.H[j * nh + l] * t[tix(q, l, i, a, b)];
        });
    if (m & CCD_T_QPART) {
        const double *Pa = M.P + (a - nh) * np, *Pb = M.P + (b - nh) * np;
        r -= 0.5 * dense_sum2<G>(1, np, g, [&](int, int d) {
            return Pa[d] * t[tix(q, i, j, nh + d, b)] - Pb[d] * t[tix(q, i, j, nh + d, a)];
        });
    }
    return r / (q.eps[i] + q.eps[j] - q.eps[a] - q.eps[b]);
}
__device__ __forceinline__ void dense_idx(const Dense& q, unsigned e, int& i, int& j, int& a, int& b) {
    const unsigned np = q.np, ij = e / (np * np), ab = e - ij * np * np;
    a = (int)(ab / np);
    b = q.nh + (int)ab - a * q.np;
    a += q.nh;
    i = (int)(ij / (unsigned)q.nh);
    j = (int)ij - i * q.nh;
}
// fixed-order sum over a block of 64 NW threads; valid in every thread
template <int NW>
__device__ __forceinline__ double dense_block_sum(double x, double* sh) {
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = x;
    __syncthreads();
    double s = 0.0;
    for (int k = 0; k < NW; k++) s += sh[k];
    return s;
}

// Model spaces whose elements, two sets of amplitudes and intermediates fit 150 KiB of
// one compute unit's LDS (all of n <= 10, and n = 11 with at most 6 holes): the sweeps
// of a whole solve in one launch of one block, up to max_sweeps of them.  A sweep is a
// chain of short sums between barriers, where the launches, copy and host read of
// separate kernels bound it at about 65 us.  The
// paper's table, 8 states and 4 particles, a solve of 21 sweeps: 1590 us by a launch
// of k_dense_sweep and a read each, 271 us here; 10 states: 2560 -> 573 us (separate
// launches of these phases: 720).  ctl: the energy before (in), the sweeps run and
// whether the last one met the stop test or left the energy not finite (out); hist:
// the energy after each sweep.
constexpr int kOneThreads = 1024, kOneG = 4;  // lanes per entry
constexpr size_t kOneLds = 150 * 1024;
__host__ __device__ inline size_t one_lds(int n, int nh) {
    const size_t nn = (size_t)n * n, np = n - nh, m = (size_t)nh * nh * np * np;
    return 8 * (nn * (nn + 1) + 2 * m + mid_doubles(nh, (int)np) + n);
}
__global__ void __launch_bounds__(kOneThreads) k_dense_one(Dense g, double* tg, double alpha, uint32_t m, double tol,
                                                           double tol_rel, int max_sweeps, double* ctl, double* hist) {
    extern __shared__ __attribute__((aligned(16))) double dl[];
    __shared__ double sh[kOneThreads / 64];
    const int n = g.n, nh = g.nh, np = g.np;
    const unsigned nn = n * n, mm = nh * nh * np * np;
    double* v = dl;
    double* t[2] = {v + nn * (nn + 1), v + nn * (nn + 1) + mm};
    const Mid M = mid_carve(t[1] + mm, nh, np);
    double* eps = t[1] + mm + mid_doubles(nh, np);
    for (unsigned e = threadIdx.x; e < nn * nn; e += kOneThreads) v[e / nn * (nn + 1) + e % nn] = g.v[e];
    for (unsigned e = threadIdx.x; e < mm; e += kOneThreads) t[0][e] = tg[e];
    for (int e = threadIdx.x; e < n; e += kOneThreads) eps[e] = g.eps[e];
    Dense q = g;
    q.v = v;
    q.eps = eps;
    q.vs = (int)nn + 1;
    __syncthreads();
    double old = ctl[0];
    int cur = 0, s = 0;
    bool stop = false;
    while (s < max_sweeps && !stop) {
        dense_mid<kOneG>(q, t[cur], M, m, threadIdx.x, kOneThreads);
        __syncthreads();
        dense_fold(q, M, m, threadIdx.x, kOneThreads);
        __syncthreads();
        double es = 0.0;
        const int g = threadIdx.x % kOneG;
        for (unsigned e = threadIdx.x / kOneG; e < mm; e += kOneThreads / kOneG) {
            int i, j, a, b;
            dense_idx(q, e, i, j, a, b);
            const double x = alpha * dense_new<kOneG>(q, t[cur], M, m, i, j, a, b, g) + (1.0 - alpha) * t[cur][e];
            if (g == 0) {
                t[cur ^ 1][e] = x;
                es += dv(q, i, j, a, b) * x;
            }
        }
        const double en = 0.25 * dense_block_sum<kOneThreads / 64>(es, sh);
        __syncthreads();
        cur ^= 1;
        if (threadIdx.x == 0) hist[s] = en;
        s++;
        stop = !isfinite(en) || ((tol > 0.0 || tol_rel > 0.0) && fabs(en - old) < tol + tol_rel * fabs(en));
        old = en;
    }
    for (unsigned e = threadIdx.x; e < mm; e += kOneThreads) tg[e] = t[cur][e];
    if (threadIdx.x == 0) {
        ctl[0] = old;
        ctl[1] = (double)s;
        ctl[2] = stop ? 1.0 : 0.0;
    }
}

// Larger model spaces: the same phases as launches, O(n_h^4 n_p^2) + O(n_h^2 n_p^4) +
// O(n_h^3 n_p^3), sixteen lanes to an entry, since one lane's sum is a serial chain
// of loads.  16 states, 4 particles, a solve of 24 sweeps: 7437 us without
// intermediates, 2426 with one lane to an entry, 696 with sixteen; one sweep of 38
// states, 14 particles: 104.9 -> 1.4 ms with its uploads.  Bound by the launches up
// to about 20 states.
constexpr int kLanes = 16;
__global__ void __launch_bounds__(256) k_dense_mid(Dense q, const double* t, Mid M, uint32_t m) {
    dense_mid<kLanes>(q, t, M, m, blockIdx.x * 256 + threadIdx.x, gridDim.x * 256);
}
__global__ void __launch_bounds__(256) k_dense_fold(Dense q, Mid M, uint32_t m) {
    dense_fold(q, M, m, blockIdx.x * 256 + threadIdx.x, gridDim.x * 256);
}
__global__ void __launch_bounds__(256) k_dense_new(Dense q, const double* t, double* tn, Mid M, double alpha,
                                                   uint32_t m, double* part) {
    __shared__ double sh[4];
    const unsigned mm = q.nh * q.nh * q.np * q.np;
    const int g = threadIdx.x % kLanes;
    double es = 0.0;
    for (unsigned e = (blockIdx.x * 256 + threadIdx.x) / kLanes; e < mm; e += gridDim.x * 256 / kLanes) {
        int i, j, a, b;
        dense_idx(q, e, i, j, a, b);
        const double x = alpha * dense_new<kLanes>(q, t, M, m, i, j, a, b, g) + (1.0 - alpha) * t[e];
        if (g == 0) {
            tn[e] = x;
            es += dv(q, i, j, a, b) * x;
        }
    }
    es = dense_block_sum<4>(es, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = 0.25 * es;
}
// the energy from the blocks' parts
__global__ void __launch_bounds__(256) k_dense_sum(const double* part, int n, double* e) {
    __shared__ double sh[4];
    double s = 0.0;
    for (int k = threadIdx.x; k < n; k += 256) s += part[k];
    s = dense_block_sum<4>(s, sh);
    if (threadIdx.x == 0) *e = s;
}

__global__ void __launch_bounds__(256) k_dense_mbpt2(Dense q, double* t) {
    const size_t m = (size_t)q.nh * q.nh * q.np * q.np;
    for (size_t e = blockIdx.x * 256 + threadIdx.x; e < m; e += (size_t)gridDim.x * 256) {
        const int b = q.nh + (int)(e % q.np), a = q.nh + (int)((e / q.np) % q.np);
        const int j = (int)((e / ((size_t)q.np * q.np)) % q.nh), i = (int)(e / ((size_t)q.np * q.np * q.nh));
        t[e] = dv(q, a, b, i, j) / (q.eps[i] + q.eps[j] - q.eps[a] - q.eps[b]);
    }
}

// ---- a sweep without intermediates ---------------------------------------------
// for work areas that hold two sets of amplitudes and no intermediates: O(n_h^4 n_p^4)
// the right-hand side of eq. ccd3 for (i, j, a, b) from amplitudes t
__device__ double ccd3_rhs(const Dense& q, const double* t, int i, int j, int a, int b, uint32_t m) {
    const int nh = q.nh, n = q.n;
    double r = dv(q, a, b, i, j);
    if (m & CCD_T_PP) {
        double s = 0.0;
        for (int c = nh; c < n; c++)
            for (int d = nh; d < n; d++) s += dv(q, a, b, c, d) * t[tix(q, i, j, c, d)];
        r += 0.5 * s;
    }
    if (m & CCD_T_HH) {
        double s = 0.0;
        for (int k = 0; k < nh; k++)
            for (int l = 0; l < nh; l++) s += dv(q, k, l, i, j) * t[tix(q, k, l, a, b)];
        r += 0.5 * s;
    }
    if (m & CCD_T_RING) {
        // P(ij|ab) f(i,j,a,b) = f(ijab) - f(jiab) - f(ijba) + f(jiba),
        // f = sum_kc <kb||cj> t_ik^ac
        auto f = [&](int i_, int j_, int a_, int b_) {
            double s = 0.0;
            for (int k = 0; k < nh; k++)
                for (int c = nh; c < n; c++) s += dv(q, k, b_, c, j_) * t[tix(q, i_, k, a_, c)];
            return s;
        };
        r += f(i, j, a, b) - f(j, i, a, b) - f(i, j, b, a) + f(j, i, b, a);
    }
    if (m & (CCD_T_QHH | CCD_T_QRING | CCD_T_QHOLE | CCD_T_QPART)) {
        double s_hh = 0.0, s_ring = 0.0, s_hole = 0.0, s_part = 0.0;
        for (int k = 0; k < nh; k++)
            for (int l = 0; l < nh; l++)
                for (int c = nh; c < n; c++)
                    for (int d = nh; d < n; d++) {
                        const double w = dv(q, k, l, c, d);
                        if (w == 0.0) continue;
                        if (m & CCD_T_QHH) s_hh += w * t[tix(q, i, j, c, d)] * t[tix(q, k, l, a, b)];
                        if (m & CCD_T_QRING)
                            s_ring += w * (t[tix(q, i, k, a, c)] * t[tix(q, j, l, b, d)] -
                                           t[tix(q, j, k, a, c)] * t[tix(q, i, l, b, d)]);
                        if (m & CCD_T_QHOLE)
                            s_hole += w * (t[tix(q, i, k, d, c)] * t[tix(q, l, j, a, b)] -
                                           t[tix(q, j, k, d, c)] * t[tix(q, l, i, a, b)]);
                        if (m & CCD_T_QPART)
                            s_part += w * (t[tix(q, l, k, a, c)] * t[tix(q, i, j, d, b)] -
                                           t[tix(q, l, k, b, c)] * t[tix(q, i, j, d, a)]);
                    }
        r += 0.25 * s_hh + s_ring - 0.5 * s_hole - 0.5 * s_part;
    }
    return r;
}

__global__ void __launch_bounds__(256) k_dense_sweep(Dense q, const double* t, double* tn, double alpha, uint32_t m) {
    const size_t mm = (size_t)q.nh * q.nh * q.np * q.np;
    for (size_t e = blockIdx.x * 256 + threadIdx.x; e < mm; e += (size_t)gridDim.x * 256) {
        const int b = q.nh + (int)(e % q.np), a = q.nh + (int)((e / q.np) % q.np);
        const int j = (int)((e / ((size_t)q.np * q.np)) % q.nh), i = (int)(e / ((size_t)q.np * q.np * q.nh));
        double tnew = 0.0;
        if (i != j && a != b) {
            const double r = ccd3_rhs(q, t, i, j, a, b, m);
            tnew = r / (q.eps[i] + q.eps[j] - q.eps[a] - q.eps[b]);
        }
        tn[e] = alpha * tnew + (1.0 - alpha) * t[e];
    }
}

// 1/4 sum <ij||ab> t_ij^ab: one partial per block (fixed order in the block)
__global__ void __launch_bounds__(256) k_dense_energy(Dense q, const double* t, double* part) {
    __shared__ double sh[256];
    const size_t mm = (size_t)q.nh * q.nh * q.np * q.np;
    const size_t e = blockIdx.x * 256 + threadIdx.x;
    double x = 0.0;
    if (e < mm) {
        const int b = q.nh + (int)(e % q.np), a = q.nh + (int)((e / q.np) % q.np);
        const int j = (int)((e / ((size_t)q.np * q.np)) % q.nh), i = (int)(e / ((size_t)q.np * q.np * q.nh));
        x = dv(q, i, j, a, b) * t[e];
    }
    sh[threadIdx.x] = x;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = 0.25 * sh[0];
}

// least: what the sweep without intermediates needs
struct DenseLayout {
    size_t v, eps, t0, t1, part, least, mid, ctl, total;
    int nblk;
};
constexpr int kDenseChunk = 64;    // sweeps between two host reads
constexpr int kDenseParts = 4096;  // energy parts of a sweep

DenseLayout dense_layout(int n, int nh) {
    const size_t np = (size_t)(n - nh), m = (size_t)nh * nh * np * np;
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    DenseLayout L;
    L.nblk = (int)((m + 255) / 256);
    L.v = 0;
    L.eps = up(L.v + 8 * (size_t)n * n * n * n);
    L.t0 = up(L.eps + 8 * (size_t)n);
    L.t1 = up(L.t0 + 8 * m);
    L.part = up(L.t1 + 8 * m);
    L.least = up(L.part + 8 * (size_t)L.nblk);
    L.mid = L.least;
    L.ctl = up(L.mid + 8 * mid_doubles(nh, (int)np));
    L.total = up(L.ctl + 8 * (size_t)(8 + kDenseChunk + kDenseParts));
    return L;
}

#define DENSE_TRY(x)                                                                 \
    do {                                                                             \
        hipError_t e_ = (x);                                                         \
        if (e_ != hipSuccess) {                                                      \
            ccd::set_error(std::string("ccd_dense_solve: ") + hipGetErrorString(e_)); \
            return CCD_EHIP;                                                         \
        }                                                                            \
    } while (0)

}  // namespace

extern "C" ccd_status ccd_dense_workspace_size(int32_t n, int32_t n_holes, size_t* bytes) {
    if (!bytes || n < 2 || n > kDenseMaxN || n_holes < 1 || n_holes >= n) {
        ccd::set_error("ccd_dense_workspace_size: need 2 <= n <= 48 and 1 <= n_holes < n");
        return CCD_EINVAL;
    }
    *bytes = dense_layout(n, n_holes).total;
    return CCD_OK;
}

// The work area of ccd_dense_solve_static (8 MiB per GPU; see
// scratch_address below for how host code reaches it).
constexpr size_t kDenseScratchBytes = CCD_DENSE_STATIC_BYTES;
static __device__ __align__(256) unsigned char scratch[kDenseScratchBytes];

namespace {

// The solve itself, on a work area `dev_work` of at least dense_layout(n,
// n_holes).least bytes (sizes and options already checked); from .total bytes on
// it goes through the intermediates.  Every byte of the area that a kernel reads
// is written first in this call: v and eps by the uploads, t0 by the MBPT2 kernel,
// t1, the intermediates, the energy partials and the energies by the sweeps'
// kernels, so a reused area needs no clearing.
ccd_status dense_solve_on(const double* h, const double* v, int32_t n, int32_t n_holes,
                          const ccd_solver_opts* o, void* dev_work, size_t work_bytes, hipStream_t s, double* e_ref,
                          double* e_mbpt2, double* e_ccd, int32_t* sweeps, double* e_hist) {
    ccd_status st = CCD_OK;
    const int nh = n_holes, np = n - n_holes;
    auto V = [&](int p, int q, int r, int s) { return v[(((size_t)p * n + q) * n + r) * n + s]; };
    // Fock energies (eq. pairingsp) and the reference energy
    std::vector<double> eps(n);
    for (int p = 0; p < n; p++) {
        double s = h[p];
        for (int i = 0; i < nh; i++) s += V(p, i, p, i);
        eps[p] = s;
    }
    double eref = 0.0, pot = 0.0;
    for (int i = 0; i < nh; i++) eref += h[i];
    for (int i = 0; i < nh; i++)
        for (int j = 0; j < nh; j++) pot += V(i, j, i, j);
    eref += 0.5 * pot;
    for (int i = 0; i < nh; i++)
        for (int a = nh; a < n; a++)
            if (!(eps[i] < eps[a])) {
                ccd::set_error("ccd_dense_solve: a hole lies at or above a particle in Fock energy");
                return CCD_EINVAL;
            }
    const DenseLayout L = dense_layout(n, nh);
    char* base = (char*)dev_work;
    DENSE_TRY(hipMemcpyAsync(base + L.v, v, 8 * (size_t)n * n * n * n, hipMemcpyHostToDevice, s));
    DENSE_TRY(hipMemcpyAsync(base + L.eps, eps.data(), 8 * (size_t)n, hipMemcpyHostToDevice, s));
    Dense q;
    q.v = (const double*)(base + L.v);
    q.eps = (const double*)(base + L.eps);
    q.n = n; q.nh = nh; q.np = np; q.vs = n * n;
    double* t[2] = {(double*)(base + L.t0), (double*)(base + L.t1)};
    double* part = (double*)(base + L.part);
    std::vector<double> ph(L.nblk);
    auto energy = [&](const double* tt, double& e) -> ccd_status {
        k_dense_energy<<<L.nblk, 256, 0, s>>>(q, tt, part);
        DENSE_TRY(hipGetLastError());
        DENSE_TRY(hipMemcpyAsync(ph.data(), part, 8 * (size_t)L.nblk, hipMemcpyDeviceToHost, s));
        DENSE_TRY(hipStreamSynchronize(s));
        e = 0.0;
        for (int b = 0; b < L.nblk; b++) e += ph[b];
        return CCD_OK;
    };
    const int grid = std::min(L.nblk, 4096);
    k_dense_mbpt2<<<grid, 256, 0, s>>>(q, t[0]);
    DENSE_TRY(hipGetLastError());
    double e2 = 0.0;
    if ((st = energy(t[0], e2)) != CCD_OK) return st;
    if (e_ref) *e_ref = eref;
    if (e_mbpt2) *e_mbpt2 = e2;
    if (e_hist)
        for (int k = 0; k < o->max_iter; k++) e_hist[k] = NAN;
    double e = e2;
    int cur = 0, done = 0;
    bool conv = false;
    const bool test = o->tol > 0.0 || o->tol_rel > 0.0;
    bool bad = false;
    // one energy more; true when the iteration ends there
    auto step = [&](double en) {
        if (e_hist) e_hist[done] = en;
        done++;
        const double de = std::fabs(en - e);
        e = en;
        bad = !std::isfinite(en);
        conv = !bad && test && de < o->tol + o->tol_rel * std::fabs(en);
        return bad || conv;
    };
    if (work_bytes < L.total) {  // no room for the intermediates
        for (bool end = false; done < o->max_iter && !end;) {
            k_dense_sweep<<<grid, 256, 0, s>>>(q, t[cur], t[cur ^ 1], o->mixing, o->terms);
            DENSE_TRY(hipGetLastError());
            cur ^= 1;
            double en = 0.0;
            if ((st = energy(t[cur], en)) != CCD_OK) return st;
            end = step(en);
        }
    } else {
        const Mid M = mid_carve((double*)(base + L.mid), nh, np);
        double* ctl = (double*)(base + L.ctl);
        double* hist = ctl + 8;
        double* parts = hist + kDenseChunk;
        double hb[8 + kDenseChunk];
        const size_t lds = one_lds(n, nh);
        const bool one = lds <= kOneLds;
        if (one) {
            DENSE_TRY(hipFuncSetAttribute((const void*)k_dense_one, hipFuncAttributeMaxDynamicSharedMemorySize,
                                          (int)kOneLds));
            DENSE_TRY(hipMemcpyAsync(ctl, &e2, 8, hipMemcpyHostToDevice, s));
        }
        // sweeps past the one that ends the iteration are thrown away: as many
        // between two reads (about 20 us) as cost no more than they save
        const double work = (double)nh * nh * np * np * ((double)np * np + (double)nh * nh + 8.0 * nh * np);
        const int chunk = one ? kDenseChunk : work < 3e7 ? 4 : 1;
        const size_t nmid = mid_doubles(nh, np);
        const int gm = (int)std::min<size_t>((kLanes * nmid + 255) / 256, 4096);
        const int gn = (int)std::min<size_t>(((size_t)kLanes * nh * nh * np * np + 255) / 256, kDenseParts);
        const int gf = ((nh * nh + np * np) + 255) / 256;
        for (bool end = false; done < o->max_iter && !end;) {
            int n_sw = std::min(chunk, o->max_iter - done);
            if (one) {
                k_dense_one<<<1, kOneThreads, lds, s>>>(q, t[0], o->mixing, o->terms, o->tol, o->tol_rel, n_sw, ctl, hist);
            } else {
                for (int k = 0; k < n_sw; k++) {
                    k_dense_mid<<<gm, 256, 0, s>>>(q, t[cur], M, o->terms);
                    k_dense_fold<<<gf, 256, 0, s>>>(q, M, o->terms);
                    k_dense_new<<<gn, 256, 0, s>>>(q, t[cur], t[cur ^ 1], M, o->mixing, o->terms, parts);
                    k_dense_sum<<<1, 256, 0, s>>>(parts, gn, hist + k);
                    cur ^= 1;
                }
            }
            DENSE_TRY(hipGetLastError());
            DENSE_TRY(hipMemcpyAsync(hb, ctl, 8 * (size_t)(8 + n_sw), hipMemcpyDeviceToHost, s));
            DENSE_TRY(hipStreamSynchronize(s));
            if (one) n_sw = (int)hb[1];
            for (int k = 0; k < n_sw && !end; k++) end = step(hb[8 + k]);
        }
    }
    if (bad) {
        if (e_ccd) *e_ccd = e;
        if (sweeps) *sweeps = done;
        ccd::set_error("ccd_dense_solve: correlation energy is not finite");
        return CCD_DIVERGED;
    }
    if (e_ccd) *e_ccd = e;
    if (sweeps) *sweeps = done;
    return test && !conv ? CCD_NOT_CONVERGED : CCD_OK;
}

ccd_status dense_check_opts(const char* who, const double* h, const double* v, const ccd_solver_opts* o) {
    if (!h || !v || !o) {
        ccd::set_error(std::string(who) + ": need h, v and opts");
        return CCD_EINVAL;
    }
    if (!(o->mixing > 0.0 && o->mixing <= 1.0) || o->max_iter < 1) {
        ccd::set_error(std::string(who) + ": need 0 < mixing <= 1 and max_iter >= 1");
        return CCD_EINVAL;
    }
    return CCD_OK;
}

// Work area of ccd_dense_solve_static: one per GPU, alive until the process
// ends.  Host code never passes `scratch` itself to a kernel or a copy (on the
// host the name is only a stand-in); it uses the device address that
// hipGetSymbolAddress returns for the current device, kept per device.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_addr[kMaxDevices] = {};

ccd_status scratch_address(void** out) {
    int dev = -1;
    DENSE_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) {
        ccd::set_error("ccd_dense_solve_static: device index out of range");
        return CCD_EINVAL;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_addr[dev]) {
        void* p = nullptr;
        DENSE_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p || (((uintptr_t)p) & 255)) {
            ccd::set_error("ccd_dense_solve_static: scratch array has no aligned device address");
            return CCD_EHIP;
        }
        g_scratch_addr[dev] = p;
    }
    *out = g_scratch_addr[dev];
    return CCD_OK;
}

}  // namespace

extern "C" ccd_status ccd_dense_solve(const double* h, const double* v, int32_t n, int32_t n_holes,
                                      const ccd_solver_opts* o, void* dev_work, size_t work_bytes, void* hip_stream,
                                      double* e_ref, double* e_mbpt2, double* e_ccd, int32_t* sweeps,
                                      double* e_hist) {
    size_t need = 0;
    ccd_status st = ccd_dense_workspace_size(n, n_holes, &need);
    if (st != CCD_OK) return st;
    if ((st = dense_check_opts("ccd_dense_solve", h, v, o)) != CCD_OK) return st;
    if (!dev_work || (((uintptr_t)dev_work) & 255) || work_bytes < dense_layout(n, n_holes).least) {
        ccd::set_error("ccd_dense_solve: need a 256-byte aligned work buffer of ccd_dense_workspace_size bytes");
        return CCD_EINVAL;
    }
    return dense_solve_on(h, v, n, n_holes, o, dev_work, work_bytes, (hipStream_t)hip_stream, e_ref, e_mbpt2, e_ccd,
                          sweeps, e_hist);
}

extern "C" ccd_status ccd_dense_solve_static(const double* h, const double* v, int32_t n, int32_t n_holes,
                                             const ccd_solver_opts* o, void* hip_stream, double* e_ref,
                                             double* e_mbpt2, double* e_ccd, int32_t* sweeps, double* e_hist) {
    size_t need = 0;
    ccd_status st = ccd_dense_workspace_size(n, n_holes, &need);
    if (st != CCD_OK) return st;
    if ((st = dense_check_opts("ccd_dense_solve_static", h, v, o)) != CCD_OK) return st;
    need = dense_layout(n, n_holes).least;
    if (need > kDenseScratchBytes) {
        ccd::set_error("ccd_dense_solve_static: this model space needs " + std::to_string(need) +
                       " bytes of work area, more than the " + std::to_string(kDenseScratchBytes) +
                       " of the static one; use ccd_dense_solve with a caller buffer");
        return CCD_EINVAL;
    }
    void* work = nullptr;
    if ((st = scratch_address(&work)) != CCD_OK) return st;
    return dense_solve_on(h, v, n, n_holes, o, work, kDenseScratchBytes, (hipStream_t)hip_stream, e_ref, e_mbpt2,
                          e_ccd, sweeps, e_hist);
}
