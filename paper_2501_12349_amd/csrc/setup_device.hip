// Setup on the device (Section 3.1), for meshes whose nodes move between
// searches: element AABB and OBB (Sections 3.1.1, 3.1.2, 4.1, 4.2) and the
// local map (Section 3.1.3), recomputed from the device copy of the nodes.
//
// Every quantity is computed with the operations of the host setup in the
// same order, and this file is compiled without floating-point contraction,
// so the boxes and the map equal those of fpts_setup on the same nodes bit
// for bit.  One wave per element: sums whose order fixes the rounding take
// a lane each; the Chebyshev-grid evaluations of the bounds run across
// lanes (each lane one grid point, the reduction is a min/max).
#include <cmath>
#include <vector>

#include "fpts_internal.hpp"

namespace fpts {
namespace {

constexpr int kLanes = 64;

// std::min / std::max semantics (first argument on ties)
__device__ __forceinline__ double mn(double a, double b) { return (b < a) ? b : a; }
__device__ __forceinline__ double mx(double a, double b) { return (a < b) ? b : a; }

__device__ __forceinline__ void wave_minmax(double &lo, double &hi)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo = mn(lo, __shfl_xor(lo, o));
        hi = mx(hi, __shfl_xor(hi, o));
    }
}

// The functions whose bounds make an element's box, per coordinate: the
// edges of a quad (4), the faces of a hex (6), the whole patch of a surface
// quad, the whole curve of a line element (1); each a function of BD = 1 or
// 2 parameters.  Function fn belongs to coordinate fn % D and side fn / D.
template <int D, int R, int N>
struct Sides {
    static constexpr int BD = (R == 3 || (R == 2 && D == 3)) ? 2 : 1;
    static constexpr int NS = R == 3 ? 6 : (R == 2 && D == 2) ? 4 : 1;   // sides
    static constexpr int NF = NS * D;
    static constexpr int PTS = BD == 2 ? N * N : N;   // nodes of a side
    static constexpr int NP = R == 3 ? N * N * N : R == 2 ? N * N : N;
    // bounds of two parameters: the sides go to G groups of NQ functions,
    // one group per lane and grid point; LDS keeps a node's NQ values
    // together (an even number of doubles, for 16-byte reads)
    static constexpr int G = R == 3 ? 2 : 1;
    static constexpr int NQ = NF / G;
    static constexpr int PQ = (NQ + 1) / 2 * 2;
    static constexpr int VALS = BD == 2 ? PTS * G * PQ : PTS * NF;
    static constexpr int MOM = BD == 2 ? 4 : 2;       // Legendre moments per function
    // node of the element at node idx of side sd
    __device__ static __forceinline__ int node(int sd, int idx)
    {
        if (NS == 1) return idx;
        const int q = (sd & 1) ? N - 1 : 0, t = sd >> 1;
        if (R == 3) {
            const int x0 = idx % N, x1 = idx / N;
            return t == 0   ? x0 + N * (x1 + N * q)
                   : t == 1 ? x0 + N * (q + N * x1)
                            : q + N * (x0 + N * x1);
        }
        return t == 0 ? idx + N * q : q + N * idx;
    }
    // where the value of function (side sd, coordinate c) at node idx is kept
    __device__ static __forceinline__ int at(int sd, int c, int idx)
    {
        if (BD == 1) return (sd * D + c) * PTS + idx;
        const int i = idx % N, j = idx / N;
        return ((i * N + j) * G + (sd & (G - 1))) * PQ + (sd / G) * D + c;
    }
};

// Bounds of an element's NF side functions, whose nodal values are in
// val (LDS), reduced to lo / hi per coordinate (uniform over the wave): the
// (bi)linear Legendre part removed, basis bounds at the M Chebyshev points
// of each parameter (eqs. eq_1D_bound_final_1/2, eq_2D_function_bound_1/2).
// The moments are sums whose order fixes the rounding: one lane per
// (function, moment).  The grid evaluations are one lane per grid point and
// group of functions, so that the products of the basis bounds at a node are
// formed once for the NQ functions of the group.
template <int D, int R, int N>
__device__ __forceinline__ void side_bounds(const BoundTables &T, double *val, double *mom,
                                            int lane, double (&lo)[3], double (&hi)[3])
{
    typedef Sides<D, R, N> S;
    constexpr int M = 2 * N;
    __syncthreads();
    for (int id = lane; id < S::NF * S::MOM; id += kLanes) {
        const int q = id % S::MOM, fn = id / S::MOM, sd = fn / D, c = fn % D;
        double a = 0.0;
        if constexpr (S::BD == 2) {
            double m0[N], m1[N];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                m0[i] = (q & 1) ? T.mom1[i] : T.mom0[i];
                m1[i] = (q & 2) ? T.mom1[i] : T.mom0[i];
            }
            const double *u = val + S::at(sd, c, 0);
#pragma unroll
            for (int j = 0; j < N; ++j) {
#pragma unroll
                for (int i = 0; i < N; ++i)
                    a += u[(i * N + j) * S::G * S::PQ] * m0[i] * m1[j];
                __builtin_amdgcn_sched_barrier(0);
            }
            mom[id] = a * (q == 0 ? 0.25 : q == 3 ? 2.25 : 0.75);
        } else {
#pragma unroll
            for (int i = 0; i < N; ++i)
                a += val[S::at(sd, c, i)] * (q ? T.mom1[i] : T.mom0[i]);
            mom[id] = a * (q ? 1.5 : 0.5);
        }
    }
    __syncthreads();
    for (int id = lane; id < S::NF * S::PTS; id += kLanes) {
        const int fn = id / S::PTS, idx = id % S::PTS, sd = fn / D, c = fn % D;
        const double *a = mom + fn * S::MOM;
        const int k = S::at(sd, c, idx);
        if constexpr (S::BD == 2) {
            const int i = idx % N, j = idx / N;
            val[k] = val[k] - (a[0] + a[1] * T.z[i] + a[2] * T.z[j] + a[3] * T.z[i] * T.z[j]);
        } else {
            val[k] = val[k] - (a[0] + a[1] * T.z[idx]);
        }
    }
    __syncthreads();
    double l[D], h[D];
#pragma unroll
    for (int c = 0; c < D; ++c) {
        l[c] = INFINITY;
        h[c] = -INFINITY;
    }
    if constexpr (S::BD == 2) {
#pragma unroll 1
        for (int it = lane; it < M * M * S::G; it += kLanes) {
            const int gp = it / S::G, grp = it % S::G, k = gp % M, ll = gp / M;
            double sl[S::NQ], sh[S::NQ], vlo[N], vhi[N];
#pragma unroll
            for (int f = 0; f < S::NQ; ++f) {
                const double *a = mom + ((f / D * S::G + grp) * D + f % D) * 4;
                sl[f] = a[0] + a[1] * T.eta[k] + a[2] * T.eta[ll] + a[3] * T.eta[k] * T.eta[ll];
                sh[f] = sl[f];
            }
#pragma unroll
            for (int j = 0; j < N; ++j) {
                vlo[j] = T.vlo[j * M + ll];
                vhi[j] = T.vhi[j * M + ll];
            }
            const double *w = val + grp * S::PQ;
#pragma unroll 1
            for (int i = 0; i < N; ++i) {
                const double ulo = T.vlo[i * M + k], uhi = T.vhi[i * M + k];
#pragma unroll
                for (int j = 0; j < N; ++j, w += S::G * S::PQ) {
                    const double p1 = ulo * vlo[j], p2 = ulo * vhi[j], p3 = uhi * vlo[j],
                                 p4 = uhi * vhi[j];
                    const double pn = fmin(fmin(p1, p2), fmin(p3, p4));
                    const double px = fmax(fmax(p1, p2), fmax(p3, p4));
                    // the smaller of w pn and w px is w pn for w >= 0, w px else
#pragma unroll
                    for (int f = 0; f < S::NQ; ++f) {
                        const double a = w[f] * pn, b = w[f] * px;
                        sl[f] += fmin(a, b);
                        sh[f] += fmax(a, b);
                    }
                    if (j % 2) __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int f = 0; f < S::NQ; ++f) {
                l[f % D] = mn(l[f % D], sl[f]);
                h[f % D] = mx(h[f % D], sh[f]);
            }
        }
    } else {
        for (int it = lane; it < M * S::NF; it += kLanes) {
            const int fn = it / M, j = it % M, cc = fn % D;
            double a = mom[2 * fn] + mom[2 * fn + 1] * T.eta[j], b = a;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const double w = val[fn * S::PTS + i];
                const double x = w * T.vlo[i * M + j], y = w * T.vhi[i * M + j];
                a += mn(x, y);
                b += mx(x, y);
            }
#pragma unroll
            for (int c = 0; c < D; ++c)
                if (cc == c) {
                    l[c] = mn(l[c], a);
                    h[c] = mx(h[c], b);
                }
        }
    }
#pragma unroll
    for (int c = 0; c < D; ++c) {
        wave_minmax(l[c], h[c]);
        lo[c] = l[c];
        hi[c] = h[c];
    }
}

// Thin-extent rule (manifolds; reference: the smallest other extent, the
// largest for lines) and expansion by tol of the extent in total.
__device__ void finish_d(int D, int R, double tol, double *lo, double *hi, const double *len)
{
    double L[3];
    for (int d = 0; d < D; ++d) L[d] = hi[d] - lo[d];
    if (R < D) {
        double P[3];
        for (int d = 0; d < D; ++d) P[d] = L[d] * len[d];
        for (int d = 0; d < D; ++d) {
            double ref = R == 1 ? 0.0 : INFINITY;
            for (int q = 0; q < D; ++q)
                if (q != d) ref = R == 1 ? mx(ref, P[q]) : mn(ref, P[q]);
            const double need = tol * ref / len[d];
            if (L[d] < need) {
                const double c = 0.5 * (lo[d] + hi[d]);
                lo[d] = c - 0.5 * need;
                hi[d] = c + 0.5 * need;
                L[d] = need;
            }
        }
    }
    for (int d = 0; d < D; ++d) {
        lo[d] -= 0.5 * tol * L[d];
        hi[d] += 0.5 * tol * L[d];
    }
}

__device__ bool invert_d(int D, const double *A, double *I)
{
    if (D == 2) {
        const double det = A[0] * A[3] - A[1] * A[2];
        if (!(det != 0.0) || !isfinite(det)) return false;
        I[0] = A[3] / det;
        I[1] = -A[1] / det;
        I[2] = -A[2] / det;
        I[3] = A[0] / det;
        return true;
    }
    const double c00 = A[4] * A[8] - A[5] * A[7], c01 = A[5] * A[6] - A[3] * A[8],
                 c02 = A[3] * A[7] - A[4] * A[6];
    const double det = A[0] * c00 + A[1] * c01 + A[2] * c02;
    if (!(det != 0.0) || !isfinite(det)) return false;
    const double id = 1.0 / det;
    I[0] = c00 * id;
    I[3] = c01 * id;
    I[6] = c02 * id;
    I[1] = (A[2] * A[7] - A[1] * A[8]) * id;
    I[4] = (A[0] * A[8] - A[2] * A[6]) * id;
    I[7] = (A[1] * A[6] - A[0] * A[7]) * id;
    I[2] = (A[1] * A[5] - A[2] * A[4]) * id;
    I[5] = (A[2] * A[3] - A[0] * A[5]) * id;
    I[8] = (A[0] * A[4] - A[1] * A[3]) * id;
    return true;
}

// AABB and OBB record (lo, hi, OBB centre, OBB inverse transform) and
// centre of every element; one wave per element.  Bound by FP64
// vector arithmetic: for a hex (2N)^2 grid points x N^2 nodes x 18 functions
// x 2 boxes x 6 operations (no contraction: the host's rounding).  Only the
// side functions' values are kept in LDS; the nodes stream through it one
// slab (k) at a time for the centre sums, whose order fixes the rounding (one
// lane per sum).  Four waves per SIMD: the element's frame waits in LDS, and
// the scheduling barriers keep the LDS reads of later rows from being hoisted
// (with 256 registers a wave had its SIMD to itself).  5832 hexes of N = 6:
// 2840 us when each function was bounded by itself, 687 with 256 registers,
// 366 now.
template <int D, int R, int N>
__global__ __launch_bounds__(kLanes) __attribute__((amdgpu_waves_per_eu(4))) void
k_elem_boxes(const BoundTables *Tg, const double *nodes, int64_t e0, int64_t nel, double tol,
             double *box, double *xc_out)
{
    typedef Sides<D, R, N> S;
    constexpr int NP = S::NP, W = 3 * D + D * D;
    constexpr int SLAB = R == 1 ? N : N * N, NSLAB = NP / SLAB;   // nodes of a slab
    constexpr int PER = (D * SLAB + kLanes - 1) / kLanes;
    static_assert(D * SLAB <= 3 * kMaxN * kMaxN, "slab");
    __shared__ __align__(16) double val[S::VALS];
    __shared__ double mom[S::NF * S::MOM], slab[D * SLAB], sc[16], frame[24];
    const BoundTables &T = *Tg;
    const int lane = threadIdx.x;
    const int64_t e = e0 + blockIdx.x;
    if (e >= nel) return;
    const double *xe = nodes + e * D * NP;
    double *rec = box + e * W;
    // centre and centre Jacobian: lane 4 c + q sums coordinate c times
    // phi phi phi (q = 0) or its derivative along direction q - 1
    {
        double pre[PER];
        auto fetch = [&](int ks) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int i = u * kLanes + lane;
                pre[u] = i < D * SLAB ? xe[i / SLAB * NP + ks * SLAB + i % SLAB] : 0.0;
            }
        };
        const int c = lane >> 2, q = lane & 3;
        double w0[N], w1[N], acc = 0.0;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            w0[i] = q == 1 ? T.d0[i] : T.v0[i];
            w1[i] = q == 2 ? T.d0[i] : T.v0[i];
        }
        fetch(0);
#pragma unroll 1
        for (int ks = 0; ks < NSLAB; ++ks) {
            __syncthreads();
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int i = u * kLanes + lane;
                if (i < D * SLAB) slab[i] = pre[u];
            }
            __syncthreads();
            if (ks + 1 < NSLAB) fetch(ks + 1);
            const double w2 = q == 3 ? T.d0[ks] : T.v0[ks];
            if (c < D && q <= R) {
                const double *u = slab + c * SLAB;
                if constexpr (R == 1) {
#pragma unroll
                    for (int i = 0; i < N; ++i) acc += u[i] * w0[i];
                } else {
#pragma unroll
                    for (int j = 0; j < N; ++j) {
#pragma unroll
                        for (int i = 0; i < N; ++i) {
                            double b = w0[i] * w1[j];
                            if (R == 3) b *= w2;
                            acc += u[i + N * j] * b;
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
        }
        __syncthreads();
        if (lane < 16) sc[lane] = acc;   // lanes without a sum: 0
        __syncthreads();
    }
    {
        double lo[3], hi[3], one[3] = {1, 1, 1};
        for (int idx = lane; idx < S::NS * S::PTS; idx += kLanes) {
            const int sd = idx / S::PTS, k = idx % S::PTS, nd = S::node(sd, k);
#pragma unroll
            for (int c = 0; c < D; ++c) val[S::at(sd, c, k)] = xe[c * NP + nd];
        }
        side_bounds<D, R, N>(T, val, mom, lane, lo, hi);
        finish_d(D, R, tol, lo, hi, one);
        if (lane == 0)
            for (int c = 0; c < D; ++c) {
                rec[c] = lo[c];
                rec[D + c] = hi[c];
                xc_out[e * D + c] = sc[4 * c];
            }
    }
    bool inv;
    {
        double Jc[9] = {0}, Ji[9] = {0}, len[3] = {1, 1, 1}, G[3][3], xc[3] = {0, 0, 0};
        for (int c = 0; c < D; ++c) {
            xc[c] = sc[4 * c];
            for (int a = 0; a < R; ++a) G[c][a] = sc[4 * c + 1 + a];
        }
        if (R == D) {
            for (int a = 0; a < D; ++a)
                for (int b = 0; b < D; ++b) Jc[a * D + b] = G[a][b];
        } else if (R == 1) {
            rodrigues_frame(D, G[0][0], G[1][0], D == 3 ? G[2][0] : 0.0, Jc);
        } else {
            const double t1[3] = {G[0][0], G[1][0], G[2][0]}, t2[3] = {G[0][1], G[1][1], G[2][1]};
            const double n[3] = {t1[1] * t2[2] - t1[2] * t2[1], t1[2] * t2[0] - t1[0] * t2[2],
                                 t1[0] * t2[1] - t1[1] * t2[0]};
            const double nn = sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
            for (int c = 0; c < 3; ++c) {
                Jc[c * 3 + 0] = t1[c];
                Jc[c * 3 + 1] = t2[c];
                Jc[c * 3 + 2] = nn > 0.0 ? n[c] / nn : 0.0;
            }
            len[0] = sqrt(t1[0] * t1[0] + t1[1] * t1[1] + t1[2] * t1[2]);
            len[1] = sqrt(t2[0] * t2[0] + t2[1] * t2[1] + t2[2] * t2[2]);
        }
        inv = invert_d(D, Jc, Ji);
        if (inv) {
            __syncthreads();   // the AABB's reads of val come first
            for (int idx = lane; idx < S::NS * S::PTS; idx += kLanes) {
                const int sd = idx / S::PTS, k = idx % S::PTS, nd = S::node(sd, k);
                double x[D];
#pragma unroll
                for (int q = 0; q < D; ++q) x[q] = xe[q * NP + nd];
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    double t = 0.0;
#pragma unroll
                    for (int q = 0; q < D; ++q) t += Ji[c * D + q] * (x[q] - xc[q]);
                    val[S::at(sd, c, k)] = t;
                }
            }
        }
        // the frame waits in LDS while the bounds are computed
        if (lane == 0)
            for (int a = 0; a < 9; ++a) {
                frame[a] = Jc[a];
                frame[9 + a] = Ji[a];
                if (a < 3) frame[18 + a] = len[a];
            }
        __syncthreads();
    }
    double *oc = rec + 2 * D, *oA = rec + 3 * D;
    if (!inv) {
        if (lane == 0) {
            for (int c = 0; c < D; ++c) oc[c] = sc[4 * c];
            for (int a = 0; a < D * D; ++a) oA[a] = 0.0;
        }
        return;
    }
    double tl[3], th[3];
    side_bounds<D, R, N>(T, val, mom, lane, tl, th);
    finish_d(D, R, tol, tl, th, frame + 18);
    if (lane == 0) {
        for (int a = 0; a < D; ++a) {
            const double half = 0.5 * (th[a] - tl[a]);
            for (int b = 0; b < D; ++b) oA[a * D + b] = frame[9 + a * D + b] / half;
        }
        for (int c = 0; c < D; ++c) {
            double s = sc[4 * c];
            for (int q = 0; q < D; ++q) s += frame[c * D + q] * 0.5 * (th[q] + tl[q]);
            oc[c] = s;
        }
    }
}

// Per block: min of the AABB lows and max of the highs over its elements.
__global__ __launch_bounds__(256) void k_union(const double *box, int64_t nel, int D,
                                              double *part)
{
    __shared__ double red[256];
    const int W = 3 * D + D * D;
    for (int q = 0; q < 2 * D; ++q) {
        const bool low = q < D;
        double v = low ? INFINITY : -INFINITY;
        for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nel;
             e += (int64_t)gridDim.x * blockDim.x) {
            const double x = box[e * W + q];
            v = low ? mn(v, x) : mx(v, x);
        }
        red[threadIdx.x] = v;
        __syncthreads();
        for (int o = blockDim.x / 2; o > 0; o >>= 1) {
            if (threadIdx.x < o)
                red[threadIdx.x] = low ? mn(red[threadIdx.x], red[threadIdx.x + o])
                                       : mx(red[threadIdx.x], red[threadIdx.x + o]);
            __syncthreads();
        }
        if (threadIdx.x == 0) part[blockIdx.x * 2 * D + q] = red[0];
        __syncthreads();
    }
}

struct MapView {
    double lo[3], del[3];
    int NL, D;
};

__device__ __forceinline__ int cell_coord_d(const MapView &v, int d, double x)
{
    double t = floor((x - v.lo[d]) / v.del[d]);
    if (t < 0.0) t = 0.0;
    if (t > v.NL - 1) t = v.NL - 1;
    return (int)t;
}

// pass 0: count the cells spanned by each element's AABB corners; pass 1:
// write the element into each of them
__global__ __launch_bounds__(256) void k_map(MapView v, const double *box, int64_t nel, int pass,
                                            int *cnt, const int *off, int *fill, int *cell_el)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nel) return;
    const int D = v.D, W = 3 * D + D * D;
    int c0[3] = {0, 0, 0}, c1[3] = {0, 0, 0};
    for (int d = 0; d < D; ++d) {
        c0[d] = cell_coord_d(v, d, box[e * W + d]);
        c1[d] = cell_coord_d(v, d, box[e * W + D + d]);
    }
    const int64_t NL = v.NL;
    for (int k = c0[2]; k <= c1[2]; ++k)
        for (int j = c0[1]; j <= c1[1]; ++j)
            for (int i = c0[0]; i <= c1[0]; ++i) {
                const int64_t c = i + NL * (j + NL * k);
                if (pass == 0) atomicAdd(&cnt[c], 1);
                else cell_el[off[c] + atomicAdd(&fill[c], 1)] = (int)e;
            }
}

// Each cell's element list in ascending id (the host registers elements in
// ascending order).  A list of up to kSortWide elements is held by kSortLanes
// lanes, and each element goes where the number of smaller ones says; longer
// lists are sorted by insertion.  (One lane per cell and insertion throughout,
// a chain of dependent loads and stores, took 66 us for 5832 elements.)
constexpr int kSortLanes = 16, kSortPer = 4, kSortWide = kSortLanes * kSortPer;
__global__ __launch_bounds__(256) void k_map_sort(const int *off, int64_t c0, int64_t ncell,
                                                 int *cell_el)
{
    const int64_t c = c0 + ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kSortLanes;
    if (c >= ncell) return;   // whole groups of lanes
    const int l = threadIdx.x % kSortLanes, first = (threadIdx.x & 63) / kSortLanes * kSortLanes;
    const int b = off[c], n = off[c + 1] - b;
    int *a = cell_el + b;
    if (n <= kSortWide) {
        int x[kSortPer], below[kSortPer];
#pragma unroll
        for (int k = 0; k < kSortPer; ++k) {
            const int i = l + k * kSortLanes;
            x[k] = i < n ? a[i] : 0;
            below[k] = 0;
        }
#pragma unroll
        for (int k = 0; k < kSortPer; ++k)
            for (int t = 0; t < min(kSortLanes, n - k * kSortLanes); ++t) {
                const int y = __shfl(x[k], first + t);
#pragma unroll
                for (int q = 0; q < kSortPer; ++q) below[q] += y < x[q];
            }
#pragma unroll
        for (int k = 0; k < kSortPer; ++k)
            if (l + k * kSortLanes < n) a[below[k]] = x[k];
        return;
    }
    if (l != 0) return;
    for (int i = 1; i < n; ++i) {
        const int x = a[i];
        int j = i - 1;
        while (j >= 0 && a[j] > x) {
            a[j + 1] = a[j];
            --j;
        }
        a[j + 1] = x;
    }
}

typedef void (*BoxKernel)(const BoundTables *, const double *, int64_t, int64_t, double, double *,
                          double *);

// Blocks of one launch at most, of up to 256 threads: a launch takes fewer than
// 2^32 threads, and a mesh may have more elements times 64 (or cells times
// kSortLanes) than that.
constexpr int64_t kLaunchBlocks = (int64_t)1 << 23;
template <int D, int R>
BoxKernel pick_boxes(int N)
{
    switch (N) {
    case 2: return k_elem_boxes<D, R, 2>;
    case 3: return k_elem_boxes<D, R, 3>;
    case 4: return k_elem_boxes<D, R, 4>;
    case 5: return k_elem_boxes<D, R, 5>;
    case 6: return k_elem_boxes<D, R, 6>;
    case 7: return k_elem_boxes<D, R, 7>;
    case 8: return k_elem_boxes<D, R, 8>;
    case 9: return k_elem_boxes<D, R, 9>;
    case 10: return k_elem_boxes<D, R, 10>;
    default: return nullptr;
    }
}

template <typename T>
struct DevBuf {
    T *p = nullptr;
    ~DevBuf() { (void)hipFree(p); }
    bool alloc(size_t n) { return hipMalloc(&p, sizeof(T) * std::max<size_t>(n, 1)) == hipSuccess; }
};

}  // namespace

int device_setup(fpts_mesh *m, hipStream_t s)
{
    const int D = m->D, R = m->R, N = m->N, W = box_words(D);
    BoundTables bt;
    bound_tables(m, &bt);
    DevBuf<BoundTables> dt;
    if (!dt.alloc(1)) return FPTS_ENOMEM;
    if (hipMemcpyAsync(dt.p, &bt, sizeof(bt), hipMemcpyHostToDevice, s) != hipSuccess)
        return FPTS_EDEVICE;
    // boxes and centres
    const BoxKernel kb = D == 2 ? (R == 2 ? pick_boxes<2, 2>(N) : pick_boxes<2, 1>(N))
                         : R == 3 ? pick_boxes<3, 3>(N)
                                  : R == 2 ? pick_boxes<3, 2>(N) : pick_boxes<3, 1>(N);
    if (!kb) return FPTS_EINVAL;
    for (int64_t e0 = 0; e0 < m->nel; e0 += kLaunchBlocks) {
        const int64_t grid = std::min<int64_t>(m->nel - e0, kLaunchBlocks);
        hipLaunchKernelGGL(kb, dim3((unsigned)grid), dim3(kLanes), 0, s, dt.p, m->d_nodes, e0,
                           (int64_t)m->nel, m->p.bbox_tol, m->d_box, m->d_xc);
        if (hipGetLastError() != hipSuccess) return FPTS_EDEVICE;
    }
    // union box
    const int ublocks = (int)std::min<int64_t>((m->nel + 255) / 256, 1024);
    DevBuf<double> part;
    if (!part.alloc((size_t)ublocks * 2 * D)) return FPTS_ENOMEM;
    hipLaunchKernelGGL(k_union, dim3(ublocks), dim3(256), 0, s, m->d_box, (int64_t)m->nel, D,
                       part.p);
    std::vector<double> hp((size_t)ublocks * 2 * D);
    if (hipGetLastError() != hipSuccess ||
        hipMemcpyAsync(hp.data(), part.p, sizeof(double) * hp.size(), hipMemcpyDeviceToHost, s) !=
            hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return FPTS_EDEVICE;
    for (int d = 0; d < D; ++d) {
        m->hlo[d] = INFINITY;
        m->hhi[d] = -INFINITY;
    }
    for (int b = 0; b < ublocks; ++b)
        for (int d = 0; d < D; ++d) {
            m->hlo[d] = std::min(m->hlo[d], hp[(size_t)b * 2 * D + d]);
            m->hhi[d] = std::max(m->hhi[d], hp[(size_t)b * 2 * D + D + d]);
        }
    for (int d = 0; d < D; ++d)
        if (!std::isfinite(m->hlo[d]) || !std::isfinite(m->hhi[d]) || !(m->hhi[d] > m->hlo[d]))
            return FPTS_EINVAL;
    // the map resolution is the mesh's (hash_n or the default, unchanged)
    const int NL = m->NL;
    for (int d = 0; d < D; ++d) m->hdel[d] = (m->hhi[d] - m->hlo[d]) / NL;
    int64_t ncell = 1;
    for (int d = 0; d < D; ++d) ncell *= NL;
    MapView v;
    for (int d = 0; d < 3; ++d) {
        v.lo[d] = d < D ? m->hlo[d] : 0.0;
        v.del[d] = d < D ? m->hdel[d] : 1.0;
    }
    v.NL = NL;
    v.D = D;
    DevBuf<int> cnt, fill, tmp;
    const int64_t tb = scan_tmp_blocks(ncell);
    if (!cnt.alloc(ncell + 1) || !fill.alloc(ncell) || !tmp.alloc(tb)) return FPTS_ENOMEM;
    const int eg = (int)((m->nel + 255) / 256);
    if (launch_zero2(cnt.p, ncell, fill.p, ncell, s) != hipSuccess) return FPTS_EDEVICE;
    hipLaunchKernelGGL(k_map, dim3(eg), dim3(256), 0, s, v, m->d_box, (int64_t)m->nel, 0, cnt.p,
                       nullptr, nullptr, nullptr);
    if (hipGetLastError() != hipSuccess ||
        launch_unit_scan(UnitScan{cnt.p, ncell, tmp.p, m->d_cell_off}, tb, s) != hipSuccess)
        return FPTS_EDEVICE;
    m->cell_off.resize(ncell + 1);
    if (hipMemcpyAsync(m->cell_off.data(), m->d_cell_off, sizeof(int) * (ncell + 1),
                       hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return FPTS_EDEVICE;
    const int64_t nnz = m->cell_off[ncell];
    if (nnz > (int64_t)m->cell_el.size()) {
        int *p = nullptr;
        if (hipMalloc(&p, sizeof(int) * nnz) != hipSuccess) return FPTS_ENOMEM;
        (void)hipFree(m->d_cell_el);
        m->d_cell_el = p;
    }
    m->cell_el.resize(std::max<int64_t>(nnz, 1));
    hipLaunchKernelGGL(k_map, dim3(eg), dim3(256), 0, s, v, m->d_box, (int64_t)m->nel, 1, nullptr,
                       m->d_cell_off, fill.p, m->d_cell_el);
    constexpr int64_t kCells = 256 / kSortLanes;   // of a block
    for (int64_t c0 = 0; c0 < ncell; c0 += kLaunchBlocks * kCells) {
        const int64_t grid = std::min((ncell - c0 + kCells - 1) / kCells, kLaunchBlocks);
        hipLaunchKernelGGL(k_map_sort, dim3((unsigned)grid), dim3(256), 0, s, m->d_cell_off, c0,
                           ncell, m->d_cell_el);
    }
    m->max_cell = 0;
    for (int64_t c = 0; c < ncell; ++c)
        m->max_cell = std::max(m->max_cell, m->cell_off[c + 1] - m->cell_off[c]);
    // host copies of the products (fpts_get_boxes, fpts_get_hash, workspace sizes)
    m->box.resize((size_t)m->nel * W);
    m->xc.resize((size_t)m->nel * D);
    if (hipGetLastError() != hipSuccess ||
        hipMemcpyAsync(m->cell_el.data(), m->d_cell_el, sizeof(int) * nnz, hipMemcpyDeviceToHost,
                       s) != hipSuccess ||
        hipMemcpyAsync(m->box.data(), m->d_box, sizeof(double) * m->box.size(),
                       hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipMemcpyAsync(m->xc.data(), m->d_xc, sizeof(double) * m->xc.size(),
                       hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return FPTS_EDEVICE;
    return FPTS_OK;
}

}  // namespace fpts
