// Trust-region Newton inversion of the element map (Section 3.2.1) for
// (point, candidate element) pairs grouped by element, with the element-map
// contraction on the matrix cores.  Instantiated in kernels_newton.hip
// (hex, quad and surface kinds); kernels_eval.hip shares its LDS layout.
//
// Task = one element and a queue of its pairs.  The wave stages the
// element's nodal coordinates in LDS and serves up to 64 pairs at a time,
// one per lane: a lane holds its pair's state and runs its Newton update.
// When a lane's pair is done it takes the next pair of the queue.
//
// The map is evaluated for 16 pairs (a column group) at a time.  The lanes
// that need an evaluation hand their reference points q over in LDS, packed
// without gaps; in column group cg, column s belongs to the four lanes
// s, s+16, s+32, s+48 (g = lane / 16 picks the quarter):
//   stage 1 (MFMA, v_mfma_{f64,f32}_16x16x4, f64_4x4x4):
//       C[row][s] = sum_i X[c][i][row] phi_i(q_s,0)   (and phi' / phi'')
//     where row = (j, k) flattened (hex) or j (quad); A = node rows from LDS,
//     B = the column's bases (lane provides phi_i for i = 4 ks + g), so the
//     16 MFMA columns are the 16 pairs and lane l receives rows of its own
//     column (four of each 16-row tile, one of each 4-row tile).
//   stage 2+3 (VALU): each lane weights its rows with phi_j(s) phi_k(t) (and
//     derivatives) of its column, read from an LDS table (for N = 4, 8
//     summed over k first, then weighted per j).
//   The sums over a column's four lanes are formed by transposition: the
//   16-lane swaps of two column groups and the 32-lane swap of two such
//   results leave the totals of column 16 cg + s in lane 16 cg + s.
// Why 16 columns of evaluation but 64 lanes of iteration: FP64 MFMA and
// vector FMA run at the same rate on gfx950, so the evaluation gains nothing
// from wider groups, while the update of a pair (some 400 FP64 instructions)
// would be issued four times if the four lanes of a column shared one pair.
// The totals of a column do not depend on which group or column it is, so a
// pair's iterates do not depend on the pairs beside it.
// Second derivatives (beta = 1 passes on faces/edges, eq. eq_newton_hessian)
// are computed in a separate sweep contracted with the pair's residual dx.
//
// Mixed precision: the FP32 phase runs every pair of the element on FP32
// nodes stored as offsets from the element centre (points shifted the same
// way in FP64 before rounding) until ||dr|| < mixed_tol (default 1e-3) or
// mixed_max_iter passes; the FP64 phase then evaluates the map at that r
// and takes one Newton step, which ends the iteration when it is at most
// kPolishTol and off the faces (the polish step), else the iteration goes
// on in FP64 from there with alpha = 1.  Codes, distances and the final
// residual come from the FP64 phase.
#pragma once
#include <cfloat>
#include <type_traits>

#include "fpts_internal.hpp"
#include "gll_table.hpp"

namespace fpts {
namespace newton {

template <typename T> struct V4;
template <> struct V4<double> { typedef double __attribute__((ext_vector_type(4))) type; };
template <> struct V4<float> { typedef float __attribute__((ext_vector_type(4))) type; };

__device__ __forceinline__ V4<double>::type mfma16(double a, double b, V4<double>::type c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ V4<float>::type mfma16(float a, float b, V4<float>::type c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// four 4x4x4 products side by side: A rows 4 (the same four for every block),
// columns 16, one row of the result per lane quarter
__device__ __forceinline__ double mfma4(double a, double b, double c)
{
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}
// (FP32 has no 4-row form of this shape; its cover is of 16-row tiles only)
template <typename T>
__device__ T mfma4(T, T, T)
{
    static_assert(std::is_same<T, double>::value, "4-row tiles are FP64");
    return T(0);
}

template <typename T> __device__ inline T eps_of();
template <> __device__ inline double eps_of<double>() { return DBL_EPSILON; }
template <> __device__ inline float eps_of<float>() { return FLT_EPSILON; }

// 1/x for a positive normal x (an LDL^T pivot): the hardware reciprocal,
// refined by two Newton steps in FP64 (its first guess is good to about 23
// bits) and used as it is in FP32 (1 ulp).  A step direction needs no
// correctly rounded quotient, and this is a third of the division sequence.
template <typename T> __device__ T rcp_pos(T x);
template <> __device__ __forceinline__ double rcp_pos<double>(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = fma(y, fma(-x, y, 1.0), y);
    return fma(y, fma(-x, y, 1.0), y);
}
template <> __device__ __forceinline__ float rcp_pos<float>(float x)
{
    return __builtin_amdgcn_rcpf(x);
}

// Square root to about 23 bits (one hardware instruction): only for the
// rounding-noise threshold of the trust-region test, a scale, not a result.
template <typename T> __device__ T sqrt_scale(T x);
template <> __device__ __forceinline__ double sqrt_scale<double>(double x)
{
    return __builtin_amdgcn_sqrt(x);
}
template <> __device__ __forceinline__ float sqrt_scale<float>(float x)
{
    return __builtin_amdgcn_sqrtf(x);
}

// Orders LDS accesses between the lanes of a wave (every workgroup here is
// one wave).  The LDS instructions of a wave complete in issue order, so only
// compiler motion has to be fenced: no wait is emitted.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The two results of v_permlane16_swap (v_permlane32_swap) applied to (x, y):
// the instruction trades rows (16-lane rows; 32-lane halves) between its two
// registers, so each result holds, row by row, values of x from one row of
// a row pair and values of y from the same row.  Used only in sums that
// come out the same whichever half of a pair moves.
template <typename T> struct Two { T a, b; };
__device__ __forceinline__ Two<float> swap16(float x, float y)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false,
                                                    false);
    return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ Two<float> swap32(float x, float y)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false,
                                                    false);
    return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ Two<double> swap16(double x, double y)
{
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(x),
                                                     (unsigned)__double2loint(y), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(x),
                                                     (unsigned)__double2hiint(y), false, false);
    return {__hiloint2double((int)hi[0], (int)lo[0]), __hiloint2double((int)hi[1], (int)lo[1])};
}
__device__ __forceinline__ Two<double> swap32(double x, double y)
{
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(x),
                                                     (unsigned)__double2loint(y), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(x),
                                                     (unsigned)__double2hiint(y), false, false);
    return {__hiloint2double((int)hi[0], (int)lo[0]), __hiloint2double((int)hi[1], (int)lo[1])};
}

// Sum of v over the four lanes of a slot (lanes l, l^16, l^32, l^48): the
// swap of v with itself gives every lane its own value and its partner's, in
// the same order in both lanes of the pair, so the four lanes end with
// bit-identical sums.
template <typename T>
__device__ __forceinline__ T slot_sum(T v)
{
    Two<T> p = swap16(v, v);
    v = p.a + p.b;
    p = swap32(v, v);
    return p.a + p.b;
}

// slot_sum of K values, four at a time by transposition: the 16-lane swap of
// (v0, v1) followed by an add leaves the row-pair sums of v0 in one row of
// each pair and those of v1 in the other; the 32-lane swap of two such
// results (v0/v1 and v2/v3) and an add complete the sums, the total of one
// value per row.  The same swaps of a total with itself then broadcast each
// row's total to the four rows.  Each total is formed once (bit-identical in
// the four lanes), with 9 swaps per four values instead of 16.
template <typename T, int K>
__device__ __forceinline__ void slot_sum_all(T (&v)[K])
{
    constexpr int Q = K / 4;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        Two<T> p = swap16(v[4 * i], v[4 * i + 1]);
        const T w01 = p.a + p.b;
        p = swap16(v[4 * i + 2], v[4 * i + 3]);
        const T w23 = p.a + p.b;
        p = swap32(w01, w23);
        const T z = p.a + p.b;
        p = swap32(z, z);
        const Two<T> h0 = swap16(p.a, p.a), h1 = swap16(p.b, p.b);
        v[4 * i] = h0.a;
        v[4 * i + 1] = h0.b;
        v[4 * i + 2] = h1.a;
        v[4 * i + 3] = h1.b;
    }
    if constexpr (K % 4 >= 2) {
        constexpr int i = 4 * Q;
        Two<T> p = swap16(v[i], v[i + 1]);
        T w = p.a + p.b;
        p = swap32(w, w);
        w = p.a + p.b;
        p = swap16(w, w);
        v[i] = p.a;
        v[i + 1] = p.b;
    }
    if constexpr (K % 2 == 1) v[K - 1] = slot_sum(v[K - 1]);
}

// Column sums by transposition.  fold16: x and y hold the partial sums of
// two column groups; the result holds, in row r of the wave, the sum over
// rows r & ~1 and r | 1 of x (r even) or of y (r odd).  fold32 of two such
// results completes them: row r holds the four-row total of group r.  Every
// total is (row 0 + row 1) + (row 2 + row 3), whichever group it is.
template <typename T, int K>
__device__ __forceinline__ void fold16(T (&x)[K], const T (&y)[K])
{
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const Two<T> p = swap16(x[k], y[k]);
        x[k] = p.a + p.b;
    }
}
template <typename T, int K>
__device__ __forceinline__ void fold32(T (&x)[K], const T (&y)[K])
{
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const Two<T> p = swap32(x[k], y[k]);
        x[k] = p.a + p.b;
    }
}

// Contraction row of the 16x16 output tile m held by lane quarter g in item
// qq: 16 m + g + 4 qq.  The FP64 instruction interleaves the tile's rows that
// way (item qq of quarter g is tile row g + 4 qq); the FP32 one gives each
// quarter four consecutive tile rows (4 g + qq), so the FP32 A operand
// supplies the rows transposed (a_row) to land on the same contraction rows.
// Both layouts checked on gfx950.
__device__ __forceinline__ int out_row(int m, int g, int qq) { return 16 * m + g + 4 * qq; }
template <typename T>
__device__ __forceinline__ int a_row(int m, int slot)
{
    return 16 * m + (std::is_same<T, double>::value ? slot : (slot >> 2) + 4 * (slot & 3));
}

template <int D, int R, int N>
struct Shape {
    static constexpr int NP = (R == 3) ? N * N * N : N * N;
    static constexpr int ROWS = (R == 3) ? N * N : N;   // contraction rows
    static constexpr int MT = (ROWS + 15) / 16;         // 16-row tiles
    static constexpr int KS = (N + 3) / 4;              // 4-wide K steps
};

// Sweep 1's cover of the contraction without (most of) its padding.  FP64:
// the rows beyond the last whole 16-row tile go to 4-row tiles
// (v_mfma_f64_4x4x4 on four column quarters: 16 columns, a quarter of the
// time), and where N is 1 or 2 above a multiple of 4 the last node indices
// are added by vector FMAs (8 or 16 per tile and coordinate against two
// MFMAs of 64 cycles, which would be padding but for them).  N = 6: 1610
// instead of 2520 cycles of stage 1 per 16 pairs; N = 10: 6.5k instead of
// 8.4k.  FP32: 16-row tiles and K steps rounded up (its MFMA is twice as
// fast against the vector FMA, and has no 4-row form of this shape).
template <typename T, int D, int R, int N>
struct Cover {
    typedef Shape<D, R, N> S;
    static constexpr bool F64 = std::is_same<T, double>::value;
    static constexpr int LEFT = S::ROWS % 16;
    static constexpr int QT = F64 && LEFT <= 12 ? (LEFT + 3) / 4 : 0;   // 4-row tiles
    static constexpr int FT = QT || !LEFT ? S::ROWS / 16 : S::MT;        // 16-row tiles
    static constexpr int KR = F64 && (N % 4 == 1 || N % 4 == 2) ? N % 4 : 0;   // by FMA
    static constexpr int KM = KR ? N / 4 : S::KS;                        // K steps by MFMA
};

// Where node (coordinate c, contraction row `row`, first index i) of the
// element sits in LDS.  The 16 lanes of a lane quarter read the A operand
// from 16 consecutive rows at one i; with rows of an even number of values
// stored back to back those reads share a few LDS banks (N = 8 doubles: two
// banks pairs for 16 lanes).  Rows of an odd length P = N + 1 spread them
// over 16; FP64 with N = 8 instead rotates each row by row / 2 positions
// (no padding: the wave's LDS stays within 20 KB, eight waves per CU).
template <typename T, int D, int R, int N>
struct NodeLds {
    typedef Shape<D, R, N> S;
    static constexpr bool ROT = std::is_same<T, double>::value && N == 8;
    static constexpr int P = (ROT || N % 2) ? N : N + 1;
    static constexpr int RP = S::ROWS * P;               // per coordinate
    static constexpr int SIZE = D * RP;
    // values from one node block to the next where a wave holds several: whole
    // 16-byte words, as stage() writes them (SIZE is odd for D = 3 and odd N)
    static constexpr int STRIDE = (SIZE * (int)sizeof(T) + 15) / 16 * 16 / (int)sizeof(T);
    static_assert(STRIDE * sizeof(T) % 16 == 0, "node blocks start on 16 bytes");
    static constexpr bool PLAIN = !ROT && P == N;        // the global layout
    __device__ static __forceinline__ int at(int c, int row, int i)
    {
        return c * RP + row * P + (ROT ? ((i + (row >> 1)) & (N - 1)) : i);
    }
};

// Packed symmetric R x R matrices: diagonal first, then the upper triangle.
template <int R> constexpr int kSym = R * (R + 1) / 2;
template <int R>
__device__ constexpr int sym(int a, int b)
{
    if (a == b) return a;
    const int lo = a < b ? a : b, hi = a < b ? b : a;
    return R == 2 ? 2 : (lo == 0 ? (hi == 1 ? 3 : 4) : 5);
}

// phi_i, phi_i', phi_i'' at x for ONE index i (runtime, per lane): the
// product over m != i of (x - z_m) carried as a jet, times w_i.
template <typename T, int N>
__device__ __forceinline__ void basis_at(T x, int i, T &v, T &d, T &dd)
{
    constexpr gll::Table<N> G = gll::Nodes<N>::t;
    T pv = T(1), pd = T(0), pdd = T(0), wi = T(0);
#pragma unroll
    for (int m = 0; m < N; ++m) {
        const bool self = (m == i);
        const T u = self ? T(1) : x - T(G.z[m]);
        const T du = self ? T(0) : T(1);
        pdd = pdd * u + T(2) * pd * du;
        pd = pd * u + pv * du;
        pv = pv * u;
        wi = self ? T(G.w[m]) : wi;
    }
    v = wi * pv;
    d = wi * pd;
    dd = wi * pdd;
}

// All N bases of one direction at x (prefix/suffix jets), written to the
// per-slot LDS table tab[kind][i][slot] (kind 0: phi, 1: phi', 2: phi'')
// when `write` holds.
template <typename T, int N, bool H2>
__device__ __forceinline__ void basis_table(T x, T *tab, int slot, bool write)
{
    constexpr gll::Table<N> G = gll::Nodes<N>::t;
    // The jets of the first one or two factors are written out (1, 0, 0),
    // (t, 1, 0), (., ., 2): products with the constants 0 and 1 would
    // otherwise be issued, since they cannot be folded for a general x.
    T pv[N], pd[N], pdd[N];
    pv[0] = T(1);
    pd[0] = T(0);
    pdd[0] = T(0);
#pragma unroll
    for (int i = 1; i < N; ++i) {
        const T t = x - T(G.z[i - 1]);
        if (H2) pdd[i] = i == 1 ? T(0) : i == 2 ? T(2) * pd[1] : pdd[i - 1] * t + T(2) * pd[i - 1];
        pd[i] = i == 1 ? T(1) : pd[i - 1] * t + pv[i - 1];
        pv[i] = i == 1 ? t : pv[i - 1] * t;
    }
    T sv = T(1), sd = T(0), sdd = T(0);
#pragma unroll
    for (int i = N - 1; i >= 0; --i) {
        const int ns = N - 1 - i;   // factors in the suffix
        if (write) {
            const T v = ns == 0 ? pv[i] : pv[i] * sv;
            const T d = ns == 0 ? pd[i] : ns == 1 ? pd[i] * sv + pv[i] : pd[i] * sv + pv[i] * sd;
            tab[(0 * N + i) * 16 + slot] = T(G.w[i]) * v;
            tab[(1 * N + i) * 16 + slot] = T(G.w[i]) * d;
            if (H2) {
                const T dd = ns == 0   ? pdd[i]
                             : ns == 1 ? pdd[i] * sv + T(2) * pd[i]
                                       : pdd[i] * sv + T(2) * pd[i] * sd + pv[i] * sdd;
                tab[(2 * N + i) * 16 + slot] = T(G.w[i]) * dd;
            }
        }
        const T t = x - T(G.z[i]);
        if (H2) sdd = ns == 0 ? T(0) : ns == 1 ? T(2) * sd : sdd * t + T(2) * sd;
        sd = ns == 0 ? T(1) : sd * t + sv;
        sv = ns == 0 ? t : sv * t;
    }
}

// LDS layout of one wave: nodes [D][NP] of type T, the basis tables of one
// column group, [R][2][N][16] (sweep 2: [R - 1][3][N][16]), then the points
// of the pairs to evaluate, [R][64] (sweep 2: [R + D][16]).  FP64 hexes with
// N <= 8 stay within 20 KB, so that eight waves fit a CU.
template <typename T, int D, int R, int N>
struct Lds {
    static constexpr int NODES = NodeLds<T, D, R, N>::STRIDE;
    static constexpr int TAB = (R == 3 ? 6 : 4) * N * 16;
    static constexpr int QB = 64 * R;
    static_assert(16 * (R + D) <= QB, "sweep 2 points");
    static constexpr size_t bytes() { return sizeof(T) * (NODES + TAB + QB); }
};

// Rows of the differentiation matrix at the GLL nodes: v[a][m] = phi_m'(z_a),
// by the same prefix/suffix product rule as the sweeps' bases (compile time).
template <typename T, int N>
struct DiffRows {
    T v[N][N];
};
template <typename T, int N>
constexpr DiffRows<T, N> make_diff()
{
    constexpr gll::Table<N> G = gll::Nodes<N>::t;
    DiffRows<T, N> d{};
    for (int a = 0; a < N; ++a) {
        const double x = G.z[a];
        double pv[N] = {}, pd[N] = {};
        pv[0] = 1.0;
        for (int i = 1; i < N; ++i) {
            const double t = x - G.z[i - 1];
            pd[i] = pd[i - 1] * t + pv[i - 1];
            pv[i] = pv[i - 1] * t;
        }
        double sv = 1.0, sd = 0.0;
        for (int i = N - 1; i >= 0; --i) {
            d.v[a][i] = T(G.w[i] * (pd[i] * sv + pv[i] * sd));
            const double t = x - G.z[i];
            sd = sd * t + sv;
            sv = sv * t;
        }
    }
    return d;
}
template <typename T, int N>
__device__ const DiffRows<T, N> kDiff = make_diff<T, N>();

// The GLL nodes, indexed per lane.
template <typename T, int N>
struct NodeRow {
    T v[N];
};
template <typename T, int N>
constexpr NodeRow<T, N> make_nodes()
{
    constexpr gll::Table<N> G = gll::Nodes<N>::t;
    NodeRow<T, N> r{};
    for (int i = 0; i < N; ++i) r.v[i] = T(G.z[i]);
    return r;
}
template <typename T, int N>
__device__ const NodeRow<T, N> kNodes = make_nodes<T, N>();

// Stage 2+3 factored by j for hexes whose 16-row tiles hold whole (j, k)
// blocks (N = 4, 8): a lane's rows 16 m + g + 4 qq have j = g + 4 (qq % NJ)
// whatever m is, so the k-weights are summed per j first and the j-weights
// applied once at the end.
template <int R, int N>
struct Factor {
    static constexpr bool ON = R == 3 && (N == 4 || N == 8);
    static constexpr int NJ = N / 4 > 0 ? N / 4 : 1;   // the lane's distinct j
};

// Sweep 1 for column group cg: each lane's partial sums of x(q) and
// G = dx/dr of its column (v: X[c], then G[c][a]); the column's totals are
// the sums over its four lanes.  NB > 1: the columns belong to NB elements
// (16 / NB consecutive columns each, the node blocks one after the other);
// every row tile is then a 4-row one, whose four products take their A rows
// from their own columns' element.  The row sums and their order are the
// same (the MFMAs of both shapes round like a chain of FMAs).
template <typename T, int D, int R, int N, int NB = 1>
__device__ __forceinline__ void sweep1(const T *xl, T *tab, const T *qb, int cg, int lane,
                                       T (&v)[D * (R + 1)])
{
    typedef Shape<D, R, N> S;
    typedef Cover<T, D, R, N> C;
    typedef Factor<R, N> F;
    typedef NodeLds<T, D, R, N> NL;
    typedef typename V4<T>::type v4;
    constexpr int FT = NB > 1 ? 0 : C::FT, QT = NB > 1 ? (S::ROWS + 3) / 4 : C::QT;
    const int slot = lane & 15, g = lane >> 4;
    if (NB > 1) xl += slot / (16 / NB) * NL::STRIDE;
    // per-column tables [direction][kind][i][column] (kinds phi, phi'): lane
    // quarter g builds direction g of its column, so the R tables of all 16
    // columns are built at once
    wave_lds_sync();   // qb is written; the previous group's reads of the tables come first
    {
        const T x = qb[(g < R ? g : 0) * 64 + 16 * cg + slot];
        basis_table<T, N, false>(x, tab + (g < R ? g : 0) * 2 * N * 16, slot, g < R);
    }
    wave_lds_sync();
    const T *tr = tab, *ts = tab + 2 * N * 16, *tt = tab + 4 * N * 16;
    // B operand: this lane's bases in direction 0 for i = 4 ks + g, and the
    // bases of the indices left to FMAs
    T b0[C::KM > 0 ? C::KM : 1], b1[C::KM > 0 ? C::KM : 1];
    T e0[C::KR > 0 ? C::KR : 1], e1[C::KR > 0 ? C::KR : 1];
#pragma unroll
    for (int ks = 0; ks < C::KM; ++ks) {
        const int i = 4 * ks + g;
        const bool ok = N % 4 == 0 || C::KR > 0 || i < N;
        b0[ks] = ok ? tr[(0 * N + i) * 16 + slot] : T(0);
        b1[ks] = ok ? tr[(1 * N + i) * 16 + slot] : T(0);
    }
#pragma unroll
    for (int u = 0; u < C::KR; ++u) {
        e0[u] = tr[(0 * N + 4 * C::KM + u) * 16 + slot];
        e1[u] = tr[(1 * N + 4 * C::KM + u) * 16 + slot];
    }
    // the lane's partial sums: X, G directly, or (factored) per j the
    // k-weighted sums Zv = sum_k C0 t_k, Zd = sum_k C1 t_k, Zt = sum_k C0 t'_k
    T X[D], G[D][R];
    T Zv[F::NJ][D], Zd[F::NJ][D], Zt[F::NJ][D];
#pragma unroll
    for (int c = 0; c < D; ++c) {
        X[c] = T(0);
#pragma unroll
        for (int a = 0; a < R; ++a) G[c][a] = T(0);
#pragma unroll
        for (int js = 0; js < F::NJ; ++js) {
            Zv[js][c] = T(0);
            Zd[js][c] = T(0);
            Zt[js][c] = T(0);
        }
    }
    // C0, C1 of one contraction row of the lane, weighted into the sums
    auto add_row = [&](int row, const T (&c0)[D], const T (&c1)[D]) __attribute__((always_inline)) {
        if constexpr (R == 3) {
            const int j = row % N, k = row / N;
            const T sv = ts[(0 * N + j) * 16 + slot], sd = ts[(1 * N + j) * 16 + slot];
            const T tv = tt[(0 * N + k) * 16 + slot], td = tt[(1 * N + k) * 16 + slot];
            const T w00 = sv * tv, w10 = sd * tv, w01 = sv * td;
#pragma unroll
            for (int c = 0; c < D; ++c) {
                X[c] = fma(c0[c], w00, X[c]);
                G[c][0] = fma(c1[c], w00, G[c][0]);
                G[c][1] = fma(c0[c], w10, G[c][1]);
                G[c][R - 1] = fma(c0[c], w01, G[c][R - 1]);
            }
        } else {
            const T sv = ts[(0 * N + row) * 16 + slot], sd = ts[(1 * N + row) * 16 + slot];
#pragma unroll
            for (int c = 0; c < D; ++c) {
                X[c] = fma(c0[c], sv, X[c]);
                G[c][0] = fma(c1[c], sv, G[c][0]);
                G[c][1] = fma(c0[c], sd, G[c][1]);
            }
        }
    };
    // A entries outside the element (rows or node indices of the padding)
    // meet a zero B entry or land in rows that are dropped; the clamped
    // address keeps the read inside the node block
    constexpr bool kFullA = (N % 4 == 0 || C::KR > 0);
    // one 16-row tile (factored: the first is issued on its own, where the
    // partial sums are still the constant 0, no registers to clear)
    auto tile = [&](int m) __attribute__((always_inline)) {
        v4 acc0[D], acc1[D];
        constexpr bool kRows = S::ROWS % 16 == 0 || C::QT > 0;   // the tile's rows all exist
        const int arow = a_row<T>(m, slot);   // A-operand row of this lane
#pragma unroll
        for (int c = 0; c < D; ++c) {
            acc0[c] = v4{0, 0, 0, 0};
            acc1[c] = v4{0, 0, 0, 0};
        }
#pragma unroll
        for (int ks = 0; ks < C::KM; ++ks) {
            const int ai = 4 * ks + g;      // A-operand column (node index i)
            const bool aok = (kFullA && kRows) || ((kRows || arow < S::ROWS) && (kFullA || ai < N));
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const T a = xl[aok ? NL::at(c, arow, ai) : 0];
                acc0[c] = mfma16(a, b0[ks], acc0[c]);
                acc1[c] = mfma16(a, b1[ks], acc1[c]);
            }
        }
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
            const int row = out_row(m, g, qq);
            if (!kRows && row >= S::ROWS) continue;
            T c0[D], c1[D];
#pragma unroll
            for (int c = 0; c < D; ++c) {
                c0[c] = acc0[c][qq];
                c1[c] = acc1[c][qq];
#pragma unroll
                for (int u = 0; u < C::KR; ++u) {
                    const T a = xl[NL::at(c, row, 4 * C::KM + u)];
                    c0[c] = fma(a, e0[u], c0[c]);
                    c1[c] = fma(a, e1[u], c1[c]);
                }
            }
            if constexpr (F::ON) {
                const int k = (16 * m + 4 * qq) / N, js = qq % F::NJ;   // row / N (g < 4)
                const T tv = tt[(0 * N + k) * 16 + slot], td = tt[(1 * N + k) * 16 + slot];
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    Zv[js][c] = fma(c0[c], tv, Zv[js][c]);
                    Zd[js][c] = fma(c1[c], tv, Zd[js][c]);
                    Zt[js][c] = fma(c0[c], td, Zt[js][c]);
                }
            } else {
                add_row(row, c0, c1);
            }
        }
    };
    if constexpr (FT > 0 && F::ON) {
        tile(0);
#pragma unroll 1
        for (int m = 1; m < FT; ++m) tile(m);
    } else if constexpr (FT > 0) {
        // (one copy: with the row weights of two the registers spill)
#pragma unroll 1
        for (int m = 0; m < FT; ++m) tile(m);
    }
    // one 4-row tile: lane quarter g receives row g, all quarters of the
    // columns read the same four A rows (of their element)
    auto quad = [&](int base, auto &&take) __attribute__((always_inline)) {
        const bool whole = S::ROWS % 4 == 0 || base + 4 <= S::ROWS;
        const int arow = base + (slot & 3), row = base + g;
        T c0[D], c1[D];
#pragma unroll
        for (int c = 0; c < D; ++c) {
            c0[c] = T(0);
            c1[c] = T(0);
        }
#pragma unroll
        for (int ks = 0; ks < C::KM; ++ks) {
            const int ai = 4 * ks + g;
            const bool aok = (whole || arow < S::ROWS) && (kFullA || ai < N);
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const T a = xl[aok ? NL::at(c, arow, ai) : 0];
                c0[c] = mfma4(a, b0[ks], c0[c]);
                c1[c] = mfma4(a, b1[ks], c1[c]);
            }
        }
        if (whole || row < S::ROWS) {
#pragma unroll
            for (int u = 0; u < C::KR; ++u)
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    const T a = xl[NL::at(c, row, 4 * C::KM + u)];
                    c0[c] = fma(a, e0[u], c0[c]);
                    c1[c] = fma(a, e1[u], c1[c]);
                }
            take(row, c0, c1);
        }
    };
    if constexpr (QT > 0 && F::ON) {
#pragma unroll 1
        for (int k = 0; k < N; ++k) {
            const T tv = tt[(0 * N + k) * 16 + slot], td = tt[(1 * N + k) * 16 + slot];
#pragma unroll
            for (int js = 0; js < F::NJ; ++js)
                quad(N * k + 4 * js, [&](int, const T (&c0)[D], const T (&c1)[D])
                                         __attribute__((always_inline)) {
#pragma unroll
                    for (int c = 0; c < D; ++c) {
                        Zv[js][c] = fma(c0[c], tv, Zv[js][c]);
                        Zd[js][c] = fma(c1[c], tv, Zd[js][c]);
                        Zt[js][c] = fma(c0[c], td, Zt[js][c]);
                    }
                });
        }
    } else if constexpr (QT > 0) {
#pragma unroll 1
        for (int t = 0; t < QT; ++t) quad(16 * FT + 4 * t, add_row);
    }
    if constexpr (F::ON) {
#pragma unroll
        for (int js = 0; js < F::NJ; ++js) {
            const int j = g + 4 * js;
            const T sv = ts[(0 * N + j) * 16 + slot], sd = ts[(1 * N + j) * 16 + slot];
#pragma unroll
            for (int c = 0; c < D; ++c) {
                X[c] = fma(Zv[js][c], sv, X[c]);
                G[c][0] = fma(Zd[js][c], sv, G[c][0]);
                G[c][1] = fma(Zv[js][c], sd, G[c][1]);
                G[c][R - 1] = fma(Zt[js][c], sv, G[c][R - 1]);
            }
        }
    }
#pragma unroll
    for (int c = 0; c < D; ++c) {
        v[c] = X[c];
#pragma unroll
        for (int a = 0; a < R; ++a) v[D + c * R + a] = G[c][a];
    }
}

// Sweep 2: S_ab = sum_c dx_c d2x_c/dr_a dr_b for 16 columns, whose points q
// and residuals dx are in qb ([R + D][16]); the four lanes of a column all
// receive its totals.  NB as in sweep 1 (one element: 16-row tiles).
template <typename T, int D, int R, int N, int NB = 1>
__device__ __forceinline__ void sweep2(const T *xl, T *tab, const T *qb, int lane,
                                       T (&Sout)[kSym<R>])
{
    typedef Shape<D, R, N> S;
    typedef Factor<R, N> F;
    typedef typename V4<T>::type v4;
    typedef NodeLds<T, D, R, N> NL;
    const int slot = lane & 15, g = lane >> 4;
    if (NB > 1) xl += slot / (16 / NB) * NL::STRIDE;
    wave_lds_sync();   // qb is written
    T q[R], dx[D];
#pragma unroll
    for (int k = 0; k < R; ++k) q[k] = qb[k * 16 + slot];
#pragma unroll
    for (int c = 0; c < D; ++c) dx[c] = qb[(R + c) * 16 + slot];
    T b0[S::KS], b1[S::KS], b2[S::KS];
#pragma unroll
    for (int ks = 0; ks < S::KS; ++ks) {
        const int i = 4 * ks + g;
        T v, d, dd;
        basis_at<T, N>(q[0], i, v, d, dd);
        b0[ks] = i < N ? v : T(0);
        b1[ks] = i < N ? d : T(0);
        b2[ks] = i < N ? dd : T(0);
    }
    // per-slot tables [direction - 1][kind][i][slot] (phi, phi', phi'') of
    // directions 1 (lane quarter 1) and 2 (lane quarter 2)
    wave_lds_sync();
    {
        const T x = (R == 3 && g == 2) ? q[R == 3 ? 2 : 0] : q[1];
        const bool w = g == 1 || (R == 3 && g == 2);
        basis_table<T, N, true>(x, tab + (g == 2 ? 3 * N * 16 : 0), slot, w);
    }
    wave_lds_sync();
    const T *tt = tab + 3 * N * 16;
    T Sa[kSym<R>];
    // factored: per j, Z[0..5] = sum_k of C2 t, C0 t, C0 t'', C1 t, C1 t',
    // C0 t' (then times s, s'', s, s', s, s' of j)
    T Z[F::NJ][6];
#pragma unroll
    for (int a = 0; a < kSym<R>; ++a) Sa[a] = T(0);
#pragma unroll
    for (int js = 0; js < F::NJ; ++js)
#pragma unroll
        for (int a = 0; a < 6; ++a) Z[js][a] = T(0);
    // a row's C0, C1, C2 = sum_c dx_c C_c[row][column] per basis kind,
    // weighted into the sums; js: the lane's j (factored), k likewise
    auto add_row = [&](int row, int k, auto jsc, T C0, T C1, T C2) __attribute__((always_inline)) {
        if constexpr (F::ON) {
            constexpr int js = decltype(jsc)::value;
            const T tv = tt[(0 * N + k) * 16 + slot], td = tt[(1 * N + k) * 16 + slot];
            const T tdd = tt[(2 * N + k) * 16 + slot];
            Z[js][0] = fma(C2, tv, Z[js][0]);
            Z[js][1] = fma(C0, tv, Z[js][1]);
            Z[js][2] = fma(C0, tdd, Z[js][2]);
            Z[js][3] = fma(C1, tv, Z[js][3]);
            Z[js][4] = fma(C1, td, Z[js][4]);
            Z[js][5] = fma(C0, td, Z[js][5]);
        } else if constexpr (R == 3) {
            const int j = row % N, kk = row / N;
            const T sv = tab[(0 * N + j) * 16 + slot], sd = tab[(1 * N + j) * 16 + slot];
            const T sdd = tab[(2 * N + j) * 16 + slot];
            const T tv = tt[(0 * N + kk) * 16 + slot], td = tt[(1 * N + kk) * 16 + slot];
            const T tdd = tt[(2 * N + kk) * 16 + slot];
            Sa[0] = fma(C2, sv * tv, Sa[0]);                                 // rr
            Sa[1] = fma(C0, sdd * tv, Sa[1]);                                // ss
            Sa[2] = fma(C0, sv * tdd, Sa[2]);                                // tt
            Sa[kSym<R> - 3] = fma(C1, sd * tv, Sa[kSym<R> - 3]);             // rs
            Sa[kSym<R> - 2] = fma(C1, sv * td, Sa[kSym<R> - 2]);             // rt
            Sa[kSym<R> - 1] = fma(C0, sd * td, Sa[kSym<R> - 1]);             // st
        } else {
            const int j = row;
            const T sv = tab[(0 * N + j) * 16 + slot], sd = tab[(1 * N + j) * 16 + slot];
            const T sdd = tab[(2 * N + j) * 16 + slot];
            Sa[0] = fma(C2, sv, Sa[0]);         // rr
            Sa[1] = fma(C0, sdd, Sa[1]);        // ss
            Sa[2] = fma(C1, sd, Sa[2]);         // rs
        }
    };
    if constexpr (NB == 1) {
        auto tile = [&](int m) __attribute__((always_inline)) {
            // the column's residual enters the B operand, so one accumulator
            // per basis kind collects the sum over the coordinates
            v4 acc0 = v4{0, 0, 0, 0}, acc1 = v4{0, 0, 0, 0}, acc2 = v4{0, 0, 0, 0};
            const int arow = a_row<T>(m, slot);
#pragma unroll
            for (int ks = 0; ks < S::KS; ++ks) {
                const int ai = 4 * ks + g;
                const bool aok =
                    ((N % 4 == 0) && (S::ROWS % 16 == 0)) || (arow < S::ROWS && ai < N);
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    const T a = xl[aok ? NL::at(c, arow, ai) : 0];
                    acc0 = mfma16(a, dx[c] * b0[ks], acc0);
                    acc1 = mfma16(a, dx[c] * b1[ks], acc1);
                    acc2 = mfma16(a, dx[c] * b2[ks], acc2);
                }
            }
            auto part = [&](auto qqc) __attribute__((always_inline)) {
                constexpr int qq = decltype(qqc)::value;
                const int row = out_row(m, g, qq);
                if (S::ROWS % 16 == 0 || row < S::ROWS)
                    add_row(row, (16 * m + 4 * qq) / N, std::integral_constant<int, qq % F::NJ>(),
                            acc0[qq], acc1[qq], acc2[qq]);
            };
            part(std::integral_constant<int, 0>());
            part(std::integral_constant<int, 1>());
            part(std::integral_constant<int, 2>());
            part(std::integral_constant<int, 3>());
        };
        tile(0);
#pragma unroll 1
        for (int m = 1; m < S::MT; ++m) tile(m);
    } else {
        auto quad = [&](int base, int k, auto jsc) __attribute__((always_inline)) {
            const bool whole = S::ROWS % 4 == 0 || base + 4 <= S::ROWS;
            const int arow = base + (slot & 3), row = base + g;
            T C0 = T(0), C1 = T(0), C2 = T(0);
#pragma unroll
            for (int ks = 0; ks < S::KS; ++ks) {
                const int ai = 4 * ks + g;
                const bool aok = (whole || arow < S::ROWS) && (N % 4 == 0 || ai < N);
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    const T a = xl[aok ? NL::at(c, arow, ai) : 0];
                    C0 = mfma4(a, dx[c] * b0[ks], C0);
                    C1 = mfma4(a, dx[c] * b1[ks], C1);
                    C2 = mfma4(a, dx[c] * b2[ks], C2);
                }
            }
            if (whole || row < S::ROWS) add_row(row, k, jsc, C0, C1, C2);
        };
        if constexpr (F::ON) {
#pragma unroll 1
            for (int k = 0; k < N; ++k) {
                quad(N * k, k, std::integral_constant<int, 0>());
                if constexpr (F::NJ > 1) quad(N * k + 4, k, std::integral_constant<int, 1>());
            }
        } else {
#pragma unroll 1
            for (int t = 0; t < (S::ROWS + 3) / 4; ++t)
                quad(4 * t, 0, std::integral_constant<int, 0>());
        }
    }
    if constexpr (F::ON) {
#pragma unroll
        for (int js = 0; js < F::NJ; ++js) {
            const int j = g + 4 * js;
            const T sv = tab[(0 * N + j) * 16 + slot], sd = tab[(1 * N + j) * 16 + slot];
            const T sdd = tab[(2 * N + j) * 16 + slot];
            Sa[0] = fma(Z[js][0], sv, Sa[0]);    // rr
            Sa[1] = fma(Z[js][1], sdd, Sa[1]);   // ss
            Sa[2] = fma(Z[js][2], sv, Sa[2]);    // tt
            Sa[3] = fma(Z[js][3], sd, Sa[3]);    // rs
            Sa[4] = fma(Z[js][4], sv, Sa[4]);    // rt
            Sa[5] = fma(Z[js][5], sd, Sa[5]);    // st
        }
    }
    slot_sum_all(Sa);
#pragma unroll
    for (int a = 0; a < kSym<R>; ++a) Sout[a] = Sa[a];
}

// Objective at a point: f = |x* - x|^2, g = G^T dx, Hgn = G^T G (packed).
template <typename T, int D, int R>
struct Obj {
    T f;
    T g[R];
    T Hgn[kSym<R>];
};

template <typename T, int D, int R>
__device__ __forceinline__ void objective(const T (&xs)[D], const T (&X)[D], const T (&G)[D][R],
                                          Obj<T, D, R> &o, T (&dx)[D])
{
    o.f = T(0);
#pragma unroll
    for (int a = 0; a < R; ++a) o.g[a] = T(0);
#pragma unroll
    for (int a = 0; a < kSym<R>; ++a) o.Hgn[a] = T(0);
#pragma unroll
    for (int c = 0; c < D; ++c) {
        dx[c] = xs[c] - X[c];
        o.f = fma(dx[c], dx[c], o.f);
#pragma unroll
        for (int a = 0; a < R; ++a) {
            o.g[a] = fma(G[c][a], dx[c], o.g[a]);
#pragma unroll
            for (int b = a; b < R; ++b)
                o.Hgn[sym<R>(a, b)] = fma(G[c][a], G[c][b], o.Hgn[sym<R>(a, b)]);
        }
    }
}

// Solve H dr = g on the free coordinates (rows/columns of held coordinates
// replaced by the identity, right-hand side 0) by LDL^T; false when a pivot
// is not positive.
template <typename T, int R>
__device__ __forceinline__ bool solve_free(const T (&H)[kSym<R>], const T (&g)[R],
                                           const bool (&held)[R], T (&x)[R])
{
    T A[R][R], b[R];
#pragma unroll
    for (int a = 0; a < R; ++a) {
        b[a] = held[a] ? T(0) : g[a];
#pragma unroll
        for (int c = 0; c < R; ++c)
            A[a][c] = (held[a] || held[c]) ? (a == c ? T(1) : T(0)) : H[sym<R>(a, c)];
    }
    T L[R][R], d[R], inv[R];
    bool ok = true;
#pragma unroll
    for (int a = 0; a < R; ++a) {
        T s = A[a][a];
#pragma unroll
        for (int k = 0; k < a; ++k) s -= L[a][k] * L[a][k] * d[k];
        d[a] = s;
        ok = ok && (s > T(0));
        inv[a] = rcp_pos(s);   // one reciprocal per pivot (unused when s <= 0)
#pragma unroll
        for (int c = a + 1; c < R; ++c) {
            T t = A[c][a];
#pragma unroll
            for (int k = 0; k < a; ++k) t -= L[c][k] * L[a][k] * d[k];
            L[c][a] = t * inv[a];
        }
    }
    T y[R];
#pragma unroll
    for (int a = 0; a < R; ++a) {
        T s = b[a];
#pragma unroll
        for (int k = 0; k < a; ++k) s -= L[a][k] * y[k];
        y[a] = s;
    }
#pragma unroll
    for (int a = R - 1; a >= 0; --a) {
        T s = y[a] * inv[a];
#pragma unroll
        for (int k = a + 1; k < R; ++k) s -= L[k][a] * x[k];
        x[a] = s;
    }
    return ok;
}

template <typename T, int R>
__device__ __forceinline__ bool on_face(const T (&r)[R])
{
    bool b = false;
#pragma unroll
    for (int a = 0; a < R; ++a) b = b || (fabs(r[a]) == T(1));
    return b;
}

struct NewtonArgs {
    const double *nodes;     // [nel][D][NP]
    const float *nodes32;    // [nel][D][NP] x - x_c (mixed mode)
    const double *near;      // [nel][4][NearLds NPAD] nearest-node score rows (FP64)
    const double *xc;        // [nel][D]     (mixed mode)
    const double *pts;       // [D][n]
    int n;
    int nel;
    NewtonIO io;             // io.r holds the start on entry, the result on exit
    int max_iter;
    double tol;
    double eps_d;
    int max_iter32;
    float tol32;
};

// Coordinate c of point p: from the packed copy when the caller made one.
template <int D>
__device__ __forceinline__ double point_coord(const NewtonArgs &a, int p, int c)
{
    return a.io.pts4 ? a.io.pts4[(size_t)p * pt_stride(D) + c] : a.pts[(size_t)c * a.n + p];
}

enum { S_FREE = 0, S_INIT = 1, S_STEP = 2, S_WAIT = 3 };

// Newton launches.  kPrimary: the primary candidates; in FP64 a pair whose
// next pass needs second derivatives is parked (NewtonIO::park_*) and the
// wave goes on with other pairs; in FP32 (mixed mode) such a pair ends the
// FP32 phase.  kResolve: the other candidates of unsettled points, second
// derivatives in the wave.  kFace: the parked pairs, resumed from their
// saved point, radius and pass count, second derivatives in the wave.
// (kResolve and kFace: a few pairs per element, run_few.)
// kPolish: the primary candidates in the FP64 phase of mixed mode (as
// kPrimary, with the polish step and the double-batch refill).
enum { kPrimary = 0, kResolve = 1, kFace = 2, kPolish = 3 };

// Free lanes that make a second refill and plan within a trip worth their
// instructions (some 250 FP64, against lanes idle for one trip).
constexpr int kReplan = 16;
// park_meta flag beside the pass count: no iteration state was saved
constexpr int kParkNoState = 1 << 30;
// State slots a wave reserves at a time: one returning atomic on the pass's
// counter for every trip that parks a pair held k_newton at 2.3 ms (N = 8,
// 5M points: about 130 thousand of them at 16 ns).  Slots left over at the
// end stay empty.
constexpr int kParkReserve = 16;
struct Reserve {
    int next = 0, left = 0;
};

// per-wave counters (scalar registers: counts of ballots)
struct Counters {
    unsigned pairs = 0, passes = 0, evals = 0, evals_h2 = 0, passes32 = 0, evals32 = 0,
             evals_h2_exec = 0, sweeps = 0, sweeps_h2 = 0, sweeps32 = 0, evals32_node = 0;
};

// Adds the wave's counters to the pass's: to the block's copy of them (an
// atomic on one address takes some 16 ns whichever wave it comes from), one
// lane per counter.
__device__ __forceinline__ void add_counters(const Counters &cn, unsigned long long *stats,
                                             int lane)
{
    const unsigned v[11] = {cn.pairs,    cn.passes,  cn.evals,         cn.evals_h2,
                            cn.passes32, cn.evals32, cn.evals_h2_exec, cn.sweeps,
                            cn.sweeps_h2, cn.sweeps32, cn.evals32_node};
    unsigned x = 0;
#pragma unroll
    for (int k = 0; k < 11; ++k) x = lane == k ? v[k] : x;
    if (x)
        atomicAdd(&stats[(blockIdx.x % kStatCopies) * kStats + lane], (unsigned long long)x);
}

// A pair's result record (NewtonIO::rec).
template <int R>
__device__ __forceinline__ void write_record(double *rec, const double (&r)[R], double dist,
                                             bool inside)
{
    typedef double v2 __attribute__((ext_vector_type(2)));
    v2 *o = reinterpret_cast<v2 *>(rec);
    o[0] = v2{r[0], r[1]};
    o[1] = v2{R == 3 ? r[R - 1] : 0.0, inside ? dist : -dist};
}

// The map at GLL node `node` (packed index i + N j + N^2 k): r, the node's
// reference point; X, the node itself; dx/dr_d = sum_m phi_m'(z_{a_d})
// x[.. m ..], an N-term sum along direction d through the node, read from
// the node block: no sweep.
template <typename T, int D, int R, int N>
__device__ __forceinline__ void node_map(const T *xl, int node, T (&r)[R], T (&X)[D], T (&G)[D][R])
{
    typedef NodeLds<T, D, R, N> NL;
    const int a0 = node % N, a1 = (node / N) % N, a2 = R == 3 ? node / (N * N) : 0;
    const int row = R == 3 ? a1 + N * a2 : a1;
#pragma unroll
    for (int c = 0; c < D; ++c) X[c] = xl[NL::at(c, row, a0)];
#pragma unroll
    for (int d = 0; d < R; ++d) {
        const int ad = d == 0 ? a0 : d == 1 ? a1 : a2;
        r[d] = kNodes<T, N>.v[ad];
        T s[D];
#pragma unroll
        for (int c = 0; c < D; ++c) s[c] = T(0);
#pragma unroll
        for (int m = 0; m < N; ++m) {
            const T w = kDiff<T, N>.v[ad][m];
            const int ii = d == 0 ? m : a0, jj = d == 1 ? m : a1, kk = d == 2 ? m : a2;
            const int at = NL::at(0, R == 3 ? jj + N * kk : jj, ii);
#pragma unroll
            for (int c = 0; c < D; ++c) s[c] = fma(w, xl[at + c * NL::RP], s[c]);
        }
#pragma unroll
        for (int c = 0; c < D; ++c) G[c][d] = s[c];
    }
}

// How a pair's start is given: the packed index of a GLL node per list
// position (io.node; the nearest node), or a point r (io.rec per list
// position, or io.r per item).
enum { kStartNode = 0, kStartPoint = 1, kStartEither = 2 };

// Run the iteration of Section 3.2.1 for every pair of element e (its queue
// [q0, q1) in io.list), in precision T, one pair per lane.  FINAL: write
// code/elem/dist/r (FP64 phase); otherwise write r only (FP32 phase of mixed
// mode).  Each trip refills free lanes, plans the trial points of the
// stepping ones, and evaluates the map (sweep 1) where that is due; pairs
// that need second derivatives leave the wave.  stage(): stages the
// element's nodes in LDS.  Returns the number of pairs parked.
template <typename T, int D, int R, int N, bool FINAL, int KIND, typename Stage>
__device__ __forceinline__ int run_element(const NewtonArgs &a, int e, int q0, int q1,
                                           const T *xl, T *tab, T *qb, int lane, int max_iter,
                                           T tol, const double *shift, Reserve &reserve,
                                           Counters &cn, Stage &&stage)
{
    typedef unsigned long long u64;
    constexpr int K = D * (R + 1);
    constexpr int START = KIND == kPolish ? kStartPoint : FINAL ? kStartNode : kStartEither;
    const NewtonIO &io = a.io;
    int state = S_FREE, item = 0, pass = 0, pos = 0, node = -1;
    bool fresh = false;   // evaluated at its start node this trip, not planned yet
    T xs[D], r[R], q[R], alpha = T(1), pred = T(0), xnorm = T(0);
    Obj<T, D, R> cur;
#pragma unroll
    for (int c = 0; c < D; ++c) xs[c] = T(0);
#pragma unroll
    for (int k = 0; k < R; ++k) {
        r[k] = T(0);
        q[k] = T(0);
        cur.g[k] = T(0);
    }
#pragma unroll
    for (int k = 0; k < kSym<R>; ++k) cur.Hgn[k] = T(0);
    cur.f = T(0);
    // Staged pairs: lane l holds the pair at list position cstart + l of the
    // batch [cstart, cend).  Batches of 64 follow each other in list order;
    // the next batch's data are loaded while the current one is handed out,
    // and the list entries of the one after are loaded with them, so that a
    // batch's gathers do not wait for its list.
    struct Batch {
        int it, node;
        double x[D], s[START == kStartNode ? 1 : R];
    };
    int head = q0, cstart = q0, cend = min(q1, q0 + kWave);
    auto load_item = [&](int b0) __attribute__((always_inline)) {
        const int idx = b0 + lane;
        return idx < q1 ? io.list[idx] : 0;
    };
    auto load_batch = [&](int b0, int it, Batch &b) __attribute__((always_inline)) {
        const int idx = b0 + lane;
        b.it = it;
        b.node = -1;
        if (idx < q1) {
            if constexpr (START != kStartPoint) {
                if (START == kStartNode || io.node) b.node = io.node[idx];
            }
            // (the items of the primary pass are the points)
#pragma unroll
            for (int c = 0; c < D; ++c) b.x[c] = point_coord<D>(a, it, c);
            if constexpr (START != kStartNode) {
                if (START == kStartPoint || !io.node) {
                    const double *src = io.rec ? io.rec + (size_t)idx * kRec : io.r + it;
                    const size_t st = io.rec ? 1 : (size_t)io.ostride;
#pragma unroll
                    for (int k = 0; k < R; ++k) b.s[k] = src[k * st];
                }
            }
        }
    };
    Batch cb = {}, nb = {};
    int it2 = 0;   // list entries of the batch after next
    int parked = 0;
    // the first batch is loaded before the nodes are staged, so that the two
    // wait together
    load_batch(q0, load_item(q0), cb);
    if (cend < q1) {
        load_batch(cend, load_item(cend), nb);
        it2 = load_item(cend + kWave);
    }
    stage();
    // Free lanes take the next pairs of the queue (wave-uniform control).
    auto refill = [&]() __attribute__((always_inline)) {
#pragma unroll 1
        for (;;) {
            const u64 freem = __ballot(state == S_FREE);
            if (!freem || head >= q1) return;
            if (head >= cend) {
                cb = nb;
                cstart = cend;
                cend = min(q1, cend + kWave);
                if (cend < q1) {
                    load_batch(cend, it2, nb);
                    it2 = load_item(cend + kWave);
                }
            }
            const int src = head - cstart + __popcll(freem & ((1ull << lane) - 1));
            const bool take = state == S_FREE && src < cend - cstart;
            const int from = min(src, kWave - 1);
            const int it = __shfl(cb.it, from);
            const int nd = START == kStartPoint ? -1 : __shfl(cb.node, from);
            T x[D], s[R];
#pragma unroll
            for (int c = 0; c < D; ++c)
                x[c] = T(__shfl(cb.x[c], from) - (shift ? shift[c] : 0.0));
#pragma unroll
            for (int k = 0; k < R; ++k)
                s[k] = START == kStartNode ? T(0) : T(__shfl(cb.s[START == kStartNode ? 0 : k], from));
            if (take) {
                item = it;
                node = nd;
                pos = cstart + src;
                T xn = T(0);
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    xs[c] = x[c];
                    xn = fma(x[c], x[c], xn);
                }
                xnorm = sqrt_scale(xn);
                // (a start node's r is set where it is evaluated)
                if (START != kStartNode) {
#pragma unroll
                    for (int k = 0; k < R; ++k) r[k] = q[k] = s[k];
                }
                state = S_INIT;
                pass = 0;
                alpha = T(1);
            }
            const int taken = min(__popcll(freem), cend - head);
            if (FINAL) cn.pairs += taken;
            head += taken;
        }
    };
    // A pair is done: results out, lane free.
    auto finish = [&](bool converged) __attribute__((always_inline)) {
        if (FINAL) {
            bool inside = true;
#pragma unroll
            for (int k = 0; k < R; ++k) inside = inside && (fabs(r[k]) < T(1));
            if (R < D) inside = inside && (cur.f < T(a.eps_d));
            double rr[R];
#pragma unroll
            for (int k = 0; k < R; ++k) rr[k] = (double)r[k];
            if (io.rec) {
                write_record<R>(io.rec + (size_t)pos * kRec, rr, sqrt((double)cur.f), inside);
            } else {
                // (the hinted search of particle tracking)
                if (io.conv) io.conv[item] = converged ? 1 : 0;
                io.code[item] = inside ? FPTS_INTERIOR : FPTS_BORDER;
                if (io.elem) io.elem[item] = e;
                io.dist[item] = sqrt((double)cur.f);
#pragma unroll
                for (int k = 0; k < R; ++k) io.r[(size_t)k * io.ostride + item] = rr[k];
            }
        } else {
#pragma unroll
            for (int k = 0; k < R; ++k) {
                if (io.rec)   // the FP64 phase's start
                    io.rec[(size_t)pos * kRec + k] = (double)r[k];
                else
                    io.r[(size_t)k * io.ostride + item] = (double)r[k];
            }
        }
        state = S_FREE;
    };
    // Lanes whose new pair starts at a GLL node: evaluated there without a
    // sweep.  They go to S_STEP with the objective at the start, as an
    // evaluation by sweep 1 would leave them.
    auto node_init = [&]() __attribute__((always_inline)) {
        fresh = false;
        if constexpr (START != kStartPoint) {
            const bool mine = state == S_INIT && node >= 0;
            const u64 minem = __ballot(mine);
            if (!minem) return;
            if (mine) {
                T X[D], Gm[D][R];
                node_map<T, D, R, N>(xl, node, r, X, Gm);
                T dx[D];
                objective<T, D, R>(xs, X, Gm, cur, dx);
                state = S_STEP;
                fresh = true;
            }
            const int cnt = __popcll(minem);
            if (FINAL) cn.evals += cnt;
            else {
                cn.evals32 += cnt;
                cn.evals32_node += cnt;
            }
        }
    };
    // Trial point of each stepping lane (only the fresh ones when asked):
    // the Newton step of Section 3.2.1 on the free coordinates, clipped to
    // the trust region and the box; a step below the tolerance ends the
    // iteration.  Returns the lanes whose pair ended.
    auto plan = [&](bool only_fresh) __attribute__((always_inline)) -> u64 {
        bool ended = false;
        if (state == S_STEP && (!only_fresh || fresh)) {
            // (beta = 0: a pair on a face after its first pass has left)
            {
                // held: at a bound of the box with the gradient pointing
                // out of it (r = +-1 exactly, so r g has the sign test)
                bool held[R];
#pragma unroll
                for (int k = 0; k < R; ++k)
                    held[k] = (fabs(r[k]) == T(1)) & (r[k] * cur.g[k] > T(0));
                T x[R];
                const bool ok = solve_free<T, R>(cur.Hgn, cur.g, held, x);
                T dr[R], dmax = T(0);
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    T d = ok ? x[k] : T(0);
                    d = fmin(fmax(d, -alpha), alpha);
                    const T t = fmin(fmax(r[k] + d, T(-1)), T(1));
                    q[k] = t;
                    dr[k] = t - r[k];
                    dmax = fmax(dmax, fabs(dr[k]));
                }
                T gd = T(0), dHd = T(0);
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    gd = fma(cur.g[k], dr[k], gd);
                    T w = T(0);   // (H dr)_k
#pragma unroll
                    for (int b = 0; b < R; ++b) w = fma(cur.Hgn[sym<R>(k, b)], dr[b], w);
                    dHd = fma(dr[k], w, dHd);
                }
                pred = T(2) * gd - dHd;
                // converged: the step is taken without evaluating the
                // map at q; the squared residual there is the model's,
                // f - pred, whose error is third order in the step.
                // Mixed mode (polish): the first FP64 step from the FP32
                // result is small and stays inside, so the start is within
                // about kPolishTol of the solution and Newton's step
                // leaves an error of second order in it; that step ends
                // the iteration, too.
                ended = dmax < tol;
                if constexpr (KIND == kPolish && R == D)
                    ended = ended || (io.polish && pass == 0 && dmax <= T(kPolishTol) &&
                                      !on_face(r) && !on_face(q));
                if (ended) {
                    ++pass;
#pragma unroll
                    for (int k = 0; k < R; ++k) r[k] = q[k];
                    cur.f = fmax(cur.f - pred, T(0));
                    finish(true);
                }
            }
        }
        const u64 em = __ballot(ended);
        if (FINAL) cn.passes += __popcll(em);
        else cn.passes32 += __popcll(em);
        return em;
    };
    // Sweep 1 at q for the lanes of evalm: their X and G in z.
    auto evaluate = [&](u64 evalm, T (&z)[K]) __attribute__((always_inline)) {
        const int ncg = (__popcll(evalm) + 15) >> 4;
        const int rank = __popcll(evalm & ((1ull << lane) - 1));
        wave_lds_sync();   // earlier reads of qb come first
        if ((evalm >> lane) & 1) {
#pragma unroll
            for (int k = 0; k < R; ++k) qb[k * 64 + rank] = q[k];
        }
        T x[K], y[K];
#pragma unroll 1
        for (int h = 0; h < 2; ++h) {
#pragma unroll 1
            for (int cg = 2 * h; cg < min(ncg, 2 * h + 2); ++cg) {
                if (cg & 1) {
#pragma unroll
                    for (int k = 0; k < K; ++k) x[k] = y[k];
                }
                sweep1<T, D, R, N>(xl, tab, qb, cg, lane, y);
            }
            // (a single group of the two: its totals come out in both rows)
            if (2 * h + 1 >= ncg) {
#pragma unroll
                for (int k = 0; k < K; ++k) x[k] = y[k];
            }
            fold16(x, y);
            if (h == 0) {
#pragma unroll
                for (int k = 0; k < K; ++k) z[k] = x[k];
                if (ncg <= 2) break;
            }
        }
        fold32(z, x);
        if (evalm & (evalm + 1)) {
            // the lanes are not the first ones: column j's totals go to the
            // j-th lane
#pragma unroll
            for (int k = 0; k < K; ++k) z[k] = __shfl(z[k], rank);
        }
        if (FINAL) cn.sweeps += ncg;
        else cn.sweeps32 += ncg;
    };
    const int guard = (q1 - q0 + 16) * (2 * max_iter + 4);
    for (int trip = 0; trip < guard; ++trip) {
        refill();
        node_init();
        if (!__ballot(state != S_FREE)) break;
        // lanes whose pair ends take new pairs at once, and get their first
        // trial point in the same trip, when that many of them are free
        const u64 em = plan(false);
        if (__popcll(em) >= kReplan && head < q1) {
            refill();
            node_init();
            plan(true);
        }
        const u64 evalm = __ballot(state == S_INIT || state == S_STEP);
        if (!evalm) continue;
        T z[K];
        evaluate(evalm, z);
        T X[D], Gm[D][R], dxn[D];
#pragma unroll
        for (int c = 0; c < D; ++c) {
            X[c] = z[c];
#pragma unroll
            for (int k = 0; k < R; ++k) Gm[c][k] = z[D + c * R + k];
        }
        Obj<T, D, R> nw;
        objective<T, D, R>(xs, X, Gm, nw, dxn);
        const u64 initm = __ballot(state == S_INIT), stepm = __ballot(state == S_STEP);
        const int ne = __popcll(stepm) + __popcll(initm);
        if (FINAL) {
            cn.evals += ne;
            cn.passes += __popcll(stepm);
        } else {
            cn.evals32 += ne;
            cn.passes32 += __popcll(stepm);
        }
        bool park = false, at_r = true;
        if (state == S_INIT) {
            cur = nw;
            state = S_STEP;
        } else if (state == S_STEP) {
            ++pass;
            // trust-region test (the step is at least the tolerance here)
            bool accept;
            const T decr = cur.f - nw.f;
            const T sf = sqrt_scale(cur.f);
            const T noise = T(64) * eps_of<T>() * sf * (xnorm + sf);
            if (pred > T(0) && pred <= noise) {
                accept = true;
            } else if (pred > T(0) && decr >= T(0.9) * pred) {
                accept = true;
                alpha *= T(2);
            } else if (pred > T(0) && decr >= T(0.01) * pred) {
                accept = true;
            } else {
                accept = false;
                alpha *= T(0.25);
            }
            if (accept) {
#pragma unroll
                for (int k = 0; k < R; ++k) r[k] = q[k];
                cur = nw;
            }
            if (pass >= max_iter) {
                finish(false);
            } else if (on_face(r)) {
                // the next pass takes second derivatives (beta = 1)
                park = true;
                at_r = accept;
            }
        }
        {
            // pairs whose next pass needs second derivatives leave the wave:
            // FP64 parks them (the face kernel resumes them, many to a wave),
            // FP32 ends its phase there (the FP64 phase takes over).  A
            // launch without a park buffer -- the hinted search of particle
            // tracking -- ends such pairs unconverged.
            const u64 pm = __ballot(park);
            if (pm) {
                if (FINAL && io.park_meta) {
                    // a record per list position, so that nothing has to be
                    // counted; a state slot from the wave's reserve
                    const int np = __popcll(pm);
                    parked += np;
                    if (np > reserve.left) {
                        reserve.left = max(kParkReserve, np);
                        int base = 0;
                        if (lane == 0) base = atomicAdd(io.park_slots, reserve.left);
                        reserve.next = __builtin_amdgcn_readfirstlane(base);
                    }
                    const int k = reserve.next + __popcll(pm & ((1ull << lane) - 1));
                    reserve.next += np;
                    reserve.left -= np;
                    if (park) {
                        // a rejected step leaves r at its start node, where
                        // the objective came from the node block: the face
                        // kernel evaluates it anew, whichever slot it got
                        const bool save = at_r && k < io.park_state_cap;
                        io.node[pos] = -1;
                        io.park_meta[pos] =
                            make_int4(item, k, e, save ? pass : pass | kParkNoState);
#pragma unroll
                        for (int j = 0; j < R; ++j)
                            io.park_r[(size_t)j * io.park_cap + pos] = (double)r[j];
                        io.park_r[(size_t)R * io.park_cap + pos] = (double)alpha;
                        static_assert(1 + R + kSym<R> + D <= kParkState, "park state");
                        if (save) {
                            // the state at r, as the evaluation there left it
                            double *ps = io.park_state + (size_t)k * kParkState;
                            ps[0] = (double)cur.f;
#pragma unroll
                            for (int j = 0; j < R; ++j) ps[1 + j] = (double)cur.g[j];
#pragma unroll
                            for (int j = 0; j < kSym<R>; ++j) ps[1 + R + j] = (double)cur.Hgn[j];
#pragma unroll
                            for (int c = 0; c < D; ++c)
                                ps[1 + R + kSym<R> + c] = (double)dxn[c];
                        }
                    }
                    if (park) state = S_FREE;
                } else if (park) {
                    finish(false);
                }
            }
        }
    }
    return parked;
}

// The iteration for pairs of few-pair elements: the pairs parked on a face
// (kFace) and the other candidates of unsettled points (kResolve), some
// three to five per element.  NB elements to a wave (their node blocks one
// after the other at xl), lanes b L .. b L + L - 1 (L = 64 / NB) for the pairs
// of element b, a pair per lane and no refill; a column group takes 16 / NB
// columns of each element, so that the sweeps and the updates of NB sparse
// elements cost what those of one do.  Second derivatives in the wave.
// has: the lane has a pair; item: kResolve, where its results go; pos: kFace,
// its list position (of its park record and its result record); node:
// kResolve, its start node; xs: its point.
template <int D, int R, int N, int KIND, int NB>
__device__ __forceinline__ void run_few(const NewtonArgs &a, const double *xl, double *tab,
                                        double *qb, int lane, bool has, int item, int pos,
                                        int node, const double (&xs)[D], Counters &cn)
{
    typedef unsigned long long u64;
    typedef NodeLds<double, D, R, N> NL;
    constexpr int K = D * (R + 1), L = kWave / NB, CB = 16 / NB;
    const NewtonIO &io = a.io;
    const int b = lane / L;
    const int max_iter = a.max_iter;
    int state = has ? S_INIT : S_FREE, pass = 0;
    double r[R], q[R], dx[D], Hs[kSym<R>], alpha = 1.0, pred = 0.0;
    Obj<double, D, R> cur;
    bool hb_ok = false;
    cur.f = 0.0;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        r[k] = 0.0;
        q[k] = 0.0;
        cur.g[k] = 0.0;
    }
#pragma unroll
    for (int k = 0; k < kSym<R>; ++k) {
        Hs[k] = 0.0;
        cur.Hgn[k] = 0.0;
    }
#pragma unroll
    for (int c = 0; c < D; ++c) dx[c] = 0.0;
    double xn = 0.0;
#pragma unroll
    for (int c = 0; c < D; ++c) xn = fma(xs[c], xs[c], xn);
    const double xnorm = sqrt_scale(xn);
    if constexpr (KIND == kFace) {
        if (has) {
            // resumed where it was parked: same point, radius and pass count
            // (the pair was counted by the primary pass)
            const int4 mt = io.park_meta[pos];
            pass = mt.w & ~kParkNoState;
            alpha = io.park_r[(size_t)R * io.park_cap + pos];
#pragma unroll
            for (int k = 0; k < R; ++k) r[k] = io.park_r[(size_t)k * io.park_cap + pos];
            if (!(mt.w & kParkNoState)) {
                // with the state the evaluation at r left: the pair waits
                // for its second derivatives at once
                const double *ps = io.park_state + (size_t)mt.y * kParkState;
                cur.f = ps[0];
#pragma unroll
                for (int j = 0; j < R; ++j) cur.g[j] = ps[1 + j];
#pragma unroll
                for (int j = 0; j < kSym<R>; ++j) cur.Hgn[j] = ps[1 + R + j];
#pragma unroll
                for (int c = 0; c < D; ++c) dx[c] = ps[1 + R + kSym<R> + c];
                state = S_WAIT;
            }
        }
    } else {
        // the start is a node: evaluated from the node block
        if (has) {
            double X[D], Gm[D][R];
            node_map<double, D, R, N>(xl + b * NL::STRIDE, node, r, X, Gm);
            objective<double, D, R>(xs, X, Gm, cur, dx);
            state = S_STEP;
        }
        const int cnt = __popcll(__ballot(has));
        cn.pairs += cnt;
        cn.evals += cnt;
    }
#pragma unroll
    for (int k = 0; k < R; ++k) q[k] = r[k];
    auto finish = [&]() __attribute__((always_inline)) {
        bool inside = true;
#pragma unroll
        for (int k = 0; k < R; ++k) inside = inside && (fabs(r[k]) < 1.0);
        if (R < D) inside = inside && (cur.f < a.eps_d);
        if constexpr (KIND == kFace) {
            write_record<R>(io.rec + (size_t)pos * kRec, r, sqrt(cur.f), inside);
        } else {
            io.code[item] = inside ? FPTS_INTERIOR : FPTS_BORDER;
            io.dist[item] = sqrt(cur.f);
#pragma unroll
            for (int k = 0; k < R; ++k) io.r[(size_t)k * io.ostride + item] = r[k];
        }
        state = S_FREE;
    };
    // A lane's place among the lanes of `mask` in its element, and the
    // column groups they make: the element's columns of group cg are those
    // of its lanes with places CB cg .. CB cg + CB - 1.
    auto place = [&](u64 mask, int &ncg) __attribute__((always_inline)) {
        constexpr u64 seg = L == 64 ? ~0ull : (1ull << (L & 63)) - 1;
        int most = 0;
#pragma unroll
        for (int u = 0; u < NB; ++u) most = max(most, __popcll((mask >> (u * L)) & seg));
        ncg = (most + CB - 1) / CB;
        return __popcll((mask >> (b * L)) & seg & ((1ull << (lane & (L - 1))) - 1));
    };
    const int guard = 2 * max_iter + 8;
    for (int trip = 0; trip < guard; ++trip) {
        if (!__ballot(state != S_FREE)) break;
        const u64 waitm = __ballot(state == S_WAIT);
        if (waitm) {
            int ncg;
            const int rank = place(waitm, ncg);
#pragma unroll 1
            for (int cg = 0; cg < ncg; ++cg) {
                const bool mine = state == S_WAIT && rank / CB == cg;
                const int col = b * CB + rank % CB;
                wave_lds_sync();   // earlier reads of qb come first
                if (mine) {
#pragma unroll
                    for (int k = 0; k < R; ++k) qb[k * 16 + col] = r[k];
#pragma unroll
                    for (int c = 0; c < D; ++c) qb[(R + c) * 16 + col] = dx[c];
                }
                double Sn[kSym<R>];
                sweep2<double, D, R, N, NB>(xl, tab, qb, lane, Sn);
#pragma unroll
                for (int k = 0; k < kSym<R>; ++k) {
                    const double v = __shfl(Sn[k], col);
                    if (mine) Hs[k] = v;
                }
                if (mine) {
                    hb_ok = true;
                    state = S_STEP;
                }
            }
            cn.sweeps_h2 += ncg;
            cn.evals_h2 += __popcll(waitm);
            cn.evals_h2_exec += __popcll(waitm);
        }
        // trial points: the Newton step of Section 3.2.1 on the free
        // coordinates, clipped to the trust region and the box; a step below
        // the tolerance ends the iteration
        bool ended = false;
        if (state == S_STEP) {
            const bool beta = (pass > 0) && on_face(r);
            if (beta && !hb_ok) {
                state = S_WAIT;   // dx at r is current: wait for sweep 2
            } else {
                double H[kSym<R>];
#pragma unroll
                for (int k = 0; k < kSym<R>; ++k) H[k] = beta ? cur.Hgn[k] - Hs[k] : cur.Hgn[k];
                // held: at a bound of the box with the gradient pointing
                // out of it (r = +-1 exactly, so r g has the sign test)
                bool held[R];
#pragma unroll
                for (int k = 0; k < R; ++k)
                    held[k] = (fabs(r[k]) == 1.0) & (r[k] * cur.g[k] > 0.0);
                double x[R];
                bool ok = solve_free<double, R>(H, cur.g, held, x);
                if (!ok && beta) {
#pragma unroll
                    for (int k = 0; k < kSym<R>; ++k) H[k] = cur.Hgn[k];
                    ok = solve_free<double, R>(H, cur.g, held, x);
                }
                double dr[R], dmax = 0.0;
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    double d = ok ? x[k] : 0.0;
                    d = fmin(fmax(d, -alpha), alpha);
                    const double t = fmin(fmax(r[k] + d, -1.0), 1.0);
                    q[k] = t;
                    dr[k] = t - r[k];
                    dmax = fmax(dmax, fabs(dr[k]));
                }
                double gd = 0.0, dHd = 0.0;
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    gd = fma(cur.g[k], dr[k], gd);
                    double w = 0.0;   // (H dr)_k
#pragma unroll
                    for (int u = 0; u < R; ++u) w = fma(H[sym<R>(k, u)], dr[u], w);
                    dHd = fma(dr[k], w, dHd);
                }
                pred = 2.0 * gd - dHd;
                if (dmax < a.tol) {
                    // converged: the step is taken without evaluating the
                    // map at q; the squared residual there is the model's,
                    // f - pred, whose error is third order in the step
                    ended = true;
                    ++pass;
#pragma unroll
                    for (int k = 0; k < R; ++k) r[k] = q[k];
                    cur.f = fmax(cur.f - pred, 0.0);
                    finish();
                }
            }
        }
        cn.passes += __popcll(__ballot(ended));
        const u64 stepm = __ballot(state == S_STEP), initm = __ballot(state == S_INIT);
        const u64 evalm = stepm | initm;
        if (!evalm) continue;
        int ncg;
        const int rank = place(evalm, ncg);
        const int col = b * CB + rank % CB;
        wave_lds_sync();   // earlier reads of qb come first
        if ((evalm >> lane) & 1) {
#pragma unroll
            for (int k = 0; k < R; ++k) qb[k * 64 + rank / CB * 16 + col] = q[k];
        }
        double z[K];
#pragma unroll
        for (int k = 0; k < K; ++k) z[k] = 0.0;
#pragma unroll 1
        for (int cg = 0; cg < ncg; ++cg) {
            double y[K];
            sweep1<double, D, R, N, NB>(xl, tab, qb, cg, lane, y);
            slot_sum_all(y);   // a column's totals in its four lanes
            const bool mine = rank / CB == cg;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const double v = __shfl(y[k], col);
                if (mine) z[k] = v;
            }
        }
        cn.sweeps += ncg;
        // a resumed pair re-evaluates the point it was parked at (the same
        // values as before): not a new evaluation of the iteration
        cn.evals += __popcll(stepm) + (KIND != kFace ? __popcll(initm) : 0);
        cn.passes += __popcll(stepm);
        double X[D], Gm[D][R], dxn[D];
#pragma unroll
        for (int c = 0; c < D; ++c) {
            X[c] = z[c];
#pragma unroll
            for (int k = 0; k < R; ++k) Gm[c][k] = z[D + c * R + k];
        }
        Obj<double, D, R> nw;
        objective<double, D, R>(xs, X, Gm, nw, dxn);
        bool moved = false;
        if (state == S_INIT) {
            moved = true;
            state = S_STEP;
        } else if (state == S_STEP) {
            ++pass;
            // trust-region test (the step is at least the tolerance here)
            const double decr = cur.f - nw.f;
            const double sf = sqrt_scale(cur.f);
            const double noise = 64.0 * eps_of<double>() * sf * (xnorm + sf);
            if (pred > 0.0 && pred <= noise) {
                moved = true;
            } else if (pred > 0.0 && decr >= 0.9 * pred) {
                moved = true;
                alpha *= 2.0;
            } else if (pred > 0.0 && decr >= 0.01 * pred) {
                moved = true;
            } else {
                alpha *= 0.25;
            }
            if (moved) {
#pragma unroll
                for (int k = 0; k < R; ++k) r[k] = q[k];
            }
        }
        if (moved) {
            cur = nw;
#pragma unroll
            for (int c = 0; c < D; ++c) dx[c] = dxn[c];
            hb_ok = false;
        }
        if (((stepm >> lane) & 1) && pass >= max_iter) finish();
        else if (moved && pass > 0 && on_face(r)) state = S_WAIT;   // next pass: beta = 1
    }
}

// Copies COUNT values of an element block from global memory to LDS (one
// wave), issuing every load before the first store, then waits for the
// workgroup.  lds starts on 16 bytes; src on a value (an element's block of an
// odd number of values puts the next one between 16-byte words).
template <typename T, int COUNT>
__device__ __forceinline__ void stage(T *lds, const T *src, int lane)
{
    typedef __attribute__((ext_vector_type(4))) unsigned int u4;
    typedef u4 __attribute__((aligned(4))) u4_at_value;   // (a float's alignment)
    constexpr int WORDS = COUNT * (int)sizeof(T) / 16;
    constexpr int PER = (WORDS + kWave - 1) / kWave;
    constexpr int BATCH = 4;   // 16-byte loads in flight per lane
    const u4_at_value *s = reinterpret_cast<const u4_at_value *>(src);
    u4 *d = reinterpret_cast<u4 *>(lds);
#pragma unroll 1
    for (int k0 = 0; k0 < PER; k0 += BATCH) {
        u4 v[BATCH];
#pragma unroll
        for (int k = 0; k < BATCH; ++k) {
            const int w = (k0 + k) * kWave + lane;
            if (w < WORDS) v[k] = s[w];
        }
#pragma unroll
        for (int k = 0; k < BATCH; ++k) {
            const int w = (k0 + k) * kWave + lane;
            if (w < WORDS) d[w] = v[k];
        }
    }
    constexpr int REST = COUNT * (int)sizeof(T) - WORDS * 16;   // 0, 4, 8 or 12 bytes
    const unsigned *s4 = reinterpret_cast<const unsigned *>(src);
    unsigned *d4 = reinterpret_cast<unsigned *>(lds);
    if (lane < REST / 4) d4[WORDS * 4 + lane] = s4[WORDS * 4 + lane];
    __syncthreads();
}

// Copies an element's node block [D][NP] (rows of N values) from global
// memory to LDS in the NodeLds layout, then waits for the workgroup.
template <typename T, int D, int R, int N>
__device__ __forceinline__ void stage_nodes(T *lds, const T *src, int lane)
{
    typedef NodeLds<T, D, R, N> L;
    constexpr int NP = Shape<D, R, N>::NP;
    if constexpr (L::PLAIN) {
        stage<T, D * NP>(lds, src, lane);
    } else {
        constexpr int COUNT = D * NP;
        constexpr int BATCH = 8;
#pragma unroll 1
        for (int v0 = 0; v0 < COUNT; v0 += BATCH * kWave) {
            T v[BATCH];
#pragma unroll
            for (int k = 0; k < BATCH; ++k) {
                const int idx = v0 + k * kWave + lane;
                if (idx < COUNT) v[k] = src[idx];
            }
#pragma unroll
            for (int k = 0; k < BATCH; ++k) {
                const int idx = v0 + k * kWave + lane;
                if (idx < COUNT) {
                    const int c = idx / NP, rem = idx - c * NP;
                    const int row = rem / N, i = rem - row * N;
                    lds[L::at(c, row, i)] = v[k];
                }
            }
        }
        __syncthreads();
    }
}

// Nearest-node contraction operands: B rows [4][NPAD] (-2 x_j, -2 y_j,
// -2 z_j, |x_j|^2 of every node j, element-local; padding columns score a
// large constant) and A rows [4][64] (x, y, z, 1 of each pair).  FP64 reads
// B from rows precomputed at setup (L2-resident per element), so its LDS
// holds only A; FP32 builds B in LDS from the FP32 nodes.
template <typename T, int D, int R, int N>
struct NearLds {
    static constexpr int NPAD = (Shape<D, R, N>::NP + 31) / 32 * 32;   // even tile count
    static constexpr bool B_IN_LDS = std::is_same<T, float>::value;
    static constexpr size_t bytes()
    {
        return sizeof(T) * (4 * ((B_IN_LDS ? NPAD : 0) + 64) + 64);
    }
};

// Nearest element node of up to 64 pairs of one element (Euclidean; among
// equal scores the lowest node index), the start of Newton (Section 3.2.1).
// The squared distance |x - x_j|^2 = |x|^2 - 2 x.x_j + |x_j|^2 has the same
// minimiser as the score |x_j|^2 - 2 x.x_j, a K = 4 contraction of
// (x, y, z, 1) with (-2 x_j, -2 y_j, -2 z_j, |x_j|^2): one 16 x 16 x 4 MFMA
// scores 16 pairs against 16 nodes.  Coordinates are element-local (node
// block minus the element centre) to keep the cancellation small.
// FP64: the accumulator starts at |x|^2, so the MFMA yields the squared
// distance itself (non-negative), and the node index replaces the low
// kNodeBits mantissa bits; one minimum per score then keeps the nearest node
// with ties (equal to 2^-42 relative) to the lowest index.
// Bound by the FP64 products and the two operations that take up each score
// (N = 8, 5M points: 390 us of the 570); the reductions over a row's 16 lanes
// are register moves, since a chain of four shuffles each, through LDS, for
// 16 scores per task cost as much as several node tiles (N = 4, 4M points 184
// -> 160 us; FP32, N = 8, 1.3M points 199 -> 183; N = 6, 27 thousand points 20
// -> 15).
constexpr int kNodeBits = 10;   // node indices below 1024 (N <= 10)
// one bit-field insert (mask from a scalar register: no literal operands
// here), in place in the low word; written out because the compiler would
// fold the node index's own arithmetic into an AND and an OR per score
__device__ __forceinline__ double with_node(double d, int node)
{
    const unsigned m = (1u << kNodeBits) - 1;
    unsigned lo = (unsigned)__double2loint(d);
    asm("v_bfi_b32 %0, %1, %2, %0" : "+v"(lo) : "s"(m), "v"(node));
    return __hiloint2double(__double2hiint(d), (int)lo);
}
// min of two keys: the keys are finite or +inf (never NaN), so the plain
// instruction serves; fmin() would first quiet both operands, which the
// compiler cannot prove to be ordinary numbers after the bit insertion.
__device__ __forceinline__ double key_min(double a, double b)
{
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float key_min(float a, float b)
{
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
// x of the lane SH places on in the row of 16 (register moves; a shuffle goes
// through LDS, and the reductions over a row are chains of four)
template <int SH>
__device__ __forceinline__ int row_ror(int x)
{
    return __builtin_amdgcn_mov_dpp(x, 0x120 + SH, 0xf, 0xf, true);
}
template <int SH>
__device__ __forceinline__ float row_ror(float x)
{
    return __int_as_float(row_ror<SH>(__float_as_int(x)));
}
template <int SH>
__device__ __forceinline__ double row_ror(double x)
{
    return __hiloint2double(row_ror<SH>(__double2hiint(x)), row_ror<SH>(__double2loint(x)));
}
template <int D, int R, int N, bool MIXED>
__device__ __forceinline__ void nearest_body(const NewtonArgs &a)
{
    typedef Shape<D, R, N> S;
    typedef NearLds<typename std::conditional<MIXED, float, double>::type, D, R, N> L;
    typedef typename std::conditional<MIXED, float, double>::type T;
    typedef typename V4<T>::type v4;
    constexpr int NT = L::NPAD / 16;   // node tiles (even)
    const T kBig = MIXED ? T(1e30f) : T(1e300);
    extern __shared__ double lds_raw[];
    T *Bt = reinterpret_cast<T *>(lds_raw);                  // [4][NPAD] (FP32)
    T *Pt = Bt + (L::B_IN_LDS ? 4 * L::NPAD : 0);            // [4][64]
    T *Xx = Pt + 4 * 64;                                     // [64] |x|^2
    const int lane = threadIdx.x, col = lane & 15, g = lane >> 4;
    const NewtonIO &io = a.io;
    const int total = io.chunk_off[a.nel];
    const int G = gridDim.x;
    // A task's inputs arrive through a chain of dependent loads (task ->
    // element offsets -> pair ids -> point coordinates).  The chain of the
    // wave's next task is started level by level while the current one is
    // scored, so that its latency hides behind the MFMA work.
    auto task_of = [&](int t, int &e, int &beg, int &cnt) __attribute__((always_inline)) {
        e = __builtin_amdgcn_readfirstlane(io.task_elem[t]);
        beg = io.elem_off[e] + (t - io.chunk_off[e]) * kChunk;
        cnt = min(io.elem_off[e + 1] - beg, kChunk);
    };
    auto pair_of = [&](int beg, int cnt) __attribute__((always_inline)) { return lane < cnt ? io.list[beg + lane] : 0; };
    // (the primary pass only: its items are the points themselves)
    auto coords_of = [&](int cnt, int item, double (&x)[D]) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < D; ++c) x[c] = lane < cnt ? point_coord<D>(a, item, c) : 0.0;
    };
    int t = task_of_block();
    if (t >= total) return;
    int e, beg, cnt;
    task_of(t, e, beg, cnt);
    int item = pair_of(beg, cnt);
    double px[D];
    coords_of(cnt, item, px);
    for (;;) {
        const int tn = t + G;
        const bool more = tn < total;
        int en = 0, begn = 0, cntn = 0;
        if (more) task_of(tn, en, begn, cntn);   // next task, level 1
        double xc[D];
#pragma unroll
        for (int c = 0; c < D; ++c) xc[c] = a.xc[(size_t)e * D + c];
        wave_lds_sync();   // the previous task's reads come first
        // B rows of the element's nodes (FP32; FP64 reads the setup rows), up
        // to eight nodes' loads per lane at once
        constexpr int AHEAD = 8;
#pragma unroll 1
        for (int j0 = lane; L::B_IN_LDS && j0 < L::NPAD; j0 += AHEAD * kWave) {
            T v[AHEAD][D];
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                const int j = min(j0 + u * kWave, S::NP - 1);
#pragma unroll
                for (int c = 0; c < D; ++c)
                    v[u][c] = MIXED ? T(a.nodes32[((size_t)e * D + c) * S::NP + j])
                                    : T(a.nodes[((size_t)e * D + c) * S::NP + j] - xc[c]);
            }
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                const int j = j0 + u * kWave;
                if (j >= L::NPAD) break;
                T r[4] = {T(0), T(0), T(0), T(0)};
                if (j < S::NP) {
                    T n2 = T(0);
#pragma unroll
                    for (int c = 0; c < D; ++c) {
                        r[c] = T(-2) * v[u][c];
                        n2 = fma(v[u][c], v[u][c], n2);
                    }
                    r[D] = n2;
                } else {
                    r[D] = kBig;
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) Bt[k * L::NPAD + j] = r[k];
            }
        }
        // A rows of the pairs
        {
            const bool has = lane < cnt;
            T pa[4] = {T(0), T(0), T(0), T(0)};
#pragma unroll
            for (int c = 0; c < D; ++c) pa[c] = has ? T(px[c] - xc[c]) : T(0);
            pa[D] = T(1);
            T xx = T(0);
#pragma unroll
            for (int c = 0; c < D; ++c) xx = fma(pa[c], pa[c], xx);
#pragma unroll
            for (int k = 0; k < 4; ++k) Pt[k * 64 + lane] = pa[k];
            Xx[lane] = xx;
        }
        wave_lds_sync();
        const int itemn = more ? pair_of(begn, cntn) : 0;   // next task, level 2
        const int ntile = (cnt + 15) >> 4;   // pair tiles of this task (wave-uniform)
        // the start of the pair at task position pl: node bi
        auto write_start = [&](int bi, int pl) __attribute__((always_inline)) {
            io.node[beg + pl] = bi;
        };
        double pxn[D];
        if constexpr (!MIXED) {
            v4 seed[4];
            double av[4], best[4][4];
#pragma unroll
            for (int pt = 0; pt < 4; ++pt) {
                av[pt] = Pt[g * 64 + 16 * pt + col];
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) {
                    seed[pt][qq] = Xx[16 * pt + g + 4 * qq];   // pair of output row g + 4 qq
                    best[pt][qq] = __builtin_huge_val();
                }
            }
            // One loop per pair-tile count, free of branches, so that the
            // tiles' MFMAs issue back to back and each result is taken up
            // after the others are issued.  Each lane's B values are loaded
            // four node tiles ahead into four registers, each reloaded right
            // after its tile's MFMAs have read it (no copy at the loop's back
            // edge, which would wait for the load); NT is even, NT >= 2.
            const double *brow = a.near + ((size_t)e * 4 + g) * L::NPAD + col;
            auto scan = [&](auto tiles) __attribute__((always_inline)) {
                constexpr int NTL = decltype(tiles)::value;
                auto tile = [&](int nt, double bv) __attribute__((always_inline)) {
                    if (nt == NT / 2 && more) coords_of(cntn, itemn, pxn);   // next task, level 3
                    const int node = 16 * nt + col;
                    v4 d[NTL];
#pragma unroll
                    for (int pt = 0; pt < NTL; ++pt) d[pt] = mfma16(av[pt], bv, seed[pt]);
#pragma unroll
                    for (int pt = 0; pt < NTL; ++pt)
#pragma unroll
                        for (int qq = 0; qq < 4; ++qq)
                            best[pt][qq] = key_min(best[pt][qq], with_node(d[pt][qq], node));
                };
                constexpr int NT4 = NT & ~3;
                double b0 = brow[0], b1 = brow[16], b2 = 0.0, b3 = 0.0;
                if constexpr (NT > 2) {
                    b2 = brow[32];
                    b3 = brow[48];
                }
                // The reloads are unconditional (past the row's end they read
                // its last tile again), so that the wait before each tile
                // counts on the three loads issued after its own.  Their
                // offsets pass through an empty asm statement: otherwise the
                // compiler proves each reload equal to the next iteration's
                // tile and loads it there, just before its use.
                auto ahead = [&](int t) __attribute__((always_inline)) {
                    int off = 16 * min(t, NT - 1);
                    asm volatile("" : "+s"(off));
                    return brow[off];
                };
#pragma unroll 1
                for (int nt = 0; nt < NT4; nt += 4) {
                    tile(nt, b0);
                    b0 = ahead(nt + 4);
                    tile(nt + 1, b1);
                    b1 = ahead(nt + 5);
                    tile(nt + 2, b2);
                    b2 = ahead(nt + 6);
                    tile(nt + 3, b3);
                    b3 = ahead(nt + 7);
                }
                if constexpr (NT4 < NT) {
                    // the last two tiles (NT = 2 mod 4), in b0 and b1
                    tile(NT4, b0);
                    tile(NT4 + 1, b1);
                }
            };
            switch (ntile) {
            case 1: scan(std::integral_constant<int, 1>()); break;
            case 2: scan(std::integral_constant<int, 2>()); break;
            case 3: scan(std::integral_constant<int, 3>()); break;
            default: scan(std::integral_constant<int, 4>()); break;
            }
#pragma unroll
            for (int pt = 0; pt < 4; ++pt) {
                if (pt >= ntile) break;
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) {
                    double k = best[pt][qq];
                    k = key_min(k, row_ror<8>(k));
                    k = key_min(k, row_ror<4>(k));
                    k = key_min(k, row_ror<2>(k));
                    best[pt][qq] = key_min(k, row_ror<1>(k));
                }
                // lane `col` < 4 writes the pair of output row g + 4 col
                // (the node index is in the low word; masks, not a select
                // chain, which the compiler would turn into a stack array)
                int lo = 0;
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) lo |= __double2loint(best[pt][qq]) & -(col == qq);
                const int pl = 16 * pt + g + 4 * col;
                if (col < 4 && pl < cnt) write_start(lo & ((1 << kNodeBits) - 1), pl);
            }
        } else {
            T av[4], best[4][4];
            int bix[4][4];
#pragma unroll
            for (int pt = 0; pt < 4; ++pt) {
                av[pt] = Pt[g * 64 + 16 * pt + col];
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) {
                    best[pt][qq] = T(__builtin_huge_valf());
                    bix[pt][qq] = 0;
                }
            }
            // node tiles outside, pair tiles inside: each B value is read once
            // per task and scores every pair tile; one branch-free loop per
            // pair-tile count, the tiles' MFMAs issued back to back
            auto scan = [&](auto tiles) __attribute__((always_inline)) {
                constexpr int NTL = decltype(tiles)::value;
#pragma unroll 2
                for (int nt = 0; nt < NT; ++nt) {
                    if (nt == NT / 2 && more) coords_of(cntn, itemn, pxn);   // next task, level 3
                    const T bv = Bt[g * L::NPAD + 16 * nt + col];
                    const int node = 16 * nt + col;
                    v4 d[NTL];
#pragma unroll
                    for (int pt = 0; pt < NTL; ++pt) d[pt] = mfma16(av[pt], bv, v4{0, 0, 0, 0});
#pragma unroll
                    for (int pt = 0; pt < NTL; ++pt)
#pragma unroll
                        for (int qq = 0; qq < 4; ++qq) {
                            const bool lt = d[pt][qq] < best[pt][qq];
                            bix[pt][qq] = lt ? node : bix[pt][qq];
                            best[pt][qq] = lt ? d[pt][qq] : best[pt][qq];
                        }
                }
            };
            switch (ntile) {
            case 1: scan(std::integral_constant<int, 1>()); break;
            case 2: scan(std::integral_constant<int, 2>()); break;
            case 3: scan(std::integral_constant<int, 3>()); break;
            default: scan(std::integral_constant<int, 4>()); break;
            }
#pragma unroll
            for (int pt = 0; pt < 4; ++pt) {
                if (pt >= ntile) break;
                // over the 16 lanes of a row: the lowest score, then the lowest
                // node among the lanes that hold it
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) {
                    T k = best[pt][qq];
                    k = key_min(k, row_ror<8>(k));
                    k = key_min(k, row_ror<4>(k));
                    k = key_min(k, row_ror<2>(k));
                    k = key_min(k, row_ror<1>(k));
                    int i = best[pt][qq] == k ? bix[pt][qq] : INT32_MAX;
                    i = min(i, row_ror<8>(i));
                    i = min(i, row_ror<4>(i));
                    i = min(i, row_ror<2>(i));
                    bix[pt][qq] = min(i, row_ror<1>(i));
                }
                // lane `col` < 4 writes the pair of its row group held in item qq = col
                int bi = bix[pt][0] * (col == 0) + bix[pt][1] * (col == 1) +
                         bix[pt][2] * (col == 2) + bix[pt][3] * (col == 3);
                const int pl = 16 * pt + 4 * g + col;   // FP32 output layout
                if (col < 4 && pl < cnt) write_start(bi, pl);
            }
        }
        if (!more) break;
        t = tn;
        e = en;
        beg = begn;
        cnt = cntn;
        item = itemn;
#pragma unroll
        for (int c = 0; c < D; ++c) px[c] = pxn[c];
    }
}

// Nearest node of x among an element's nodes staged in LDS at xl (FP64,
// NodeLds layout), by a segment of L lanes together (j: the lane's place in
// it): the squared distance summed over the coordinates in order, the lowest
// node index among equal distances (Section 3.2.1 starts Newton there).
// (The same reduction, and four nodes' reads at once: k_newton_resolve, N = 8,
// 5M points 431 -> 415 us; surface, N = 7, 2M points 174 -> 161.)
template <int D, int R, int N, int L>
__device__ __forceinline__ int nearest_staged(const double *xl, const double (&x)[D], int j)
{
    double bd = __builtin_huge_val();
    int bi = 0;
#pragma unroll(N <= 8 ? 4 : 1)
    for (int n = j; n < Shape<D, R, N>::NP; n += L) {
        double d2 = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const double t = x[d] - xl[NodeLds<double, D, R, N>::at(d, n / N, n % N)];
            d2 = fma(t, t, d2);
        }
        if (d2 < bd) {
            bd = d2;
            bi = n;
        }
    }
    // the lowest distance, then the lowest node among the lanes that hold it
    // (rows of 16 by register moves, the rest of the segment by shuffles)
    double k = bd;
    k = key_min(k, row_ror<8>(k));
    k = key_min(k, row_ror<4>(k));
    k = key_min(k, row_ror<2>(k));
    k = key_min(k, row_ror<1>(k));
    if (L >= 32) k = key_min(k, __shfl_xor(k, 16));
    if (L >= 64) k = key_min(k, __shfl_xor(k, 32));
    bi = bd == k ? bi : INT32_MAX;
    bi = min(bi, row_ror<8>(bi));
    bi = min(bi, row_ror<4>(bi));
    bi = min(bi, row_ror<2>(bi));
    bi = min(bi, row_ror<1>(bi));
    if (L >= 32) bi = min(bi, __shfl_xor(bi, 16));
    if (L >= 64) bi = min(bi, __shfl_xor(bi, 32));
    return bi;
}

// Newton over the element queues in precision T.  Tasks are the parts of an
// element's queue: io.newt_off[e] .. io.newt_off[e + 1] - 1 are element e's,
// io.newt_task[t] is task t's element, and the element's pairs are divided
// evenly among its tasks: one task per element would leave most waves idle
// at the end where elements hold many pairs (2 million particles in 3888
// elements, N = 8: 2.37 ms so).  The primary and polish passes and the FP32
// phase divide the tasks among the XCDs, a contiguous range each; a wave's
// first task is its own place in its XCD's range, the others come from the
// XCD's counter (io.counter, kXcdCounter ints apart; the FP32 phase's after
// the FP64 kernels').  (One counter for all: an atomic on one address takes
// some 16 ns, 1.05 ms for the 64 thousand tasks of 4M points, N = 4.)
template <typename T, int D, int R, int N, int KIND>
__device__ __forceinline__ void newton_body(const NewtonArgs &a)
{
    typedef Shape<D, R, N> S;
    typedef Lds<T, D, R, N> L;
    constexpr bool FINAL = std::is_same<T, double>::value;
    extern __shared__ double lds_raw[];
    const int lane = threadIdx.x;
    const NewtonIO &io = a.io;
    T *xl = reinterpret_cast<T *>(lds_raw);
    T *tab = xl + L::NODES;
    T *qb = tab + L::TAB;
    Counters cn;
    const int *off = io.newt_off, *elem = io.newt_task;
    const int all = off[a.nel];
    // (the grid is a multiple of the XCD count)
    const int xcd = blockIdx.x % kXcd, waves = gridDim.x / kXcd;
    const int share = (all + kXcd - 1) / kXcd;
    const int first = xcd * share, total = min(all, first + share);
    int *ctr = io.counter + ((FINAL ? 0 : kXcd) + xcd) * kXcdCounter;
    // the ticket of the wave's next task is taken one task ahead, so that
    // its atomic completes while the current one is processed (every ticket
    // of the range is processed by the wave that took it)
    auto take = [&]() __attribute__((always_inline)) {
        int v = 0;
        if (lane == 0) v = atomicAdd(ctr, 1);
        return first + waves + v;
    };
    int ticket = first + (int)blockIdx.x / kXcd;
    int parked = 0;
    Reserve reserve;
    for (;;) {
        const int t = __builtin_amdgcn_readfirstlane(ticket);
        if (t >= total) break;
        ticket = take();
        const int e = __builtin_amdgcn_readfirstlane(elem[t]);
        // part t - off[e] of the queue's nt even parts
        const int nt = off[e + 1] - off[e];
        int q0 = io.elem_off[e], q1 = io.elem_off[e + 1];
        const int per = (q1 - q0 + nt - 1) / nt;
        q0 += (t - off[e]) * per;
        q1 = min(q1, q0 + per);
        __syncthreads();
        // the nodes are staged after the first batch of pairs has been asked
        // for
        if constexpr (FINAL) {
            const double *src = a.nodes + (size_t)e * D * S::NP;
            parked += run_element<double, D, R, N, true, KIND>(
                a, e, q0, q1, xl, tab, qb, lane, a.max_iter, a.tol, nullptr, reserve, cn,
                [&] { stage_nodes<double, D, R, N>(xl, src, lane); });
        } else {
            const float *src = a.nodes32 + (size_t)e * D * S::NP;
            run_element<float, D, R, N, false, KIND>(
                a, e, q0, q1, xl, tab, qb, lane, a.max_iter32, a.tol32, a.xc + (size_t)e * D,
                reserve, cn, [&] { stage_nodes<float, D, R, N>(xl, src, lane); });
        }
    }
    if (FINAL && lane == 0 && parked) atomicAdd(io.park_count, parked);
    add_counters(cn, io.stats, lane);
}

// The face and resolve kernels: waves stride over the tasks of io.task_elem
// (up to few_lanes pairs of one element each; io.chunk_off their offsets per
// element), up to NB of them at a time, consecutive ones.  kResolve finds the
// starts of its pairs itself, from the nodes it stages anyway: a separate
// nearest-node pass would read every such element's node data once more for
// a few pairs, and score them on matrix tiles of 16.
template <int D, int R, int N, int KIND>
__device__ __forceinline__ void few_body(const NewtonArgs &a)
{
    typedef Shape<D, R, N> S;
    typedef NodeLds<double, D, R, N> NL;
    constexpr int NB = few_elems(R, N), L = few_lanes(R, N);
    extern __shared__ double lds_raw[];
    double *xl = lds_raw;
    double *tab = xl + NB * NL::STRIDE;
    double *qb = tab + Lds<double, D, R, N>::TAB;
    const int lane = threadIdx.x, b = lane / L, j = lane % L;
    const NewtonIO &io = a.io;
    Counters cn;
    const int total = io.chunk_off[a.nel];
    // elements per trip: fewer than NB where the launch's waves are more than
    // total / NB (a wave with one element is done sooner than one with NB)
    const int nb = min(NB, (total + (int)gridDim.x - 1) / (int)gridDim.x);
    for (int64_t t0 = (int64_t)task_of_block() * nb; t0 < total; t0 += (int64_t)gridDim.x * nb) {
        const int t = (int)t0 + b;
        const bool on = b < nb && t < total;
        const int e = on ? io.task_elem[t] : -1;
        int q = 0;
        bool has = false;
        if (on) {
            q = io.elem_off[e] + (t - io.chunk_off[e]) * L + j;
            has = q < io.elem_off[e + 1];
        }
        // kFace: the list holds the pairs' positions in the primary list
        const int pos = has ? io.list[q] : 0;
        int item = pos, p = 0;
        if (has) {
            if constexpr (KIND == kFace) item = p = io.park_meta[pos].x;
            else p = io.slot_pt[item];
        }
        double xs[D];
#pragma unroll
        for (int d = 0; d < D; ++d) xs[d] = has ? point_coord<D>(a, p, d) : 0.0;
        __syncthreads();   // the previous elements' reads come first
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int eu = __builtin_amdgcn_readlane(e, u * L);
            if (eu >= 0)
                stage_nodes<double, D, R, N>(xl + u * NL::STRIDE, a.nodes + (size_t)eu * D * S::NP,
                                             lane);
        }
        int node = 0;
        if constexpr (KIND == kResolve) {
            // every segment finds its pairs' nearest nodes one after the other
            const unsigned long long hm = __ballot(has);
            int most = 0;
#pragma unroll
            for (int u = 0; u < NB; ++u)
                most = max(most, __popcll(L == 64 ? hm : (hm >> (u * L)) & ((1ull << (L & 63)) - 1)));
            for (int k = 0; k < most; ++k) {
                double x[D];
#pragma unroll
                for (int d = 0; d < D; ++d) x[d] = __shfl(xs[d], b * L + k);
                const int bi = nearest_staged<D, R, N, L>(xl + b * NL::STRIDE, x, j);
                if (j == k) node = bi;
            }
        }
        run_few<D, R, N, KIND, NB>(a, xl, tab, qb, lane, has, item, pos, node, xs, cn);
    }
    add_counters(cn, io.stats, lane);
}

// Waves per SIMD of the Newton and resolve kernels (the launch takes four times
// as many blocks per CU).  Two parameters leave room for three, with a few
// spilled registers at most, which cover more of each other's latencies
// (k_newton, surface, N = 7, 2M points 485 -> 431 us; quads, N = 6, 1.5M
// points 213 -> 179; k_newton_resolve, surface, N = 6, 1M points 135 -> 90;
// at N = 10 it spills, 216 -> 238, and stays at two).  Three parameters need
// all 256 registers (N = 4 at three waves: 2251 instead of 768 us).
constexpr int newton_waves(int R) { return R == 2 ? 3 : 2; }
constexpr int resolve_waves(int R, int N) { return R == 2 && N <= 9 ? 3 : 2; }

// (at least three waves per SIMD: the register budget then stays within the
// 256 VGPRs, and the compiler gives the MFMA results VGPRs, not AGPRs that
// the selection would first have to copy out)
template <int D, int R, int N, bool MIXED>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3))) void
k_nearest(NewtonArgs a)
{
    nearest_body<D, R, N, MIXED>(a);
}
template <int D, int R, int N>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(
    newton_waves(R), newton_waves(R)))) void
k_newton(NewtonArgs a)
{
    newton_body<double, D, R, N, kPrimary>(a);
}
template <int D, int R, int N>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(
    newton_waves(R), newton_waves(R)))) void
k_newton_polish(NewtonArgs a)
{
    newton_body<double, D, R, N, kPolish>(a);
}
template <int D, int R, int N>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(
    resolve_waves(R, N), resolve_waves(R, N)))) void
k_newton_resolve(NewtonArgs a)
{
    few_body<D, R, N, kResolve>(a);
}
template <int D, int R, int N>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void
k_newton_face(NewtonArgs a)
{
    few_body<D, R, N, kFace>(a);
}
template <int D, int R, int N>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3, 3))) void
k_newton32(NewtonArgs a)
{
    newton_body<float, D, R, N, kPrimary>(a);
}

// Phase D for the points whose other candidates found no room in the slot
// array (more candidate pairs than the workspace holds): one wavefront per
// point, its other candidates in ascending id order, each started from its
// nearest node (squared distances to every node of the element, ties to the
// lowest index) and iterated by the code of the resolve kernel, with one lane's
// pair; then the selection rule of Section 3.2 over the primary and them.  One
// pair per wavefront: a path for rare overloads only.
template <int D, int R, int N>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void
k_resolve_overflow(NewtonArgs a, HashView h)
{
    typedef Shape<D, R, N> S;
    extern __shared__ double lds_raw[];
    double *xl = lds_raw;
    double *tab = xl + Lds<double, D, R, N>::NODES;
    double *qb = tab + Lds<double, D, R, N>::TAB;
    const int lane = threadIdx.x, b = blockIdx.x, G = gridDim.x;
    const NewtonIO &io = a.io;
    const int cnt = *io.ocount;
    // a pair's result goes to item b of the block's scratch
    int *ov_code = io.ov_int;
    NewtonArgs la = a;
    la.io.code = ov_code;
    la.io.r = io.ov_dbl;
    la.io.ostride = G;
    la.io.dist = io.ov_dbl + (size_t)R * G;
    Counters cn;
    for (int i = b; i < cnt; i += G) {
        const int p = io.list[i];
        const int prim = io.cand[p].y, c = io.cellpt[p];
        double x[D];
#pragma unroll
        for (int d = 0; d < D; ++d) x[d] = point_coord<D>(a, p, d);
        // the primary's result is the best so far
        int bcode = io.code[p], belem = prim;
        double bdist = io.dist[p], br[R];
#pragma unroll
        for (int k = 0; k < R; ++k) br[k] = io.r[(size_t)k * io.ostride + p];
        bool changed = false;
        for (int q = h.cell_off[c]; q < h.cell_off[c + 1]; ++q) {
            const int e = h.cell_el[q];
            double depth;
            if (e == prim || !box_pass<D>(h.box + (size_t)e * (3 * D + D * D), x, depth))
                continue;
            __syncthreads();
            stage_nodes<double, D, R, N>(xl, a.nodes + (size_t)e * D * S::NP, lane);
            const int bi = nearest_staged<D, R, N, kWave>(xl, x, lane);
            run_few<D, R, N, kResolve, 1>(la, xl, tab, qb, lane, lane == 0, b, 0, bi, x, cn);
            // lane 0, the pair's lane, wrote the result
            int cd = 0;
            double dd = 0.0, rr[R];
            if (lane == 0) {
                cd = ov_code[b];
                dd = la.io.dist[b];
            }
#pragma unroll
            for (int k = 0; k < R; ++k) rr[k] = lane == 0 ? la.io.r[(size_t)k * G + b] : 0.0;
            cd = __shfl(cd, 0);
            dd = __shfl(dd, 0);
#pragma unroll
            for (int k = 0; k < R; ++k) rr[k] = __shfl(rr[k], 0);
            // Section 3.2: the lowest-id INTERIOR candidate, else the
            // smallest distance, the lower id on ties
            bool take;
            if (bcode == FPTS_INTERIOR) take = cd == FPTS_INTERIOR && e < belem;
            else if (cd == FPTS_INTERIOR) take = true;
            else take = dd < bdist || (dd == bdist && e < belem);
            if (take) {
                bcode = cd;
                belem = e;
                bdist = dd;
#pragma unroll
                for (int k = 0; k < R; ++k) br[k] = rr[k];
                changed = true;
            }
        }
        if (lane == 0 && changed) {
            io.code[p] = bcode;
            io.elem[p] = belem;
            io.dist[p] = bdist;
#pragma unroll
            for (int k = 0; k < R; ++k) io.r[(size_t)k * io.ostride + p] = br[k];
        }
    }
    add_counters(cn, io.stats, lane);
}

typedef void (*KernelFn)(NewtonArgs);
typedef void (*OverflowFn)(NewtonArgs, HashView);

struct Kernels {
    KernelFn nearest = nullptr, newton32 = nullptr, newton = nullptr, warm = nullptr,
             face = nullptr;
    OverflowFn overflow = nullptr;
    size_t lds_nearest = 0, lds_newton32 = 0, lds_newton = 0, lds_few = 0;
};

template <int D, int R, bool MIXED>
Kernels pick_kernels(int N, bool resolve)
{
    typedef typename std::conditional<MIXED, float, double>::type TN;
    Kernels k;
#define FPTS_CASE(NN)                                                                       \
    case NN:                                                                                \
        k.nearest = resolve ? nullptr : k_nearest<D, R, NN, MIXED>;                          \
        k.newton = resolve ? k_newton_resolve<D, R, NN> : k_newton<D, R, NN>;               \
        k.warm = k_newton_polish<D, R, NN>;                                                 \
        k.face = k_newton_face<D, R, NN>;                                                   \
        k.overflow = k_resolve_overflow<D, R, NN>;                                          \
        if (MIXED && !resolve) {                                                            \
            k.newton32 = k_newton32<D, R, NN>;                                              \
        }                                                                                   \
        k.lds_nearest = NearLds<TN, D, R, NN>::bytes();                                     \
        k.lds_newton32 = Lds<float, D, R, NN>::bytes();                                     \
        k.lds_newton = Lds<double, D, R, NN>::bytes();                                      \
        k.lds_few = k.lds_newton + sizeof(double) * (few_elems(R, NN) - 1) *                \
                                       NodeLds<double, D, R, NN>::STRIDE;                   \
        break;
    switch (N) {
        FPTS_CASE(2)
        FPTS_CASE(3)
        FPTS_CASE(4)
        FPTS_CASE(5)
        FPTS_CASE(6)
        FPTS_CASE(7)
        FPTS_CASE(8)
        FPTS_CASE(9)
        FPTS_CASE(10)
    default:
        break;
    }
#undef FPTS_CASE
    return k;
}

// Launches on the caller's stream: nearest nodes (which & 1; task grid of
// 64-pair tasks over io.chunk_off, io.task_elem; not for the *_resolve
// kernels, which find them from the nodes they stage), then Newton (which & 2;
// the tasks of io.newt_off, io.newt_task: in mixed mode the FP32 phase, then
// the FP64 kernel); which & 4 runs the face kernel over the parked pairs
// (io.list = their list positions binned by element, io.elem_off / chunk_off
// / task_elem their buckets and tasks).  io.counter must be zero
// (kNewtonCounters ints).  A list with io.slot_pt set (other candidates) selects
// the *_resolve kernels, whose waves stride over tasks of up to few_lanes pairs,
// like those of the face kernel.
template <int D, int R>
hipError_t launch_newton_kind(const fpts_mesh *m, bool mixed, int64_t n, const double *pts,
                              const NewtonIO &io, int which, hipStream_t s)
{
    const bool resolve = io.slot_pt != nullptr;
    const Kernels k = mixed ? pick_kernels<D, R, true>(m->N, resolve)
                            : pick_kernels<D, R, false>(m->N, resolve);
    if ((!k.nearest && !resolve) || !k.newton) return hipErrorInvalidValue;
    NewtonArgs a;
    a.nodes = m->d_nodes;
    a.nodes32 = m->d_nodes32;
    a.near = m->d_near;
    if (m->near_npad != (m->NP + 31) / 32 * 32) return hipErrorInvalidValue;
    a.xc = m->d_xc;
    a.pts = pts;
    a.n = (int)n;
    a.nel = (int)m->nel;
    a.io = io;
    a.max_iter = io.max_iter > 0 ? io.max_iter : m->p.max_iter;
    a.tol = m->p.newton_tol;
    a.eps_d = m->p.surf_eps_d;
    a.max_iter32 = m->p.mixed_max_iter;
    a.tol32 = (float)m->p.mixed_tol;
    // the other candidates' Newton kernel finds their starts itself
    if ((which & 1) && !resolve) {
        hipLaunchKernelGGL(k.nearest, dim3(task_grid(io.task_bound, m->cus)), dim3(64),
                           k.lds_nearest, s, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (which & 2) {
        if (k.newton32) {
            // three waves per SIMD, as the kernel's register budget allows
            hipLaunchKernelGGL(k.newton32, dim3(xcd_grid((int64_t)m->cus * 12)), dim3(64),
                               k.lds_newton32, s, a);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        // starts given as points (the FP32 phase's results, or the hinted
        // search of particle tracking) take the warm-start kernel
        const KernelFn kn = resolve || (io.node && !mixed) ? k.newton : k.warm;
        const int waves = resolve ? resolve_waves(m->R, m->N) : newton_waves(m->R);
        hipLaunchKernelGGL(kn, dim3(xcd_grid((int64_t)m->cus * 4 * waves)), dim3(64),
                           resolve ? k.lds_few : k.lds_newton, s, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (which & 4) {
        if (!k.face) return hipErrorInvalidValue;
        hipLaunchKernelGGL(k.face, dim3(xcd_grid((int64_t)m->cus * 8)), dim3(64), k.lds_few, s,
                           a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (which & 8) {
        // grid = the scratch's block count (io.task_bound)
        if (!k.overflow || io.task_bound < 1) return hipErrorInvalidValue;
        hipLaunchKernelGGL(k.overflow, dim3((unsigned)io.task_bound), dim3(64), k.lds_newton, s,
                           a, hash_view(m));
        return hipGetLastError();
    }
    return hipSuccess;
}

}  // namespace newton
}  // namespace fpts
