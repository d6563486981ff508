// Interpolate (Section 3.3): u_f(r*) = sum_ijk u_f,ijk phi_i(r) phi_j(s)
// phi_k(t) (eq. eq_u_tensor) at the computational coordinates from Find.
//
// Points are first counted and scattered into per-element buckets (the
// grouping by element the paper's CPU code uses, Section 5 remark), then a
// wavefront takes up to 64 points of ONE element, stages the element's nodal
// values in LDS (once per wave, not once per point) and each lane contracts
// them sum-factorised: N^3 + N^2 + N FMAs per field and point.  On quad, hex
// and surface meshes the first contraction runs on the matrix cores, 16
// points at a time (k_eval_mfma): every lane reading the same staged value
// (a broadcast, 64 copies per read) left the per-lane form bound by LDS
// bandwidth.  Line meshes keep the per-lane form.
// Also: the FP32 element-local node copy used by mixed-precision Newton.
#include "fpts_internal.hpp"
#include "gll_table.hpp"
#include "newton_mfma.hpp"

namespace fpts {
namespace {

// fields per launch from which, nodes per direction up to which and points
// from which the values go through list order (launch_eval; the points for an
// Interpolate call and for the first pass of the fused call)
constexpr int kSpreadFields = 3, kSpreadNodes = 6;
constexpr int64_t kSpreadPoints = 2500000, kSpreadFusedPoints = 500000;

// fused find + interpolate: elements holding at most this many of the
// remaining points have them interpolated one lane per point
constexpr int kSparseMax = 4;

// pass 0: count points per element, keep each point's rank in its bucket
// (-1 for points not binned) and write NaN for NOT_FOUND points; pass 1:
// place point ids (with their r, as records, unless erec is null) at their
// ranks in their element's bucket.  With `cand`
// (fused find + interpolate) the points that their primary result settled
// are left out: the fused pass over Find's primary list has them.
__global__ __launch_bounds__(256) void k_eval_bin(int pass, int n, int nel, int es, int R,
                                                 const int32_t *code, const int32_t *elem,
                                                 const double *r, const int2 *cand,
                                                 int n_fields, double *out, int *elem_cnt,
                                                 const int *elem_off, int *rank,
                                                 int *sorted, double *erec)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const bool in = p < n;
    if (pass == 1) {
        // rank[p] < 0: not binned
        if (!in) return;
        const int k = rank[p], e = elem[p];
        if (erec) {
            // volume and surface meshes: r and the id as one record (a
            // scattered write of 32 bytes costs what one of 4 does, and the
            // interpolation then reads its points in order)
            double rr[3] = {0.0, 0.0, 0.0};
#pragma unroll
            for (int a = 0; a < 3; ++a)
                if (a < R) rr[a] = r[(size_t)a * n + p];
            if (k >= 0) {
                typedef double v2 __attribute__((ext_vector_type(2)));
                v2 *o = reinterpret_cast<v2 *>(erec + (size_t)(elem_off[e] + k) * kRec);
                o[0] = v2{rr[0], rr[1]};
                o[1] = v2{rr[2], __hiloint2double(0, p)};
            }
        } else if (k >= 0) {
            sorted[elem_off[e] + k] = p;
        }
        return;
    }
    // pass 0, no early exit (wave_inc needs every lane); all of a point's
    // loads are issued at once
    int e = -1, pr = -1;
    int32_t cd = FPTS_NOT_FOUND;
    double rr[3] = {0.0, 0.0, 0.0};
    if (in) {
        e = elem[p];
        cd = code[p];
        if (cand) {
            pr = cand[p].y;
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (k < R) rr[k] = r[(size_t)k * n + p];
        }
    }
    const bool found = in && cd != FPTS_NOT_FOUND && e >= 0 && e < nel;
    bool done = false;
    if (cand && found && cd == FPTS_INTERIOR && pr == e) {
        double mg = 1.0;
        for (int k = 0; k < R; ++k) mg = fmin(mg, 1.0 - fabs(rr[k]));
        done = mg > kSettleGuard;
    }
    const bool bin = found && !done;
    const int k = wave_inc(elem_cnt, e * es, bin);
    if (in) rank[p] = bin ? k : -1;
    if (in && !found)
        for (int f = 0; f < n_fields; ++f) out[(size_t)f * n + p] = __builtin_nan("");
}

// k_eval_bin over a list of found points (grid-stride; the loop bound is
// uniform per wavefront, as wave_inc needs)
__global__ __launch_bounds__(256) void k_eval_bin_list(int pass, const int *list,
                                                      const int *count, int nel, int es,
                                                      const int32_t *elem, int *elem_cnt,
                                                      const int *elem_off, int *rank,
                                                      int *sorted)
{
    const int cnt = *count;
    const int lane = threadIdx.x & 63;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i - lane < cnt;
         i += gridDim.x * blockDim.x) {
        const bool act = i < cnt;
        const int p = act ? list[i] : 0;
        const int e = act ? elem[p] : -1;
        const bool ok = act && e >= 0 && e < nel;
        if (pass == 0) {
            const int k = wave_inc(elem_cnt, e * es, ok);
            if (act) rank[i] = ok ? k : -1;
        } else if (ok && rank[i] >= 0) {
            sorted[elem_off[e] + rank[i]] = p;
        }
    }
}

template <int N>
__device__ __forceinline__ void basis_v(double r, const double *z, const double *w, double (&v)[N])
{
    double pv[N];
    pv[0] = 1.0;
#pragma unroll
    for (int i = 1; i < N; ++i) pv[i] = pv[i - 1] * (r - z[i - 1]);
    double sv = 1.0;
#pragma unroll
    for (int i = N - 1; i >= 0; --i) {
        v[i] = w[i] * (pv[i] * sv);
        sv *= r - z[i];
    }
}

struct EvalArgs {
    const double *r;        // [R][n]
    int n;
    int nel;
    int n_fields;
    const double *field;    // [n_fields][nel][NP]
    double *out;            // [n_fields][n]
    const int *sorted;
    const int *elem_off;
    const int *chunk_off;   // task offsets per element
    const int *task_elem;   // task -> element
    Basis basis;
    // where r comes from, by list position (first one that is not null):
    // erec, records (r, id) of k_eval_bin; rec, Find's result records of its
    // primary list (NewtonIO::rec; with deep_only those that are not INTERIOR
    // at least kSettleGuard inside are skipped); rs, the same of line meshes
    // (NaN skips the point).  Else r
    const double *erec;
    const double *rec;
    bool deep_only;
    const double *rs;
    // k_eval_mfma: values by list position, tmp[4 q + f] (k_eval_spread
    // brings them into point order), instead of out
    double *tmp;
    int f0;                 // first field of this launch (k_eval_mfma)
};

typedef const __attribute__((address_space(4))) double cdouble;

// sum over the element's nodal values u of one field times the tensor bases
template <int R, int N, typename P>
__device__ __forceinline__ double contract(P u, const double (&v0)[N], const double (&v1)[N],
                                           const double (&v2)[N])
{
    double acc = 0.0;
    if constexpr (R == 3) {
#pragma unroll
        for (int k = 0; k < N; ++k) {
            double B = 0.0;
#pragma unroll
            for (int j = 0; j < N; ++j) {
                double A = 0.0;
#pragma unroll
                for (int i = 0; i < N; ++i) A = fma(u[i + N * (j + N * k)], v0[i], A);
                B = fma(A, v1[j], B);
            }
            acc = fma(B, v2[k], acc);
        }
    } else if constexpr (R == 2) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            double A = 0.0;
#pragma unroll
            for (int i = 0; i < N; ++i) A = fma(u[i + N * j], v0[i], A);
            acc = fma(A, v1[j], acc);
        }
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) acc = fma(u[i], v0[i], acc);
    }
    return acc;
}

// LDS: the element's nodal values of each field are staged in LDS with
// coalesced loads and read by every lane at the same address (broadcast);
// otherwise they are read with scalar loads.  Staging wins when an element
// holds few points (its values are cold, and scalar loads of them stall on
// latency); when many tasks share an element its values stay in the scalar
// cache and the scalar operands save the LDS reads.  The staged loads are
// software-pipelined: the values of the next field (or of the next task's
// first field) are loaded into registers while the current field is
// contracted, so their latency hides behind the arithmetic.
template <int R, int N, bool LDS>
__global__ __launch_bounds__(64) void k_eval(EvalArgs a)
{
    constexpr int NP = (R == 3) ? N * N * N : (R == 2) ? N * N : N;
    constexpr int PER = (NP + 63) / 64;   // staged values per lane
    extern __shared__ double ldsu[];   // [NP] (LDS staging)
    const int lane = threadIdx.x;
    const int total = a.chunk_off[a.nel];
    const int G = gridDim.x;
    double pre[PER];
    // the nodal values of field f of element e into pre
    auto fetch = [&](int e, int f) {
        const double *src = a.field + ((size_t)f * a.nel + e) * NP;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int j = lane + 64 * k;
            pre[k] = (NP % 64 == 0 || j < NP) ? src[j] : 0.0;
        }
    };
    int t = task_of_block();
    if (LDS && t < total && a.n_fields > 0)
        fetch(__builtin_amdgcn_readfirstlane(a.task_elem[t]), 0);
    for (; t < total; t += G) {
        const int e = __builtin_amdgcn_readfirstlane(a.task_elem[t]);
        const int beg = a.elem_off[e] + (t - a.chunk_off[e]) * kChunk;
        const int end = min(a.elem_off[e + 1], beg + kChunk);
        const int idx = beg + lane;
        bool has = idx < end;
        const int p = has ? a.sorted[idx] : 0;
        double rr[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < R; ++k)
            if (has) rr[k] = a.rs ? a.rs[(size_t)k * a.n + idx] : a.r[(size_t)k * a.n + p];
        if (a.rs) has = has && !__builtin_isnan(rr[0]);
        double v0[N], v1[N], v2[N];
        basis_v<N>(has ? rr[0] : 0.0, a.basis.z, a.basis.w, v0);
        if (R >= 2) basis_v<N>(has ? rr[1] : 0.0, a.basis.z, a.basis.w, v1);
        if (R == 3) basis_v<N>(has ? rr[2] : 0.0, a.basis.z, a.basis.w, v2);
        for (int f = 0; f < a.n_fields; ++f) {
            double acc;
            if constexpr (LDS) {
                __syncthreads();   // the previous field's reads come first
#pragma unroll
                for (int k = 0; k < PER; ++k) {
                    const int j = lane + 64 * k;
                    if (NP % 64 == 0 || j < NP) ldsu[j] = pre[k];
                }
                __syncthreads();
                if (f + 1 < a.n_fields) fetch(e, f + 1);
                else if (t + G < total) fetch(__builtin_amdgcn_readfirstlane(a.task_elem[t + G]), 0);
                acc = contract<R, N>((const double *)ldsu, v0, v1, v2);
            } else {
                acc = contract<R, N>((cdouble *)(a.field + ((size_t)f * a.nel + e) * NP), v0, v1,
                                     v2);
            }
            if (has) a.out[(size_t)f * a.n + p] = acc;
        }
    }
}

// Waves per SIMD of k_eval_mfma: four where the fields loaded ahead leave the
// contraction enough of 128 registers, else two, with all they can use (N = 6,
// four fields, 3M points: 250 us so, 373 held to four with 108 spilled
// registers; N = 8, three fields, 5M points: 423 us, 468 with three waves, which
// get in each other's way with their scattered writes).  Calls of 2M points, N = 3
// to 10, one to four fields, each with two, three and four waves: the rule's choice
// is the fastest or within 3 % of it, but for quads of N = 9 and 10 with four
// fields (266 us, 248 with four waves; 270, 258).  On either side of its lines:
// hexes, N = 7, one field 230 us (248 with two waves), two 283 (313 with four);
// N = 9 and 10, one field 346 (391), 466 (492); quads, N = 10, three fields 224
// (250), N = 8, four 237 (234).
template <int R, int N, int FC>
constexpr int eval_waves_per_eu()
{
    return (R == 2 ? FC * N <= 30 : FC * N * N <= 90) ? 4 : 2;
}

// Fields of a launch at most: four, but three on hexes of ten nodes per
// direction, where the products of four spill 14 registers (13824 elements, four
// fields in one launch and in two: 3M points 2011 and 1710 us, 20 thousand 219
// and 175; on 512 elements, 20 thousand points 45 and 53).
constexpr int most_fields(int R, int N) { return R == 3 && N == 10 ? 3 : 4; }

// Interpolation with the first contraction on the matrix cores (quad, hex
// and surface meshes; FC fields a.f0 .. a.f0 + FC - 1 per launch).  One
// wavefront per task, one of the even parts of an element's list (one wave
// for each element left most of the chip idle where the points crowd: 2M
// points in the wake of a channel, N = 8, three fields, 679 -> 201 us): the
// FC fields of the element are staged in LDS once (layout of the Newton
// kernels' node block, one field per coordinate slot), and the task's points
// are taken 64 and then 16 at a time, one per slot of four lanes (slot = lane
// % 16, quarter g = lane / 16).  Quarter g builds the bases of direction g of
// its slot's point; then C_f[row][s] = sum_i u_f[i][row] phi_i(r_s) on the
// matrix cores (A = the element's values, row = (j, k) or j; B = the slots'
// phi_i; tiles of 16 rows, the last rows in tiles of four), each lane weights
// its rows with phi_j(s) phi_k(t) of its slot (hexes with N = 4, 8: summed
// over k first, then weighted per j), and the four lanes of a slot are
// summed.  A point's value depends on its own coordinates and element only,
// not on the group or task it lands in.
// The fields of the wave's next task, the next 64 points and the offsets of
// the task after are loaded while the current ones are contracted.
// Bound by FP64 arithmetic at large N (N = 8, 5M points, three fields: 423
// us, with the matrix cores 63% and the vector units another 27% of the time
// busy, against 240 for the products alone) and by the scattered writes of
// its values at small N (N = 4, 4M points, one field: 107 us, 37 G/s).
template <int R, int N, int FC>
__global__ __launch_bounds__(64)
__attribute__((amdgpu_waves_per_eu(eval_waves_per_eu<R, N, FC>(),
                                   eval_waves_per_eu<R, N, FC>()))) void
k_eval_mfma(EvalArgs a)
{
    typedef newton::Shape<3, R, N> S;
    typedef newton::NodeLds<double, FC, R, N> L;
    typedef newton::Factor<R, N> F;
    typedef newton::V4<double>::type v4;
    constexpr int NP = S::NP, ROWS = S::ROWS, KS = S::KS;
    constexpr int PER = (NP + 63) / 64;
    // row tiles: FT of 16 rows, QT of four (a 16-row tile takes as long as
    // four of those)
    constexpr int FT = ROWS / 16 + (ROWS % 16 > 12 ? 1 : 0);
    constexpr int QT = ROWS > 16 * FT ? (ROWS - 16 * FT + 3) / 4 : 0;
    constexpr bool kFullK = N % 4 == 0;
    constexpr bool kRows = ROWS >= 16 * FT;   // the 16-row tiles' rows all exist
    // what the A operand's padding reads: a zero of its own, behind the tables.
    // (A field's value there, times the zero of the B operand, would carry a
    // NaN or an infinity of one field into the others.)
    constexpr int kZero = L::SIZE + R * N * 16;
    extern __shared__ double lds_eval[];
    const int lane = threadIdx.x, slot = lane & 15, g = lane >> 4;
    double *xl = lds_eval;        // the FC fields, NodeLds layout
    double *tab = xl + L::SIZE;   // [R][N][16] bases of the group's points
    if (N % 4 && lane == 0) xl[kZero] = 0.0;   // (read after stage_fields' barriers)
    const int G = gridDim.x, nel = a.nel;
    double v[FC][PER];
    auto load_fields = [&](int en) __attribute__((always_inline)) {
#pragma unroll
        for (int f = 0; f < FC; ++f) {
            const double *src = a.field + ((size_t)(a.f0 + f) * nel + en) * NP;
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int j = lane + 64 * k;
                v[f][k] = (NP % 64 == 0 || j < NP) ? src[j] : 0.0;
            }
        }
    };
    // the element's FC fields, from v into LDS
    auto stage_fields = [&]() __attribute__((always_inline)) {
        __syncthreads();   // the previous element's reads come first
#pragma unroll
        for (int f = 0; f < FC; ++f)
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int j = lane + 64 * k;
                if (NP % 64 == 0 || j < NP) xl[L::at(f, j / N, j % N)] = v[f][k];
            }
        __syncthreads();
    };
    // the lane's point: list position beg + lane (< end)
    struct Pt {
        double r[3], sd;
        int p;
    };
    auto load_point = [&](int beg, int end, Pt &q) __attribute__((always_inline)) {
        const int idx = beg + lane;
        q.p = 0;
        q.sd = 0.0;
        q.r[0] = q.r[1] = q.r[2] = 0.0;
        if (idx >= end) return;
        if (a.erec || a.rec) {
            typedef double v2 __attribute__((ext_vector_type(2)));
            const v2 *src = reinterpret_cast<const v2 *>((a.erec ? a.erec : a.rec) +
                                                         (size_t)idx * kRec);
            const v2 lo = src[0], hi = src[1];
            q.r[0] = lo[0];
            q.r[1] = lo[1];
            q.r[2] = hi[0];
            q.sd = hi[1];
            if (!a.erec && !a.tmp) q.p = a.sorted[idx];
        } else {
            q.p = a.sorted[idx];
#pragma unroll
            for (int k = 0; k < R; ++k) q.r[k] = a.r[(size_t)k * a.n + q.p];
        }
    };
    Pt nx;   // the next points
    // the points of the staged element: list positions [ebeg, eend), the
    // first of them in nx
    auto points = [&](int ebeg, int eend, int nbeg, int nend) __attribute__((always_inline)) {
#pragma unroll 1
        for (int beg = ebeg; beg < eend; beg += kChunk) {
            const int end = min(eend, beg + kChunk);
            const Pt cur = nx;
            if (end < eend) load_point(end, eend, nx);
            else load_point(nbeg, nend, nx);
            bool has = beg + lane < end;
            int p = cur.p;
            if (a.erec) {
                p = __double2loint(cur.sd);
            } else if (a.rec && a.deep_only) {
                double mg = 1.0;
#pragma unroll
                for (int k = 0; k < R; ++k) mg = fmin(mg, 1.0 - fabs(cur.r[k]));
                has = has && !__builtin_signbit(cur.sd) && mg > kSettleGuard;
            }
#pragma unroll 1
            for (int grp = 0; beg + 16 * grp < end; ++grp) {
                const int first = beg + 16 * grp;   // the group's positions
                const int pl = 16 * grp + slot;   // the lane with this slot's point
                // coordinate g of that point (each coordinate shuffled, then
                // the quarter's one selected)
                const double c0 = __shfl(cur.r[0], pl);
                const double c1 = R >= 2 ? __shfl(cur.r[1], pl) : 0.0;
                const double c2 = R == 3 ? __shfl(cur.r[2], pl) : 0.0;
                const double x = g == 0 ? c0 : g == 1 ? c1 : c2;
                newton::wave_lds_sync();   // the previous group's table reads come first
                if (g < R) {
                    double pv[N];
                    pv[0] = 1.0;
#pragma unroll
                    for (int i = 1; i < N; ++i) pv[i] = pv[i - 1] * (x - a.basis.z[i - 1]);
                    double sv = 1.0;
#pragma unroll
                    for (int i = N - 1; i >= 0; --i) {
                        tab[(g * N + i) * 16 + slot] = a.basis.w[i] * (pv[i] * sv);
                        sv *= x - a.basis.z[i];
                    }
                }
                newton::wave_lds_sync();
                const double *ts = tab + N * 16, *tt = tab + 2 * N * 16;
                double b0[KS];
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const int i = 4 * ks + g;
                    b0[ks] = kFullK || i < N ? tab[i * 16 + slot] : 0.0;
                }
                double X[FC], Z[F::NJ][FC];
#pragma unroll
                for (int f = 0; f < FC; ++f) {
                    X[f] = 0.0;
#pragma unroll
                    for (int js = 0; js < F::NJ; ++js) Z[js][f] = 0.0;
                }
                // one contraction row of the lane, weighted into the sums
                auto weight = [&](int row) __attribute__((always_inline)) {
                    return R == 3 ? ts[(row % N) * 16 + slot] * tt[(row / N) * 16 + slot]
                                  : ts[row * 16 + slot];
                };
#pragma unroll(FT <= 4 ? (FT > 0 ? FT : 1) : 1)
                for (int m = 0; m < FT; ++m) {
                    v4 acc[FC];
#pragma unroll
                    for (int f = 0; f < FC; ++f) acc[f] = v4{0, 0, 0, 0};
                    const int arow = 16 * m + slot;
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        const int ai = 4 * ks + g;
                        const bool aok = (kRows || arow < ROWS) && (kFullK || ai < N);
#pragma unroll
                        for (int f = 0; f < FC; ++f)
                            acc[f] = newton::mfma16(xl[aok ? L::at(f, arow, ai) : kZero],
                                                    b0[ks], acc[f]);
                    }
#pragma unroll
                    for (int qq = 0; qq < 4; ++qq) {
                        const int row = newton::out_row(m, g, qq);
                        if (!kRows && row >= ROWS) continue;
                        if constexpr (F::ON) {
                            const int k = (16 * m + 4 * qq) / N, js = qq % F::NJ;
                            const double tv = tt[k * 16 + slot];
#pragma unroll
                            for (int f = 0; f < FC; ++f) Z[js][f] = fma(acc[f][qq], tv, Z[js][f]);
                        } else {
                            const double w = weight(row);
#pragma unroll
                            for (int f = 0; f < FC; ++f) X[f] = fma(acc[f][qq], w, X[f]);
                        }
                    }
                }
#pragma unroll
                for (int t = 0; t < QT; ++t) {
                    const int base = 16 * FT + 4 * t;
                    const bool whole = base + 4 <= ROWS;
                    const int arow = base + (slot & 3), row = base + g;
                    double c[FC];
#pragma unroll
                    for (int f = 0; f < FC; ++f) c[f] = 0.0;
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        const int ai = 4 * ks + g;
                        const bool aok = (whole || arow < ROWS) && (kFullK || ai < N);
#pragma unroll
                        for (int f = 0; f < FC; ++f)
                            c[f] = newton::mfma4(xl[aok ? L::at(f, arow, ai) : kZero], b0[ks],
                                                 c[f]);
                    }
                    if (whole || row < ROWS) {
                        const double w = weight(row);
#pragma unroll
                        for (int f = 0; f < FC; ++f) X[f] = fma(c[f], w, X[f]);
                    }
                }
                if constexpr (F::ON) {
#pragma unroll
                    for (int js = 0; js < F::NJ; ++js) {
                        const double sv = ts[(g + 4 * js) * 16 + slot];
#pragma unroll
                        for (int f = 0; f < FC; ++f) X[f] = fma(Z[js][f], sv, X[f]);
                    }
                }
                newton::slot_sum_all(X);
                // quarter g writes field g of its slot's point
                double u = X[0];
#pragma unroll
                for (int f = 1; f < FC; ++f) u = g == f ? X[f] : u;
                if (a.tmp) {
                    if (g < FC && first + slot < end) a.tmp[(size_t)(first + slot) * 4 + g] = u;
                } else {
                    const bool hp = __shfl((int)has, pl) != 0;
                    const int pp = __shfl(p, pl);
                    if (hp && g < FC) a.out[(size_t)(a.f0 + g) * a.n + pp] = u;
                }
            }
        }
    };
    const int total = a.chunk_off[nel];
    // task t's list positions from its element's offsets (loaded a task ahead)
    struct Offs {
        int c0, c1, o0, o1;
    };
    auto load_offs = [&](int e, Offs &o) __attribute__((always_inline)) {
        o.c0 = a.chunk_off[e];
        o.c1 = a.chunk_off[e + 1];
        o.o0 = a.elem_off[e];
        o.o1 = a.elem_off[e + 1];
    };
    auto range_of = [&](int t, const Offs &o, int &q0, int &q1) __attribute__((always_inline)) {
        const int k = __builtin_amdgcn_readfirstlane(t - o.c0);
        const int nt = __builtin_amdgcn_readfirstlane(o.c1 - o.c0);
        const int b = __builtin_amdgcn_readfirstlane(o.o0);
        const int cnt = __builtin_amdgcn_readfirstlane(o.o1) - b;
        const int per = ((cnt + nt - 1) / nt + 15) / 16 * 16;   // whole groups
        q0 = b + min(cnt, k * per);
        q1 = b + min(cnt, (k + 1) * per);
    };
    int t = task_of_block();
    if (t >= total) return;
    // e: the task's element, e1: the next one's, e2: that of the one after,
    // each loaded a task before its offsets are
    int q0, q1, e1 = 0, e2 = 0;
    Offs of;
    {
        const int e = __builtin_amdgcn_readfirstlane(a.task_elem[t]);
        if (t + G < total) e1 = a.task_elem[t + G];
        if (t + 2 * G < total) e2 = a.task_elem[t + 2 * G];
        load_offs(e, of);
        range_of(t, of, q0, q1);
        load_fields(e);
        load_point(q0, q1, nx);
        e1 = __builtin_amdgcn_readfirstlane(e1);
        if (t + G < total) load_offs(e1, of);
    }
    for (;;) {
        stage_fields();   // loaded during the previous task
        const int tn = t + G;
        int n0 = 0, n1 = 0;
        if (tn < total) {
            range_of(tn, of, n0, n1);
            load_fields(e1);
            e1 = __builtin_amdgcn_readfirstlane(e2);
            if (tn + G < total) load_offs(e1, of);
            if (tn + 2 * G < total) e2 = a.task_elem[tn + 2 * G];
        }
        if (q0 < q1) points(q0, q1, n0, n1);
        else load_point(n0, n1, nx);
        if (tn >= total) break;
        t = tn;
        q0 = n0;
        q1 = n1;
    }
}

// Values by list position (tmp[4 q + f], FC fields from f0 on) into point
// order: a 32-byte gather per point and coalesced writes, instead of a
// scattered 8-byte write per point and field (some 30 G/s on this GPU).  The
// list position of point p: elem_off[elem] + rank (rank < 0: not in the
// list), or, with cand, its place in Find's primary list (points that the
// list's results do not settle get values that the interpolation of the
// rest overwrites).
template <int FC>
__global__ __launch_bounds__(256) void k_eval_spread(int n, const int2 *cand, const int32_t *elem,
                                                    const int *rank, const int *elem_off,
                                                    const double *tmp, int f0, double *out)
{
    typedef double v2 __attribute__((ext_vector_type(2)));
    constexpr int U = 4;
    const int64_t base = (int64_t)blockIdx.x * U * 256 + threadIdx.x;
    int64_t pos[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t p = base + u * 256;
        int e = -1;
        unsigned k = 0;
        if (p < n) {
            if (cand) {
                const int2 cd = cand[p];
                e = cd.y;
                k = (unsigned)cd.x >> 1;
            } else {
                const int rk = rank[p];
                e = rk < 0 ? -1 : elem[p];
                k = (unsigned)rk;
            }
        }
        pos[u] = e < 0 ? -1 : (int64_t)elem_off[e] + k;
    }
    v2 lo[U], hi[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        lo[u] = v2{0.0, 0.0};
        hi[u] = v2{0.0, 0.0};
        if (pos[u] >= 0) {
            const v2 *src = reinterpret_cast<const v2 *>(tmp + pos[u] * 4);
            lo[u] = src[0];
            if (FC > 2) hi[u] = src[1];
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t p = base + u * 256;
        if (pos[u] < 0) continue;
        const double x[4] = {lo[u][0], lo[u][1], hi[u][0], hi[u][1]};
#pragma unroll
        for (int f = 0; f < FC; ++f) out[(size_t)(f0 + f) * n + p] = x[f];
    }
}

// Line meshes: points of elements that hold at most kSparseMax of the
// points to interpolate, one lane per point: a wavefront per element task
// would run the whole element's contraction for one or two points.  Each
// lane reads its own element's nodal values (global loads), with the
// arithmetic of k_eval, so both give the same bits.  Grid-stride over the
// list.
template <int R, int N>
__global__ __launch_bounds__(256) void k_eval_sparse(EvalArgs a, const int32_t *elem,
                                                    const int *list, const int *count)
{
    constexpr int NP = (R == 3) ? N * N * N : (R == 2) ? N * N : N;
    const int cnt = *count;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < cnt; i += gridDim.x * blockDim.x) {
        const int p = list[i];
        const int e = elem[p];
        double rr[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < R; ++k) rr[k] = a.r[(size_t)k * a.n + p];
        double v0[N], v1[N], v2[N];
        basis_v<N>(rr[0], a.basis.z, a.basis.w, v0);
        if (R >= 2) basis_v<N>(rr[1], a.basis.z, a.basis.w, v1);
        if (R == 3) basis_v<N>(rr[2], a.basis.z, a.basis.w, v2);
        for (int f = 0; f < a.n_fields; ++f) {
            const double *src = a.field + ((size_t)f * a.nel + e) * NP;
            a.out[(size_t)f * a.n + p] = contract<R, N>(src, v0, v1, v2);
        }
    }
}

// Elements with at most kSparseMax binned points drop out of the bucket
// counts (their points go to the per-point list).
__global__ __launch_bounds__(256) void k_eval_dense(int nel, int es, int *elem_cnt)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < nel && elem_cnt[e * es] <= kSparseMax) elem_cnt[e * es] = 0;
}

// Pass 1 with the split: a binned point (rank >= 0) of a dense element goes
// to its bucket, one of a sparse element to the list.  A block takes
// kSplitChunk consecutive points, gathers its listed points in LDS and
// reserves their places with one atomic (same-address device atomics
// serialise).
constexpr int kSplitChunk = 4096;

__global__ __launch_bounds__(256) void k_eval_split(int n, const int32_t *elem, const int *rank,
                                                   const int *dense_cnt, int es, const int *elem_off,
                                                   int *sorted, int *list, int *count)
{
    __shared__ int lst[kSplitChunk];
    __shared__ int lcnt, gbase;
    const int lane = threadIdx.x & 63;
    if (threadIdx.x == 0) lcnt = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kSplitChunk;
    for (int it = 0; it < kSplitChunk / 256; ++it) {
        const int64_t q = base + it * 256 + threadIdx.x;
        const int p = (int)q;
        bool sp = false;
        if (q < n) {
            const int k = rank[p], e = elem[p];
            if (k >= 0) {
                if (dense_cnt[e * es] > 0) sorted[elem_off[e] + k] = p;
                else sp = true;
            }
        }
        const unsigned long long m = __ballot(sp);
        if (m) {
            int at = 0;
            if (lane == 0) at = atomicAdd(&lcnt, __popcll(m));
            at = __shfl(at, 0, 64);
            if (sp) lst[at + __popcll(m & ((1ull << lane) - 1))] = p;
        }
    }
    __syncthreads();
    const int cnt = lcnt;
    if (cnt == 0) return;
    if (threadIdx.x == 0) gbase = atomicAdd(count, cnt);
    __syncthreads();
    for (int i = threadIdx.x; i < cnt; i += 256) list[gbase + i] = lst[i];
}

__global__ void k_nodes32(const double *nodes, const double *xc, float *out, int64_t nel, int D,
                          int NP)
{
    const int64_t total = nel * D * NP;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t e = i / ((int64_t)D * NP);
        const int c = (int)((i / NP) % D);
        out[i] = (float)(nodes[i] - xc[e * D + c]);
    }
}

__global__ void k_near_rows(const double *nodes, const double *xc, double *rows, int64_t nel,
                            int D, int NP, int npad)
{
    const int64_t total = nel * npad;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t e = i / npad;
        const int j = (int)(i % npad);
        double b[4] = {0.0, 0.0, 0.0, 0.0};
        if (j < NP) {
            double n2 = 0.0;
            for (int c = 0; c < D; ++c) {
                const double v = nodes[(e * D + c) * NP + j] - xc[e * D + c];
                b[c] = -2.0 * v;
                n2 = fma(v, v, n2);
            }
            b[D] = n2;
        } else {
            b[D] = 1e300;
        }
        for (int k = 0; k < 4; ++k) rows[(e * 4 + k) * npad + j] = b[k];
    }
}

typedef void (*EvalFn)(EvalArgs);

template <int R, bool LDS>
EvalFn pick_eval(int N)
{
    switch (N) {
    case 2: return k_eval<R, 2, LDS>;
    case 3: return k_eval<R, 3, LDS>;
    case 4: return k_eval<R, 4, LDS>;
    case 5: return k_eval<R, 5, LDS>;
    case 6: return k_eval<R, 6, LDS>;
    case 7: return k_eval<R, 7, LDS>;
    case 8: return k_eval<R, 8, LDS>;
    case 9: return k_eval<R, 9, LDS>;
    case 10: return k_eval<R, 10, LDS>;
    default: return nullptr;
    }
}

typedef void (*SparseFn)(EvalArgs, const int32_t *, const int *, const int *);

template <int R>
SparseFn pick_sparse(int N)
{
    switch (N) {
    case 2: return k_eval_sparse<R, 2>;
    case 3: return k_eval_sparse<R, 3>;
    case 4: return k_eval_sparse<R, 4>;
    case 5: return k_eval_sparse<R, 5>;
    case 6: return k_eval_sparse<R, 6>;
    case 7: return k_eval_sparse<R, 7>;
    case 8: return k_eval_sparse<R, 8>;
    case 9: return k_eval_sparse<R, 9>;
    case 10: return k_eval_sparse<R, 10>;
    default: return nullptr;
    }
}

template <int R, int FC>
EvalFn pick_eval_mfma(int N, size_t *lds)
{
    switch (N) {
#define FPTS_CASE(NN)                                                                      \
    case NN:                                                                               \
        if constexpr (FC <= most_fields(R, NN)) {                                          \
            *lds = sizeof(double) * (newton::NodeLds<double, FC, R, NN>::SIZE +            \
                                     R * NN * 16 + (NN % 4 ? 1 : 0));                      \
            return k_eval_mfma<R, NN, FC>;                                                 \
        }                                                                                  \
        return nullptr;
        FPTS_CASE(2)
        FPTS_CASE(3)
        FPTS_CASE(4)
        FPTS_CASE(5)
        FPTS_CASE(6)
        FPTS_CASE(7)
        FPTS_CASE(8)
        FPTS_CASE(9)
        FPTS_CASE(10)
#undef FPTS_CASE
    default: return nullptr;
    }
}

template <int R>
EvalFn pick_eval_mfma_fc(int N, int fc, size_t *lds)
{
    switch (fc) {
    case 4: return pick_eval_mfma<R, 4>(N, lds);
    case 3: return pick_eval_mfma<R, 3>(N, lds);
    case 2: return pick_eval_mfma<R, 2>(N, lds);
    default: return pick_eval_mfma<R, 1>(N, lds);
    }
}

template <bool LDS>
EvalFn pick_eval_r(int R, int N)
{
    return R == 1 ? pick_eval<1, LDS>(N) : nullptr;   // line meshes
}

}  // namespace

hipError_t launch_eval_bin_list(const fpts_mesh *m, int pass, const int *list, const int *count,
                                int64_t cap, const int32_t *elem, int *elem_cnt, int es,
                                const int *elem_off, int *rank, int *sorted, hipStream_t s)
{
    if (cap <= 0) return hipSuccess;
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((cap + 255) / 256,
                                                                 (int64_t)m->cus * 16));
    hipLaunchKernelGGL(k_eval_bin_list, dim3(grid), dim3(256), 0, s, pass, list, count,
                       (int)m->nel, es, elem, elem_cnt, elem_off, rank, sorted);
    return hipGetLastError();
}

hipError_t launch_eval_bin(const fpts_mesh *m, int pass, int64_t n, const int32_t *code,
                           const int32_t *elem, const double *r, const int2 *cand,
                           int n_fields, double *out, int *elem_cnt, int es,
                           const int *elem_off, int *rank, int *sorted, double *erec,
                           hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_eval_bin, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, pass,
                       (int)n, (int)m->nel, es, m->R, code, elem, r, cand, n_fields, out,
                       elem_cnt, elem_off, rank, sorted, erec);
    return hipGetLastError();
}

hipError_t launch_eval(const fpts_mesh *m, int64_t n, int n_fields, int field_n,
                       const double *field, double *out, const EvalList &l, hipStream_t s)
{
    EvalArgs a{};
    a.r = l.r;
    a.n = (int)n;
    a.nel = (int)m->nel;
    a.n_fields = n_fields;
    a.field = field;
    a.out = out;
    a.sorted = l.sorted;
    a.elem_off = l.elem_off;
    a.chunk_off = l.chunk_off;
    a.task_elem = l.task_elem;
    a.erec = l.erec;
    a.rec = l.rec;
    a.deep_only = l.deep_only;
    a.rs = l.rs;
    if (field_n == m->N) a.basis = m->basis;
    else gll::fill(field_n, a.basis.z, a.basis.w);
    if (m->R >= 2) {
        // matrix cores, up to most_fields per launch, evenly
        const int most = most_fields(m->R, field_n);
        const int launches = (n_fields + most - 1) / most;
        const dim3 grid(xcd_grid(std::min<int64_t>(l.task_bound, (int64_t)m->cus * 16)));
        for (int k = 0, f0 = 0; k < launches; ++k) {
            size_t lds = 0;
            const int fc = (n_fields - f0 + launches - k - 1) / (launches - k);
            EvalFn fn = m->R == 3 ? pick_eval_mfma_fc<3>(field_n, fc, &lds)
                                  : pick_eval_mfma_fc<2>(field_n, fc, &lds);
            if (!fn) return hipErrorInvalidValue;
            a.f0 = f0;
            // three or four fields of up to six nodes per direction go through
            // list order where the points are many: a gather per point and
            // coalesced writes take less than that many scattered writes (some
            // 28 us per 1M values; N = 6, four fields, 3M points: 250 + 77 us,
            // scattered 360).  At larger N the writes hide behind the arithmetic
            // (N = 8, three fields, 5M points: 420 + 121 us, scattered 423), with
            // two fields the gather costs as much (N = 4, 2M points: call 237 us,
            // 214), and where the values of few points stay in the caches
            // scattered writes cost little: geometric means of the calls' times
            // over N = 2 to 6, list order against scattered, hexes (and quads) of
            // 512 to 90000 elements: 100 thousand points 1.16 (1.16), 1 million
            // 1.05 (1.05), 3 million 0.98 (0.91).  The fused call's first pass
            // (four fields, N = 4): 200 thousand points 1.01, 1 million 0.98, 4
            // million 0.92 (quads 1.01, 0.96, 0.84).
            const bool spread = l.tmp && fc >= kSpreadFields && field_n <= kSpreadNodes &&
                                n >= (l.cand ? kSpreadFusedPoints : kSpreadPoints);
            a.tmp = spread ? l.tmp : nullptr;
            hipLaunchKernelGGL(fn, grid, dim3(64), lds, s, a);
            if (spread) {
                auto sp = fc == 4 ? k_eval_spread<4> : k_eval_spread<3>;
                hipLaunchKernelGGL(sp, dim3((unsigned)((n + 1023) / 1024)), dim3(256), 0, s,
                                   (int)n, l.cand, l.elem, l.rank, l.elem_off, l.tmp, f0, out);
            }
            f0 += fc;
        }
        return hipGetLastError();
    }
    // line meshes: stage in LDS unless elements hold many points (several
    // tasks each)
    const dim3 grid(task_grid(l.task_bound, m->cus));
    const bool lds = n <= (int64_t)4 * kChunk * m->nel;
    EvalFn fn = lds ? pick_eval_r<true>(m->R, field_n) : pick_eval_r<false>(m->R, field_n);
    if (!fn) return hipErrorInvalidValue;
    hipLaunchKernelGGL(fn, grid, dim3(64), lds ? sizeof(double) * field_n : 0, s, a);
    return hipGetLastError();
}

hipError_t launch_eval_split(const fpts_mesh *m, int64_t n, const int32_t *elem, const int *rank,
                             int *elem_cnt, int es, const int *elem_off, int *sorted,
                             int *list, int *count, int phase, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    if (phase == 0) {
        hipLaunchKernelGGL(k_eval_dense, dim3((unsigned)((m->nel + 255) / 256)), dim3(256), 0, s,
                           (int)m->nel, es, elem_cnt);
    } else {
        hipLaunchKernelGGL(k_eval_split, dim3((unsigned)((n + kSplitChunk - 1) / kSplitChunk)),
                           dim3(256), 0, s, (int)n, elem, rank, elem_cnt, es, elem_off, sorted,
                           list, count);
    }
    return hipGetLastError();
}

hipError_t launch_eval_sparse(const fpts_mesh *m, int64_t n, const double *r, int n_fields,
                              int field_n, const double *field, double *out,
                              const int32_t *elem, const int *list, const int *count,
                              hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    // line meshes only: the other meshes interpolate every point on the
    // matrix cores (the same bits in both calls need the same arithmetic)
    SparseFn fn = m->R == 1 ? pick_sparse<1>(field_n) : nullptr;
    if (!fn) return hipErrorInvalidValue;
    EvalArgs a{};
    a.r = r;
    a.n = (int)n;
    a.nel = (int)m->nel;
    a.n_fields = n_fields;
    a.field = field;
    a.out = out;
    if (field_n == m->N) a.basis = m->basis;
    else gll::fill(field_n, a.basis.z, a.basis.w);
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, m->cus * 8));
    hipLaunchKernelGGL(fn, dim3(grid), dim3(256), 0, s, a, elem, list, count);
    return hipGetLastError();
}

hipError_t launch_near_rows(const fpts_mesh *m, hipStream_t s)
{
    const int64_t total = m->nel * m->near_npad;
    const int grid = (int)std::min<int64_t>((total + 255) / 256, 65536);
    hipLaunchKernelGGL(k_near_rows, dim3(grid), dim3(256), 0, s, m->d_nodes, m->d_xc, m->d_near,
                       (int64_t)m->nel, m->D, m->NP, m->near_npad);
    return hipGetLastError();
}

hipError_t launch_nodes32(const fpts_mesh *m, hipStream_t s)
{
    hipLaunchKernelGGL(k_nodes32, dim3(4096), dim3(256), 0, s, m->d_nodes, m->d_xc,
                       m->d_nodes32, (int64_t)m->nel, m->D, m->NP);
    return hipGetLastError();
}

}  // namespace fpts
