// Find, outside Newton (Section 3.2): points are binned by cell of the local
// map (Section 3.1.3); each cell's candidates are tested with the AABB and
// OBB tests (eqs. eq_AABB_test, eq_OBB_test); the primary candidate of each
// point is bucketed by element for Newton; points the primary does not
// settle get their other candidates in a second pass and the selection rule
// of Section 3.2.  Also the scans used by find and eval and the copies of a
// serving batch.
#include "fpts_internal.hpp"

namespace fpts {
namespace {

// Zeroes [a, a + na) and [b, b + nb).
__global__ __launch_bounds__(256) void k_zero2(int *a, int64_t na, int *b, int64_t nb)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < na + nb; i += stride) {
        if (i < na) a[i] = 0;
        else b[i - na] = 0;
    }
}

// Exclusive scans of the counts of a bucketing, all in one pass over them:
// off (items before each unit), choff (tasks of up to len items before it,
// with the map task -> unit) and off2 (tasks of up to len2 items, with their map).
// A block scans a tile of 8192 counts; where there are several tiles,
// k_unit_sums has left their sums in tile_sum (3 per tile) and every block
// adds up those before its own (no block waits for another).  A kernel of a
// few microseconds costs about 4.6 us of the stream on this GPU whatever it
// does, so the three scans and their maps as kernels of their own (eight
// launches) took 37 us per bucketing, six bucketings per call.
constexpr int kUsThreads = 1024;
constexpr int kUsItems = 8;
constexpr int kUsTile = kUsThreads * kUsItems;
constexpr int kUsWaves = kUsThreads / kWave;

__device__ __forceinline__ int tasks_of(int cnt, int len) { return (cnt + len - 1) / len; }

__device__ __forceinline__ void load_counts(const UnitScan &u, int64_t base, int (&v)[kUsItems])
{
    if (u.stride > 1) {
#pragma unroll
        for (int k = 0; k < kUsItems; ++k)
            v[k] = base + k < u.n ? u.cnt[(base + k) * u.stride] : 0;
    } else if (base + kUsItems <= u.n) {
        const int4 *p = reinterpret_cast<const int4 *>(u.cnt + base);   // 256-byte aligned arrays
        const int4 x = p[0], y = p[1];
        v[0] = x.x;
        v[1] = x.y;
        v[2] = x.z;
        v[3] = x.w;
        v[4] = y.x;
        v[5] = y.y;
        v[6] = y.z;
        v[7] = y.w;
    } else {
#pragma unroll
        for (int k = 0; k < kUsItems; ++k) v[k] = base + k < u.n ? u.cnt[base + k] : 0;
    }
}

__device__ __forceinline__ void sum_counts(const UnitScan &u, const int (&v)[kUsItems],
                                           int (&s)[3])
{
    s[0] = s[1] = s[2] = 0;
#pragma unroll
    for (int k = 0; k < kUsItems; ++k) {
        s[0] += v[k];
        if (u.choff) s[1] += tasks_of(v[k], u.len);
        if (u.off2) s[2] += tasks_of(v[k], u.len2);
    }
}

// Block sums of three values, in every thread.
__device__ __forceinline__ void block_sum3(int (&s)[3], int (*red)[kUsWaves])
{
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) s[q] += __shfl_xor(s[q], o, kWave);
    __syncthreads();
    if (lane == 0) {
#pragma unroll
        for (int q = 0; q < 3; ++q) red[q][wid] = s[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        s[q] = 0;
#pragma unroll
        for (int w = 0; w < kUsWaves; ++w) s[q] += red[q][w];
    }
    __syncthreads();
}

__global__ __launch_bounds__(kUsThreads) void k_unit_sums(UnitScan u)
{
    __shared__ int red[3][kUsWaves];
    int v[kUsItems], s[3];
    load_counts(u, (int64_t)blockIdx.x * kUsTile + (int64_t)threadIdx.x * kUsItems, v);
    sum_counts(u, v, s);
    block_sum3(s, red);
    if (threadIdx.x < 3) u.tile_sum[3 * (int64_t)blockIdx.x + threadIdx.x] = s[threadIdx.x];
}

// The maps' entries of the wave's units: task[base ..] = unit, cnt of them.
// Units with many tasks are written by the whole wave.
__device__ __forceinline__ void write_tasks(int *task, int base, int cnt, int unit)
{
    constexpr int kOwn = 8;
    const int lane = threadIdx.x & (kWave - 1);
    if (cnt <= kOwn)
        for (int t = 0; t < cnt; ++t) task[base + t] = unit;
    unsigned long long big = __ballot(cnt > kOwn);
    while (big) {
        const int l = __builtin_ctzll(big);
        big &= big - 1;
        const int b = __shfl(base, l), c = __shfl(cnt, l), un = __shfl(unit, l);
        for (int t = lane; t < c; t += kWave) task[b + t] = un;
    }
}

// (parts = 1 or kUsItems blocks scan each tile and write a share of the
// results each: the scattered stores of the task maps of one tile keep one
// CU's address unit busy for 20 us)
__global__ __launch_bounds__(kUsThreads) void k_unit_scan(UnitScan u, int parts)
{
    __shared__ int red[3][kUsWaves];
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    const int tile = blockIdx.x / parts, part = blockIdx.x % parts;
    const int64_t base = (int64_t)tile * kUsTile + (int64_t)threadIdx.x * kUsItems;
    // items and tasks of the earlier tiles
    int pre[3] = {0, 0, 0};
    if (tile > 0) {
        for (int64_t i = threadIdx.x; i < tile; i += kUsThreads)
#pragma unroll
            for (int q = 0; q < 3; ++q) pre[q] += u.tile_sum[3 * i + q];
        block_sum3(pre, red);
    }
    int v[kUsItems], s[3];
    load_counts(u, base, v);
    sum_counts(u, v, s);
    // exclusive scan of the threads' sums over the block
    int at[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        int incl = s[q];
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int t = __shfl_up(incl, o, kWave);
            if (lane >= o) incl += t;
        }
        at[q] = incl - s[q];
        if (lane == kWave - 1) red[q][wid] = incl;
    }
    __syncthreads();
    // totals of the earlier waves: lane w holds wave w's
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        int t = lane < wid ? red[q][lane] : 0;
#pragma unroll
        for (int o = kUsWaves / 2; o > 0; o >>= 1) t += __shfl_xor(t, o, kWave);
        at[q] += pre[q] + __shfl(t, 0, kWave);
    }
#pragma unroll
    for (int k = 0; k < kUsItems; ++k) {
        const int64_t i = base + k;
        const bool in = i < u.n;
        const int t1 = in && u.choff ? tasks_of(v[k], u.len) : 0;
        const int t2 = in && u.off2 ? tasks_of(v[k], u.len2) : 0;
        const bool mine = parts == 1 || k == part;
        if (in && mine) {
            u.off[i] = at[0];
            if (u.choff) u.choff[i] = at[1];
            if (u.off2) u.off2[i] = at[2];
        }
        if (u.choff && mine) write_tasks(u.task, at[1], t1, (int)i);
        if (u.off2 && mine) write_tasks(u.task2, at[2], t2, (int)i);
        at[0] += in ? v[k] : 0;
        at[1] += t1;
        at[2] += t2;
        if (i == u.n - 1 && mine) {
            u.off[u.n] = at[0];
            if (u.choff) u.choff[u.n] = at[1];
            if (u.off2) u.off2[u.n] = at[2];
        }
    }
}

// Cell of x in the local map, or -1 when x is not finite or outside the
// union of the boxes.  Same operations as the host registration of element
// boxes (subtract, divide, floor, clamp), so a point inside an element's AABB
// always lands in a cell that lists the element.
template <int D>
__device__ inline int cell_of(const HashView &h, const double *x)
{
    int cell = 0, mul = 1;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        if (!__builtin_isfinite(x[d]) || !(x[d] >= h.lo[d] && x[d] <= h.hi[d])) return -1;
        double t = floor((x[d] - h.lo[d]) / h.del[d]);
        t = fmin(fmax(t, 0.0), (double)(h.NL - 1));
        cell += mul * (int)t;
        mul *= h.NL;
    }
    return cell;
}

__device__ inline void write_not_found(int p, int n, int R, int32_t *code, int32_t *elem,
                                       double *r, double *dist)
{
    code[p] = FPTS_NOT_FOUND;
    elem[p] = -1;
    dist[p] = __builtin_huge_val();
    for (int a = 0; a < R; ++a) r[(size_t)a * n + p] = 0.0;
}

// Phase A for one point: its cell (-1 for a kept point, whose result is
// already final, and for a point outside the map), the packed copy of its
// coordinates (pts4 not null), defined candidate data, and NOT_FOUND for a
// point outside the map.
template <int D>
__device__ inline int bin_point(const HashView &h, int p, int n, int R, const double *pts,
                                double *pts4, const int *keep, int *cellpt, int2 *cand,
                                int32_t *code, int32_t *elem, double *r, double *dist)
{
    int c = -1;
    const bool kept = keep && keep[p];
    if (!kept) {
        double x[D];
#pragma unroll
        for (int d = 0; d < D; ++d) x[d] = pts[(size_t)d * n + p];
        c = cell_of<D>(h, x);
        if (pts4) {
            // the packed copy (one cache line per point for the kernels that
            // visit points in bucket order)
            typedef double v2 __attribute__((ext_vector_type(2)));
            v2 *o = reinterpret_cast<v2 *>(pts4 + (size_t)p * pt_stride(D));
            o[0] = v2{x[0], x[1]};
            if (D == 3) o[1] = v2{x[D - 1], 0.0};
        }
    }
    cellpt[p] = c;
    cand[p] = make_int2(0, -1);
    if (c < 0 && !kept) write_not_found(p, n, R, code, elem, r, dist);
    return c;
}

// Phase A with one atomic per point (bin_shift: few points, or more than
// kBinMaxCells cells); the cells' counters lie cs ints apart.  pass 0: bin_point
// and the count per cell; pass 1: scatter point ids into their cell's bucket.
template <int D>
__global__ __launch_bounds__(256) void k_cell_bin(HashView h, int pass, int n, int R,
                                                 const double *pts, double *pts4, const int *keep,
                                                 int *cellpt, int *cell_cnt, int cs,
                                                 const int *cell_poff, int *rank,
                                                 int *pbin, int2 *cand, int32_t *code,
                                                 int32_t *elem, double *r, double *dist)
{
    // no early exit: wave_inc needs every lane
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const bool in = p < n;
    if (pass == 0) {
        const int c =
            in ? bin_point<D>(h, p, n, R, pts, pts4, keep, cellpt, cand, code, elem, r, dist) : -1;
        const int k = wave_inc(cell_cnt, c * cs, c >= 0);
        if (c >= 0) rank[p] = k;
    } else {
        const int c = in ? cellpt[p] : -1;
        if (c >= 0) pbin[cell_poff[c] + rank[p]] = p;
    }
}

// Phase A without per-point atomics.  Points arrive in any order (uniformly
// random in the benchmarks), so a count per cell by atomics costs one
// device atomic per point (about 26 G/s on this GPU) and the scatter into
// cell buckets one write at a random place per point.  Instead the cells
// are grouped into coarse buckets of 2^shift consecutive cells (at most
// kBinMaxBuckets buckets):
//  tiles:   per tile of points, bin_point and the tile's histogram
//           over the buckets (LDS atomics), stored bucket-major in bh; an
//           exclusive scan of bh gives each (bucket, tile) its range;
//  coarse:  each tile writes its points as (cell, id) pairs into those
//           ranges: pairs sorted by bucket, one short run per (tile, bucket);
//  rank:    windows of as many consecutive pairs (cells of at most two
//           buckets, unless the buckets are sparse) count their cells in LDS
//           and take one atomic per cell on cell_cnt for a block of ranks;
//  scatter: after the scan of cell_cnt, pbin[cell_poff[c] + rank] = id in
//           pair order, so a window's writes fall in the cells of one or two
//           buckets.
// The scatter's ranges go to the XCDs in contiguous blocks (task_of_block),
// so that an XCD's writes stay within a few buckets and partly written cache
// lines meet in one L2 (the same mapping for the tiles measured slower).
// A tile or window is 256 threads times 4 to 32 items (bin_items): long runs
// per bucket where there are many points, and enough blocks to fill the chip
// where there are few (20 thousand points in tiles of 8192, three blocks, took
// the tile pass 31 us).
constexpr int kBinThreads = 256;
constexpr int kBinItems = 32;   // at most

template <int D>
__global__ __launch_bounds__(kBinThreads) void k_bin_tiles(HashView h, int n, int R,
                                                          const double *pts, double *pts4,
                                                          const int *keep, int *cellpt,
                                                          int2 *cand,
                                                          int32_t *code, int32_t *elem, double *r,
                                                          double *dist, int shift, int nb,
                                                          int ntile, int items, int *bh)
{
    extern __shared__ int hist[];   // [nb]
    const int tile = blockIdx.x;
    for (int i = threadIdx.x; i < nb; i += kBinThreads) hist[i] = 0;
    __syncthreads();
    const int64_t base = (int64_t)tile * items * kBinThreads;
    for (int k = 0; k < items; ++k) {
        const int64_t q = base + (int64_t)k * kBinThreads + threadIdx.x;
        if (q < n) {
            const int c = bin_point<D>(h, (int)q, n, R, pts, pts4, keep, cellpt, cand, code,
                                       elem, r, dist);
            if (c >= 0) atomicAdd(&hist[c >> shift], 1);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nb; i += kBinThreads)
        bh[(int64_t)i * ntile + tile] = hist[i];
}

__global__ __launch_bounds__(kBinThreads) void k_bin_coarse(int n, const int *cellpt, int shift,
                                                           int nb, int ntile, int items,
                                                           const int *boff, int2 *pairs)
{
    extern __shared__ int off[];   // [nb] next free place of each bucket's range
    const int tile = blockIdx.x;
    for (int i = threadIdx.x; i < nb; i += kBinThreads)
        off[i] = boff[(int64_t)i * ntile + tile];
    __syncthreads();
    const int64_t base = (int64_t)tile * items * kBinThreads;
    for (int k = 0; k < items; ++k) {
        const int64_t q = base + (int64_t)k * kBinThreads + threadIdx.x;
        if (q < n) {
            const int c = cellpt[q];
            if (c >= 0) pairs[atomicAdd(&off[c >> shift], 1)] = make_int2(c, (int)q);
        }
    }
}

template <int ITEMS>
__global__ __launch_bounds__(kBinThreads) void k_bin_rank(const int *total_p, int shift,
                                                         const int2 *pairs, int *cell_cnt,
                                                         int *rank)
{
    constexpr int kBinItems = ITEMS, kBinTile = kBinThreads * ITEMS;
    extern __shared__ int cnt[];   // [2 << shift] cells of buckets hA, hA + 1
    const int total = *total_p;
    const int64_t w0 = (int64_t)task_of_block() * kBinTile;
    if (w0 >= total) return;   // the whole block
    const int w1 = (int)(w0 + kBinTile < total ? w0 + kBinTile : total);
    const int hA = pairs[w0].x >> shift, hB = pairs[w1 - 1].x >> shift;
    if (hB - hA > 1) {
        // sparse buckets: few pairs per cell, one atomic each
        for (int64_t i = w0 + threadIdx.x; i < w1; i += kBinThreads)
            rank[i] = atomicAdd(&cell_cnt[pairs[i].x], 1);
        return;
    }
    const int c0 = hA << shift, nbin = 2 << shift;
    for (int i = threadIdx.x; i < nbin; i += kBinThreads) cnt[i] = 0;
    __syncthreads();
    int bin[kBinItems], lr[kBinItems];
#pragma unroll
    for (int k = 0; k < kBinItems; ++k) {
        const int64_t i = w0 + (int64_t)k * kBinThreads + threadIdx.x;
        bin[k] = 0;
        lr[k] = 0;
        if (i < w1) {
            bin[k] = pairs[i].x - c0;
            lr[k] = atomicAdd(&cnt[bin[k]], 1);
        }
    }
    __syncthreads();
    // the window's block of ranks in each of its cells
    for (int j = threadIdx.x; j < nbin; j += kBinThreads) {
        const int v = cnt[j];
        if (v > 0) cnt[j] = atomicAdd(&cell_cnt[c0 + j], v);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kBinItems; ++k) {
        const int64_t i = w0 + (int64_t)k * kBinThreads + threadIdx.x;
        if (i < w1) rank[i] = cnt[bin[k]] + lr[k];
    }
}

__global__ __launch_bounds__(kBinThreads) void k_bin_scatter(const int *total_p, const int2 *pairs,
                                                            const int *rank,
                                                            const int *cell_poff, int *pbin)
{
    const int64_t total = *total_p;
    const int64_t per = (total + gridDim.x - 1) / gridDim.x;   // pairs per block
    const int64_t b0 = task_of_block() * per, b1 = b0 + per < total ? b0 + per : total;
    for (int64_t i = b0 + threadIdx.x; i < b1; i += kBinThreads) {
        const int2 cp = pairs[i];
        pbin[cell_poff[cp.x] + rank[i]] = cp.y;
    }
}

// Phase B: one wavefront per task of up to 64 points of one cell (task
// grid); every lane tests its own point against the cell's candidates.  The
// candidates' box records are loaded into registers with vector loads, up to
// kLocChunk at a time (lane j holds the first half of candidate j's record,
// lane 32 + j the second), and each candidate's record is then broadcast to
// scalar registers with lane reads.  A task's inputs come through dependent
// loads (task -> cell -> point ids and candidate ids -> coordinates and
// records): those of the wave's next task are issued while the current one
// is tested, level by level, so that their latency hides behind the tests.
// Per point: primary candidate (smallest OBB depth, lowest id on ties), its
// rank in the primary's bucket, and whether there are other candidates.
constexpr int kLocChunk = 32;

__device__ __forceinline__ double read_lane(double v, int l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}

template <int D, bool PACKED>
__global__ __launch_bounds__(64) void k_locate_cells(HashView h, int n, int R, const double *pts,
                                                    const double *pts4,
                                                    const int *pbin, const int *cell_poff,
                                                    const int *cell_choff, int ncell,
                                                    const int *task_cell, int2 *cand,
                                                    int *elem_cnt, int es, int *rank,
                                                    int *bin_prim, int32_t *code, int32_t *elem,
                                                    double *r, double *dist)
{
    constexpr int RS = 3 * D + D * D;   // doubles per box record
    constexpr int HR = (RS + 1) / 2;    // record doubles per lane (half a record)
    const int lane = threadIdx.x;
    const int total = cell_choff[ncell];
    const int G = gridDim.x;
    struct Task {
        int c, beg, end, q0, q1;
    };
    // level 1: the task's cell, its points' range and its candidates' range
    auto task_of = [&](int t) __attribute__((always_inline)) {
        Task k;
        k.c = __builtin_amdgcn_readfirstlane(task_cell[t]);
        k.beg = cell_poff[k.c] + (t - cell_choff[k.c]) * kChunk;
        k.end = min(cell_poff[k.c + 1], k.beg + kChunk);
        k.q0 = __builtin_amdgcn_readfirstlane(h.cell_off[k.c]);
        k.q1 = __builtin_amdgcn_readfirstlane(h.cell_off[k.c + 1]);
        return k;
    };
    // level 2: this lane's point id and candidate id (candidate qb + lane % 32)
    auto ids_of = [&](const Task &k, int qb, int &p, int &mine) __attribute__((always_inline)) {
        p = k.beg + lane < k.end ? pbin[k.beg + lane] : 0;
        const int j = lane & (kLocChunk - 1);
        mine = j < min(kLocChunk, k.q1 - qb) ? h.cell_el[qb + j] : 0;
    };
    // level 3: the point's coordinates and this lane's half record
    auto data_of = [&](const Task &k, int qb, int p, int mine, double (&x)[D],
                       double (&rv)[HR]) __attribute__((always_inline)) {
        const bool has = k.beg + lane < k.end;
#pragma unroll
        for (int d = 0; d < D; ++d)
            x[d] = !has    ? 0.0
                   : PACKED ? pts4[(size_t)p * pt_stride(D) + d]
                            : pts[(size_t)d * n + p];
        const bool live = (lane & (kLocChunk - 1)) < min(kLocChunk, k.q1 - qb);
        const int f0 = (lane >> 5) * HR;
        const double *src = h.box + (size_t)mine * RS + f0;
#pragma unroll
        for (int u = 0; u < HR; ++u) rv[u] = (live && f0 + u < RS) ? src[u] : 0.0;
    };
    int t = task_of_block();
    if (t >= total) return;
    Task cur = task_of(t);
    int p, mine;
    double x[D], rv[HR];
    ids_of(cur, cur.q0, p, mine);
    data_of(cur, cur.q0, p, mine, x, rv);
    for (;;) {
        const int tn = t + G;
        const bool more = tn < total;
        Task nxt = cur;
        if (more) nxt = task_of(tn);   // next task, level 1
        int pn = 0, minen = 0;
        double xn[D], rvn[HR];
        bool l2 = !more, l3 = !more;
        const bool has = cur.beg + lane < cur.end;
        int cnt = 0, prim = -1;
        double best = __builtin_huge_val();
        for (int qb = cur.q0; qb < cur.q1; qb += kLocChunk) {
            const int nb = min(kLocChunk, cur.q1 - qb);
            if (qb != cur.q0) {
                // more candidates than one chunk: the next chunk, loaded now
                int pq;
                double xq[D];
                ids_of(cur, qb, pq, mine);
                data_of(cur, qb, pq, mine, xq, rv);
            }
            if (!l2) {
                ids_of(nxt, nxt.q0, pn, minen);   // next task, level 2
                l2 = true;
            }
            for (int j = 0; j < nb; ++j) {
                if (!l3 && j == nb / 2) {
                    data_of(nxt, nxt.q0, pn, minen, xn, rvn);   // next task, level 3
                    l3 = true;
                }
                // candidate j's record, broadcast to scalar registers: the
                // AABB first; when no point of the wave lies inside it (a
                // box that only grazes the cell) the OBB part is neither
                // read nor tested
                double rec[RS];
#pragma unroll
                for (int f = 0; f < 2 * D; ++f) rec[f] = read_lane(rv[f % HR], j + 32 * (f / HR));
                const bool in = has && aabb_in<D>(rec, x);
                if (!__ballot(in)) continue;
#pragma unroll
                for (int f = 2 * D; f < RS; ++f) rec[f] = read_lane(rv[f % HR], j + 32 * (f / HR));
                const int e = __builtin_amdgcn_readlane(mine, j);
                const double depth = obb_depth<D>(rec, x);
                if (in && depth <= 1.0) {
                    ++cnt;
                    if (depth < best) {
                        best = depth;
                        prim = e;
                    }
                }
            }
        }
        if (!l2) ids_of(nxt, nxt.q0, pn, minen);   // a cell without candidates
        if (!l3) data_of(nxt, nxt.q0, pn, minen, xn, rvn);
        const int k = wave_inc(elem_cnt, prim * es, has && prim >= 0);
        if (has) {
            // one scattered write per point
            cand[p] = make_int2((int)((unsigned)k << 1 | (cnt > 1)), prim);
            if (prim < 0) write_not_found(p, n, R, code, elem, r, dist);
        }
        // primary and rank in bin order (coalesced), for the scatter by bins
        if (has) {
            bin_prim[cur.beg + lane] = prim;
            rank[cur.beg + lane] = k;
        }
        if (!more) break;
        t = tn;
        cur = nxt;
        p = pn;
        mine = minen;
#pragma unroll
        for (int d = 0; d < D; ++d) x[d] = xn[d];
#pragma unroll
        for (int u = 0; u < HR; ++u) rv[u] = rvn[u];
    }
}

__global__ __launch_bounds__(256) void k_primary_scatter(int n, int nel, const int2 *cand,
                                                        const int *elem_off, const int *rank,
                                                        int *sorted)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const int e = p < n ? cand[p].y : -1;
    if (e >= 0 && e < nel) sorted[elem_off[e] + rank[p]] = p;
}

// Primary buckets from the bin-ordered output of k_locate_cells: the point
// at bin position i goes to sorted[elem_off[bin_prim[i]] + rank[i]].
__global__ __launch_bounds__(256) void k_primary_scatter_bins(int n, const int *nbinned,
                                                             const int *pbin,
                                                             const int *bin_prim,
                                                             const int *rank,
                                                             const int *elem_off, int *sorted)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n || i >= *nbinned) return;
    const int e = bin_prim[i];
    if (e >= 0) sorted[elem_off[e] + rank[i]] = pbin[i];
}

// A primary result settles the point when it is INTERIOR at least `guard`
// inside the reference box: no other element can then hold the point in its
// interior (it would overlap the primary), so the paper's rule -- first
// INTERIOR candidate in ascending id order -- picks the same element.

__device__ inline bool deep_interior(bool interior, const double (&rr)[3], int R)
{
    if (!interior) return false;
    double m = 1.0;
    for (int a = 0; a < R; ++a) m = fmin(m, 1.0 - fabs(rr[a]));
    return m > kSettleGuard;
}

// Phase D, marking: every point whose primary result leaves the search open
// (a primary, other candidates and not settled) is appended to ulist, in no
// particular order, *ucount of them.  The other candidates of the few listed
// points are then handled by dense wavefronts: tested where they lie among
// all points, their candidate loops (dependent loads) kept whole wavefronts
// waiting.  A block marks up to kMarkChunk consecutive points, gathers its
// listed points in LDS and reserves their places with one atomic:
// device-scope atomics on one address serialise (some 16 ns each), so one
// per wavefront with a listed point would take longer than the loads.  Four
// points' loads per thread are issued at once.
constexpr int kMarkChunk = 4096;
constexpr int kMarkAhead = 4;

__device__ inline void list_append(bool take, int p, int lane, int *lst, int &lcnt)
{
    const unsigned long long m = __ballot(take);
    if (m) {
        int at = 0;
        if (lane == 0) at = atomicAdd(&lcnt, __popcll(m));
        at = __shfl(at, 0, 64);
        if (take) lst[at + __popcll(m & ((1ull << lane) - 1))] = p;
    }
}

// Line meshes: the marking pass over the outputs.
__global__ __launch_bounds__(256) void k_unsettled(int n, const int2 *cand, const int32_t *code,
                                                  const double *r, int *ulist, int *ucount,
                                                  int items)
{
    __shared__ int lst[kMarkChunk];
    __shared__ int lcnt, gbase;
    const int lane = threadIdx.x & 63;
    if (threadIdx.x == 0) lcnt = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * items * 256 + threadIdx.x;
    for (int it = 0; it < items; it += kMarkAhead) {
        int2 cd[kMarkAhead];
        int32_t co[kMarkAhead];
        double rr[kMarkAhead];
#pragma unroll
        for (int u = 0; u < kMarkAhead; ++u) {
            const int64_t p = base + (int64_t)(it + u) * 256;
            const bool in = it + u < items && p < n;
            cd[u] = in ? cand[p] : make_int2(0, -1);
            co[u] = in ? code[p] : FPTS_NOT_FOUND;
            rr[u] = in ? r[p] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kMarkAhead; ++u) {
            const double r3[3] = {rr[u], 0.0, 0.0};
            const bool todo = cd[u].y >= 0 && (cd[u].x & 1) &&
                              !deep_interior(co[u] == FPTS_INTERIOR, r3, 1);
            list_append(todo, (int)(base + (int64_t)(it + u) * 256), lane, lst, lcnt);
        }
    }
    __syncthreads();
    const int cnt = lcnt;
    if (threadIdx.x == 0 && cnt) gbase = atomicAdd(ucount, cnt);
    __syncthreads();
    for (int i = threadIdx.x; i < cnt; i += 256) ulist[gbase + i] = lst[i];
}

// Volume and surface meshes: the result records of the primary pass are
// brought into point order -- one 32-byte gather per point, then coalesced
// writes of the outputs -- and the points marked in the same pass.  With
// rest.out (fused find + interpolate) the interpolated values of NOT_FOUND
// points become NaN, and with rest.list the points that the interpolation
// over the primary list leaves out are listed too -- found, but not INTERIOR
// at least kSettleGuard inside by the primary result (the listed points
// among them) --, so that the interpolation needs no pass over all points of
// its own.
// Points without a primary (NOT_FOUND, or kept from a hinted search) hold
// their results already.
template <int R>
__global__ __launch_bounds__(256) void k_settle(int n, const int2 *cand, const int *elem_off,
                                               const double *rec, int32_t *code, int32_t *elem,
                                               double *r, double *dist, int *ulist, int *ucount,
                                               int items, EvalRest rest)
{
    typedef double v2 __attribute__((ext_vector_type(2)));
    __shared__ int lst[kMarkChunk], elst[kMarkChunk];
    __shared__ int lcnt, ecnt, gbase, ebase;
    const int lane = threadIdx.x & 63;
    if (threadIdx.x == 0) {
        lcnt = 0;
        ecnt = 0;
    }
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * items * 256 + threadIdx.x;
    for (int it = 0; it < items; it += kMarkAhead) {
        int2 cd[kMarkAhead];
        v2 lo[kMarkAhead], hi[kMarkAhead];
        bool in[kMarkAhead];
#pragma unroll
        for (int u = 0; u < kMarkAhead; ++u) {
            const int64_t p = base + (int64_t)(it + u) * 256;
            in[u] = it + u < items && p < n;
            cd[u] = in[u] ? cand[p] : make_int2(0, -1);
        }
#pragma unroll
        for (int u = 0; u < kMarkAhead; ++u) {
            lo[u] = v2{0.0, 0.0};
            hi[u] = v2{0.0, 0.0};
            if (cd[u].y >= 0) {
                const int64_t pos = (int64_t)elem_off[cd[u].y] + ((unsigned)cd[u].x >> 1);
                const v2 *src = reinterpret_cast<const v2 *>(rec + pos * kRec);
                lo[u] = src[0];
                hi[u] = src[1];
            }
        }
#pragma unroll
        for (int u = 0; u < kMarkAhead; ++u) {
            const int64_t q = base + (int64_t)(it + u) * 256;
            const int p = (int)q;
            const bool has = cd[u].y >= 0;
            const bool interior = has && !__builtin_signbit(hi[u][1]);
            const double rr[3] = {lo[u][0], lo[u][1], R == 3 ? hi[u][0] : 0.0};
            if (has) {
                code[p] = interior ? FPTS_INTERIOR : FPTS_BORDER;
                elem[p] = cd[u].y;
                dist[p] = fabs(hi[u][1]);
#pragma unroll
                for (int a = 0; a < R; ++a) r[(size_t)a * n + p] = rr[a];
            }
            const bool deep = deep_interior(interior, rr, R);
            list_append(has && (cd[u].x & 1) && !deep, p, lane, lst, lcnt);
            if (rest.list) list_append(has && !deep, p, lane, elst, ecnt);
            if (rest.out && in[u] && !has)
                for (int f = 0; f < rest.n_fields; ++f)
                    rest.out[(size_t)f * n + p] = __builtin_nan("");
        }
    }
    __syncthreads();
    const int cnt = lcnt, ec = ecnt;
    if (threadIdx.x == 0) {
        if (cnt) gbase = atomicAdd(ucount, cnt);
        if (ec) ebase = atomicAdd(rest.count, ec);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < cnt; i += 256) ulist[gbase + i] = lst[i];
    for (int i = threadIdx.x; i < ec; i += 256) rest.list[ebase + i] = elst[i];
}

// Phase D over the listed points, a contiguous range of the list per block,
// kResLanes lanes to a point: they test its cell's candidates side by side
// (a point per lane walked some 20 of them one dependent load after the
// other, twice: 50 us a pass whatever the number of points).  pass 0: count
// each point's other candidates (ucnt) and give the point a block of that
// many slots, uoff[i] .. uoff[i] + ucnt[i] - 1 (one atomic per block on
// *slot_total), and count them per element; a point whose block would end
// beyond the slot capacity cap2 gets none (ucnt[i] = 0, uoff[i] = -1) and
// goes to the overflow list instead (olist, *ocount: searched one point per wavefront).
// pass 1: write the slots (k-th other candidate in ascending id at uoff[i] +
// k) and bucket them by element.
constexpr int kResLanes = 16;
constexpr int kResGroups = 256 / kResLanes;

template <int D>
__global__ __launch_bounds__(256) void k_resolve(HashView h, int pass, int n, const double *pts,
                                                const int *cellpt, const int2 *cand,
                                                const int *ulist, const int *ucount,
                                                int *uoff, int *ucnt,
                                                unsigned long long *slot_total,
                                                int *elem_cnt2, const int *elem_off2,
                                                int *slot_pt, int *slot_elem, int *sorted2,
                                                int64_t cap2, int *olist, int *ocount)
{
    __shared__ int wsum[4];
    __shared__ unsigned long long sbase;
    const int cnt = *ucount;
    // (at least two points per group: the blocks' atomics on *slot_total, some
    // 16 ns each, come one after the other)
    const int per = max((int)((cnt + gridDim.x - 1) / gridDim.x), 2 * kResGroups);
    const int i0 = min((int64_t)cnt, (int64_t)blockIdx.x * per);
    const int i1 = min((int64_t)cnt, (int64_t)i0 + per);
    if (i0 >= i1) return;   // the whole block
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    const int gl = threadIdx.x % kResLanes, grp = threadIdx.x / kResLanes;
    const int shift = lane / kResLanes * kResLanes;   // the group's lanes in its wave
    // calls hit(e, k) for the point's k-th other candidate e, in ascending
    // id (every lane of the group takes part; the hitting lane calls);
    // returns their number
    auto others = [&](int i, auto &&hit) __attribute__((always_inline)) {
        const int p = ulist[i], prim = cand[p].y, c = cellpt[p];
        double x[D];
#pragma unroll
        for (int d = 0; d < D; ++d) x[d] = pts[(size_t)d * n + p];
        int k = 0;
        const int q1 = h.cell_off[c + 1];
        for (int q = h.cell_off[c]; q < q1; q += kResLanes) {
            const int e = q + gl < q1 ? h.cell_el[q + gl] : prim;
            double depth;
            const bool ok =
                e != prim && box_pass<D>(h.box + (size_t)e * (3 * D + D * D), x, depth);
            const unsigned m =
                (unsigned)(__ballot(ok) >> shift) & ((1u << kResLanes) - 1);
            if (ok) hit(p, e, k + __popc(m & ((1u << gl) - 1)));
            k += __popc(m);
        }
        return k;
    };
    if (pass == 1) {
        for (int i = i0 + grp; i < i1; i += kResGroups) {
            if (ucnt[i] == 0) continue;
            const int s0 = uoff[i];
            others(i, [&](int p, int e, int k) __attribute__((always_inline)) {
                slot_pt[s0 + k] = p;
                slot_elem[s0 + k] = e;
                sorted2[elem_off2[e] + atomicSub(&elem_cnt2[e], 1) - 1] = s0 + k;
            });
        }
        return;
    }
    int sum = 0;
    for (int i = i0 + grp; i < i1; i += kResGroups) {
        const int k = others(i, [&](int, int e, int) __attribute__((always_inline)) {
            atomicAdd(&elem_cnt2[e], 1);
        });
        if (gl == 0) {
            ucnt[i] = k;
            sum += k;
        }
    }
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
    if (lane == 0) wsum[wid] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        const int tot = wsum[0] + wsum[1] + wsum[2] + wsum[3];
        sbase = tot ? atomicAdd(slot_total, (unsigned long long)tot) : 0;
    }
    __syncthreads();
    // the points' places in the block's slots, 256 at a time
    unsigned long long base = sbase;
    for (int c0 = i0; c0 < i1; c0 += 256) {
        const int i = c0 + threadIdx.x;
        const int k = i < i1 ? ucnt[i] : 0;
        int incl = k;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int t = __shfl_up(incl, o);
            if (lane >= o) incl += t;
        }
        __syncthreads();   // earlier reads of wsum come first
        if (lane == kWave - 1) wsum[wid] = incl;
        __syncthreads();
        int before = incl - k, all = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w < wid) before += wsum[w];
            all += wsum[w];
        }
        const unsigned long long at = base + (unsigned long long)before;
        const bool fits = at + (unsigned long long)k <= (unsigned long long)cap2;
        if (i < i1) {
            if (!fits) {
                ucnt[i] = 0;
                if (k > 0) olist[atomicAdd(ocount, 1)] = ulist[i];
            }
            uoff[i] = fits ? (int)at : k > 0 ? -1 : 0;
        }
        base += (unsigned long long)all;
    }
    if (base <= (unsigned long long)cap2) return;   // (base is uniform over the block)
    // points without room: their candidates are counted back out
    __syncthreads();
    for (int i = i0 + grp; i < i1; i += kResGroups) {
        if (uoff[i] >= 0) continue;
        others(i, [&](int, int e, int) __attribute__((always_inline)) {
            atomicSub(&elem_cnt2[e], 1);
        });
    }
}

// Section 3.2 selection over the primary and the other candidates of a
// listed point: the lowest-id INTERIOR candidate, else the smallest
// distance (lowest id on ties).
__global__ __launch_bounds__(256) void k_select2(int n, int R, const int *ulist,
                                                const int *ucount, const int *uoff,
                                                const int *ucnt, const int2 *cand,
                                                const int *slot_elem, int64_t cap2,
                                                const double *res_r, const double *res_dist,
                                                const int *res_code, int32_t *code,
                                                int32_t *elem, double *r, double *dist)
{
    const int cnt = *ucount;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < cnt; i += gridDim.x * blockDim.x) {
        const int p = ulist[i];
        const int s0 = uoff[i], s1 = s0 + ucnt[i];
        if (s0 == s1) continue;
        // best so far: the primary (slot -1)
        int best = -1;
        int bcode = code[p], belem = cand[p].y;
        double bdist = dist[p];
        for (int s = s0; s < s1; ++s) {
            const int e = slot_elem[s], cd = res_code[s];
            const double dd = res_dist[s];
            bool take;
            if (bcode == FPTS_INTERIOR) take = cd == FPTS_INTERIOR && e < belem;
            else if (cd == FPTS_INTERIOR) take = true;
            else take = dd < bdist || (dd == bdist && e < belem);
            if (take) {
                best = s;
                bcode = cd;
                belem = e;
                bdist = dd;
            }
        }
        if (best < 0) continue;
        code[p] = bcode;
        elem[p] = belem;
        dist[p] = bdist;
        for (int a = 0; a < R; ++a) r[(size_t)a * n + p] = res_r[(size_t)a * cap2 + best];
    }
}

inline int grid_for(int64_t n, int block) { return (int)((n + block - 1) / block); }

// Search hints (points that move a little between searches): pass 0 takes
// the previous element of every point whose previous code was INTERIOR as
// its only candidate and counts it per element; pass 1 marks the points
// whose hinted search converged (keep[p] holds the Newton convergence flag
// on entry) INTERIOR at least kSettleGuard inside the reference box: no
// other element can hold them in its interior, so that result is the one
// the full search gives, and they are kept.
__global__ __launch_bounds__(256) void k_hint(int pass, int n, int nel, int es, int R,
                                             const int32_t *code, const int32_t *elem,
                                             const double *r, int2 *cand, int *elem_cnt,
                                             int *rank, int *keep)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const bool in = p < n;
    if (pass == 0) {
        const int e = in && code[p] == FPTS_INTERIOR ? elem[p] : -1;
        const bool ok = e >= 0 && e < nel;
        if (in) cand[p] = make_int2(ok ? 1 : 0, ok ? e : -1);
        const int k = wave_inc(elem_cnt, e * es, ok);
        if (ok) rank[p] = k;
    } else if (in) {
        bool k = cand[p].y >= 0 && code[p] == FPTS_INTERIOR && keep[p] == 1;
        double mg = 1.0;
        for (int a = 0; a < R; ++a) mg = fmin(mg, 1.0 - fabs(r[(size_t)a * n + p]));
        keep[p] = k && mg > kSettleGuard;
    }
}

// Parked pairs of the primary Newton pass, binned by element (their queue
// for the face kernel).  A fixed grid strides over the pass's list
// positions; the loop bound is uniform per wavefront, as wave_inc needs.
__global__ __launch_bounds__(256) void k_park_bin(int pass, const int4 *meta, const int *total_p,
                                                 int cap, int *node, int *elem_cnt,
                                                 const int *elem_off, int *sorted)
{
    const int total = min(*total_p, cap);
    const int lane = threadIdx.x & 63;
    for (int64_t k0 = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63); k0 < total;
         k0 += (int64_t)gridDim.x * blockDim.x) {
        const int k = (int)k0 + lane;
        const int nd = k < total ? node[k] : 0;
        const bool active = nd < 0;
        if (!__ballot(active)) continue;
        const int e = active ? meta[k].z : 0;
        if (pass == 0) {
            const int rk = wave_inc(elem_cnt, e, active);
            if (active) node[k] = -2 - rk;
        } else if (active) {
            sorted[elem_off[e] - 2 - nd] = k;
        }
    }
}

// Points of a serving batch's requests gathered, and its results handed
// back: one launch for up to kBatchReqs requests, a thread per point (a copy
// per request and component, 70 of them for eight requests in three batches,
// took the host and the stream about 3 us each).
__global__ __launch_bounds__(256) void k_batch_copy(int which, BatchArrays b, BatchReqs reqs,
                                                   int64_t p0, int64_t p1)
{
    const int64_t p = p0 + (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= p1) return;
    for (int k = 0; k < reqs.count; ++k) {
        const BatchReq &q = reqs.q[k];
        const int64_t i = p - q.off;
        if (i < 0 || i >= q.n) continue;
        if (which == 0) {
            for (int d = 0; d < b.D; ++d) b.pts[d * b.n + p] = q.pts[d * q.n + i];
            return;
        }
        q.code[i] = b.code[p];
        q.elem[i] = b.elem[p];
        q.dist[i] = b.dist[p];
        for (int a = 0; a < b.R; ++a) q.r[a * q.n + i] = b.r[a * b.n + p];
        for (int f = 0; f < b.n_fields; ++f) q.out[f * q.n + i] = b.out[f * b.n + p];
        return;
    }
}

}  // namespace

hipError_t launch_zero2(int *a, int64_t na, int *b, int64_t nb, hipStream_t s)
{
    if (na + nb <= 0) return hipSuccess;
    const int grid = (int)std::min<int64_t>((na + nb + 1023) / 1024, 4096);
    hipLaunchKernelGGL(k_zero2, dim3(grid), dim3(256), 0, s, a, na, b, nb);
    return hipGetLastError();
}

int64_t scan_tmp_blocks(int64_t n) { return 3 * ((n + kUsTile - 1) / kUsTile) + 1; }

hipError_t launch_unit_scan(UnitScan u, int64_t tmp_blocks, hipStream_t s)
{
    const int64_t tiles = (u.n + kUsTile - 1) / kUsTile;
    if (u.n < 1 || 3 * tiles > tmp_blocks || ((uintptr_t)u.cnt & 15) != 0)
        return hipErrorInvalidValue;
    // a single tile: as many threads as it has counts for (a block of few
    // waves is launched and synchronised sooner)
    int threads = kUsThreads;
    if (tiles > 1)
        hipLaunchKernelGGL(k_unit_sums, dim3((unsigned)tiles), dim3(kUsThreads), 0, s, u);
    else
        threads = (int)((u.n + kUsItems * kWave - 1) / (kUsItems * kWave)) * kWave;
    // (in place, off aliasing cnt, a tile's counts are read by one block only)
    const int parts = u.n >= 512 && u.off != u.cnt ? kUsItems : 1;
    hipLaunchKernelGGL(k_unit_scan, dim3((unsigned)(tiles * parts)), dim3(threads), 0, s, u,
                       parts);
    return hipGetLastError();
}

hipError_t launch_park_bin(int pass, const int4 *meta, const int *total, int64_t cap,
                           int *node, int *elem_cnt, const int *elem_off, int *sorted, int cus,
                           hipStream_t s)
{
    if (cap <= 0) return hipSuccess;
    const int grid = (int)std::min<int64_t>(grid_for(cap, 256), (int64_t)cus * 8);
    hipLaunchKernelGGL(k_park_bin, dim3(grid), dim3(256), 0, s, pass, meta, total, (int)cap,
                       node, elem_cnt, elem_off, sorted);
    return hipGetLastError();
}

hipError_t launch_cell_bin(const fpts_mesh *m, int pass, int64_t n, const double *pts,
                           double *pts4, const int *keep, int *cellpt, int *cell_cnt, int cs,
                           const int *cell_poff, int *rank, int *pbin, int2 *cand,
                           int32_t *code, int32_t *elem, double *r, double *dist, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    HashView h = hash_view(m);
    const int grid = grid_for(n, 256);
    auto k = m->D == 2 ? k_cell_bin<2> : k_cell_bin<3>;
    hipLaunchKernelGGL(k, dim3(grid), dim3(256), 0, s, h, pass, (int)n, m->R, pts, pts4, keep,
                       cellpt, cell_cnt, cs, cell_poff, rank, pbin, cand, code, elem, r, dist);
    return hipGetLastError();
}

// Up to kCellBinPoints points go to their cells with one atomic each: three
// launches instead of six (of 3 to 5 us each), and with the counters spread over
// at least 512 cache lines a few thousand atomics take a few microseconds.  The
// line is a cautious one: find + interpolate took 5 to 17 us less so at every
// size measured, 500 to 32000 points, all over the mesh or all in one cell (256
// quads, N = 5: 1000 points 104 against 115 us, 4000 109 and 121, 16000 122 and
// 132; 512 hexes, N = 8: 160 and 172, 193 and 205, 249 and 263); beyond, points
// that crowd in cells of one line wait for each other's atomics, 16 ns each.
int bin_shift(int64_t n, int64_t ncell)
{
    if (n <= kCellBinPoints || ncell > kBinMaxCells) return -1;
    // buckets of at least 512 cells: a tile's run per bucket is then tens
    // of pairs long (whole cache lines) at a few points per cell
    int shift = 9;
    while ((ncell + (1ll << shift) - 1) >> shift > kBinMaxBuckets) ++shift;
    return shift;
}

// items per thread of a tile: 32 from about 6 million points on, fewer
// below so that some three blocks per CU have work, as long as the bucket
// histograms (one per tile) stay below an eighth of the points.  (At 4
// million points 8 items took the tile pass from 74 to 64 us, but the pass
// that writes the shorter runs from 26 to 33.)  The second condition, once
// met, holds for every larger n, so that the items grow with n at the ends of
// the ranges only.
static int64_t bin_items_end(int items) { return (int64_t)kBinThreads * items * 768; }
static int bin_items(int64_t n, int nb)
{
    int items = kBinItems;
    while (items > 4 && n < bin_items_end(items) &&
           nb * (n + kBinThreads / 2 * items) <= kBinThreads / 16 * items * n)
        items /= 2;
    return items;
}
static int64_t tiles_for(int64_t n, int items)
{
    return (n + (int64_t)kBinThreads * items - 1) / ((int64_t)kBinThreads * items);
}
static int bin_buckets(int64_t ncell, int shift)
{
    return (int)((ncell + (1ll << shift) - 1) >> shift);
}
int64_t bin_hist_size(int64_t n, int64_t ncell, int shift)
{
    const int nb = bin_buckets(ncell, shift);
    return nb * tiles_for(n, bin_items(n, nb));
}
int64_t bin_hist_bound(int64_t n, int64_t ncell, int shift)
{
    // the histograms shrink where the items grow: the last size before it
    int64_t most = bin_hist_size(n, ncell, shift);
    for (int items = kBinItems; items > 4; items /= 2)
        if (n >= bin_items_end(items))
            most = std::max(most, bin_hist_size(bin_items_end(items) - 1, ncell, shift));
    return most;
}

hipError_t launch_bin_tiles(const fpts_mesh *m, int64_t n, const double *pts, double *pts4,
                            const int *keep, int *cellpt, int2 *cand,
                            int32_t *code, int32_t *elem, double *r, double *dist, int shift,
                            int *bh, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    HashView h = hash_view(m);
    const int nb = bin_buckets(bin_cells(m), shift), items = bin_items(n, nb);
    const int ntile = (int)tiles_for(n, items);
    auto k = m->D == 2 ? k_bin_tiles<2> : k_bin_tiles<3>;
    hipLaunchKernelGGL(k, dim3(ntile), dim3(kBinThreads), sizeof(int) * nb, s, h, (int)n, m->R,
                       pts, pts4, keep, cellpt, cand, code, elem, r, dist, shift, nb,
                       ntile, items, bh);
    return hipGetLastError();
}

hipError_t launch_bin_coarse(const fpts_mesh *m, int64_t n, const int *cellpt, int shift,
                             const int *boff, int2 *pairs, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int nb = bin_buckets(bin_cells(m), shift), items = bin_items(n, nb);
    const int ntile = (int)tiles_for(n, items);
    hipLaunchKernelGGL(k_bin_coarse, dim3(ntile), dim3(kBinThreads), sizeof(int) * nb, s, (int)n,
                       cellpt, shift, nb, ntile, items, boff, pairs);
    return hipGetLastError();
}

hipError_t launch_bin_rank(const fpts_mesh *m, int64_t n, const int *total, int shift,
                           const int2 *pairs, int *cell_cnt, int *rank, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int items = bin_items(n, bin_buckets(bin_cells(m), shift));
    auto k = items == 4 ? k_bin_rank<4> : items == 8 ? k_bin_rank<8>
             : items == 16 ? k_bin_rank<16> : k_bin_rank<32>;
    hipLaunchKernelGGL(k, dim3(xcd_grid(tiles_for(n, items))), dim3(kBinThreads),
                       sizeof(int) * (2 << shift), s, total, shift, pairs, cell_cnt, rank);
    return hipGetLastError();
}

hipError_t launch_bin_scatter(int64_t n, const int *total, const int2 *pairs, const int *rank,
                              const int *cell_poff, int *pbin, int cus, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int grid = xcd_grid(std::min<int64_t>(grid_for(n, kBinThreads), (int64_t)cus * 16));
    hipLaunchKernelGGL(k_bin_scatter, dim3(grid), dim3(kBinThreads), 0, s, total, pairs, rank,
                       cell_poff, pbin);
    return hipGetLastError();
}

hipError_t launch_locate_cells(const fpts_mesh *m, int64_t n, const double *pts,
                               const double *pts4,
                               const int *pbin, const int *cell_poff, const int *cell_choff,
                               int64_t ncell, const int *task_cell, int64_t task_bound,
                               int2 *cand, int *elem_cnt, int *rank,
                               int *bin_prim, int32_t *code, int32_t *elem, double *r,
                               double *dist, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    HashView h = hash_view(m);
    auto k = m->D == 2 ? (pts4 ? k_locate_cells<2, true> : k_locate_cells<2, false>)
                       : (pts4 ? k_locate_cells<3, true> : k_locate_cells<3, false>);
    hipLaunchKernelGGL(k, dim3(task_grid(task_bound, m->cus)), dim3(64), 0, s, h, (int)n, m->R,
                       pts, pts4, pbin, cell_poff, cell_choff, (int)ncell, task_cell, cand,
                       elem_cnt, find_stride(m->nel, n), rank, bin_prim, code, elem, r, dist);
    return hipGetLastError();
}

hipError_t launch_primary_scatter_bins(int64_t n, const int *nbinned, const int *pbin,
                                       const int *bin_prim, const int *rank,
                                       const int *elem_off, int *sorted, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_primary_scatter_bins, dim3(grid_for(n, 256)), dim3(256), 0, s, (int)n,
                       nbinned, pbin, bin_prim, rank, elem_off, sorted);
    return hipGetLastError();
}

hipError_t launch_primary_scatter(int64_t n, int64_t nel, const int2 *cand,
                                  const int *elem_off, const int *rank, int *sorted,
                                  hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_primary_scatter, dim3(grid_for(n, 256)), dim3(256), 0, s, (int)n,
                       (int)nel, cand, elem_off, rank, sorted);
    return hipGetLastError();
}

// a marking block's items per thread: 16 (4096 points) where that still
// leaves two blocks per CU, else fewer (a block of 16 takes 19 us however few
// points there are)
static int mark_items(const fpts_mesh *m, int64_t n)
{
    return (int)std::min<int64_t>(std::max<int64_t>(n / ((int64_t)m->cus * 2 * 256), 1),
                                  kMarkChunk / 256);
}

hipError_t launch_unsettled(const fpts_mesh *m, int64_t n, const int2 *cand,
                            const int32_t *code, const double *r, int *ulist,
                            int *ucount, hipStream_t s)
{
    if (n <= 0 || m->R != 1) return n <= 0 ? hipSuccess : hipErrorInvalidValue;
    const int items = mark_items(m, n);
    hipLaunchKernelGGL(k_unsettled, dim3(grid_for(n, 256 * items)), dim3(256), 0, s, (int)n, cand,
                       code, r, ulist, ucount, items);
    return hipGetLastError();
}

hipError_t launch_settle(const fpts_mesh *m, int64_t n, const int2 *cand, const int *elem_off,
                         const double *rec, int32_t *code, int32_t *elem, double *r, double *dist,
                         int *ulist, int *ucount, const EvalRest &rest, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int items = mark_items(m, n);
    auto k = m->R == 3 ? k_settle<3> : k_settle<2>;
    hipLaunchKernelGGL(k, dim3(grid_for(n, 256 * items)), dim3(256), 0, s, (int)n, cand, elem_off,
                       rec, code, elem, r, dist, ulist, ucount, items, rest);
    return hipGetLastError();
}

hipError_t launch_batch_copy(int which, const BatchArrays &b, const BatchReqs &reqs,
                             hipStream_t s)
{
    // (the requests of a launch lie one after the other in the batch)
    if (reqs.count < 1 || reqs.count > kBatchReqs) return hipErrorInvalidValue;
    const BatchReq &z = reqs.q[reqs.count - 1];
    const int64_t p0 = reqs.q[0].off, p1 = z.off + z.n;
    if (p1 <= p0) return hipSuccess;
    hipLaunchKernelGGL(k_batch_copy, dim3(grid_for(p1 - p0, 256)), dim3(256), 0, s, which, b, reqs,
                       p0, p1);
    return hipGetLastError();
}

// grid-stride kernels over the unsettled list: enough blocks to fill the
// chip when the list is long, few to launch when it is short
static int list_grid(const fpts_mesh *m, int64_t n)
{
    return std::max(1, (int)std::min<int64_t>(grid_for(n, 256), (int64_t)m->cus * 16));
}

hipError_t launch_resolve(const fpts_mesh *m, int pass, int64_t n, const double *pts,
                          const int *cellpt, const int2 *cand, const int *ulist,
                          const int *ucount, int *uoff, int *ucnt, unsigned long long *slot_total,
                          int *elem_cnt2, const int *elem_off2, int *slot_pt,
                          int *slot_elem, int *sorted2, int64_t cap2, int *olist, int *ocount,
                          hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    HashView h = hash_view(m);
    auto k = m->D == 2 ? k_resolve<2> : k_resolve<3>;
    const int grid = std::max(
        1, (int)std::min<int64_t>((n + kResGroups - 1) / kResGroups, (int64_t)m->cus * 4));
    hipLaunchKernelGGL(k, dim3(grid), dim3(256), 0, s, h, pass, (int)n, pts, cellpt,
                       cand, ulist, ucount, uoff, ucnt, slot_total, elem_cnt2, elem_off2,
                       slot_pt, slot_elem, sorted2, cap2, olist, ocount);
    return hipGetLastError();
}

hipError_t launch_select2(const fpts_mesh *m, int64_t n, const int *ulist, const int *ucount,
                          const int *uoff, const int *ucnt, const int2 *cand,
                          const int *slot_elem, int64_t cap2, const double *res_r,
                          const double *res_dist, const int *res_code, int32_t *code,
                          int32_t *elem, double *r, double *dist, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_select2, dim3(list_grid(m, n)), dim3(256), 0, s, (int)n, m->R, ulist,
                       ucount, uoff, ucnt, cand, slot_elem, cap2, res_r, res_dist, res_code,
                       code, elem, r, dist);
    return hipGetLastError();
}

}  // namespace fpts

namespace fpts {

hipError_t launch_hint(const fpts_mesh *m, int pass, int64_t n, const int32_t *code,
                       const int32_t *elem, const double *r, int2 *cand, int *elem_cnt,
                       int *rank, int *keep, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_hint, dim3(grid_for(n, 256)), dim3(256), 0, s, pass, (int)n,
                       (int)m->nel, find_stride(m->nel, n), m->R, code, elem, r, cand, elem_cnt,
                       rank, keep);
    return hipGetLastError();
}

}  // namespace fpts
