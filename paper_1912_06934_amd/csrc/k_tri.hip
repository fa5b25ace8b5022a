// Triangular smoothers of the two-stage preconditioner: ILU(0) (Sec. 3.2,
// Sec. 4.1), IC(0) (Sec. 4.1, Sec. 4.2) and symmetric Gauss-Seidel (Sec. 3.2,
// Sec. 4.2), each in a sweep order: the natural order, or a multicolour
// order (first-fit colouring in ascending row order on the symmetrised
// pattern, rows sorted by colour, ascending within a colour).
//
// The factorisations run on A's own CSR pattern in its original numbering; the
// order only decides which stored entries count as "earlier" (lower) or
// "later" (upper).  The solves read the factors (or A) packed level by level.
// Rows are grouped into dependency levels of the lower and
// of the upper triangle in that order.  A level with many rows is one launch
// across the whole GPU (thread per row); consecutive levels with few rows are
// walked by a single work-group with a barrier between levels.  In the
// multicolour order every colour is one level, so a sweep is a handful of
// wide launches; in the natural order a 2D grid has a few hundred narrow
// levels.  Either way every row sees its predecessors final, so the factors
// and solves equal the sequential algorithm in that order (up to the
// rounding of the sums).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <numeric>

#include "internal.h"

namespace msrsb {
namespace {

constexpr int kNarrowThreads = 1024;
constexpr int kWideRows = 2048;  // a level with at least this many rows gets its own launch

// --- per-row device work ---

// position of column col in row i (columns ascending), or -1
__device__ __forceinline__ int find_col(const int *__restrict__ ci, int e0, int e1, int col)
{
    int lo = e0, hi = e1 - 1;
    while (lo <= hi) {
        const int mid = (lo + hi) >> 1;
        const int c = ci[mid];
        if (c == col) return mid;
        if (c < col) lo = mid + 1;
        else hi = mid - 1;
    }
    return -1;
}

struct TriArgs {
    const int *rp, *ci, *dpos;
    const int8_t *side;  // -1 earlier column, 0 diagonal, +1 later
    const int *lord;     // earlier entries of each row, sorted by the column's rank
    const int *nlow;     // their count per row
};

// IKJ elimination of row i in the order (earlier neighbours k by rank)
__device__ void ilu_row(const TriArgs &t, int i, double *__restrict__ lu, int *__restrict__ flag)
{
    const int e0 = t.rp[i], e1 = t.rp[i + 1], nl = t.nlow[i];
    for (int u = 0; u < nl; ++u) {
        const int e = t.lord[e0 + u];
        const int k = t.ci[e];
        const double piv = lu[t.dpos[k]];
        if (piv == 0.0) flag[0] = 1;
        const double lik = lu[e] / piv;
        lu[e] = lik;
        for (int q = t.rp[k]; q < t.rp[k + 1]; ++q) {
            if (t.side[q] <= 0) continue;  // only entries later than k
            const int f = find_col(t.ci, e0, e1, t.ci[q]);
            if (f >= 0) lu[f] -= lik * lu[q];
        }
    }
}

// IC(0) row i: L_ij = (A_ij - sum_k L_ik L_jk) / L_jj over earlier j by rank,
// then L_ii = sqrt(A_ii - sum_k L_ik^2)
__device__ void ic_row(const TriArgs &t, int i, const double *__restrict__ a,
                       double *__restrict__ l, int *__restrict__ flag)
{
    const int e0 = t.rp[i], nl = t.nlow[i];
    for (int u = 0; u < nl; ++u) {
        const int e = t.lord[e0 + u];
        const int j = t.ci[e];
        double s = a[e];
        const int j0 = t.rp[j], j1 = t.rp[j + 1];
        for (int w = 0; w < u; ++w) {  // k earlier than j, stored in row i
            const int p = t.lord[e0 + w];
            const int f = find_col(t.ci, j0, j1, t.ci[p]);
            if (f >= 0) s -= l[p] * l[f];
        }
        l[e] = s / l[t.dpos[j]];
    }
    double s = a[t.dpos[i]];
    for (int u = 0; u < nl; ++u) {
        const double v = l[t.lord[e0 + u]];
        s -= v * v;
    }
    if (!(s > 0.0)) {
        flag[0] = 1;
        s = 1.0;
    }
    l[t.dpos[i]] = sqrt(s);
}

// --- factorisation kernels: wide (one level, thread per row) and narrow
// (levels walked by one work-group) ---

enum { OP_ILU = 0, OP_IC = 1 };

struct RowOp {
    int op = OP_ILU;
    const double *a = nullptr;  // IC(0): A's values
    double *f = nullptr;        // factor values
    int *flag = nullptr;
};

__device__ __forceinline__ void do_row(const TriArgs &t, const RowOp &r, int i)
{
    if (r.op == OP_ILU) ilu_row(t, i, r.f, r.flag);
    else ic_row(t, i, r.a, r.f, r.flag);
}

__global__ __launch_bounds__(256) void k_tri_wide(TriArgs t, RowOp r,
                                                  const int *__restrict__ rows, int count)
{
    const int u = blockIdx.x * 256 + threadIdx.x;
    if (u < count) do_row(t, r, rows[u]);
}

__global__ __launch_bounds__(kNarrowThreads) void k_tri_narrow(TriArgs t, RowOp r,
                                                               const int *__restrict__ lev_ptr,
                                                               const int *__restrict__ rows,
                                                               int lev0, int lev1)
{
    for (int l = lev0; l < lev1; ++l) {
        for (int u = lev_ptr[l] + threadIdx.x; u < lev_ptr[l + 1]; u += kNarrowThreads)
            do_row(t, r, rows[u]);
        __syncthreads();
    }
}

// ILU(0) of a run of narrow levels by one work-group, kIluLanes lanes per row
// (rows of at most that many entries, at most kIluLow of them earlier): a lane
// holds one entry of its row, and everything the row needs of its earlier
// neighbours (the pivots and the entries that meet the row's columns, found
// once per pattern by k_ilu_map) is loaded at once when the level starts.  A
// thread per row walked the neighbours' rows with a search per entry: 6.17 ms
// for the 298 levels of 100 x 100 cells and nine entries, bound by the chain
// of dependent loads; 0.68 ms this way.  Same operations in the same order.
constexpr int kIluLanes = 16;
constexpr int kIluLow = 8;

// of the u-th row's w-th earlier neighbour k: the row's entry of that
// column, k's diagonal entry and first entry (at[u * kIluLow + w], x < 0:
// none), and per entry f of the row the offset in row k of its column when
// that comes later than k, else -1 (map[(u * kIluLow + w) * kIluLanes + f])
__global__ __launch_bounds__(256) void k_ilu_map(TriArgs t, const int *__restrict__ rows, int n,
                                                 int4 *__restrict__ at, int8_t *__restrict__ map)
{
    const int64_t g = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int f = static_cast<int>(g % kIluLanes);
    const int64_t uw = g / kIluLanes;
    const int u = static_cast<int>(uw / kIluLow), w = static_cast<int>(uw % kIluLow);
    if (u >= n) return;
    const int i = rows[u], e0 = t.rp[i], len = t.rp[i + 1] - e0;
    int m = -1;
    int4 a = make_int4(-1, 0, 0, 0);
    if (w < t.nlow[i]) {
        const int e = t.lord[e0 + w], k = t.ci[e], k0 = t.rp[k];
        a = make_int4(e - e0, t.dpos[k], k0, 0);
        if (f < len) {
            const int q = find_col(t.ci, k0, t.rp[k + 1], t.ci[e0 + f]);
            if (q >= 0 && t.side[q] > 0) m = q - k0;
        }
    }
    map[g] = static_cast<int8_t>(m);
    if (f == 0) at[uw] = a;
}

template <int LOW>
__global__ __launch_bounds__(kNarrowThreads) void k_ilu_run(TriArgs t,
                                                            const int *__restrict__ rows,
                                                            const int *__restrict__ lev, int lev0,
                                                            int lev1,
                                                            const int4 *__restrict__ at,
                                                            const int8_t *__restrict__ map,
                                                            double *lu, int *__restrict__ flag)
{
    const int f = threadIdx.x % kIluLanes, g = threadIdx.x / kIluLanes;
    constexpr int ROWS = kNarrowThreads / kIluLanes;
    const int first = lev[lev0];  // the maps' row 0
    for (int l = lev0; l < lev1; ++l) {
        for (int u = lev[l] + g; u < lev[l + 1]; u += ROWS) {
            const int i = rows[u], e0 = t.rp[i], len = t.rp[i + 1] - e0;
            const bool own = f < len;
            int4 a[LOW];
            int m[LOW];
#pragma unroll
            for (int w = 0; w < LOW; ++w) {
                const int64_t uw = static_cast<int64_t>(u - first) * kIluLow + w;
                a[w] = at[uw];
                m[w] = map[uw * kIluLanes + f];
            }
            double v = own ? lu[e0 + f] : 0.0;
            double piv[LOW], x[LOW];
#pragma unroll
            for (int w = 0; w < LOW; ++w) {
                piv[w] = a[w].x >= 0 ? lu[a[w].y] : 1.0;
                x[w] = m[w] >= 0 ? lu[a[w].z + m[w]] : 0.0;
            }
#pragma unroll
            for (int w = 0; w < LOW; ++w) {
                if (a[w].x < 0) continue;  // the same for a row's lanes
                if (piv[w] == 0.0) flag[0] = 1;
                const double lik = __shfl(v, a[w].x, kIluLanes) / piv[w];
                if (f == a[w].x) v = lik;
                else if (m[w] >= 0) v -= lik * x[w];
            }
            if (own) lu[e0 + f] = v;
        }
        __syncthreads();
    }
}

// --- solves on the packed sides (TriSide, TriValues) ---
//
// One side's pass: x_i = (in_i - sum val x_col) / diag, with `in` the right-hand
// side of the first pass or the first pass's x for the second.  A level's
// columns, values and rows are packed level by level, so a row costs two
// memory round trips (its packed data, then x at its columns) instead of four
// dependent ones through the CSR arrays.  Three launches fewer per
// application than a launch per level and triangle plus the copy and the sum:
// - rows of the second level take what they need of the first from `in`
//   (marked columns; the first level's division is folded into the values),
//   so the first two levels go together;
// - a row with nothing on the upper side (the upper triangle's first level)
//   needs no second pass: the first one ends with its division (fold);
// - the last pass adds x to z (or sets it).
// The coloured ILU(0) on 65,536 rows of nine entries: 8 launches of 5.2 us, a
// copy and a sum -> 6 launches of 3.4 us per application; the coloured IC(0)
// on 215,025 rows of seven: 4 launches of 7.9 us, a copy and a sum -> 2 of 6.5.
constexpr int kTriFirst = INT32_MIN;

struct TriPass {
    const int *row, *col;
    const double *val, *diag, *fold;  // diag: null for a unit one; fold: null unless
                                      // this pass ends some rows
    const double *in;
    double *x, *z;
    bool last;  // every row of the pass ends here (z is written)
    bool set;   // z = x instead of z += x
};

__device__ __forceinline__ void tri_end(const TriPass &p, int i, double s)
{
    p.z[i] = p.set ? s : p.z[i] + s;
}

// positions [u0, u0 + skip + cnt): `skip` rows without entries (level 0, when
// the first two levels go together), then the cnt rows of one level with their
// entries from place `at` on.  W: the width, or 0 for any; tail: null unless
// rows of the level are longer.  FIRST: a first pass (marked columns are read
// from `in`; a second pass has in = x).
template <int W, bool FIRST>
__global__ __launch_bounds__(256) void k_tri_level(TriPass p, int u0, int skip, int cnt,
                                                   int64_t at, int width,
                                                   const int64_t *__restrict__ tail)
{
    const int tt = blockIdx.x * 256 + threadIdx.x, t = tt - skip;
    if (t >= cnt) return;
    constexpr int C = W > 0 ? W : 8;  // entries per step
    const int n = t < 0 ? 0 : W > 0 ? W : width;
    int c[C];
    double v[C];
    // (the entries before the row that everything else waits for; rows without
    // entries read the level's first ones and leave them)
    auto fetch = [&](int k0) {
#pragma unroll
        for (int k = 0; k < C; ++k) {
            // a step past the width repeats its last entry
            const int kk = W > 0 ? k : min(k0 + k, width - 1);
            const int64_t e = at + static_cast<int64_t>(kk) * cnt + max(t, 0);
            c[k] = p.col[e];
            v[k] = p.val[e];
        }
    };
    if (W > 0 || n > 0) fetch(0);
    const int u = u0 + tt, i = p.row[u];
    const double di = p.diag ? p.diag[u] : 1.0, fo = p.fold ? p.fold[u] : 0.0;
    double s = p.in[i];
    for (int k0 = 0; k0 < n; k0 += C) {
        double xv[C];
        if (W == 0 && k0 > 0) fetch(k0);
#pragma unroll
        for (int k = 0; k < C; ++k)
            xv[k] = FIRST && c[k] < 0 ? p.in[c[k] & ~kTriFirst] : p.x[c[k] & ~kTriFirst];
        // (what fills a row has the value 0 and its own column: 0 times an
        // infinity would not be nothing)
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const bool fill = (c[k] & ~kTriFirst) == i || (W == 0 && k0 + k >= width);
            s -= fill ? 0.0 : v[k] * xv[k];
        }
    }
    if (tail && t >= 0) {
        const int64_t e1 = tail[u + 1];
#pragma unroll 8
        for (int64_t e = tail[u]; e < e1; ++e) {
            const int c = p.col[e];
            s -= p.val[e] * (FIRST && c < 0 ? p.in : p.x)[c & ~kTriFirst];
        }
    }
    if (p.diag) s /= di;
    const bool end = p.last || fo != 0.0;
    if (fo != 0.0) s /= fo;
    p.x[i] = s;
    if (end) tri_end(p, i, s);
}

// a run of narrow levels by one work-group with a barrier between levels; x
// in LDS for systems of at most kNarrowLdsRows rows.  The first kRowRegs
// entries of a thread's first row of a level are loaded while the previous
// level is still being solved.
constexpr int kNarrowLdsRows = 16384;  // 128 KB of LDS
constexpr int kRowRegs = 8;

// TAIL: rows of these levels may have tails, whose entries need registers too.
template <bool LDS, bool TAIL>
__global__ __launch_bounds__(kNarrowThreads) void k_tri_run(TriPass p,
                                                            const int *__restrict__ lev,
                                                            const int *__restrict__ width,
                                                            const int64_t *__restrict__ off,
                                                            const int64_t *__restrict__ tail,
                                                            int lev0, int lev1, int n, bool second)
{
    constexpr int REGS = TAIL ? kRowRegs / 2 : kRowRegs;
    extern __shared__ double sx[];
    const int tid = threadIdx.x;
    double *x = LDS ? sx : p.x;
    if (LDS && (lev0 > 0 || second)) {
        for (int i = tid; i < n; i += kNarrowThreads) sx[i] = p.x[i];
        __syncthreads();
    }
    const double *in = second ? x : p.in;
    struct Row {
        int i, c[REGS];
        double v[REGS], d, fo;
    };
    auto load = [&](int l, int t, Row &q) {
        q.i = -1;
        if (l >= lev1) return;
        const int u0 = lev[l], cnt = lev[l + 1] - u0, w = width[l];
        if (t >= cnt) return;
        const int64_t at = off[l] + t;
        q.i = p.row[u0 + t];
        q.d = p.diag ? p.diag[u0 + t] : 1.0;
        q.fo = p.fold ? p.fold[u0 + t] : 0.0;
#pragma unroll
        for (int k = 0; k < REGS; ++k) {
            // (marked: padding; the first level's columns are marked in wide
            // levels only)
            q.c[k] = k < w ? p.col[at + static_cast<int64_t>(k) * cnt] : kTriFirst;
            q.v[k] = k < w ? p.val[at + static_cast<int64_t>(k) * cnt] : 0.0;
        }
    };
    auto solve = [&](int l, int t, const Row &q) {
        double s = in[q.i];
        const int w = width[l];
#pragma unroll
        for (int k = 0; k < REGS; ++k)
            if (q.c[k] >= 0) s -= q.v[k] * x[q.c[k]];
        if (w > REGS) {
            const int cnt = lev[l + 1] - lev[l];
            for (int k = REGS; k < w; ++k) {
                const int64_t e = off[l] + static_cast<int64_t>(k) * cnt + t;
                const int c = p.col[e];
                if (c >= 0) s -= p.val[e] * x[c];
            }
        }
        if constexpr (TAIL) {
            const int u = lev[l] + t;
            const int64_t e1 = tail[u + 1];
#pragma unroll 4
            for (int64_t e = tail[u]; e < e1; ++e) s -= p.val[e] * x[p.col[e]];
        }
        if (p.diag) s /= q.d;
        const bool end = p.last || q.fo != 0.0;
        if (q.fo != 0.0) s /= q.fo;
        x[q.i] = s;
        if (LDS) p.x[q.i] = s;
        if (end) tri_end(p, q.i, s);
    };
    Row cur, nxt;
    load(lev0, tid, cur);
    for (int l = lev0; l < lev1; ++l) {
        load(l + 1, tid, nxt);  // independent of x
        if (cur.i >= 0) solve(l, tid, cur);
        for (int t = tid + kNarrowThreads; t < lev[l + 1] - lev[l]; t += kNarrowThreads) {
            Row q;
            load(l, t, q);
            solve(l, t, q);
        }
        __syncthreads();
        cur = nxt;
    }
}

// Both triangles (or one) of a system of narrow levels in the natural order
// by one wavefront, with no barrier between levels: a wavefront's LDS
// operations complete in order, so a level reads the x values the previous
// levels wrote.  Levels of at most 64 rows per H, rows of at most kTriWaveW
// entries per side (2D 9-point stencils and narrower): each level is H x 64
// records of 80 bytes (LDS offsets, values, the diagonal and its reciprocal;
// lanes without a row work on the spare slot), stored lane by lane and loaded
// kTriDepth levels ahead, so a level costs one LDS round trip, its products
// and the instructions of one row per lane: the wavefront is alone on its
// SIMD and bound by their issue.  The other wavefronts of the work-group only
// move x in and z out.
// 2 x 134 us (rows of two per lane, 128-byte records with counts and level
// pointers, a division per row) + 2 x 5.8 us (records packed on each call) ->
// 66 us per application of ILU(0) on 100 x 100 cells (298 levels a side).
typedef __attribute__((address_space(3))) double lds_double;
constexpr int kTriWaveW = 4;
constexpr int kTriDepth = 6;    // levels loaded ahead
constexpr int kTriTrip = 24;    // levels per loop trip (a multiple of kTriDepth)

struct alignas(16) WaveRec {
    int c[4];       // LDS byte offsets of the columns
    double v[4];
    double d, r;    // the diagonal and its reciprocal
    int i, pad[3];  // LDS byte offset of the row
};
// the records' five 16-byte parts of the 64 lanes one after another: all within
// reach of one address, the third part's
constexpr int kWaveParts = 5;
struct WaveLevel {
    int4 q[kWaveParts][64];
};

template <int H>
__device__ __forceinline__ void tri_wave_side(const WaveLevel *__restrict__ rec, int nlev)
{
    auto x = [](int at) -> lds_double & { return *reinterpret_cast<lds_double *>(at); };
    const int lane = threadIdx.x;
    union Slot {
        int4 q[kWaveParts - 1];
        WaveRec r;
        __device__ Slot() {}
    };
    Slot ring[kTriDepth][H];
    int row[kTriDepth][H];
    auto load = [&](int l, Slot(&s)[H], int(&i)[H]) {
#pragma unroll
        for (int h = 0; h < H; ++h) {
            typedef __attribute__((address_space(1))) const int4 global_int4;
            global_int4 *at = (global_int4 *)&rec[l * H + h].q[2][lane];
            asm("" : "+v"(at));  // (not taken apart into one address per part)
#pragma unroll
            for (int k = 0; k < kWaveParts - 1; ++k) {
                const int *part = (const int *)(at + 64 * (k - 2));
                s[h].q[k] = *(const int4 *)part;
            }
            i[h] = *(const int *)(at + 64 * 2);
        }
    };
#pragma unroll
    for (int k = 0; k < kTriDepth; ++k) load(k, ring[k], row[k]);
    // the records hold a multiple of kTriTrip levels and kTriDepth more
    for (int l = 0; l < nlev; l += kTriTrip) {
#pragma unroll
        for (int kk = 0; kk < kTriTrip; ++kk) {
            Slot(&cur)[H] = ring[kk % kTriDepth];
            int(&at)[H] = row[kk % kTriDepth];
            // (the scheduling barriers keep a later level's arithmetic, and
            // with it the wait for its records, below this level's)
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const WaveRec &r = cur[h].r;
                double s = x(at[h]);
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    s -= r.v[k] * x(r.c[k]);
                // s / d: the product with the reciprocal and one correction (and
                // what zeros and infinities give)
                const double q = s * r.r;
                x(at[h]) = __builtin_amdgcn_div_fixup(fma(fma(-q, r.d, s), r.r, q), r.d, s);
            }
            load(l + kk + kTriDepth, cur, at);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// (one wavefront per SIMD: to make room for more, the compiler would read a
// level's columns from LDS one after another)
template <int H>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_tri_wave(
    int n, const double *__restrict__ in, double *__restrict__ z, bool set,
    const WaveLevel *__restrict__ rec0, int nlev0, const WaveLevel *__restrict__ rec1, int nlev1)
{
    extern __shared__ double sx[];  // x and a spare slot
    for (int i = threadIdx.x; i < n; i += 256) sx[i] = in[i];
    if (threadIdx.x == 0) sx[n] = 0.0;
    __syncthreads();
    // The records' offsets are used as LDS addresses: sx is the kernel's only LDS
    // and begins at address 0 (adding its base took 5 instructions a level, 75.3
    // against 70.5 us).  The compiler is told that sx is reached by addresses.
    asm volatile("" ::"v"(sx) : "memory");
    if (threadIdx.x < 64) {
        if (rec0) tri_wave_side<H>(rec0, nlev0);
        if (rec1) tri_wave_side<H>(rec1, nlev1);
    }
    asm volatile("" ::: "memory");
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += 256) z[i] = set ? sx[i] : z[i] + sx[i];
}

// --- packing of the pattern, once per order ---

// columns and sources of position u (see TriSide; want: the side's sign in
// t.side), and with fold the diagonal's entry of rows with nothing later.  In
// the second level of a side whose first two go together every column is one
// of the first level.  First application on a new pattern, against packing by
// one host thread and a copy: coloured, 215,025 rows of seven 17.1 -> 13.5 ms,
// 65,536 rows of nine 7.9 -> 5.6 ms.
__global__ __launch_bounds__(256) void k_tri_fill(TriArgs t, int n, int want, int nlev, bool merged,
                                                  const int *__restrict__ lev,
                                                  const int *__restrict__ width,
                                                  const int64_t *__restrict__ off,
                                                  const int64_t *__restrict__ tail,
                                                  const int *__restrict__ row,
                                                  int *__restrict__ col, int *__restrict__ src,
                                                  int *__restrict__ fold)
{
    const int u = blockIdx.x * 256 + threadIdx.x;
    if (u >= n) return;
    int l = 0;
    for (int hi = nlev - 1; l < hi;) {  // the last level that starts at u or before
        const int mid = (l + hi + 1) >> 1;
        if (lev[mid] <= u) l = mid;
        else hi = mid - 1;
    }
    const int i = row[u], cnt = lev[l + 1] - lev[l], w = width[l];
    const int mark = merged && l == 1 ? kTriFirst : 0;
    const int64_t at = off[l] + u - lev[l];
    int k = 0;
    bool later = false;
    for (int e = t.rp[i]; e < t.rp[i + 1]; ++e) {
        later |= t.side[e] > 0;
        if (t.side[e] != want) continue;
        const int64_t p = k < w ? at + static_cast<int64_t>(k) * cnt : tail[u] + k - w;
        col[p] = t.ci[e] | mark;
        src[p] = e;
        ++k;
    }
    for (; k < w; ++k) {
        col[at + static_cast<int64_t>(k) * cnt] = i | kTriFirst;
        src[at + static_cast<int64_t>(k) * cnt] = -1;
    }
    if (fold) fold[u] = later ? -1 : t.dpos[i];
}

// --- packing of the values ---

// entries: f's value, with scale (first passes with a diagonal) the first
// level's division folded into the marked columns' values; padding: 0
__global__ __launch_bounds__(256) void k_tri_pack(int64_t m, const int *__restrict__ src,
                                                  const int *__restrict__ col,
                                                  const int *__restrict__ dpos, bool scale,
                                                  const double *__restrict__ f,
                                                  double *__restrict__ val)
{
    const int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (e >= m) return;
    const int q = src[e], c = col[e];
    double v = q < 0 ? 0.0 : f[q];
    if (q >= 0 && c < 0 && scale) v /= f[dpos[c & ~kTriFirst]];
    val[e] = v;
}

__global__ __launch_bounds__(256) void k_tri_pack_diag(int n, const int *__restrict__ row,
                                                       const int *__restrict__ dpos,
                                                       const int *__restrict__ foldsrc, bool unit,
                                                       const double *__restrict__ f,
                                                       double *__restrict__ diag,
                                                       double *__restrict__ fold)
{
    const int u = blockIdx.x * 256 + threadIdx.x;
    if (u >= n) return;
    diag[u] = unit ? 1.0 : f[dpos[row[u]]];
    if (fold) fold[u] = foldsrc[u] < 0 ? 0.0 : f[foldsrc[u]];
}

// the wavefront's records of level blockIdx.x (levels past nlev: no rows)
template <int H>
__global__ __launch_bounds__(64 * H) void k_tri_pack_wave(int n, int nlev,
                                                          const int *__restrict__ lev,
                                                          const int *__restrict__ width,
                                                          const int64_t *__restrict__ off,
                                                          const int *__restrict__ row,
                                                          const int *__restrict__ col,
                                                          const double *__restrict__ val,
                                                          const double *__restrict__ diag,
                                                          WaveLevel *__restrict__ rec)
{
    const int l = blockIdx.x, t = threadIdx.x;
    union {
        int4 q[kWaveParts];
        WaveRec r;
    } s;
    s.r.i = 8 * n;
    s.r.pad[0] = s.r.pad[1] = s.r.pad[2] = 0;
    s.r.d = s.r.r = 1.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        s.r.c[k] = 8 * n;
        s.r.v[k] = 0.0;
    }
    if (l < nlev && t < lev[l + 1] - lev[l]) {
        const int u = lev[l] + t, cnt = lev[l + 1] - lev[l], w = width[l];
        s.r.i = 8 * row[u];
        s.r.d = diag[u];
        s.r.r = 1.0 / diag[u];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t e = off[l] + static_cast<int64_t>(k) * cnt + t;
            if (k < w && val[e] != 0.0) {
                s.r.c[k] = 8 * (col[e] & ~kTriFirst);
                s.r.v[k] = val[e];
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kWaveParts; ++k) rec[l * H + t / 64].q[k][t & 63] = s.q[k];
}

// upper entries of the IC(0) array take the factor value of their transpose
__global__ __launch_bounds__(256) void k_ic_mirror(int64_t nnz, const int8_t *__restrict__ side,
                                                   const int *__restrict__ tpos,
                                                   double *__restrict__ l)
{
    const int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (e < nnz && side[e] > 0) l[e] = l[tpos[e]];
}

__global__ __launch_bounds__(256) void k_copy_vals(int64_t m, const double *__restrict__ a,
                                                   double *__restrict__ b)
{
    const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (t < m) b[t] = a[t];
}

// --- host: colouring, levels, launch segments ---

// first fit in ascending row order on the symmetrised pattern
int first_fit_colours(int n, const std::vector<int> &rp, const std::vector<int> &ci,
                      std::vector<int> &colour)
{
    std::vector<int> trp(n + 1, 0), tci(ci.size());
    for (int c : ci) trp[c + 1]++;
    for (int i = 0; i < n; ++i) trp[i + 1] += trp[i];
    {
        std::vector<int> pos(trp.begin(), trp.end() - 1);
        for (int i = 0; i < n; ++i)
            for (int e = rp[i]; e < rp[i + 1]; ++e) tci[pos[ci[e]]++] = i;
    }
    colour.assign(n, 0);
    std::vector<int> seen(n + 1, -1);
    int ncol = 0;
    for (int i = 0; i < n; ++i) {
        for (int e = rp[i]; e < rp[i + 1]; ++e)
            if (ci[e] < i) seen[colour[ci[e]]] = i;
        for (int e = trp[i]; e < trp[i + 1]; ++e)
            if (tci[e] < i) seen[colour[tci[e]]] = i;
        int c = 0;
        while (seen[c] == i) ++c;
        colour[i] = c;
        ncol = std::max(ncol, c + 1);
    }
    return ncol;
}

// rows grouped by dependency level (lower: on earlier entries, visited in
// order; upper: on later entries, visited backwards); rows ascending within
// a level
void level_sets(int n, const std::vector<int> &rp, const std::vector<int> &ci,
                const std::vector<int> &order, const std::vector<int> &rank, bool lower,
                std::vector<int> &ptr, std::vector<int> &rows)
{
    std::vector<int> lev(n, 0);
    int maxl = 0;
    for (int t = 0; t < n; ++t) {
        const int i = order[lower ? t : n - 1 - t];
        int l = 0;
        for (int e = rp[i]; e < rp[i + 1]; ++e) {
            const int j = ci[e];
            if (lower ? rank[j] < rank[i] : rank[j] > rank[i]) l = std::max(l, lev[j] + 1);
        }
        lev[i] = l;
        maxl = std::max(maxl, l);
    }
    ptr.assign(maxl + 2, 0);
    for (int i = 0; i < n; ++i) ptr[lev[i] + 1]++;
    for (int l = 0; l <= maxl; ++l) ptr[l + 1] += ptr[l];
    rows.resize(n);
    std::vector<int> pos(ptr.begin(), ptr.end() - 1);
    for (int i = 0; i < n; ++i) rows[pos[lev[i]]++] = i;
}

void segments(const std::vector<int> &ptr, std::vector<TriSegment> &seg)
{
    seg.clear();
    const int nlev = static_cast<int>(ptr.size()) - 1;
    for (int l = 0; l < nlev; ++l) {
        const bool wide = ptr[l + 1] - ptr[l] >= kWideRows;
        if (!wide && !seg.empty() && !seg.back().wide && seg.back().lev1 == l) {
            seg.back().lev1 = l + 1;
            continue;
        }
        seg.push_back(TriSegment{l, l + 1, wide, 0});
    }
}

// The packed width of a level of cnt rows with sum entries, the longest row
// `widest`; len gives a row's entries.  A level is padded to its longest row
// where that takes no more than kRowRegs places a row or three per entry; else
// to the width that all but an eighth of its rows keep to, at most eight places
// per entry, and the longer rows' further entries go to the tails.
// A row of 2,500 entries in a level of 20,001 short ones: padded to it, 50 M
// places (2.3 GB with the values of ILU(0) and SGS in two orders), 160 ms for a
// first ILU(0) application and 375 us for each; with tails 18 MB, 13 ms and 100 us.
template <typename Len>
int level_width(int cnt, int64_t sum, int widest, std::vector<int> &lengths, Len len)
{
    if (widest <= kRowRegs || static_cast<int64_t>(cnt) * widest <= 3 * sum) return widest;
    lengths.assign(widest + 1, 0);  // rows of each length
    for (int u = 0; u < cnt; ++u) lengths[len(u)]++;
    int w = widest;
    for (int longer = 0; w > 0 && longer + lengths[w] <= cnt / 8; --w) longer += lengths[w];
    return w;
}

// Arrays that live and die together, in one device allocation (the host
// vectors must outlive upload()); room() is left for a kernel to fill.
struct Slab {
    struct Place {
        void **dst;
        const void *src;
        size_t at, len;
    };
    std::vector<Place> places;
    size_t bytes = 0;
    template <typename T>
    void add(T **dst, const std::vector<T> &h)
    {
        room(dst, h.size());
        places.back().src = h.data();
    }
    template <typename T>
    void room(T **dst, size_t count)
    {
        places.push_back({reinterpret_cast<void **>(dst), nullptr, bytes, count * sizeof(T)});
        bytes += (count * sizeof(T) + 255) / 256 * 256;
    }
    bool upload(void **slab)
    {
        bool ok = hipMalloc(slab, std::max<size_t>(bytes, 1)) == hipSuccess;
        for (const Place &p : places) {
            if (!ok) break;
            *p.dst = static_cast<char *>(*slab) + p.at;
            ok = !p.src || p.len == 0 ||
                 hipMemcpy(*p.dst, p.src, p.len, hipMemcpyHostToDevice) == hipSuccess;
        }
        return ok;
    }
};

// the maps of k_ilu_run, once per pattern, of the rows in runs of narrow levels:
// natural order, rows that fit its lanes, and at most 512 MB of them.  Without
// them, also where they cannot be allocated, the runs take k_tri_narrow.
void ilu_maps(hipStream_t s, TriOrder &t)
{
    TriSide &q = t.s[0];
    if (t.ilu_at || t.ncolours > 0 || t.max_row > kIluLanes || q.max_w > kIluLow) return;
    int64_t m = 0;
    for (TriSegment &g : q.seg)
        if (!g.wide) {
            g.map0 = m;
            m += q.lev[g.lev1] - q.lev[g.lev0];
        }
    const size_t at = m * kIluLow * sizeof(int4), map = m * kIluLow * kIluLanes;
    if (m == 0 || at + map > (size_t(1) << 29)) return;
    if (hipMalloc(&t.ilu_at, at) != hipSuccess || hipMalloc(&t.ilu_map, map) != hipSuccess) {
        (void)hipGetLastError();
        if (t.ilu_at) hipFree(t.ilu_at);
        t.ilu_at = nullptr;
        t.ilu_map = nullptr;
        return;
    }
    const TriArgs a{t.rp, t.ci, t.dpos, t.side, t.lord, t.nlow};
    for (const TriSegment &g : q.seg) {
        if (g.wide) continue;
        const int64_t cnt = q.lev[g.lev1] - q.lev[g.lev0];
        k_ilu_map<<<static_cast<int>((cnt * kIluLow * kIluLanes + 255) / 256), 256, 0, s>>>(
            a, q.row + q.lev[g.lev0], static_cast<int>(cnt), t.ilu_at + g.map0 * kIluLow,
            t.ilu_map + g.map0 * kIluLow * kIluLanes);
    }
}

void run_factor(hipStream_t s, const TriOrder &t, const RowOp &r)
{
    const TriArgs a{t.rp, t.ci, t.dpos, t.side, t.lord, t.nlow};
    const TriSide &q = t.s[0];
    for (const TriSegment &g : q.seg) {
        if (g.wide) {
            const int cnt = q.lev[g.lev0 + 1] - q.lev[g.lev0];
            k_tri_wide<<<(cnt + 255) / 256, 256, 0, s>>>(a, r, q.row + q.lev[g.lev0], cnt);
        } else if (r.op == OP_ILU && t.ilu_map) {
            auto kern = q.max_w <= 4 ? k_ilu_run<4> : k_ilu_run<kIluLow>;
            kern<<<1, kNarrowThreads, 0, s>>>(a, q.row, q.d_lev, g.lev0, g.lev1,
                                              t.ilu_at + g.map0 * kIluLow,
                                              t.ilu_map + g.map0 * kIluLow * kIluLanes, r.f,
                                              r.flag);
        } else {
            k_tri_narrow<<<1, kNarrowThreads, 0, s>>>(a, r, q.d_lev, q.row, g.lev0, g.lev1);
        }
    }
}

// levels of a side's records: its own, rounded up to whole loop trips
int wave_levels(const TriSide &q)
{
    const int nlev = static_cast<int>(q.lev.size()) - 1;
    return (nlev + kTriTrip - 1) / kTriTrip * kTriTrip;
}
int wave_rows(const TriOrder &t) { return std::max(t.s[0].max_cnt, t.s[1].max_cnt) <= 64 ? 1 : 2; }

void launch_level(hipStream_t s, const TriPass &p, bool first, int u0, int skip, int cnt,
                  int64_t at, int width, const int64_t *tail)
{
    auto go = [&](auto w) {
        constexpr int W = decltype(w)::value;
        const int nb = (skip + cnt + 255) / 256;
        if (first) k_tri_level<W, true><<<nb, 256, 0, s>>>(p, u0, skip, cnt, at, width, tail);
        else k_tri_level<W, false><<<nb, 256, 0, s>>>(p, u0, skip, cnt, at, width, tail);
    };
    using std::integral_constant;
    switch (width) {
    case 1: go(integral_constant<int, 1>{}); break;
    case 2: go(integral_constant<int, 2>{}); break;
    case 3: go(integral_constant<int, 3>{}); break;
    case 4: go(integral_constant<int, 4>{}); break;
    case 5: go(integral_constant<int, 5>{}); break;
    case 6: go(integral_constant<int, 6>{}); break;
    case 7: go(integral_constant<int, 7>{}); break;
    case 8: go(integral_constant<int, 8>{}); break;
    default: go(integral_constant<int, 0>{}); break;
    }
}

// one side's pass; second: the other side's pass came first (p.in == p.x) and,
// with a symmetric pattern, has ended the rows of this side's level 0
void run_side(hipStream_t s, const TriOrder &t, const TriSide &q, const TriPass &p, bool second)
{
    const int from = second && t.sym_pattern ? 1 : 0;
    for (const TriSegment &g : q.seg) {
        const int lev0 = std::max(g.lev0, from);
        if (lev0 >= g.lev1) continue;
        if (g.wide) {
            const bool merged = q.merged && !second;
            if (merged && lev0 == 0) continue;  // in level 1's launch
            const int skip = merged && lev0 == 1 ? q.lev[1] : 0;
            launch_level(s, p, !second, q.lev[lev0] - skip, skip, q.lev[lev0 + 1] - q.lev[lev0],
                         q.off[lev0], q.width[lev0], q.tails[lev0] ? q.tail : nullptr);
            continue;
        }
        const size_t sh = t.n <= kNarrowLdsRows ? static_cast<size_t>(t.n) * sizeof(double) : 0;
        auto go = [&](auto kern) {
            if (sh > 65536)
                hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                    hipFuncAttributeMaxDynamicSharedMemorySize,
                                    static_cast<int>(sh));
            kern<<<1, kNarrowThreads, sh, s>>>(p, q.d_lev, q.d_width, q.d_off, q.tail, lev0, g.lev1,
                                               t.n, second);
        };
        if (std::find(q.tails.begin() + lev0, q.tails.begin() + g.lev1, 1) !=
            q.tails.begin() + g.lev1)
            sh ? go(k_tri_run<true, true>) : go(k_tri_run<false, true>);
        else
            sh ? go(k_tri_run<true, false>) : go(k_tri_run<false, false>);
    }
}

// room for the packed sides' values of one smoother, allocated once
bool alloc_values(const TriOrder &t, TriValues &v)
{
    if (v.slab) return true;
    size_t bytes = 0;
    auto place = [&](size_t m) {
        const size_t at = bytes;
        bytes += (m + 255) / 256 * 256;
        return at;
    };
    size_t val[2], diag[2], wave[2];
    for (int side = 0; side < 2; ++side) {
        const TriSide &q = t.s[side];
        val[side] = place(q.places * sizeof(double));
        diag[side] = place(t.n * sizeof(double));
        wave[side] = place(!t.wave ? 0
                                   : static_cast<size_t>(wave_levels(q) + kTriDepth) *
                                         wave_rows(t) * sizeof(WaveLevel));
    }
    const size_t fold = place(t.n * sizeof(double));
    if (hipMalloc(&v.slab, bytes) != hipSuccess) return false;
    char *base = static_cast<char *>(v.slab);
    for (int side = 0; side < 2; ++side) {
        v.val[side] = reinterpret_cast<double *>(base + val[side]);
        v.diag[side] = reinterpret_cast<double *>(base + diag[side]);
        v.wave[side] = base + wave[side];
    }
    v.fold = reinterpret_cast<double *>(base + fold);
    return true;
}

void pack_values(hipStream_t s, TriOrder &t, int kind, const double *f)
{
    TriValues &v = t.v[kind];
    for (int side = 0; side < 2; ++side) {
        const TriSide &q = t.s[side];
        const bool unit = kind == TRI_ILU && side == 0;
        const bool first = side == 0 || kind == TRI_GS;
        const int64_t m = q.places;
        if (m > 0)
            k_tri_pack<<<static_cast<int>((m + 255) / 256), 256, 0, s>>>(
                m, q.src, q.col, t.dpos, first && !unit, f, v.val[side]);
        const bool fold = side == 0 && kind != TRI_GS && t.sym_pattern;
        k_tri_pack_diag<<<(t.n + 255) / 256, 256, 0, s>>>(t.n, q.row, t.dpos, q.fold, unit, f,
                                                          v.diag[side], fold ? v.fold : nullptr);
        if (!t.wave) continue;
        const int nlev = static_cast<int>(q.lev.size()) - 1, nl = wave_levels(q) + kTriDepth;
        auto *rec = static_cast<WaveLevel *>(v.wave[side]);
        if (wave_rows(t) == 1)
            k_tri_pack_wave<1><<<nl, 64, 0, s>>>(t.n, nlev, q.d_lev, q.d_width, q.d_off, q.row,
                                                 q.col, v.val[side], v.diag[side], rec);
        else
            k_tri_pack_wave<2><<<nl, 128, 0, s>>>(t.n, nlev, q.d_lev, q.d_width, q.d_off, q.row,
                                                  q.col, v.val[side], v.diag[side], rec);
    }
    v.ok = true;
}

// z (+)= the solve of the sides [side0, side1] with the values of a kind
void run_solve(hipStream_t s, const TriOrder &t, int kind, int side0, int side1,
               const double *res, double *z, bool set, double *x)
{
    const TriValues &v = t.v[kind];
    if (t.wave) {
        const size_t sh = static_cast<size_t>(t.n + 1) * sizeof(double);
        const bool both = side0 != side1;
        auto go = [&](auto kern) {
            if (sh > 65536)
                hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                    hipFuncAttributeMaxDynamicSharedMemorySize,
                                    static_cast<int>(sh));
            kern<<<1, 256, sh, s>>>(t.n, res, z, set,
                                    static_cast<const WaveLevel *>(v.wave[side0]),
                                    wave_levels(t.s[side0]),
                                    both ? static_cast<const WaveLevel *>(v.wave[side1]) : nullptr,
                                    both ? wave_levels(t.s[side1]) : 0);
        };
        if (wave_rows(t) == 1) go(k_tri_wave<1>);
        else go(k_tri_wave<2>);
        return;
    }
    for (int side = side0;; side = side1) {
        const TriSide &q = t.s[side];
        const bool second = side != side0, last = side == side1;
        const bool unit = kind == TRI_ILU && side == 0;
        const TriPass p{q.row, q.col, v.val[side], unit ? nullptr : v.diag[side],
                        !last && t.sym_pattern ? v.fold : nullptr,
                        second ? x : res, x, z, last, set};
        run_side(s, t, q, p, second);
        if (last) break;
    }
}

}  // namespace

void free_tri_order(TriOrder &t)
{
    for (void *p : {t.slab, static_cast<void *>(t.ilu_at), static_cast<void *>(t.ilu_map),
                    t.v[0].slab, t.v[1].slab, t.v[2].slab})
        if (p) hipFree(p);
    t = TriOrder();
}

msrsb_status tri_order_setup(msrsb_ctx *c, int ordering)
{
    TriOrder &t = c->tri[ordering];
    if (t.built) return MSRSB_OK;
    const int n = c->n;
    const std::vector<int> &rp = c->h_rp, &ci = c->h_ci;
    std::vector<int> order(n), rank(n);
    if (ordering == MSRSB_ORDER_MULTICOLOR) {
        std::vector<int> colour;
        const int ncol = first_fit_colours(n, rp, ci, colour);
        std::vector<int> start(ncol + 1, 0);
        for (int i = 0; i < n; ++i) start[colour[i] + 1]++;
        for (int k = 0; k < ncol; ++k) start[k + 1] += start[k];
        for (int i = 0; i < n; ++i) order[start[colour[i]]++] = i;
        t.ncolours = ncol;
    } else {
        std::iota(order.begin(), order.end(), 0);
        t.ncolours = 0;
    }
    t.n = n;
    for (int k = 0; k < n; ++k) rank[order[k]] = k;
    const int64_t nnz = c->nnz;
    std::vector<int8_t> side(nnz);
    std::vector<int> lord(nnz, 0), nlow(n, 0), tpos(nnz, -1);
    std::vector<std::pair<int, int>> low;
    std::vector<int> count[2];  // entries of a row on each side
    count[0].assign(n, 0);
    count[1].assign(n, 0);
    for (int i = 0; i < n; ++i) {
        low.clear();
        for (int e = rp[i]; e < rp[i + 1]; ++e) {
            const int j = ci[e];
            side[e] = j == i ? 0 : (rank[j] < rank[i] ? -1 : 1);
            if (side[e] < 0) low.emplace_back(rank[j], e);
            // the transposed entry (j, i), when stored
            const int *b = ci.data() + rp[j], *en = ci.data() + rp[j + 1];
            const int *it = std::lower_bound(b, en, i);
            if (it != en && *it == i) tpos[e] = static_cast<int>(it - ci.data());
        }
        if (t.ncolours > 0) std::sort(low.begin(), low.end());  // (ascending already if natural)
        t.max_row = std::max(t.max_row, rp[i + 1] - rp[i]);
        nlow[i] = static_cast<int>(low.size());
        for (size_t u = 0; u < low.size(); ++u) lord[rp[i] + u] = low[u].second;
        count[0][i] = nlow[i];
        count[1][i] = rp[i + 1] - rp[i] - 1 - nlow[i];
    }
    t.sym_pattern = std::all_of(tpos.begin(), tpos.end(), [](int p) { return p >= 0; });
    Slab slab;
    std::vector<int> rows_of[2], lengths;
    std::vector<int64_t> tail_of[2];
    slab.add(&t.side, side);
    slab.add(&t.lord, lord);
    slab.add(&t.nlow, nlow);
    slab.add(&t.tpos, tpos);
    for (int sd = 0; sd < 2; ++sd) {
        TriSide &q = t.s[sd];
        std::vector<int> &rows = rows_of[sd];
        level_sets(n, rp, ci, order, rank, sd == 0, q.lev, rows);
        segments(q.lev, q.seg);
        const int nlev = static_cast<int>(q.lev.size()) - 1;
        q.merged = nlev >= 2 && q.seg[0].wide && q.seg[1].wide;
        q.width.assign(nlev, 0);
        q.off.assign(nlev + 1, 0);
        q.tails.assign(nlev, 0);
        std::vector<int64_t> &tail = tail_of[sd];
        for (int l = 0; l < nlev; ++l) {
            const int cnt = q.lev[l + 1] - q.lev[l];
            auto len = [&](int u) { return count[sd][rows[q.lev[l] + u]]; };
            int widest = 0;
            int64_t sum = 0;
            for (int u = 0; u < cnt; ++u) {
                widest = std::max(widest, len(u));
                sum += len(u);
            }
            q.width[l] = level_width(cnt, sum, widest, lengths, len);
            q.off[l + 1] = q.off[l] + static_cast<int64_t>(cnt) * q.width[l];
            q.max_w = std::max(q.max_w, widest);
            q.max_cnt = std::max(q.max_cnt, cnt);
            if (q.width[l] == widest) continue;
            q.tails[l] = 1;
            tail.resize(n + 1);
        }
        q.places = q.off[nlev];
        if (!tail.empty()) {
            for (int l = 0; l < nlev; ++l)
                for (int u = q.lev[l]; u < q.lev[l + 1]; ++u) {
                    tail[u] = q.places;
                    q.places += std::max(count[sd][rows[u]] - q.width[l], 0);
                }
            tail[n] = q.places;
            slab.add(&q.tail, tail);
        }
        slab.room(&q.col, q.places);
        slab.room(&q.src, q.places);
        if (sd == 0) slab.room(&q.fold, n);
        slab.add(&q.d_lev, q.lev);
        slab.add(&q.d_width, q.width);
        slab.add(&q.d_off, q.off);
        slab.add(&q.row, rows);
    }
    t.rp = c->rp;
    t.ci = c->ci;
    t.dpos = c->diag_pos;
    // one wavefront walks both triangles of a small system in the natural order
    t.wave = t.ncolours == 0 && n <= kNarrowLdsRows &&
             std::max(t.s[0].max_w, t.s[1].max_w) <= kTriWaveW &&
             std::max(t.s[0].max_cnt, t.s[1].max_cnt) <= 128;
    // (SGS needs no factors, so the allocation-free application takes it on any
    // order that is set up: its room comes with the order)
    if (!slab.upload(&t.slab) || !alloc_values(t, t.v[TRI_GS])) {
        free_tri_order(t);
        return MSRSB_E_NOMEM;
    }
    const TriArgs a{t.rp, t.ci, t.dpos, t.side, t.lord, t.nlow};
    for (int sd = 0; sd < 2; ++sd) {
        const TriSide &q = t.s[sd];
        k_tri_fill<<<(n + 255) / 256, 256, 0, c->stream>>>(
            a, n, sd == 0 ? -1 : 1, static_cast<int>(q.lev.size()) - 1, q.merged, q.d_lev,
            q.d_width, q.d_off, q.tail, q.row, q.col, q.src, q.fold);
    }
    t.built = true;
    return MSRSB_OK;
}

msrsb_status tri_factor(msrsb_ctx *c, int ordering, int kind)
{
    hipStream_t s = c->stream;
    TriOrder &t = c->tri[ordering];
    const int k = kind == MSRSB_SMOOTH_ILU0 ? TRI_ILU : TRI_IC;
    double *&f = k == TRI_ILU ? c->ilu_f[ordering] : c->ic_f[ordering];
    if (!f && hipMalloc(&f, c->nnz * sizeof(double)) != hipSuccess) return MSRSB_E_NOMEM;
    if (!alloc_values(t, t.v[k])) return MSRSB_E_NOMEM;
    int *flag = c->dev_flag;
    hipMemsetAsync(flag, 0, sizeof(int), s);
    RowOp r;
    r.f = f;
    r.flag = flag;
    const int nb = static_cast<int>((c->nnz + 255) / 256);
    if (k == TRI_ILU) {
        ilu_maps(s, t);
        k_copy_vals<<<nb, 256, 0, s>>>(c->nnz, c->a, f);
        r.op = OP_ILU;
        run_factor(s, t, r);
    } else {
        r.op = OP_IC;
        r.a = c->a;
        run_factor(s, t, r);
        k_ic_mirror<<<nb, 256, 0, s>>>(c->nnz, t.side, t.tpos, f);
    }
    pack_values(s, t, k, f);
    int hflag = 0;
    hipMemcpyAsync(&hflag, flag, sizeof(int), hipMemcpyDeviceToHost, s);
    if (hipStreamSynchronize(s) != hipSuccess) return MSRSB_E_HIP;
    return hflag ? MSRSB_E_BREAKDOWN : MSRSB_OK;
}

void tri_apply(msrsb_ctx *c, int ordering, int kind, const double *res, double *z, bool set,
               double *x)
{
    run_solve(c->stream, c->tri[ordering], kind == MSRSB_SMOOTH_ILU0 ? TRI_ILU : TRI_IC, 0, 1, res,
              z, set, x);
}

// A's values are packed by the first half sweep of an order and from then on
// whenever they change, so that a graph that holds this launch and not the
// packing follows them
void tri_gs_half(msrsb_ctx *c, int ordering, bool lower, const double *res, double *z, bool set,
                 double *x)
{
    TriOrder &t = c->tri[ordering];
    if (!t.v[TRI_GS].ok) {
        pack_values(c->stream, t, TRI_GS, c->a);
        t.gs_used = true;
        // (recorded into a graph, the packing has not been done yet)
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(c->stream, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone)
            t.v[TRI_GS].ok = false;
    }
    const int side = lower ? 0 : 1;
    run_solve(c->stream, t, TRI_GS, side, side, res, z, set, x);
}

void tri_values_changed(msrsb_ctx *c)
{
    for (TriOrder &t : c->tri)
        if (t.gs_used) pack_values(c->stream, t, TRI_GS, c->a);
}

}  // namespace msrsb
