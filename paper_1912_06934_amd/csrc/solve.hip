// Two-stage preconditioner (Alg. 3, Alg. 4) and the Krylov drivers (PCG with
// the flexible Polak-Ribiere beta, right-preconditioned restarted GMRES).
// All vector arithmetic runs in device kernels; the host only queues work and
// reads the residual norm to decide when to stop.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstring>
#include <new>
#include <type_traits>

#include "internal.h"
#include "solve.h"

namespace msrsb {
namespace {

// --- GMRES orthogonalisation (classical Gram-Schmidt applied twice) ---
//
// For the first kOrthoCols columns of a cycle the whole step after w = A B v
// is four launches (15 to 30 us a step on 65,536 rows from the first to the
// 30th column, bound by the latency of the partial sums and by the vectors'
// passes through the L2; a launch per product, sum, update and scalar took
// eleven, 28 to 40 us):
//   dots     part = V^T w by work-group
//   update   h = the sum of part; w -= V h; part = V^T w again
//   norm     h2 = the sum of part; w -= V h2; ||w||^2 by work-group
//   finish   v_next = w / ||w||; one wavefront: the Hessenberg column h + h2,
//            its Givens rotations and the residual posted to the host
// A work-group holds kOrthoThreads rows per pass and at most kOrthoBlocks
// work-groups share the rows, so that every consumer can add the producers'
// partial sums by itself (at most 256 per column, read from the L2) instead
// of waiting for a launch that does; sums in a fixed order (reproducible).
constexpr int kOrthoCols = 32;
constexpr int kOrthoThreads = 512;
constexpr int kOrthoBlocks = 256;
constexpr int kOrthoWaves = kOrthoThreads / 64;

// v[q] summed over the wavefront for q < K (K a power of two up to 32): lane
// pairs exchange halves of the values, so that lane l ends with the total of
// value l / (64 / K) in v[0]
template <int K, int M = K / 2, int OFF = 32>
__device__ __forceinline__ void wave_sums(double (&v)[K])
{
    if constexpr (M >= 1) {
        const bool hi = (threadIdx.x & OFF) != 0;
#pragma unroll
        for (int q = 0; q < M; ++q) {
            const double keep = hi ? v[q + M] : v[q], send = hi ? v[q] : v[q + M];
            v[q] = keep + __shfl_xor(send, OFF, 64);
        }
        wave_sums<K, M / 2, OFF / 2>(v);
    } else if constexpr (OFF >= 1) {
        v[0] += __shfl_xor(v[0], OFF, 64);
        wave_sums<K, 0, OFF / 2>(v);
    }
}

// part[t * gridDim.x + b] = the work-group's sum of acc[t], t < k
template <int K>
__device__ __forceinline__ void store_sums(double (&acc)[K], int k, double *__restrict__ part)
{
    __shared__ double sh[kOrthoWaves][K];
    wave_sums<K>(acc);
    constexpr int G = 64 / K;  // lanes per value
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane % G == 0) sh[w][lane / G] = acc[0];
    __syncthreads();
    if (static_cast<int>(threadIdx.x) < k) {
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < kOrthoWaves; ++q) s += sh[q][threadIdx.x];
        part[static_cast<int64_t>(threadIdx.x) * gridDim.x + blockIdx.x] = s;
    }
}

// h[t] = sum over the nb work-groups of part[t * nb + b] for t < k, 0 for the
// other t < K, in LDS
template <int K>
__device__ __forceinline__ void load_sums(int k, int nb, const double *__restrict__ part,
                                          double *__restrict__ h)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    constexpr int T = (K + kOrthoWaves - 1) / kOrthoWaves;
    double v[T];
#pragma unroll
    for (int q = 0; q < T; ++q) {
        const int t = w + q * kOrthoWaves;
        v[q] = 0.0;
        if (t < k)
#pragma unroll
            for (int b = 0; b < kOrthoBlocks / 64; ++b)
                if (lane + 64 * b < nb) v[q] += part[static_cast<int64_t>(t) * nb + lane + 64 * b];
    }
#pragma unroll
    for (int q = 0; q < T; ++q) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v[q] += __shfl_xor(v[q], off, 64);
        const int t = w + q * kOrthoWaves;
        if (lane == 0 && t < K) h[t] = v[q];
    }
    __syncthreads();
}

// UPDATE: first w -= V h with h summed from pin (work-group 0 writes it to
// hout, added to what is there with ADD).  DOTS: pout = V^T w, else ||w||^2.
template <int K, bool UPDATE, bool ADD, bool DOTS>
__global__ __launch_bounds__(kOrthoThreads) void k_ortho(int n, int k, int nbin, int64_t ldv,
                                                         const double *__restrict__ V,
                                                         double *__restrict__ w,
                                                         const double *__restrict__ pin,
                                                         double *__restrict__ hout,
                                                         double *__restrict__ pout)
{
    __shared__ double h[K];
    int i = blockIdx.x * kOrthoThreads + threadIdx.x;
    double v[K], x;
    // (columns past k repeat the last one: no branches between the loads)
    auto load = [&](int r) {
#pragma unroll
        for (int t = 0; t < K; ++t) v[t] = V[min(t, k - 1) * ldv + r];
        x = w[r];
    };
    // without products the registers hold the first rows while the sums are
    // formed (9.2 -> 7.9 us at 32 columns; with them, they spill: 16 us)
    constexpr bool AHEAD = UPDATE && !DOTS;
    if constexpr (AHEAD) load(min(i, n - 1));
    if constexpr (UPDATE) {
        load_sums<K>(k, nbin, pin, h);
        if (blockIdx.x == 0 && static_cast<int>(threadIdx.x) < k)
            hout[threadIdx.x] = ADD ? hout[threadIdx.x] + h[threadIdx.x] : h[threadIdx.x];
    }
    constexpr int A = DOTS ? K : 1;
    double acc[A];
#pragma unroll
    for (int t = 0; t < A; ++t) acc[t] = 0.0;
    for (bool first = true; i < n; i += gridDim.x * kOrthoThreads, first = false) {
        if (!AHEAD || !first) load(i);
        if constexpr (UPDATE) {
            double s = 0.0;
#pragma unroll
            for (int t = 0; t < K; ++t) s += h[t] * v[t];
            x -= s;
            w[i] = x;
        }
        if constexpr (DOTS) {
#pragma unroll
            for (int t = 0; t < K; ++t) acc[t] += v[t] * x;
        } else {
            acc[0] += x * x;
        }
    }
    store_sums<A>(acc, DOTS ? k : 1, pout);
}

// Apply the previous Givens rotations to the new Hessenberg column (h[0..j]
// from the Gram-Schmidt, the norm below), form the new rotation, update g and
// write |g[j+1]| and the rotated diagonal to res.  One wavefront; lane i holds
// entry i of the column (j < 64) and of the rotations, which thread by thread
// follow each other through lane reads instead of memory.
// With host_out (coherent pinned memory) the residual estimate and the
// denominator also go to the host's mailbox.
__device__ void gmres_givens(int j, int m, double *__restrict__ H, const double *__restrict__ h,
                             double norm, double *__restrict__ cs, double *__restrict__ sn,
                             double *__restrict__ g, double *__restrict__ res,
                             double *__restrict__ host_out, double tag)
{
    const int lane = threadIdx.x & 63;
    const double hl = lane <= j ? h[lane] : 0.0;
    const double cl = lane < j ? cs[lane] : 0.0, sl = lane < j ? sn[lane] : 0.0;
    const double gj = g[j];
    double a = __shfl(hl, 0, 64), mine = 0.0;  // a: the running entry i
    for (int i = 0; i < j; ++i) {
        const double b = __shfl(hl, i + 1, 64), c = __shfl(cl, i, 64), s = __shfl(sl, i, 64);
        const double top = c * a + s * b;
        a = -s * a + c * b;
        if (lane == i) mine = top;
    }
    const double den = sqrt(a * a + norm * norm);
    double c = 1.0, s = 0.0;
    if (den > 0.0) {
        c = a / den;
        s = norm / den;
    }
    if (lane == j) mine = den;
    if (lane <= j) H[static_cast<int64_t>(lane) * m + j] = mine;
    if (lane != 0) return;
    cs[j] = c;
    sn[j] = s;
    const double gn = -s * gj;
    g[j + 1] = gn;
    g[j] = c * gj;
    res[0] = fabs(gn);
    res[1] = den;
    if (host_out) post_mail(host_out, fabs(gn), den, tag);
}

struct GivensArgs {
    int j, m;
    double *H;
    const double *h;
    double *cs, *sn, *g, *res, *host_out;
    double tag;
};

// (columns past kOrthoCols: the norm comes from launch_norm_scale)
__global__ __launch_bounds__(64) void k_gmres_givens(GivensArgs a, const double *__restrict__ nrm2)
{
    gmres_givens(a.j, a.m, a.H, a.h, sqrt(nrm2[0]), a.cs, a.sn, a.g, a.res, a.host_out, a.tag);
}

// v = w / ||w|| (0 when the norm is 0), with ||w||^2 summed from nb partials;
// the last work-group has no rows: its first wavefront does the Givens step
__global__ __launch_bounds__(kOrthoThreads) void k_ortho_finish(int n, int nb,
                                                                const double *__restrict__ part,
                                                                const double *__restrict__ w,
                                                                double *__restrict__ v,
                                                                GivensArgs a)
{
    __shared__ double h[1];
    load_sums<1>(1, nb, part, h);
    const double nr = sqrt(h[0]);
    const int rows = gridDim.x - 1;
    if (static_cast<int>(blockIdx.x) == rows) {
        if (threadIdx.x < 64)
            gmres_givens(a.j, a.m, a.H, a.h, nr, a.cs, a.sn, a.g, a.res, a.host_out, a.tag);
        return;
    }
    for (int i = blockIdx.x * kOrthoThreads + threadIdx.x; i < n; i += rows * kOrthoThreads)
        v[i] = nr > 0.0 ? w[i] / nr : 0.0;
}

// y = H(0:k,0:k)^{-1} g(0:k) (upper triangular back substitution): lane i
// holds g_i and reads its row of H ahead of the column that needs it
__global__ __launch_bounds__(64) void k_gmres_solve(int k, int m, const double *__restrict__ H,
                                                    const double *__restrict__ g,
                                                    double *__restrict__ y)
{
    __shared__ double U[64][65];
    const int lane = threadIdx.x;
    for (int r = 0; r < k; ++r)
        if (lane < k) U[r][lane] = H[static_cast<int64_t>(r) * m + lane];
    __syncthreads();
    double s = lane < k ? g[lane] : 0.0;
    for (int r = k - 1; r >= 0; --r) {
        const double yr = __shfl(s, r, 64) / U[r][r];
        if (lane < r) s -= U[lane][r] * yr;
        if (lane == r) s = yr;
    }
    if (lane < k) y[lane] = s;
}

__global__ void k_gmres_init_g(int m, double *__restrict__ g, const double *__restrict__ nrm2)
{
    if (threadIdx.x != 0) return;
    for (int i = 0; i <= m; ++i) g[i] = 0.0;
    g[0] = sqrt(nrm2[0]);
}

__global__ void k_vec_add(int k, double *__restrict__ a, const double *__restrict__ b)
{
    const int t = threadIdx.x;
    if (t < k) a[t] += b[t];
}

// the orthogonalisation of one step with k <= kOrthoCols columns
void ortho(hipStream_t s, int n, int k, int64_t ldv, const double *V, double *w, double *vnext, double *h,
           double *const part[2], const GivensArgs &g)
{
    const int nb = std::min(kOrthoBlocks, (n + kOrthoThreads - 1) / kOrthoThreads);
    auto go = [&](auto kk) {
        constexpr int K = decltype(kk)::value;
        k_ortho<K, false, false, true>
            <<<nb, kOrthoThreads, 0, s>>>(n, k, nb, ldv, V, w, nullptr, nullptr, part[0]);
        k_ortho<K, true, false, true>
            <<<nb, kOrthoThreads, 0, s>>>(n, k, nb, ldv, V, w, part[0], h, part[1]);
        k_ortho<K, true, true, false>
            <<<nb, kOrthoThreads, 0, s>>>(n, k, nb, ldv, V, w, part[1], h, part[0]);
    };
    using std::integral_constant;
    if (k <= 4) go(integral_constant<int, 4>{});
    else if (k <= 8) go(integral_constant<int, 8>{});
    else if (k <= 16) go(integral_constant<int, 16>{});
    else go(integral_constant<int, kOrthoCols>{});
    k_ortho_finish<<<nb + 1, kOrthoThreads, 0, s>>>(n, nb, part[0], w, vnext, g);
}

// out = a x + b y + c w (w may be null); out may alias x, y or w
__global__ __launch_bounds__(kBlock) void k_lincomb(int n, double a, const double *x, double b,
                                                    const double *y, double c, const double *w,
                                                    double *out)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    double v = a * x[i] + b * y[i];
    if (w) v += c * w[i];
    out[i] = v;
}

void lincomb(hipStream_t s, int n, double a, const double *x, double b, const double *y,
             double c, const double *w, double *out)
{
    k_lincomb<<<(n + kBlock - 1) / kBlock, kBlock, 0, s>>>(n, a, x, b, y, c, w, out);
}

// The fine operator (A, or A^T for the transposed solve) in its CSR and,
// when available, DIA forms, with the diagonal inverses of its smoothers.
struct Op {
    const int *rp, *ci;
    const double *a;
    const float *a32;
    DiaOffsets d;
    const double *ad;
    const float *ad32;
    const double *dj, *dl1;
    const float *dj32, *dl132;
    NodeStencil ns;            // NBS form (ns.n == 0: none)
    const double *nv;
    const float *nv32;
};

Op fine_op(msrsb_ctx *c, bool trans)
{
    Op o;
    if (!trans || c->a_symmetric) {  // A^T = A: share A's data
        o.rp = c->rp;
        o.ci = c->ci;
        o.a = c->a;
        o.a32 = c->a32;
        o.d = c->a_off;
        o.ad = c->a_dia;
        o.ad32 = c->a_dia32;
        o.dj = c->dinv_jac;
        o.dl1 = c->dinv_l1;
        o.dj32 = c->dinv_jac32;
        o.dl132 = c->dinv_l1_32;
        o.ns = c->a_ns;
        o.nv = c->a_ns_val;
        o.nv32 = c->a_ns_val32;
    } else {
        o.rp = c->at_rp;
        o.ci = c->at_ci;
        o.a = c->at;
        o.a32 = c->at32;
        o.d = c->at_off;
        o.ad = c->at_dia;
        o.ad32 = c->at_dia32;
        o.dj = c->dinv_jac_t;
        o.dl1 = c->dinv_l1_t;
        o.dj32 = c->dinv_jac32_t;
        o.dl132 = c->dinv_l1_32_t;
        o.ns = NodeStencil();
        o.nv = nullptr;
        o.nv32 = nullptr;
    }
    return o;
}

// r = f - A x; fp32 (inside the preconditioner of the precision form) uses
// the FP32 copy of A's stencil values when there is one
void op_residual(hipStream_t s, int n, const Op &o, const double *f, const double *x, double *r,
                 bool fp32 = false)
{
    if (o.d.n > 0)
        launch_dia_residual(s, n, o.d, o.ad, fp32 ? o.ad32 : nullptr, f, x, r);
    else if (o.ns.n > 0)
        launch_nbs_residual(s, n, o.ns, o.nv, fp32 ? o.nv32 : nullptr, f, x, r);
    else
        launch_residual(s, n, o.rp, o.ci, o.a, f, x, r);
}

void op_spmv(hipStream_t s, int n, const Op &o, const double *x, double *y)
{
    if (o.d.n > 0)
        launch_dia_spmv(s, n, o.d, o.ad, x, y);
    else if (o.ns.n > 0)
        launch_nbs_spmv(s, n, o.ns, o.nv, x, y);
    else
        launch_spmv(s, n, o.rp, o.ci, o.a, x, y);
}

// p = z + beta p_old, q = A p (PCG); returns the number of p.q partials left
// for the update to add, 0 when alpha has been formed
int p_spmv(hipStream_t s, int n, const Op &o, const double *z, const double *pold, double *pnew,
           double *q, double *pq, const PcgSums &sums)
{
    int nb;
    if (o.d.n == 0 && o.ns.n > 0)
        nb = launch_nbs_pcg_p_spmv(s, n, o.ns, o.nv, z, pold, pnew, q, pq, sums);
    else
        nb = launch_pcg_p_spmv(s, n, o.d, o.ad, o.rp, o.ci, o.a, z, pold, pnew, q, pq, sums);
    if (nb <= kSumBlocks) return nb;
    launch_fin_alpha(s, nb, pq, sums.scal, sums.rz_new, sums.tag + 1.0);
    return 0;
}

template <typename T>
msrsb_status dev_alloc(T **p, size_t count)
{
    if (*p) return MSRSB_OK;
    if (hipMalloc(reinterpret_cast<void **>(p), std::max<size_t>(count, 1) * sizeof(T)) !=
        hipSuccess)
        return MSRSB_E_NOMEM;
    return MSRSB_OK;
}

bool is_diag(int kind) { return kind == MSRSB_SMOOTH_JACOBI || kind == MSRSB_SMOOTH_L1JACOBI; }

// one smoothing sweep z += M^{-1} (v - A z); with zero, z is known to be zero
// and is not read.  The result may land in *spare, in which case the two
// pointers are exchanged.  ord: sweep order of the triangular smoothers.
void sweep(msrsb_ctx *c, const Op &o, int kind, bool fp32, const double *v, double **z,
           double **spare, bool zero, double *tmp, int ord)
{
    hipStream_t s = c->stream;
    const int n = c->n;
    if (is_diag(kind)) {
        const bool l1 = kind == MSRSB_SMOOTH_L1JACOBI;
        const double *d64 = l1 ? o.dl1 : o.dj;
        const float *d32 = l1 ? o.dl132 : o.dj32;
        if (o.d.n > 0 && !zero)
            launch_dia_sweep(s, n, o.d, fp32, o.ad, o.ad32, d64, d32, v, *z, *spare, false);
        else if (o.ns.n > 0)
            launch_nbs_sweep(s, n, o.ns, fp32, o.nv, o.nv32, d64, d32, v, *z, *spare, zero);
        else
            launch_sweep(s, n, o.rp, o.ci, o.a, o.a32, d64, d32, fp32, v, *z, *spare, zero);
        std::swap(*z, *spare);
    } else if (is_tri(kind)) {
        // residual, then the triangular solves in the order; SGS is a forward
        // sweep (D + L)^{-1} and a backward one (D + U)^{-1}, each on the
        // residual of the current iterate
        const double *res = v;
        if (!zero) {
            op_residual(s, n, o, v, *z, tmp);
            res = tmp;
        }
        if (kind == MSRSB_SMOOTH_SGS) {
            tri_gs_half(c, ord, true, res, *z, zero, *spare);
            op_residual(s, n, o, v, *z, tmp);
            tri_gs_half(c, ord, false, tmp, *z, false, *spare);
        } else {
            tri_apply(c, ord, kind, res, *z, zero, *spare);
        }
    }
}

}  // namespace

bool is_tri(int kind)
{
    return kind == MSRSB_SMOOTH_ILU0 || kind == MSRSB_SMOOTH_IC0 || kind == MSRSB_SMOOTH_SGS;
}

msrsb_status ensure_workspace(msrsb_ctx *c)
{
    const size_t n = static_cast<size_t>(c->n);
    for (auto &p : c->w)
        if (dev_alloc(&p, n)) return MSRSB_E_NOMEM;
    for (auto &p : c->wf)
        if (dev_alloc(&p, n)) return MSRSB_E_NOMEM;
    // (PCG: two products' partials, then the p.q ones, at most one per 128 rows: the
    // 64 nodes of a work-group at two components each)
    const size_t np = std::max<size_t>({pq_offset(n) + n / 128 + 16, 2 * static_cast<size_t>(kReduceBlocks),
                                        64 * static_cast<size_t>(std::max(c->nc, 1)) + 64,
                                        static_cast<size_t>(64 * 66),
                                        static_cast<size_t>(3 * 2048)});
    // (the r.r ones: at most one per 64 rows and 16 more, where a 2D grid's tiles
    // are mostly edge)
    if (dev_alloc(&c->partials, np) || dev_alloc(&c->partials_rr, n / 64 + 16) ||
        dev_alloc(&c->scal, S_COUNT) ||
        dev_alloc(&c->vc, std::max(c->nc, 1)) || dev_alloc(&c->wc, std::max(c->nc, 1)) ||
        dev_alloc(&c->eit_val, 1) || dev_alloc(&c->dev_flag, 4))
        return MSRSB_E_NOMEM;
    if (!c->h_pinned && hipHostMalloc(reinterpret_cast<void **>(&c->h_pinned), 64 * sizeof(double),
                                      hipHostMallocCoherent) != hipSuccess)
        return MSRSB_E_NOMEM;
    return MSRSB_OK;
}

msrsb_status ensure_smoother(msrsb_ctx *c, const msrsb_solve_opts *o, bool trans)
{
    const int kinds[2] = {o->pre_sweeps > 0 ? o->pre_smoother : MSRSB_SMOOTH_NONE,
                          o->post_sweeps > 0 ? o->post_smoother : MSRSB_SMOOTH_NONE};
    const bool need_tri = is_tri(kinds[0]) || is_tri(kinds[1]);
    if (need_tri && trans) {
        c->err = "ILU(0), IC(0) and SGS are not available for the transposed solve";
        return MSRSB_E_ARG;
    }
    const bool fp32 = o->fp32_smoother != 0;
    const size_t n = static_cast<size_t>(c->n);
    hipStream_t s = c->stream;
    if (c->a_symmetric) trans = false;  // the smoothers of A^T are those of A
    const int noff = trans ? c->at_off.n : c->a_off.n;
    if (!trans) {
        if (!c->smoother_valid || (fp32 && !c->smoother32_valid)) {
            if (dev_alloc(&c->dinv_jac, n) || dev_alloc(&c->dinv_l1, n)) return MSRSB_E_NOMEM;
            // A's FP32 values: of its stencil form, or of the CSR entries
            const size_t nslot = static_cast<size_t>(c->a_ns.n) * c->a_ns.bs;
            const bool csr = noff == 0 && nslot == 0;
            if (fp32 && (dev_alloc(&c->dinv_jac32, n) || dev_alloc(&c->dinv_l1_32, n) ||
                         (csr && dev_alloc(&c->a32, static_cast<size_t>(c->nnz)))))
                return MSRSB_E_NOMEM;
            if (fp32 && noff > 0 && dev_alloc(&c->a_dia32, n * noff)) return MSRSB_E_NOMEM;
            if (fp32 && nslot > 0 && dev_alloc(&c->a_ns_val32, n * nslot)) return MSRSB_E_NOMEM;
            launch_diag_inverses(s, c->n, c->rp, c->ci, c->a, c->a_off, c->a_dia, c->a_ns,
                                 c->a_ns_val, c->dinv_jac, c->dinv_l1,
                                 fp32 ? c->dinv_jac32 : nullptr, fp32 ? c->dinv_l1_32 : nullptr,
                                 fp32 && csr ? c->a32 : nullptr, c->dev_flag);
            if (fp32 && noff > 0)
                launch_p_convert_down(s, static_cast<int64_t>(n) * noff, c->a_dia, c->a_dia32);
            if (fp32 && nslot > 0)
                launch_p_convert_down(s, static_cast<int64_t>(n * nslot), c->a_ns_val,
                                      c->a_ns_val32);
            c->smoother_valid = true;
            c->smoother32_valid = fp32;
        }
    } else {
        if (!c->smoother_t_valid || (fp32 && !c->smoother32_t_valid)) {
            if (dev_alloc(&c->dinv_jac_t, n) || dev_alloc(&c->dinv_l1_t, n)) return MSRSB_E_NOMEM;
            if (fp32 && (dev_alloc(&c->dinv_jac32_t, n) || dev_alloc(&c->dinv_l1_32_t, n) ||
                         (noff == 0 && dev_alloc(&c->at32, static_cast<size_t>(c->nnz)))))
                return MSRSB_E_NOMEM;
            if (fp32 && noff > 0 && dev_alloc(&c->at_dia32, n * noff)) return MSRSB_E_NOMEM;
            launch_diag_inverses(s, c->n, c->at_rp, c->at_ci, c->at, c->at_off, c->at_dia,
                                 NodeStencil(), nullptr, c->dinv_jac_t, c->dinv_l1_t,
                                 fp32 ? c->dinv_jac32_t : nullptr,
                                 fp32 ? c->dinv_l1_32_t : nullptr,
                                 fp32 && noff == 0 ? c->at32 : nullptr, c->dev_flag);
            if (fp32 && noff > 0)
                launch_p_convert_down(s, static_cast<int64_t>(n) * noff, c->at_dia, c->at_dia32);
            c->smoother_t_valid = true;
            c->smoother32_t_valid = fp32;
        }
    }
    if (need_tri) {
        const int ord = o->ordering;
        msrsb_status st;
        try {
            st = tri_order_setup(c, ord);
        } catch (const std::bad_alloc &) {
            free_tri_order(c->tri[ord]);
            st = MSRSB_E_NOMEM;
        }
        if (st) {
            c->err = "sweep order set-up failed";
            return st;
        }
        for (int k : kinds) {
            if (k == MSRSB_SMOOTH_IC0 &&
                (!c->a_symmetric || c->made_symmetric || !c->tri[ord].sym_pattern)) {
                c->err = "IC(0) needs a symmetric matrix";
                return MSRSB_E_ARG;
            }
            bool &ok = k == MSRSB_SMOOTH_ILU0 ? c->ilu_ok[ord] : c->ic_ok[ord];
            if ((k != MSRSB_SMOOTH_ILU0 && k != MSRSB_SMOOTH_IC0) || ok) continue;
            st = tri_factor(c, ord, k);
            if (st) {
                c->err = st == MSRSB_E_BREAKDOWN
                             ? (k == MSRSB_SMOOTH_ILU0 ? "zero pivot in ILU(0)"
                                                       : "non-positive pivot in IC(0)")
                             : "smoother factorisation failed";
                return st;
            }
            ok = true;
        }
    }
    return MSRSB_OK;
}

// z = B v (Alg. 4): z = 0; pre-smoothing; z += P M_c^{-1} R (v - A z);
// post-smoothing.  With trans the preconditioner of A^T is applied: A^T, the
// smoothers of A^T, pre and post exchanged, and A_c^{-T}.  With dots (inside
// PCG) the partials of r.z and r.(z - zold) are formed as well, in the last
// sweep when possible, and left to the next direction, or to the one-block
// kernel that forms beta.
// wc = A_c^{-1} vc (A_c^{-T} for trans): the SPD path's symmetric inverse
// from its packed lower tiles, otherwise the dense product
static void coarse_apply(msrsb_ctx *c, bool trans, const ApplyBufs &b)
{
    if (c->child) {  // multilevel: w_c = B_next v_c (the next level's workspace)
        apply_two_stage(c->child, &c->child_opts, b.vc, b.wc, trans, nullptr);
        return;
    }
    if (c->acinv_sym)
        launch_symv_packed(c->stream, c->nc, c->acinv_pk, b.vc, b.wc, c->symv_part);
    else
        launch_gemv(c->stream, c->nc, c->acinv, b.vc, b.wc, trans, b.part);
}

ApplyBufs ctx_apply_bufs(msrsb_ctx *c)
{
    ApplyBufs b;
    b.z = c->w[8];
    b.spare = c->w[9];
    b.tmp = c->w[10];
    for (int k = 0; k < 3; ++k) b.f[k] = c->wf[k];
    b.vc = c->vc;
    b.wc = c->wc;
    b.part = c->partials;
    return b;
}

// The FP64 prolongation reads P's split form while it holds the current P
// (fewer bytes: the zero slots of rows with fewer than 8 entries are not
// stored).  The FP32 one keeps the padded rows, which it reads as fast.
// prolong_p64 / prolong_p32 return the matching values.
static bool prolong_split(const msrsb_ctx *c)
{
    return c->paxes && c->ps_valid && c->pw == 8 && !c->p_is32;
}
static ProlongAxes prolong_axes(const msrsb_ctx *c)
{
    ProlongAxes a;
    if (c->paxes) {
        a.tab = c->paxes;
        a.nx = c->tdims[0];
        a.ny = c->tdims[1];
        a.ncx = c->pax_ncx;
        a.ncxy = c->pax_ncxy;
        if (prolong_split(c)) {
            a.wtab = c->psplit_wtab;
            a.n8 = c->psplit.n8;
        }
    }
    return a;
}
static const double *prolong_p64(const msrsb_ctx *c)
{
    return prolong_split(c) ? c->ps64[c->pcur] : c->p64[c->pcur];
}
static const float *prolong_p32(const msrsb_ctx *c)
{
    return c->p32[c->pcur];
}

static RestrictBoxes restrict_boxes(const msrsb_ctx *c)
{
    RestrictBoxes b;
    b.maxlen = c->rmaxlen;
    if (c->rbox) {
        b.box = c->rbox;
        b.nx = c->tdims[0];
        b.nxy = c->tdims[0] * c->tdims[1];
    }
    return b;
}

void apply_two_stage(msrsb_ctx *c, const msrsb_solve_opts *o, const double *v, double *zout,
                     bool trans, PcgDots *dots, const UpdArgs *upd, const ApplyBufs *bufs)
{
    const ApplyBufs b = bufs ? *bufs : ctx_apply_bufs(c);
    hipStream_t s = c->stream;
    const int n = c->n;
    const Op op = fine_op(c, trans);
    const bool fp32 = o->fp32_smoother != 0;
    int pre_k = o->pre_smoother, pre_n = o->pre_sweeps;
    int post_k = o->post_smoother, post_n = o->post_sweeps;
    if (trans) {
        std::swap(pre_k, post_k);
        std::swap(pre_n, post_n);
    }
    if (pre_k == MSRSB_SMOOTH_NONE) pre_n = 0;
    if (post_k == MSRSB_SMOOTH_NONE) post_n = 0;
    // the stages after the coarse solve, and the update with two pre-sweeps and
    // their residual, in one launch each, inside PCG on a 2D grid.  In FP64 they
    // are faster from 64 x 64 (18.5 us an iteration, 23.9 without the one and 20.4
    // without the other) to 2000 x 2000 (288 us, 309 and 303) and on long narrow
    // grids; in FP32 not on large grids whose tiles are half empty (30 x 33,334:
    // 74 us, 72 without the first; 1000 x 1000: 64.7, 70.7 and 69.8).
    bool grid2d = dots && o->use_multiscale && c->a_grid_nx > 0 && op.d.n == c->a_off.n &&
                  (!fp32 || n <= 200000 ||
                   2 * static_cast<int64_t>(tile_pre_groups(n, c->a_grid_nx)) * kTileCells <=
                       3 * static_cast<int64_t>(n));
    for (int k = 0; grid2d && k < op.d.n; ++k) grid2d = op.d.off[k] == c->a_off.off[k];
    const bool post_tile = grid2d && c->pw == 4 && c->pcol16 && is_diag(post_k) && post_n >= 1 &&
                           post_n <= kPostSweeps;
    const bool pre_tile = grid2d && upd && is_diag(pre_k) && pre_n == 2;
    double *z = b.z, *spare = b.spare, *tmp = b.tmp;
    // the sweeps that exchange z and spare are known beforehand, so the last
    // one can write zout itself (unless v, read until then, lies there).  Where
    // the end of the post-sweeps writes it anyway, z and spare stay the
    // application's own: PCG's two z vectors are a step old, and the memory-side
    // cache has lost them (2.1 M rows: update with two sweeps 36.7 -> 36.1 us,
    // prolongation 28.2 -> 27.5)
    const bool fused_end = dots && is_diag(post_k) && (op.d.n > 0 || op.ns.n > 0) &&
                           post_n > (o->use_multiscale || pre_n > 0 ? 0 : 1);
    if (!fused_end && (zout + n <= v || v + n <= zout)) {
        int swaps = is_diag(post_k) ? post_n : 0;
        if (is_diag(pre_k)) swaps += pre_n - (pre_n >= 2 && op.d.n > 0 ? 2 : 0);
        (swaps & 1 ? spare : z) = zout;
    }
    // precision form inside PCG with two Jacobi-type sweeps on each side of a
    // stencil operator: FP32 intermediate vectors (launch_prec_f32_*)
    const bool f32_path = fp32 && dots && o->use_multiscale && op.d.n > 0 && c->pcol16 &&
                          c->p_is32 && (c->pw == 4 || c->pw == 8) && is_diag(pre_k) &&
                          pre_n == 2 && pre_k == post_k && post_n == 2;
    const bool sweep2 = pre_n >= 2 && is_diag(pre_k) && op.d.n > 0;
    // beta of the products just formed (nb partials each): left to the next
    // direction's kernel when it can add them itself
    auto finish = [&](int nb) {
        dots->sums.dots = dots->part;
        dots->sums.ndots = nb;
        if (nb <= kSumBlocks && !dots->last) return;
        launch_fin_beta(s, dots->sums, dots->last ? dots->post : PostArgs{});
        dots->sums.ndots = 0;
    };
    // the step's post goes with the restriction, or right after the update
    if (dots) {
        const bool tiles = pre_tile && !f32_path;
        dots->post.nrr = tiles ? tile_pre_groups(n, c->a_grid_nx) : (n + kBlock - 1) / kBlock;
    }
    const PostArgs post = dots && !dots->last ? dots->post : PostArgs{};
    if (f32_path) {
        const float *dinv = pre_k == MSRSB_SMOOTH_L1JACOBI ? op.dl132 : op.dj32;
        float *z1 = b.f[0], *z2 = b.f[1], *tf = b.f[2];
        launch_prec_f32_pre(s, n, op.d, op.ad32, dinv, v, z1, tf, c->nc, c->rrp, c->rci,
                            c->roff16, c->rbase, c->r32, b.vc, restrict_boxes(c), upd, post);
        coarse_apply(c, trans, b);
        finish(launch_prec_f32_post(s, n, op.d, op.ad32, dinv, v, z1, z2, c->pw, c->pcol16,
                                    prolong_p32(c), b.wc, zout, dots->zold, dots->part,
                                    prolong_axes(c)));
        return;
    }
    bool zero = true;
    int t = 0;
    // the PCG update that produces v: inside the first two-sweep kernel, with
    // the first Jacobi-type sweep from zero, or on its own
    if (upd && !sweep2) {
        if (pre_n > 0 && is_diag(pre_k)) {
            const bool l1 = pre_k == MSRSB_SMOOTH_L1JACOBI;
            launch_pcg_update(s, n, *upd, spare, l1 ? op.dl1 : op.dj,
                              fp32 ? (l1 ? op.dl132 : op.dj32) : nullptr);
            std::swap(z, spare);
            zero = false;
            t = 1;
        } else {
            launch_pcg_update(s, n, *upd);
        }
    }
    if (pre_tile) {
        const bool l1 = pre_k == MSRSB_SMOOTH_L1JACOBI;
        launch_tile_pre(s, n, op.d, op.ad, fp32 ? op.ad32 : nullptr, l1 ? op.dl1 : op.dj,
                        l1 ? op.dl132 : op.dj32, c->a_grid_nx, z, tmp, *upd);
        zero = false;
        t = 2;
    } else if (sweep2) {
        const bool l1 = pre_k == MSRSB_SMOOTH_L1JACOBI;
        launch_dia_sweep(s, n, op.d, fp32, op.ad, op.ad32, l1 ? op.dl1 : op.dj,
                         l1 ? op.dl132 : op.dj32, v, nullptr, z, true, upd);
        zero = false;
        t = 2;
    }
    if (post.host_out && !o->use_multiscale) launch_post(s, post);
    for (; t < pre_n; ++t) {
        sweep(c, op, pre_k, fp32, v, &z, &spare, zero, tmp, o->ordering);
        zero = false;
    }
    if (o->use_multiscale) {
        const double *res = v;
        if (!zero) {
            if (!pre_tile) op_residual(s, n, op, v, z, tmp, fp32);
            res = tmp;
        }
        launch_restrict(s, c->nc, c->rrp, c->rci, c->roff16, c->rbase, c->p_is32, c->r64, c->r32,
                        res, b.vc, restrict_boxes(c), post);
        coarse_apply(c, trans, b);
        if (post_tile) {
            // (z is not zout, whose neighbouring rows it would still read)
            const bool l1 = post_k == MSRSB_SMOOTH_L1JACOBI;
            finish(launch_tile_post(s, n, op.d, op.ad, fp32 ? op.ad32 : nullptr,
                                    l1 ? op.dl1 : op.dj, l1 ? op.dl132 : op.dj32, v,
                                    zero ? nullptr : z, c->p64[c->pcur],
                                    c->p_is32 ? c->p32[c->pcur] : nullptr, c->pcol16, b.wc,
                                    c->a_grid_nx, post_n, zout, dots->zold, dots->part));
            return;
        }
        launch_prolong_ell(s, n, c->pw, c->pcol_ell, c->pcol16, c->p_is32, prolong_p64(c),
                           prolong_p32(c),
                           b.wc, z, zero, prolong_axes(c));
        zero = false;
    }
    for (t = 0; t < post_n; ++t) {
        const bool last = t == post_n - 1;
        if (last && dots && is_diag(post_k) && op.d.n > 0 && !zero) {
            const bool l1 = post_k == MSRSB_SMOOTH_L1JACOBI;
            finish(launch_dia_sweep_dots(s, n, op.d, fp32, op.ad, op.ad32, l1 ? op.dl1 : op.dj,
                                         l1 ? op.dl132 : op.dj32, v, z, zout, dots->zold,
                                         dots->part));
            return;
        }
        if (last && dots && is_diag(post_k) && op.ns.n > 0 && !zero) {
            const bool l1 = post_k == MSRSB_SMOOTH_L1JACOBI;
            finish(launch_nbs_sweep_dots(s, n, op.ns, fp32, op.nv, op.nv32, l1 ? op.dl1 : op.dj,
                                         l1 ? op.dl132 : op.dj32, v, z, zout, dots->zold,
                                         dots->part));
            return;
        }
        sweep(c, op, post_k, fp32, v, &z, &spare, zero, tmp, o->ordering);
        zero = false;
    }
    if (zero)
        launch_fill(s, n, zout, 0.0);
    else if (z != zout)
        launch_copy(s, n, z, zout);
    if (dots) finish(launch_dots(s, n, v, zout, dots->zold, dots->part));
}

// Wait until the mailbox mb (two values, the step's tag and the word of all
// three, see post_mail) holds the post tagged `tag`; val receives the values.
// Only plain reads of pinned memory while the device works: a
// stream query puts a marker into the stream, and the barrier behind it
// leaves the device idle for several microseconds.  After a second without
// the post the stream is queried, and if it has finished or failed without
// the post arriving the wait reports failure instead of spinning on.  One
// Krylov step takes milliseconds at most, so a post still missing after
// kMailboxDeadline means the device is stuck: the wait gives up with an
// error rather than holding the host forever.
constexpr auto kMailboxDeadline = std::chrono::seconds(120);

static bool wait_mailbox(hipStream_t s, volatile double *mb, int tag, double (&val)[2])
{
    const double want = tag;
    auto arrived = [&] {
        if (mb[2] != want) return false;
        val[0] = mb[0];
        val[1] = mb[1];
        const unsigned long long w = *reinterpret_cast<volatile unsigned long long *>(mb + 3);
        return w == mail_word(val[0], val[1], want);
    };
    const auto start = std::chrono::steady_clock::now();
    auto t0 = start;
    for (unsigned spin = 1;; ++spin) {
        if (arrived()) return true;
        if ((spin & 0xFFFFu) == 0 &&
            std::chrono::steady_clock::now() - t0 > std::chrono::seconds(1)) {
            if (hipStreamQuery(s) != hipErrorNotReady) return arrived();
            t0 = std::chrono::steady_clock::now();
            if (t0 - start > kMailboxDeadline) return false;
        }
    }
}

static msrsb_status read_scalars(msrsb_ctx *c, int first, int count)
{
    hipMemcpyAsync(c->h_pinned, c->scal + first, count * sizeof(double), hipMemcpyDeviceToHost,
                   c->stream);
    return hipStreamSynchronize(c->stream) == hipSuccess ? MSRSB_OK : MSRSB_E_HIP;
}

// Whether PCG runs in one work-group (k_small.hip): a stencil operator with
// Jacobi-type sweeps in FP64 and a coarse stage that is symmetric and dense,
// up to the sizes at which that is faster (both sides' times stand there).
static bool pcg_fits_small(const msrsb_ctx *c, const Op &op, const msrsb_solve_opts *o)
{
    auto diag = [](int k, int sweeps) {
        return sweeps == 0 || k == MSRSB_SMOOTH_NONE || is_diag(k);
    };
    return op.d.n > 0 && op.d.n <= kSmallDiags && c->n <= kSmallRows && !o->fp32_smoother &&
           diag(o->pre_smoother, o->pre_sweeps) && diag(o->post_smoother, o->post_sweeps) &&
           (!o->use_multiscale ||
            (!c->child && c->acinv_sym && c->nc <= kSmallCoarse && !c->p_is32 && c->pcol16 &&
             (c->pw == 4 || c->pw == 8)));
}

static msrsb_status pcg_small(msrsb_ctx *c, const Op &op, const double *f, double *x,
                              const msrsb_solve_opts *o, msrsb_solve_info *info, bool trans)
{
    hipStream_t s = c->stream;
    SmallPcg a{};
    a.n = c->n;
    a.nd = op.d.n;
    for (int k = 0; k < a.nd; ++k) a.off[k] = op.d.off[k];
    a.ad = op.ad;
    auto dinv = [&](int k) { return k == MSRSB_SMOOTH_L1JACOBI ? op.dl1 : op.dj; };
    a.npre = is_diag(o->pre_smoother) ? o->pre_sweeps : 0;
    a.npost = is_diag(o->post_smoother) ? o->post_sweeps : 0;
    a.dpre = dinv(o->pre_smoother);
    a.dpost = dinv(o->post_smoother);
    if (trans) {
        std::swap(a.npre, a.npost);
        std::swap(a.dpre, a.dpost);
    }
    a.coarse = o->use_multiscale != 0;
    if (a.coarse) {
        a.nc = c->nc;
        a.p = c->p64[c->pcur];
        a.pc = c->pcol16;
        a.rrp = c->rrp;
        a.rc = c->rci;
        a.rv = c->r64;
        a.inv = c->acinv_pk;
    }
    a.f = f;
    a.x = x;
    for (int k = 0; k < 3; ++k) a.state[k] = c->w[k];
    a.out = c->scal;
    a.hist = c->partials;
    a.rtol = o->rtol;
    a.max_iter = o->max_iter;
    a.steps = kSmallSteps;
    a.fresh = true;
    double *hist = info ? info->history : nullptr;
    const int hcap = info ? info->history_cap : 0;
    for (;;) {
        launch_pcg_small(s, a, a.coarse ? c->pw : 4);
        if (read_scalars(c, 0, 6)) return MSRSB_E_HIP;
        const double *out = c->h_pinned;
        const int code = static_cast<int>(out[0]), it = static_cast<int>(out[1]);
        const double fn = out[2] == 0.0 ? 1.0 : std::sqrt(out[2]);
        const int m = hist ? std::min(it + 1, hcap) - a.it0 : 0;
        if (m > 0) {
            // (each step's entry, the last one's not yet where more follow)
            hipMemcpyAsync(hist + a.it0, a.hist, m * sizeof(double), hipMemcpyDeviceToHost, s);
            if (hipStreamSynchronize(s) != hipSuccess) return MSRSB_E_HIP;
            for (int k = 0; k < m; ++k) hist[a.it0 + k] = std::sqrt(hist[a.it0 + k]) / fn;
        }
        if (code == kSmallMore) {
            a.it0 = it;
            a.ff = out[2];
            a.rz = out[4];
            a.bad_alpha = out[5] != 0.0;
            a.fresh = false;
            continue;
        }
        if (info) {
            info->iters = it;
            info->true_rel_res = std::sqrt(out[3]) / fn;
        }
        return code == kSmallDone      ? MSRSB_OK
               : code == kSmallMaxIter ? MSRSB_E_NOT_CONVERGED
                                       : MSRSB_E_BREAKDOWN;
    }
}

// Preconditioned CG with flexible beta.  f, x device pointers (x = x0 on entry).
// r.r of iteration k is posted by the restriction of its preconditioner, and
// the host queues iteration k+1 while the rest of iteration k (the coarse
// solve, the post-sweeps and the next direction, 15 us and more) still runs,
// so the device never waits for the host.
msrsb_status pcg(msrsb_ctx *c, const double *f, double *x, const msrsb_solve_opts *o,
                 msrsb_solve_info *info, bool trans)
{
    hipStream_t s = c->stream;
    const int n = c->n;
    const Op op = fine_op(c, trans);
    if (pcg_fits_small(c, op, o)) return pcg_small(c, op, f, x, o, info, trans);
    // r and p each alternate between two buffers: the kernels that update
    // them read the old values at neighbouring rows
    double *r = c->w[0], *z = c->w[1], *zold = c->w[2], *p = c->w[3], *q = c->w[4],
           *p2 = c->w[7], *r2 = c->w[12];
    double *sc = c->scal;
    launch_fill(s, S_COUNT, sc, 0.0);
    launch_dot(s, n, f, f, c->partials, sc + S_FF);
    if (read_scalars(c, S_FF, 1)) return MSRSB_E_HIP;
    double fn = std::sqrt(c->h_pinned[0]);
    if (fn == 0.0) fn = 1.0;
    const double thr2 = (o->rtol * fn) * (o->rtol * fn);
    int it = 0;
    msrsb_status rc = MSRSB_E_NOT_CONVERGED;
    bool restart = true, queued = false;
    double *hist = info ? info->history : nullptr;
    const int hcap = info ? info->history_cap : 0;
    // r.r, the breakdown flag and the iteration tag, posted by the device
    volatile double *hmon = c->h_pinned + 8;
    hmon[2] = -1.0;
    // r.z of step k in scal, and the partials of p.q behind those of the dots
    auto rz = [](int k) { return S_RZ_SLOT + (k & 1); };
    double *pq = c->partials + pq_offset(static_cast<size_t>(n));
    int npq = 0;
    PcgDots dots{};
    dots.part = c->partials;
    dots.sums.scal = sc;
    dots.post.rr = c->partials_rr;
    dots.post.scal = sc;
    dots.post.host_out = c->h_pinned + 8;
    while (it <= o->max_iter) {
        if (restart) {
            op_residual(s, n, op, f, x, r);
            launch_dot(s, n, r, r, c->partials, sc + S_RR);
            if (read_scalars(c, S_RR, 1)) { rc = MSRSB_E_HIP; break; }
            const double rr = c->h_pinned[0];
            if (hist && it < hcap) hist[it] = std::sqrt(rr) / fn;
            if (!std::isfinite(rr)) { rc = MSRSB_E_BREAKDOWN; break; }
            if (rr <= thr2) { rc = MSRSB_OK; break; }
            if (it == o->max_iter) break;
            apply_two_stage(c, o, r, z, trans, nullptr);
            launch_dot(s, n, r, z, c->partials, sc + rz(it));
            launch_fill(s, 1, sc + S_BETA, 0.0);   // p = z
            launch_fill(s, 2, sc + S_BREAK, 0.0);  // a queued-ahead step may have set them
            restart = false;
            queued = false;
        }
        if (!queued) {
            PcgSums first;
            first.scal = sc;
            first.rz_new = rz(it);
            first.tag = it;
            npq = p_spmv(s, n, op, z, p, p2, q, pq, first);
            std::swap(p, p2);
        }
        ++it;
        // x += alpha p and r2 = r - alpha q (inside the preconditioner's first
        // kernel where it can be), the next preconditioner application and
        // the next step's p = z + beta p, q = A p, all queued while the host
        // waits for r.r (the last two touch neither x nor r, so their work is
        // merely dropped if this step turns out to be the last)
        const UpdArgs upd{x, r, p, q, r2, c->partials_rr, sc, pq, npq, rz(it - 1),
                          static_cast<double>(it)};
        std::swap(r, r2);
        std::swap(z, zold);
        queued = it < o->max_iter;
        dots.zold = zold;
        dots.last = !queued;
        dots.sums.tag = dots.post.tag = it;
        dots.sums.rz_old = rz(it - 1);
        dots.sums.rz_new = rz(it);
        apply_two_stage(c, o, r, z, trans, &dots, &upd);
        if (queued) {
            npq = p_spmv(s, n, op, z, p, p2, q, pq, dots.sums);
            std::swap(p, p2);
        }
        double mail[2];
        if (!wait_mailbox(s, hmon, it, mail)) {
            c->err = "the device did not report the residual of a Krylov step";
            return MSRSB_E_HIP;
        }
        const double rr = mail[0];
        // the step that broke down: this one, or the last one's beta
        const int brk = static_cast<int>(mail[1]);
        if (brk != 0 && brk < it) {
            it = brk;
            rc = MSRSB_E_BREAKDOWN;
            break;
        }
        if (hist && it < hcap) hist[it] = std::sqrt(rr) / fn;
        if (brk != 0 || !std::isfinite(rr)) { rc = MSRSB_E_BREAKDOWN; break; }
        if (rr <= thr2) { restart = true; continue; }
        if (it >= o->max_iter) break;
    }
    // true residual at exit
    op_residual(s, n, op, f, x, r);
    launch_dot(s, n, r, r, c->partials, sc + S_TMP0);
    if (read_scalars(c, S_TMP0, 1)) return MSRSB_E_HIP;
    if (info) {
        info->iters = it;
        info->true_rel_res = std::sqrt(c->h_pinned[0]) / fn;
    }
    return rc;
}

// Right-preconditioned GMRES(m) with classical Gram-Schmidt applied twice.
msrsb_status gmres(msrsb_ctx *c, const double *f, double *x, const msrsb_solve_opts *o,
                   msrsb_solve_info *info, bool trans)
{
    hipStream_t s = c->stream;
    const int n = c->n;
    const int m = std::max(1, std::min(o->restart, 64));
    const Op op = fine_op(c, trans);
    // the basis vectors' stride: whole 256-byte blocks, an odd number of them,
    // so that the same rows of all vectors spread over the memory channels and
    // cache sets (at 65,536 rows a stride of 512 KB put them all in one set:
    // 18 us per pass over 31 vectors)
    const int64_t ldv = ((n + 31) / 32 | 1) * static_cast<int64_t>(32);
    if (c->gm_cap < m) {
        if (c->gm_v) hipFree(c->gm_v);
        if (c->gm_h) hipFree(c->gm_h);
        c->gm_v = c->gm_h = nullptr;
        if (dev_alloc(&c->gm_v, static_cast<size_t>(m + 1) * ldv) ||
            dev_alloc(&c->gm_h, static_cast<size_t>(m + 1) * m + 8 * (m + 2) +
                                    2 * kOrthoCols * kOrthoBlocks))
            return MSRSB_E_NOMEM;
        c->gm_cap = m;
    }
    double *V = c->gm_v;
    double *H = c->gm_h;                        // (m+1) x m
    double *cs = H + (m + 1) * m, *sn = cs + (m + 2), *g = sn + (m + 2), *y = g + (m + 2);
    double *hc = y + (m + 2), *h2 = hc + (m + 2), *gsc = h2 + (m + 2);  // gsc: 2 scalars
    // partial sums of the orthogonalisation: two arrays in turn
    double *part[2] = {gsc + (m + 2), gsc + (m + 2) + kOrthoCols * kOrthoBlocks};
    double *w = c->w[0], *zt = c->w[1], *r = c->w[2];
    double *sc = c->scal;
    // two mailbox slots in coherent pinned memory (steps alternate).  The tags
    // number the steps queued in all cycles: a cycle that ends early leaves the
    // post of the step queued ahead, which is no step of the next cycle
    volatile double *mbox[2] = {c->h_pinned + 16, c->h_pinned + 24};
    mbox[0][2] = mbox[1][2] = -1.0;
    int posts = 0, want[2] = {0, 0};
    launch_dot(s, n, f, f, c->partials, sc + S_FF);
    if (read_scalars(c, S_FF, 1)) return MSRSB_E_HIP;
    double fn = std::sqrt(c->h_pinned[0]);
    if (fn == 0.0) fn = 1.0;
    int it = 0;
    msrsb_status rc = MSRSB_E_NOT_CONVERGED;
    double *hist = info ? info->history : nullptr;
    const int hcap = info ? info->history_cap : 0;
    for (;;) {
        op_residual(s, n, op, f, x, r);
        launch_dot(s, n, r, r, c->partials, sc + S_RR);
        if (read_scalars(c, S_RR, 1)) return MSRSB_E_HIP;
        const double beta = std::sqrt(c->h_pinned[0]);
        if (hist && it < hcap) hist[it] = beta / fn;
        if (!std::isfinite(beta)) { rc = MSRSB_E_BREAKDOWN; break; }
        if (beta <= o->rtol * fn) { rc = MSRSB_OK; break; }
        if (it >= o->max_iter) break;
        launch_norm_scale(s, n, r, V, c->partials, sc + S_RR);
        k_gmres_init_g<<<1, 64, 0, s>>>(m, g, sc + S_RR);
        // one Arnoldi step: v_{j+1} and column j of H, its Givens rotation,
        // and the residual estimate posted to mailbox slot j mod 2
        auto step = [&](int jj) {
            const double *vj = V + jj * ldv;
            double *vn = V + (jj + 1) * ldv;
            apply_two_stage(c, o, vj, zt, trans, nullptr);
            op_spmv(s, n, op, zt, w);
            // CGS2: h = V^T w; w -= V h; h2 = V^T w; w -= V h2; h += h2
            want[jj & 1] = ++posts;
            const GivensArgs ga{jj, m, H, hc, cs, sn, g, gsc, const_cast<double *>(mbox[jj & 1]),
                                static_cast<double>(posts)};
            if (jj < kOrthoCols) {
                ortho(s, n, jj + 1, ldv, V, w, vn, hc, part, ga);
                return;
            }
            launch_multi_dot(s, n, jj + 1, V, ldv, w, c->partials, hc);
            launch_multi_axpy(s, n, jj + 1, V, ldv, hc, w, -1.0);
            launch_multi_dot(s, n, jj + 1, V, ldv, w, c->partials, h2);
            launch_multi_axpy(s, n, jj + 1, V, ldv, h2, w, -1.0);
            k_vec_add<<<1, 64, 0, s>>>(jj + 1, hc, h2);
            launch_norm_scale(s, n, w, vn, c->partials, sc + S_TMP1);
            k_gmres_givens<<<1, 64, 0, s>>>(ga, sc + S_TMP1);
        };
        int j = 0;
        bool brk = false;
        if (it < o->max_iter) step(0);
        for (j = 0; j < m && it < o->max_iter; ++j) {
            // step j + 1 goes into the queue before step j's residual is read,
            // so the device does not wait for the host; it writes only column
            // j + 1 of H, g[j + 1 ..] and v_{j + 2}, none of which the solution
            // after step j uses
            if (j + 1 < m && it + 1 < o->max_iter) step(j + 1);
            double mail[2];
            if (!wait_mailbox(s, mbox[j & 1], want[j & 1], mail)) {
                c->err = "the device did not report the residual of a Krylov step";
                return MSRSB_E_HIP;
            }
            ++it;
            const double res = mail[0], den = mail[1];
            if (hist && it < hcap) hist[it] = res / fn;
            if (!std::isfinite(res) || !(den > 0.0)) { brk = true; break; }
            if (res <= o->rtol * fn) { ++j; break; }
        }
        if (j > 0) {
            k_gmres_solve<<<1, 64, 0, s>>>(j, m, H, g, y);
            launch_fill(s, n, w, 0.0);
            launch_multi_axpy(s, n, j, V, ldv, y, w, 1.0);
            apply_two_stage(c, o, w, zt, trans, nullptr);
            launch_axpy(s, n, 1.0, zt, x);
        }
        if (brk) { rc = MSRSB_E_BREAKDOWN; break; }
    }
    op_residual(s, n, op, f, x, r);
    launch_dot(s, n, r, r, c->partials, sc + S_TMP0);
    if (read_scalars(c, S_TMP0, 1)) return MSRSB_E_HIP;
    const double tr = std::sqrt(c->h_pinned[0]) / fn;
    if (info) {
        info->iters = it;
        info->true_rel_res = tr;
    }
    if (rc == MSRSB_OK && !(tr <= o->rtol)) rc = MSRSB_E_NOT_CONVERGED;
    return rc;
}

// The stand-alone iteration of Sec. 3.2 (Richardson): x += B (f - A x) until
// the true residual meets the tolerance; iterations count applications of B.
msrsb_status richardson(msrsb_ctx *c, const double *f, double *x, const msrsb_solve_opts *o,
                        msrsb_solve_info *info, bool trans)
{
    hipStream_t s = c->stream;
    const int n = c->n;
    const Op op = fine_op(c, trans);
    double *r = c->w[0], *z = c->w[1];
    double *sc = c->scal;
    launch_dot(s, n, f, f, c->partials, sc + S_FF);
    if (read_scalars(c, S_FF, 1)) return MSRSB_E_HIP;
    double fn = std::sqrt(c->h_pinned[0]);
    if (fn == 0.0) fn = 1.0;
    double *hist = info ? info->history : nullptr;
    const int hcap = info ? info->history_cap : 0;
    int it = 0;
    double rel = 0.0;
    msrsb_status rc = MSRSB_E_NOT_CONVERGED;
    for (;;) {
        op_residual(s, n, op, f, x, r);
        launch_dot(s, n, r, r, c->partials, sc + S_RR);
        if (read_scalars(c, S_RR, 1)) return MSRSB_E_HIP;
        rel = std::sqrt(c->h_pinned[0]) / fn;
        if (hist && it < hcap) hist[it] = rel;
        if (!std::isfinite(rel)) { rc = MSRSB_E_BREAKDOWN; break; }
        if (rel <= o->rtol) { rc = MSRSB_OK; break; }
        if (it >= o->max_iter) break;
        apply_two_stage(c, o, r, z, trans, nullptr);
        launch_axpy(s, n, 1.0, z, x);
        ++it;
    }
    if (info) {
        info->iters = it;
        info->true_rel_res = rel;
    }
    return rc;
}

// Right-preconditioned BiCGStab (two applications of B per iteration,
// Sec. 4.1).  Scalars are read back on the host after each product; a pass
// that meets the tolerance after its first half ends there.  Convergence of
// the recursive residual is confirmed on the true residual, and the method
// starts again from x if that is still above the tolerance.  Breakdown:
// |rhat^T r| <= 1e-14 ||rhat|| ||r|| (an exact zero is hidden by rounding),
// or rhat^T v or t^T t zero.
msrsb_status bicgstab(msrsb_ctx *c, const double *f, double *x, const msrsb_solve_opts *o,
                      msrsb_solve_info *info, bool trans)
{
    hipStream_t s = c->stream;
    const int n = c->n;
    const Op op = fine_op(c, trans);
    // (w[5] and w[6] hold f and x of a host-staged solve)
    double *r = c->w[0], *rh = c->w[1], *p = c->w[2], *v = c->w[3], *y = c->w[4],
           *sv = c->w[7], *z = c->w[12], *t = c->w[13];
    double *sc = c->scal;
    auto dot = [&](const double *a, const double *b, double &out) {
        launch_dot(s, n, a, b, c->partials, sc + S_TMP0);
        if (read_scalars(c, S_TMP0, 1)) return false;
        out = c->h_pinned[0];
        return true;
    };
    double ff = 0.0;
    if (!dot(f, f, ff)) return MSRSB_E_HIP;
    double fn = std::sqrt(ff);
    if (fn == 0.0) fn = 1.0;
    double *hist = info ? info->history : nullptr;
    const int hcap = info ? info->history_cap : 0;
    int it = 0;
    msrsb_status rc = MSRSB_E_NOT_CONVERGED;
    bool restart = true;
    double rho = 1.0, alpha = 1.0, omega = 1.0, rhn = 0.0, rn = 0.0;
    while (it <= o->max_iter) {
        if (restart) {
            op_residual(s, n, op, f, x, r);
            double rr = 0.0;
            if (!dot(r, r, rr)) return MSRSB_E_HIP;
            const double rel = std::sqrt(rr) / fn;
            if (hist && it < hcap) hist[it] = rel;
            if (!std::isfinite(rel)) { rc = MSRSB_E_BREAKDOWN; break; }
            if (rel <= o->rtol) { rc = MSRSB_OK; break; }
            if (it >= o->max_iter) break;
            launch_copy(s, n, r, rh);
            launch_copy(s, n, r, p);
            rho = rr;
            rhn = std::sqrt(rr);
            restart = false;
        } else {
            double rho_new = 0.0;
            if (!dot(rh, r, rho_new)) return MSRSB_E_HIP;
            if (!(std::fabs(rho_new) > 1e-14 * rhn * rn)) { rc = MSRSB_E_BREAKDOWN; break; }
            const double beta = (rho_new / rho) * (alpha / omega);
            lincomb(s, n, 1.0, r, beta, p, -beta * omega, v, p);  // p = r + beta (p - omega v)
            rho = rho_new;
        }
        apply_two_stage(c, o, p, y, trans, nullptr);
        op_spmv(s, n, op, y, v);
        double sig = 0.0;
        if (!dot(rh, v, sig)) return MSRSB_E_HIP;
        if (sig == 0.0 || !std::isfinite(sig)) { rc = MSRSB_E_BREAKDOWN; break; }
        alpha = rho / sig;
        lincomb(s, n, 1.0, r, -alpha, v, 0.0, nullptr, sv);  // s = r - alpha v
        ++it;
        double ss = 0.0;
        if (!dot(sv, sv, ss)) return MSRSB_E_HIP;
        if (std::sqrt(ss) <= o->rtol * fn) {
            lincomb(s, n, 1.0, x, alpha, y, 0.0, nullptr, x);
            if (hist && it < hcap) hist[it] = std::sqrt(ss) / fn;
            restart = true;
            continue;
        }
        apply_two_stage(c, o, sv, z, trans, nullptr);
        op_spmv(s, n, op, z, t);
        double tt = 0.0, ts = 0.0;
        if (!dot(t, t, tt) || !dot(t, sv, ts)) return MSRSB_E_HIP;
        if (tt == 0.0 || !std::isfinite(tt)) { rc = MSRSB_E_BREAKDOWN; break; }
        omega = ts / tt;
        lincomb(s, n, 1.0, x, alpha, y, omega, z, x);        // x += alpha y + omega z
        lincomb(s, n, 1.0, sv, -omega, t, 0.0, nullptr, r);  // r = s - omega t
        double rr = 0.0;
        if (!dot(r, r, rr)) return MSRSB_E_HIP;
        rn = std::sqrt(rr);
        const double rel = rn / fn;
        if (hist && it < hcap) hist[it] = rel;
        if (!std::isfinite(rel)) { rc = MSRSB_E_BREAKDOWN; break; }
        if (rel <= o->rtol) { restart = true; continue; }
        if (omega == 0.0) { rc = MSRSB_E_BREAKDOWN; break; }
        if (it >= o->max_iter) break;
    }
    op_residual(s, n, op, f, x, r);
    double rr = 0.0;
    if (!dot(r, r, rr)) return MSRSB_E_HIP;
    if (info) {
        info->iters = it;
        info->true_rel_res = std::sqrt(rr) / fn;
    }
    return rc;
}

}  // namespace msrsb
