// PCG on small stencil problems in one launch: one work-group holds the whole
// iteration, so a step costs work-group barriers and not kernel launches.
//
// A step on a few thousand rows is seven launches of 2 to 4 us each whatever
// the size, of which the reads and the arithmetic are well below one.  Here
// the vectors of the iteration live in registers (thread t has rows t and
// t + T), neighbours are exchanged through two LDS buffers in turn (one
// barrier per product or sweep), and sums go over the wavefront by DPP and
// over the wavefronts through LDS.  With one row per thread (REG) the rows'
// coefficients, P entries and the wavefront's part of R stay in registers as
// well; with two the 128 registers a thread has do not hold them, and they are
// read from the L2 in each product.  Bound by the barriers and the dependent
// latencies between them.  Per step, no pre-sweep and one post-sweep / two and
// two, launches against this kernel:
//   32 x 32, 5 diagonals      20.3 / 28.8 us    4.2 /  6.0 us
//   45 x 45, 5 diagonals      21.2 / 29.1      10.2 / 15.6
//   10 x 10 x 10, 7 diagonals 22.2 / 31.0       6.5 /  9.2
//   12 x 12 x 12, 7 diagonals 22.9 / 32.4      14.1 / 21.5
// Four rows per thread were slower where P is wide (16 x 16 x 16: 24.2 / 34.1
// us against 38.0 / 54.2) and little faster elsewhere (64 x 64: 21.7 / 29.9
// against 17.5 / 27.4), and 256 coarse unknowns cost 20 us more than 64, so
// the line lies at 2048 rows and 64 coarse unknowns.
#include "internal.h"

#include <algorithm>
#include <type_traits>

namespace msrsb {

namespace {

constexpr int kT = kSmallThreads;
constexpr int kR = 6;       // entries of R a lane keeps

template <int CTRL>
__device__ __forceinline__ double dpp_add(double v)
{
    union { double d; int i[2]; } a, b;
    a.d = v;
    b.i[0] = __builtin_amdgcn_update_dpp(0, a.i[0], CTRL, 0xf, 0xf, true);
    b.i[1] = __builtin_amdgcn_update_dpp(0, a.i[1], CTRL, 0xf, 0xf, true);
    return v + b.d;
}
// sum over each 16 lanes, the same bits in all of them
__device__ __forceinline__ double row_sum(double v)
{
    v = dpp_add<0xB1>(v);   // lane ^ 1
    v = dpp_add<0x4E>(v);   // lane ^ 2
    v = dpp_add<0x141>(v);  // the other four of eight
    return dpp_add<0x140>(v);  // the other eight of 16
}
__device__ __forceinline__ double lane_of(double v, int l)
{
    union { double d; int i[2]; } a;
    a.d = v;
    a.i[0] = __builtin_amdgcn_readlane(a.i[0], l);
    a.i[1] = __builtin_amdgcn_readlane(a.i[1], l);
    return a.d;
}
__device__ __forceinline__ double wave_sum(double v)
{
    v = row_sum(v);
    return (lane_of(v, 0) + lane_of(v, 16)) + (lane_of(v, 32) + lane_of(v, 48));
}

// NDT: room for diagonals; PW: width of P's rows; RPT: rows per thread.
template <int NDT, int PW, int RPT>
__global__ __launch_bounds__(kT) void k_pcg_small(SmallPcg a)
{
    constexpr bool REG = RPT == 1;
    extern __shared__ double lds[];
    __shared__ double red[2][3][kT / 64];
    const int n = a.n, T = blockDim.x, t = threadIdx.x, lane = t & 63, w = t >> 6, nw = T >> 6;
    // lds: two exchange buffers, then the coarse vectors
    double *const vc = lds + 2 * n, *const wc = vc + a.nc;
    int cur = 0, phase = 0;
    for (int e = t; e < 6 * (kT / 64); e += T) (&red[0][0][0])[e] = 0.0;  // (absent wavefronts)
    __syncthreads();

    double av[REG ? RPT : 1][NDT], pv[REG ? RPT : 1][PW], dpre[RPT], dpost[RPT];
    unsigned pc[REG ? RPT : 1][PW / 2];
    double x[RPT], r[RPT], z[RPT], p[RPT];
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        const int i = t + k * T;
        const bool in = i < n;
        x[k] = in ? a.x[i] : 0.0;
        dpre[k] = in && a.npre ? a.dpre[i] : 0.0;
        dpost[k] = in && a.npost ? a.dpost[i] : 0.0;
        r[k] = z[k] = p[k] = 0.0;
        if (!a.fresh && in) {
            r[k] = a.state[0][i];
            z[k] = a.state[1][i];
            p[k] = a.state[2][i];
        }
        if constexpr (REG) {
#pragma unroll
            for (int o = 0; o < NDT; ++o) {
                const int q = i + a.off[o];
                av[k][o] = in && o < a.nd && q >= 0 && q < n
                               ? a.ad[static_cast<int64_t>(o) * n + i] : 0.0;
            }
            if (a.coarse) {
#pragma unroll
                for (int s = 0; s < PW; s += 2) {
                    const int64_t e = static_cast<int64_t>(in ? i : 0) * PW + s;
                    unsigned c0 = a.pc[e], c1 = a.pc[e + 1];
                    pv[k][s] = in && c0 != 0xFFFFu ? a.p[e] : 0.0;
                    pv[k][s + 1] = in && c1 != 0xFFFFu ? a.p[e + 1] : 0.0;
                    c0 = c0 == 0xFFFFu ? 0 : c0;
                    c1 = c1 == 0xFFFFu ? 0 : c1;
                    pc[k][s / 2] = c0 | c1 << 16;
                }
            }
        }
    }
    // the first entries of the wavefront's first row of R, and the thread's
    // four of A_c^{-1} where each row has its 16 lanes
    double rv[kR];
    int rc[kR], r0 = 0, r1 = 0;
    double m4[4];
    const bool keep4 = a.coarse && a.nc <= T / 16;
    if (a.coarse) {
        if (w < a.nc) {
            r0 = a.rrp[w];
            r1 = a.rrp[w + 1];
        }
        if constexpr (REG) {
#pragma unroll
            for (int u = 0; u < kR; ++u) {
                const int e = r0 + lane + 64 * u;
                rv[u] = e < r1 ? a.rv[e] : 0.0;
                rc[u] = e < r1 ? a.rc[e] : 0;
            }
        }
        if (keep4) {
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                m4[b] = a.inv[min(t >> 4, a.nc - 1) * 64 + 4 * (t & 15) + b];
            }
        }
    }

    // (A y)_i of the thread's k-th row, y in the current exchange buffer; an
    // offset that leaves the rows reads y_i with a zero coefficient
    auto row_dot = [&](int k) {
        int i = t + k * T < n ? t + k * T : 0;
        asm volatile("" : "+v"(i));  // (addresses are formed anew, not kept)
        const double *y = lds + cur;
        double s = 0.0;
#pragma unroll
        for (int o = 0; o < NDT; ++o) {
            if (!REG && o >= a.nd) break;
            const int q = i + a.off[o];
            const bool in = q >= 0 && q < n;
            double c;
            if constexpr (REG) c = av[k][o];
            else c = in ? a.ad[o * n + i] : 0.0;
            s += c * y[in ? q : i];
        }
        return s;
    };
    auto put = [&](const double (&v)[RPT]) {
        cur = n - cur;
#pragma unroll
        for (int k = 0; k < RPT; ++k)
            if (t + k * T < n) lds[cur + t + k * T] = v[k];
        __syncthreads();
    };
    auto sums = [&](auto &v) {  // v: the threads' parts, then the totals
        constexpr int NV = sizeof(v) / sizeof(double);
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const double s = wave_sum(v[q]);
            if (lane == 0) red[phase][q][w] = s;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] = row_sum(red[phase][q][lane & (kT / 64 - 1)]);
        phase ^= 1;
    };

    double ff = a.ff;
    if (a.fresh) {
        double s[1] = {0.0};
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            const double fk = t + k * T < n ? a.f[t + k * T] : 0.0;
            s[0] += fk * fk;
        }
        sums(s);
        ff = s[0];
    }
    const double fn = ff == 0.0 ? 1.0 : sqrt(ff);
    const double thr2 = (a.rtol * fn) * (a.rtol * fn);
    auto residual = [&]() {  // r = f - A x, returns r.r
        put(x);
        double s[1] = {0.0};
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            r[k] = t + k * T < n ? a.f[t + k * T] - row_dot(k) : 0.0;
            s[0] += r[k] * r[k];
        }
        sums(s);
        return s[0];
    };

    int it = a.it0, code = kSmallMaxIter;
    bool restart = a.fresh, leave = false, bad_alpha = a.bad_alpha;
    double rz = a.rz, rr = 0.0;
    for (;;) {
        if (restart || leave) {
            rr = residual();
            if (leave) break;  // the true residual at exit
            if (t == 0) a.hist[it - a.it0] = rr;
            if (!isfinite(rr)) { code = kSmallBreakdown; break; }
            if (rr <= thr2) { code = kSmallDone; break; }
            if (it >= a.max_iter) break;
        } else if (it - a.it0 == a.steps) {
            code = kSmallMore;
            break;
        }
        double zold[RPT];
#pragma unroll
        for (int k = 0; k < RPT; ++k) zold[k] = z[k];
        // z = B r
        bool zero = true;
        for (int s = 0; s < a.npre; ++s) {
            if (!zero) put(z);
#pragma unroll
            for (int k = 0; k < RPT; ++k)
                z[k] = zero ? dpre[k] * r[k] : z[k] + dpre[k] * (r[k] - row_dot(k));
            zero = false;
        }
        if (a.coarse) {
            if (zero) {
                put(r);
            } else {
                put(z);
                double res[RPT];
#pragma unroll
                for (int k = 0; k < RPT; ++k) res[k] = r[k] - row_dot(k);
                put(res);
            }
            const double *y = lds + cur;
            for (int j = w; j < a.nc; j += nw) {
                const int e0 = j == w ? r0 : a.rrp[j], e1 = j == w ? r1 : a.rrp[j + 1];
                double s = 0.0;
                int e = e0 + lane;
                if constexpr (REG) {
                    if (j == w) {
#pragma unroll
                        for (int u = 0; u < kR; ++u) s += rv[u] * y[rc[u]];
                        e += 64 * kR;
                    }
                }
                for (; e + 192 < e1; e += 256) {
                    double g[4], h[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        g[u] = a.rv[e + 64 * u];
                        h[u] = y[a.rc[e + 64 * u]];
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) s += g[u] * h[u];
                }
                for (; e < e1; e += 64) s += a.rv[e] * y[a.rc[e]];
                s = wave_sum(s);
                if (lane == 0) vc[j] = s;
            }
            __syncthreads();
            // A_c^{-1} (its one tile, zero past nc), 16 lanes to a row
            const int h = t & 15;
            for (int j = t >> 4; j < a.nc; j += T >> 4) {
                double s = 0.0;
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    s += (keep4 ? m4[b] : a.inv[j * 64 + 4 * h + b]) * vc[min(4 * h + b, a.nc - 1)];
                s = row_sum(s);
                if (h == 0) wc[j] = s;
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < RPT; ++k) {
                double s = 0.0;
                int i = t + k * T < n ? t + k * T : 0;
                asm volatile("" : "+v"(i));
#pragma unroll
                for (int q = 0; q < PW; ++q) {
                    if constexpr (REG) {
                        s += pv[k][q] * wc[(pc[k][q / 2] >> (16 * (q & 1))) & 0xFFFFu];
                    } else {
                        const unsigned c = a.pc[i * PW + q];
                        const double v = a.p[i * PW + q];
                        s += c != 0xFFFFu ? v * wc[c] : 0.0;
                    }
                }
                z[k] = zero ? s : z[k] + s;
            }
            zero = false;
        }
        for (int s = 0; s < a.npost; ++s) {
            if (!zero) put(z);
#pragma unroll
            for (int k = 0; k < RPT; ++k)
                z[k] = zero ? dpost[k] * r[k] : z[k] + dpost[k] * (r[k] - row_dot(k));
            zero = false;
        }
        double d[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            const bool in = t + k * T < n;
            z[k] = zero || !in ? 0.0 : z[k];
            d[0] += r[k] * z[k];
            d[1] += r[k] * (z[k] - zold[k]);
            d[2] += r[k] * r[k];
        }
        sums(d);
        double beta = 0.0;
        if (!restart) {
            // (r.r of the step, known only here: its sum goes with the others')
            if (t == 0) a.hist[it - a.it0] = d[2];
            bool bad;
            beta = beta_of(d[1], rz, bad);
            const bool broken = bad_alpha || !isfinite(d[2]);
            restart = !broken && d[2] <= thr2;
            leave = broken || (!restart && (it >= a.max_iter || bad));
            if (broken || (leave && bad)) code = kSmallBreakdown;
            if (restart || leave) continue;
        }
        restart = false;
        rz = d[0];
#pragma unroll
        for (int k = 0; k < RPT; ++k) p[k] = beta == 0.0 ? z[k] : z[k] + beta * p[k];
        put(p);
        double q[RPT], s[1] = {0.0};
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            q[k] = t + k * T < n ? row_dot(k) : 0.0;
            s[0] += p[k] * q[k];
        }
        sums(s);
        const double alpha = alpha_of(rz, s[0], bad_alpha);
        ++it;
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            x[k] += alpha * p[k];
            r[k] -= alpha * q[k];
        }
    }
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        const int i = t + k * T;
        if (i >= n) continue;
        a.x[i] = x[k];
        if (code == kSmallMore) {
            a.state[0][i] = r[k];
            a.state[1][i] = z[k];
            a.state[2][i] = p[k];
        }
    }
    if (t == 0) {
        a.out[0] = code;
        a.out[1] = it;
        a.out[2] = ff;
        a.out[3] = rr;
        a.out[4] = rz;
        a.out[5] = bad_alpha;
    }
}

// a row of 4 slots, 16 bytes at a time
template <typename T>
__device__ __forceinline__ void load_slots(const T *__restrict__ at, T (&v)[4])
{
    constexpr int L = 16 / sizeof(T);
    typedef T vec __attribute__((ext_vector_type(L)));
#pragma unroll
    for (int q = 0; q < 4 / L; ++q) {
        const vec x = reinterpret_cast<const vec *>(at)[q];
#pragma unroll
        for (int l = 0; l < L; ++l) v[q * L + l] = x[l];
    }
}
template <typename T>
__device__ __forceinline__ void store_slots(T *__restrict__ at, const T (&v)[4])
{
    constexpr int L = 16 / sizeof(T);
    typedef T vec __attribute__((ext_vector_type(L)));
#pragma unroll
    for (int q = 0; q < 4 / L; ++q) {
        vec x;
#pragma unroll
        for (int l = 0; l < L; ++l) x[l] = v[q * L + l];
        reinterpret_cast<vec *>(at)[q] = x;
    }
}

// J's coefficient o of row i (column k, inside the matrix or not; si: the row's
// scale where J is factored)
template <typename T>
__device__ __forceinline__ T smooth_weight(const SmoothArgs &a, const T *__restrict__ jv, int i,
                                           int o, int k, bool inside, T si)
{
    const int mid = a.jw / 2;
    if (a.sym && o == mid) return si == T(0) ? T(1) : static_cast<T>(1.0 - a.omega);
    if (a.sym && o < mid)
        return inside ? si * jv[static_cast<int64_t>(a.jw - 1 - o) * a.n + k] : T(0);
    const T v = jv[static_cast<int64_t>(o) * a.n + i];
    return a.sym ? si * v : v;
}

// Smoothing of P on small problems, all steps in one launch (the arithmetic of
// k_smooth_map, in its order): P lies in LDS, slot-major and with a zero row
// for absent slots, in two buffers in turn; a thread keeps its rows' weights
// and, two to a register, the places of its neighbours' slots.  Bound by the
// LDS reads, one per coefficient and slot, against a launch per step before:
// see smooth_fits_small.
template <typename T, int NDT, int PW, int RPT>
__global__ __launch_bounds__(kT) void k_smooth_small(SmoothArgs a, const T *__restrict__ jv,
                                                     T *__restrict__ p, int steps, int eit_step)
{
    extern __shared__ char lds_raw[];
    __shared__ double red[kT / 64];
    T *const lds = reinterpret_cast<T *>(lds_raw);
    const int n = a.n, W = blockDim.x, t = threadIdx.x, lane = t & 63;
    const int half = (PW + 1) * n;  // one buffer
    const uint8_t *jmap = static_cast<const uint8_t *>(a.jmap_idx);
    T w[RPT][NDT];
    unsigned at[RPT][NDT][PW / 2];
    bool inner[RPT];
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int i = t + q * W;
        const bool in = i < n;
        const T si = in && a.sym ? jv[static_cast<int64_t>(a.jw / 2) * n + i] : T(0);
        inner[q] = in && a.interior[in ? i : 0] != 0;
#pragma unroll
        for (int o = 0; o < NDT; ++o) {
            const bool have = in && o < a.jw;
            const int64_t e = static_cast<int64_t>(o) * n + i;
            const uint32_t m = have ? a.jmap_tab[jmap[e]] : 0xFFFFFFFFu;
            int k = !have ? 0 : a.jcol ? a.jcol[e] : i + a.joff.off[o];
            const bool inside = k >= 0 && k < n;
            w[q][o] = have ? smooth_weight(a, jv, i, o, k, inside, si) : T(0);
            if (!inside) k = in ? i : 0;
#pragma unroll
            for (int s = 0; s < PW; s += 2) {
                const int c0 = min(static_cast<int>(m >> (4 * s) & 0xFu), PW);
                const int c1 = min(static_cast<int>(m >> (4 * s + 4) & 0xFu), PW);
                at[q][o][s / 2] = static_cast<unsigned>(c0 * n + k) |
                                  static_cast<unsigned>(c1 * n + k) << 16;
            }
        }
        if (!in) continue;
#pragma unroll
        for (int s = 0; s < PW; ++s) lds[s * n + i] = p[static_cast<int64_t>(i) * PW + s];
        lds[PW * n + i] = lds[half + PW * n + i] = T(0);
    }
    int cur = 0;
    for (int step = 0; step < steps; ++step) {
        __syncthreads();
        const T *from = lds + cur;
        T *to = lds + (half - cur);
        double emax = 0.0;
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const int i = t + q * W;
            T acc[PW];
#pragma unroll
            for (int s = 0; s < PW; ++s) acc[s] = T(0);
#pragma unroll
            for (int o = 0; o < NDT; ++o) {  // (past a.jw: zeros)
#pragma unroll
                for (int s = 0; s < PW; ++s)
                    acc[s] += w[q][o] * from[at[q][o][s / 2] >> (16 * (s & 1)) & 0xFFFFu];
            }
            if (i >= n) continue;
            double rs = 0.0;
#pragma unroll
            for (int s = 0; s < PW; ++s) rs += static_cast<double>(acc[s]);
            const double rinv = 1.0 / rs;
#pragma unroll
            for (int s = 0; s < PW; ++s) {
                if (step == eit_step && inner[q]) {
                    const double dlt = fabs(static_cast<double>(acc[s]) -
                                            static_cast<double>(from[s * n + i]));
                    emax = (dlt > emax || dlt != dlt) ? dlt : emax;
                }
                to[s * n + i] = static_cast<T>(static_cast<double>(acc[s]) * rinv);
            }
        }
        cur = half - cur;
        if (step != eit_step) continue;
        auto larger = [](double x, double y) { return (y > x || y != y) ? y : x; };
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) emax = larger(emax, __shfl_xor(emax, off, 64));
        if (lane == 0) red[t >> 6] = emax;
        __syncthreads();
        if (t == 0) {
            for (int u = 1; u < W >> 6; ++u) emax = larger(emax, red[u]);
            a.eit_out[0] = emax;
        }
    }
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int i = t + q * W;
        if (i >= n) continue;
#pragma unroll
        for (int s = 0; s < PW; ++s) p[static_cast<int64_t>(i) * PW + s] = lds[cur + s * n + i];
    }
}

// Several smoothing steps per launch on a 2D grid (rows x + nx y, couplings to
// the eight neighbours at most, rows of 4 slots): a work-group takes a tile of
// kTile x kTile cells with kHalo more on every side, a cell per thread, and
// each step is right one cell further from the edge less, so that after kHalo
// steps the tile itself still is.  Held as in k_smooth_small; the halo costs
// 1.8 times the arithmetic and saves three of four launches and of four
// passes over P, J and the maps.
// Bound by the launch and the LDS reads.  A step in FP64, before and now:
// 250 x 187, five neighbours 4.7 -> 2.1 us; 256 x 256, nine 6.9 -> 3.3 us;
// 100 x 100, nine 6.5 -> 3.1 us.
constexpr int kHalo = 4, kTile = 32 - 2 * kHalo;
template <typename T, int ND>
__global__ __launch_bounds__(kT) void k_smooth_tile(SmoothArgs a, const T *__restrict__ jv,
                                                    const T *__restrict__ pin,
                                                    T *__restrict__ pout, int nx, int ny, int ntx,
                                                    int steps, int eit_step)
{
    constexpr int PW = 4, ZERO = PW * kT;  // one buffer: slot-major, then a zero
    __shared__ T lds[2][ZERO + 1];
    __shared__ double red[kT / 64];
    const int n = a.n, t = threadIdx.x, tx = t & 31, ty = t >> 5;
    const int b = xcd_group(blockIdx.x, gridDim.x);
    const int x = b % ntx * kTile - kHalo + tx, y = b / ntx * kTile - kHalo + ty;
    const bool in = x >= 0 && x < nx && y >= 0 && y < ny;
    const int i = in ? x + nx * y : 0;
    const bool own = in && tx >= kHalo && tx < 32 - kHalo && ty >= kHalo && ty < 32 - kHalo;
    const uint8_t *jmap = static_cast<const uint8_t *>(a.jmap_idx);
    T w[ND];
    unsigned at[ND][PW / 2];
    const T si = a.sym ? jv[static_cast<int64_t>(ND / 2) * n + i] : T(0);
    T p[PW];
    load_slots(pin + static_cast<int64_t>(i) * PW, p);
#pragma unroll
    for (int o = 0; o < ND; ++o) {
        const int k = i + a.joff.off[o];
        const bool inside = k >= 0 && k < n;
        w[o] = in ? smooth_weight(a, jv, i, o, k, inside, si) : T(0);
        const uint32_t m = in ? a.jmap_tab[jmap[static_cast<int64_t>(o) * n + i]] : 0xFFFFFFFFu;
        // the neighbour's thread (past the edge: its own, and not right any more)
        const int dx = ND == 5 ? (o == 1 ? -1 : o == 3 ? 1 : 0) : o % 3 - 1;
        const int dy = ND == 5 ? (o == 0 ? -1 : o == 4 ? 1 : 0) : o / 3 - 1;
        const bool there = tx + dx >= 0 && tx + dx < 32 && ty + dy >= 0 && ty + dy < 32;
        const int q = there ? t + dx + 32 * dy : t;
        auto place = [&](int s) {
            const unsigned c = m >> (4 * s) & 0xFu;
            return c < PW ? c * kT + q : ZERO;
        };
#pragma unroll
        for (int s = 0; s < PW; s += 2) at[o][s / 2] = place(s) | place(s + 1) << 16;
    }
#pragma unroll
    for (int s = 0; s < PW; ++s) lds[0][s * kT + t] = p[s];
    if (t < 2) lds[t][ZERO] = T(0);
    const bool inner = own && eit_step >= 0 && a.interior[i] != 0;
    double emax = 0.0;
    for (int step = 0; step < steps; ++step) {
        __syncthreads();
        const T *from = lds[step & 1];
        T acc[PW];
#pragma unroll
        for (int s = 0; s < PW; ++s) acc[s] = T(0);
#pragma unroll
        for (int o = 0; o < ND; ++o)
#pragma unroll
            for (int s = 0; s < PW; ++s)
                acc[s] += w[o] * from[at[o][s / 2] >> (16 * (s & 1)) & 0xFFFFu];
        double rs = 0.0;
#pragma unroll
        for (int s = 0; s < PW; ++s) rs += static_cast<double>(acc[s]);
        const double rinv = 1.0 / rs;
#pragma unroll
        for (int s = 0; s < PW; ++s) {
            if (step == eit_step && inner) {
                const double dlt = fabs(static_cast<double>(acc[s]) - static_cast<double>(p[s]));
                emax = (dlt > emax || dlt != dlt) ? dlt : emax;
            }
            p[s] = static_cast<T>(static_cast<double>(acc[s]) * rinv);
            lds[~step & 1][s * kT + t] = p[s];
        }
    }
    if (own) store_slots(pout + static_cast<int64_t>(i) * PW, p);
    if (eit_step < 0) return;
    auto larger = [](double u, double v) { return (v > u || v != v) ? v : u; };
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) emax = larger(emax, __shfl_xor(emax, off, 64));
    if ((t & 63) == 0) red[t >> 6] = emax;
    __syncthreads();
    if (t == 0) {
        for (int u = 1; u < kT >> 6; ++u) emax = larger(emax, red[u]);
        a.eit_part[blockIdx.x] = emax;
    }
}

template <typename T, int NDT, int PW>
void smooth_small(hipStream_t s, const SmoothArgs &a, const T *jv, T *p, int steps, int eit_step)
{
    const int W = std::min(kT, (a.n + 63) / 64 * 64);
    const int lds = 2 * (PW + 1) * a.n * static_cast<int>(sizeof(T));
    auto go = [&](auto kern) {
        if (lds > 60000)
            hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        kern<<<1, W, lds, s>>>(a, jv, p, steps, eit_step);
    };
    if constexpr (PW == 4) {
        if (a.n > kT) return go(k_smooth_small<T, NDT, PW, 2>);
    }
    go(k_smooth_small<T, NDT, PW, 1>);
}

int smooth_tiles(int n, int nx)
{
    return ((nx + kTile - 1) / kTile) * ((n / nx + kTile - 1) / kTile);
}

template <int NDT, int PW>
void launch_small(hipStream_t s, const SmallPcg &a)
{
    const int T = std::min(kT, (a.n + 63) / 64 * 64);  // whole wavefronts
    const size_t lds = (2 * static_cast<size_t>(a.n) + 2 * a.nc) * sizeof(double);  // 33 KB at most
    if (a.n <= kT) k_pcg_small<NDT, PW, 1><<<1, T, lds, s>>>(a);
    else k_pcg_small<NDT, PW, 2><<<1, T, lds, s>>>(a);
}

// The end of the preconditioner on a 2D grid (as k_smooth_tile's: rows
// x + nx y, rows of P of 4 slots) in one launch: z1 = z + P w_c, one or two
// sweeps z + dinv (r - A z), and the partials of r.z and r.(z - z_old).  A
// work-group takes a tile with a halo of two cells, which its two sweeps use
// up; z and the coefficients are read 1.5 times instead of once per stage.
// Bound by the launch and three dependent round trips.
// 250 x 187 in FP64, two sweeps: 3.0 + 3.0 + 3.7 us in three launches, 3.9 here.
constexpr int kPostX = 32, kPostY = 16, kPostHalo = 2, kPostT = kPostX * kPostY;
static_assert((kPostX - 2 * kPostHalo) * (kPostY - 2 * kPostHalo) == kTileCells);
template <int ND, bool SYM, typename MT, typename PT>
__global__ __launch_bounds__(kPostT) void k_tile_post(
    int n, DiaOffsets d, const MT *__restrict__ a, const MT *__restrict__ dinv,
    const double *__restrict__ r, const double *__restrict__ zin, const PT *__restrict__ pv,
    const uint16_t *__restrict__ pcol, const double *__restrict__ wc, int nx, int ny, int ntx,
    int sweeps, double *__restrict__ zout, const double *__restrict__ zold,
    double *__restrict__ part)
{
    __shared__ double ex[2][kPostT];
    __shared__ double red[2][kPostT / 64];
    constexpr int TX = kPostX - 2 * kPostHalo, TY = kPostY - 2 * kPostHalo;
    const int t = threadIdx.x, tx = t % kPostX, ty = t / kPostX;
    const int b = xcd_group(blockIdx.x, gridDim.x);
    const int x = b % ntx * TX - kPostHalo + tx, y = b / ntx * TY - kPostHalo + ty;
    const bool in = x >= 0 && x < nx && y >= 0 && y < ny;
    const int i = in ? x + nx * y : 0;
    const bool own = in && tx >= kPostHalo && tx < kPostX - kPostHalo && ty >= kPostHalo &&
                     ty < kPostY - kPostHalo;
    typedef uint16_t c4 __attribute__((ext_vector_type(4)));
    const c4 cs = reinterpret_cast<const c4 *>(pcol)[i];
    PT p[4];
    load_slots(pv + static_cast<int64_t>(i) * 4, p);
    double z = zin ? zin[i] : 0.0;
    const MT ri = static_cast<MT>(r[i]);
    const MT di = dinv[i];
    const double zo = zold[i], rd = r[i];
    MT av[ND];
    int at[ND];
#pragma unroll
    for (int o = 0; o < ND; ++o) {
        const int k = i + d.off[o];
        const bool have = in && k >= 0 && k < n;
        MT v;
        if constexpr (SYM) {
            v = o < ND / 2 ? a[static_cast<int64_t>(ND - 1 - o) * n + (have ? k : i)]
                           : a[static_cast<int64_t>(o) * n + i];
        } else {
            v = a[static_cast<int64_t>(o) * n + i];
        }
        av[o] = have ? v : MT(0);
        const int dx = ND == 5 ? (o == 1 ? -1 : o == 3 ? 1 : 0) : o % 3 - 1;
        const int dy = ND == 5 ? (o == 0 ? -1 : o == 4 ? 1 : 0) : o / 3 - 1;
        const bool there = tx + dx >= 0 && tx + dx < kPostX && ty + dy >= 0 && ty + dy < kPostY;
        at[o] = there ? t + dx + kPostX * dy : t;
    }
    double g[4], s = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) g[q] = wc[cs[q] == 0xFFFFu ? 0 : cs[q]];
#pragma unroll
    for (int q = 0; q < 4; ++q) s += cs[q] == 0xFFFFu ? 0.0 : static_cast<double>(p[q]) * g[q];
    z = zin ? z + s : s;
    if (!in) z = 0.0;
    for (int k = 0; k < sweeps; ++k) {
        ex[k & 1][t] = z;
        __syncthreads();
        MT dot = MT(0);
#pragma unroll
        for (int o = 0; o < ND; ++o) dot += av[o] * static_cast<MT>(ex[k & 1][at[o]]);
        z += static_cast<double>(di * (ri - dot));
    }
    double v[2] = {0.0, 0.0};
    if (own) {
        zout[i] = z;
        v[0] = rd * z;
        v[1] = rd * (z - zo);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const double w = wave_sum(v[q]);
        if ((t & 63) == 0) red[q][t >> 6] = w;
    }
    __syncthreads();
    if (t < 2) {
        double w = 0.0;
        for (int u = 0; u < kPostT / 64; ++u) w += red[t][u];
        part[static_cast<int64_t>(t) * gridDim.x + blockIdx.x] = w;
    }
}

}  // namespace

// 100 steps, launch by launch against one launch, set-up of J and the
// statistics included (FP64 / FP32):
//   32 x 32, 5 slots of J, rows of 4      0.46 / 0.42 ms   0.14 / 0.13 ms
//   45 x 43, 5 slots, rows of 4           0.48 / 0.47      0.22 / 0.21
//   10 x 10 x 10, 7 slots, rows of 8      0.67 / 0.59      0.36 / 0.24
// The limits are LDS (two buffers) and registers: two rows per thread of 8
// slots, or 9 slots of J by 8, would be held in scratch memory.
bool smooth_fits_small(const SmoothArgs &a, bool fp32)
{
    return a.n <= (a.pw == 8 ? kSmallThreads : kSmallRows) && (a.pw == 4 || a.pw == 8) &&
           a.jw <= (a.pw == 8 ? 7 : kSmallDiags) && a.jmap_kind == 1 &&
           2 * (a.pw + 1) * a.n * (fp32 ? 4 : 8) <= 155000;  // of 160 KB of LDS
}

void launch_smooth_small(hipStream_t s, const SmoothArgs &a, bool fp32, const double *jv64,
                         const float *jv32, double *p64, float *p32, int steps, int eit_step)
{
    auto go = [&](auto nd, auto pw) {
        constexpr int N = decltype(nd)::value, PW = decltype(pw)::value;
        if (fp32) smooth_small<float, N, PW>(s, a, jv32, p32, steps, eit_step);
        else smooth_small<double, N, PW>(s, a, jv64, p64, steps, eit_step);
    };
    typedef std::integral_constant<int, 4> c4;
    typedef std::integral_constant<int, 5> c5;
    typedef std::integral_constant<int, 7> c7;
    typedef std::integral_constant<int, 8> c8;
    typedef std::integral_constant<int, 9> c9;
    if (a.jw <= 5) a.pw == 8 ? go(c5{}, c8{}) : go(c5{}, c4{});
    else if (a.jw <= 7) a.pw == 8 ? go(c7{}, c8{}) : go(c7{}, c4{});
    else go(c9{}, c4{});
}

// Where the launches no longer bound the steps, the tiles' arithmetic (1.8 times
// a step's, and more where the last tile of a line is nearly empty) does.
// Microseconds a step, launch by launch / tiles:
//   five neighbours   FP64                     FP32
//   512 x 512         6.8 /  4.2 (484 tiles)   5.3 /  3.0
//   25 x 10,900       7.3 /  7.1 (910)         5.3 /  4.8
//   1000 x 1000      22.6 / 15.0 (1,764)      11.1 /  8.9
//   49 x 20,400      21.1 / 19.7 (2,550)      11.1 / 11.6   tiles 1.5 times the grid
//   30 x 33,334      21.6 / 20.8 (2,778)      11.0 / 12.5   1.6 times
//   25 x 40,000      21.7 / 25.0 (3,334)      10.9 / 15.0   1.9 times
//   nine neighbours
//   512 x 512        13.9 /  6.9               6.6 /  5.4
//   25 x 6,250        8.8 /  8.1 (522)         5.7 /  7.2
//   600 x 600        19.0 / 10.5 (625)         7.8 /  7.8
//   1000 x 1000      54.5 / 23.9              14.1 / 21.7
//   25 x 40,000      54.5 / 39.6              13.7 / 36.7
// So nine neighbours in FP32 take the tiles while all of them run at once (two to
// each of 256 compute units), five neighbours up to twice that or while the tiles
// are little larger than the grid, nine in FP64 always.
int smooth_tile_steps(const SmoothArgs &a, int nx, bool fp32)
{
    if (nx <= 0 || a.pw != 4 || a.jmap_kind != 1 || (a.jw != 5 && a.jw != 9)) return 0;
    const int64_t tiles = smooth_tiles(a.n, nx);
    if (a.jw == 9) return !fp32 || tiles <= 512 ? kHalo : 0;
    const bool close = 10 * tiles * kTile * kTile <= (fp32 ? 13 : 17) * static_cast<int64_t>(a.n);
    return tiles <= 1024 || close ? kHalo : 0;
}

void launch_smooth_tile(hipStream_t s, const SmoothArgs &a, int nx, bool fp32, const double *jv64,
                        const float *jv32, const double *pin64, double *pout64,
                        const float *pin32, float *pout32, int steps, int eit_step)
{
    const int ny = a.n / nx, ntx = (nx + kTile - 1) / kTile;
    const int grid = smooth_tiles(a.n, nx);
    auto go = [&](auto nd) {
        constexpr int ND = decltype(nd)::value;
        if (fp32)
            k_smooth_tile<float, ND><<<grid, kT, 0, s>>>(a, jv32, pin32, pout32, nx, ny, ntx, steps,
                                                         eit_step);
        else
            k_smooth_tile<double, ND><<<grid, kT, 0, s>>>(a, jv64, pin64, pout64, nx, ny, ntx,
                                                          steps, eit_step);
    };
    if (a.jw == 5) go(std::integral_constant<int, 5>{});
    else go(std::integral_constant<int, 9>{});
    if (eit_step >= 0) launch_eit_final(s, grid, a.eit_part, a.eit_out);
}

int launch_tile_post(hipStream_t s, int n, const DiaOffsets &d, const double *a, const float *a32,
                     const double *dinv, const float *dinv32, const double *r, const double *zin,
                     const double *p64, const float *p32, const uint16_t *pcol, const double *wc,
                     int nx, int sweeps, double *zout, const double *zold, double *part)
{
    constexpr int TX = kPostX - 2 * kPostHalo, TY = kPostY - 2 * kPostHalo;
    const int ny = n / nx, ntx = (nx + TX - 1) / TX, grid = ntx * ((ny + TY - 1) / TY);
    auto go = [&](auto nd, auto sym, auto *ap, auto *dp, auto *pp) {
        k_tile_post<decltype(nd)::value, decltype(sym)::value><<<grid, kPostT, 0, s>>>(
            n, d, ap, dp, r, zin, pp, pcol, wc, nx, ny, ntx, sweeps, zout, zold, part);
    };
    auto with_types = [&](auto nd, auto sym) {
        if (a32 && p32) go(nd, sym, a32, dinv32, p32);
        else if (a32) go(nd, sym, a32, dinv32, p64);
        else if (p32) go(nd, sym, a, dinv, p32);
        else go(nd, sym, a, dinv, p64);
    };
    auto with_sym = [&](auto nd) {
        if (d.sym) with_types(nd, std::true_type{});
        else with_types(nd, std::false_type{});
    };
    if (d.n == 5) with_sym(std::integral_constant<int, 5>{});
    else with_sym(std::integral_constant<int, 9>{});
    return grid;
}

int grid2d_width(const DiaOffsets &d, int n)
{
    if (d.n != 5 && d.n != 9) return 0;
    const int nx = d.off[d.n - 1] - (d.n == 9 ? 1 : 0);
    if (nx < 16 || n % nx != 0 || n / nx < 16) return 0;
    for (int o = 0; o < d.n; ++o) {
        const int dx = d.n == 5 ? (o == 1 ? -1 : o == 3 ? 1 : 0) : o % 3 - 1;
        const int dy = d.n == 5 ? (o == 0 ? -1 : o == 4 ? 1 : 0) : o / 3 - 1;
        if (d.off[o] != dx + nx * dy) return 0;
    }
    return nx;
}

void launch_pcg_small(hipStream_t s, const SmallPcg &a, int pw)
{
    if (a.nd <= 5) pw == 8 ? launch_small<5, 8>(s, a) : launch_small<5, 4>(s, a);
    else pw == 8 ? launch_small<9, 8>(s, a) : launch_small<9, 4>(s, a);
}

}  // namespace msrsb
