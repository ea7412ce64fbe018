// Levels of at most 64^2 (2D) or 16^3 (3D) cells in one workgroup, every level in
// LDS: the end of a larger grid's V-cycle (k_tail, and kb_tail of the batched
// solver), and whole FP64 solves of grids that small (k_solve1).
// What bounds it: one CU does all the work, so each stage costs its LDS and
// FP64 issue (64^2 in FP64: 4096 cells, about 1300 cycles of LDS reads a sweep)
// and, on the smaller levels, one LDS round trip, one chain of dependent
// operations and one barrier.  So every level is a template instance: a thread's
// run of cells along the last axis has a compile-time length and all its loads
// are issued before the first use, neighbours along x come from lane rotations
// where a grid row is a whole wavefront or a DPP row (64 or 16 cells), and the
// levels of at most 64 cells run on one wavefront without barriers.  Measured against
// run-time loops over the levels: twelve FP64 cycles at 128^2 443 -> 360 us, at 32^3 614 ->
// 528 us, so about 7 us of a tail of 15 to 20.
#pragma once

#include "mg_block2.h"
#include "mg_fused3.h"

namespace np {

// Cells of the levels coarser than LG in the LDS arrays (coarsest level, 4^D, first).
template <int D> constexpr int tail_off(int lg) { return ((1 << (D * lg)) - (1 << (2 * D))) / ((1 << D) - 1); }

// The operators of the tail's levels: at<LG>() gives a level's.  LapTail: -Lap_h with the finest tail level's weights; on a
// level 2^k times coarser 1/h^2 scales by 4^-k and the Jacobi weight by 4^k, both exactly.
template <int D, class C> struct LapTail {
    double inv_h2, wd;
    int lg_t;
    template <int LG> __device__ __forceinline__ auto at() const {
        const double q = double(1 << (2 * (lg_t - LG)));
        if constexpr (D == 2) return Lap2<C>{C(inv_h2 / q), C(wd * q)};
        else return Lap3<C>{C(inv_h2 / q), C(wd * q)};
    }
};
// A barrier among the NT threads at work: one wavefront needs only its LDS accesses kept in order.
template <int NT> __device__ __forceinline__ void tail_sync() {
    if constexpr (NT == 64) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    } else {
        __syncthreads();
    }
}

// The values of the lanes at x - 1 and x + 1 of a grid row of 2^LG cells (64: the wavefront, 16: a
// DPP row), wrapped.
template <int LG, bool UP> __device__ __forceinline__ uint32_t row_lane(uint32_t v) {
    static_assert(LG == 6 || LG == 4, "a row is a wavefront or a DPP row");
    constexpr int ctrl = LG == 6 ? (UP ? 0x134 : 0x13c) : (UP ? 0x12f : 0x121);  // wave_rol/ror:1, row_ror:15/1
    return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), ctrl, 0xf, 0xf, true));
}
template <int LG, bool UP> __device__ __forceinline__ float row_lane(float v) {
    return __uint_as_float(row_lane<LG, UP>(__float_as_uint(v)));
}
template <int LG, bool UP> __device__ __forceinline__ double row_lane(double v) {
    return __hiloint2double(int(row_lane<LG, UP>(uint32_t(__double2hiint(v)))),
                            int(row_lane<LG, UP>(uint32_t(__double2loint(v)))));
}

// One stage of a level on NT threads: T = X + wd (F - A X) (SWEEP), the sweep after a first one from
// zero (ZERO2: its iterate w f is formed from F), or the residual T = F - A X (RESID).  Returns this
// thread's share of |F - A X|^2.  Each thread marches along the last axis over `len` cells.
enum TailStage { kTailSweep, kTailZero2, kTailResid };
template <int D, class C, int NT, int LG, TailStage ST, class OP, class TO>
__device__ __forceinline__ double tail_stage(const C *X, const C *F, TO *T, int bc, const OP &op) {
    constexpr int n = 1 << LG, last = n - 1, sm = D == 3 ? n * n : n;
    static_assert(sm <= NT, "a thread per cell of a plane");
    constexpr int chunks = NT / sm < n ? NT / sm : n, len = n / chunks;
    double acc = 0.0;
    const int t = int(threadIdx.x);
    if (sm * chunks == NT || t < sm * chunks) {
        const bool per = bc != 0;
        const int i = t & last, j = D == 3 ? (t >> LG) & last : 0, z0 = (t / sm) * len;
        const int c = z0 * sm + (t & (sm - 1));
        auto xv = [&](int q) -> C { return ST == kTailZero2 ? op.wd * F[q] : X[q]; };
        const bool gxm = i == 0 && !per, gxp = i == last && !per;  // Dirichlet ghosts: minus the own value
        const bool gzm = z0 == 0 && !per, gzp = z0 + len == n && !per;
        C xc[len + 2], xm[len], xp[len], ym[len], yp[len], f[len];
        xc[0] = xv(z0 > 0 ? c - sm : (per ? c + last * sm : c));
        xc[len + 1] = xv(z0 + len < n ? c + len * sm : (per ? c + (len - n) * sm : c));
#pragma unroll
        for (int u = 0; u < len; ++u) xc[u + 1] = xv(c + u * sm);
        constexpr bool lanes = LG == 6 || LG == 4;
        if constexpr (!lanes) {
            const int om = i > 0 ? -1 : (per ? last : 0), op_ = i < last ? 1 : (per ? -last : 0);
#pragma unroll
            for (int u = 0; u < len; ++u) {
                xm[u] = xv(c + om + u * sm);
                xp[u] = xv(c + op_ + u * sm);
            }
        }
        bool gym = false, gyp = false;
        if constexpr (D == 3) {
            const int om = j > 0 ? -n : (per ? last * n : 0), op_ = j < last ? n : (per ? -last * n : 0);
            gym = j == 0 && !per;
            gyp = j == last && !per;
#pragma unroll
            for (int u = 0; u < len; ++u) {
                ym[u] = xv(c + om + u * sm);
                yp[u] = xv(c + op_ + u * sm);
            }
        }
#pragma unroll
        for (int u = 0; u < len; ++u) f[u] = F[c + u * sm];
        if constexpr (lanes) {
#pragma unroll
            for (int u = 0; u < len; ++u) {
                xm[u] = row_lane<LG, false>(xc[u + 1]);
                xp[u] = row_lane<LG, true>(xc[u + 1]);
            }
        }
#pragma unroll
        for (int u = 0; u < len; ++u) {
            const C v = xc[u + 1];
            const C wm = gxm ? -v : xm[u], wp = gxp ? -v : xp[u];
            const C am = u == 0 && gzm ? -v : xc[u], ap = u == len - 1 && gzp ? -v : xc[u + 2];
            C r;
            if constexpr (D == 3) r = op.resid(f[u], v, wm, wp, gym ? -v : ym[u], gyp ? -v : yp[u], am, ap);
            else r = op.resid(f[u], v, wm, wp, am, ap);
            acc += double(r) * double(r);
            T[c + u * sm] = TO(ST == kTailResid ? r : v + op.wd * r);
        }
    }
    return acc;
}

// X += P E (E: the next coarser level); terms and order of k_prolong_add.
template <int D, class C, int NT, int LG>
__device__ __forceinline__ void tail_prolong(const C *E, C *X, int bc) {
    constexpr int n = 1 << LG, last = n - 1, LC = LG - 1, nc = n >> 1, sm = D == 3 ? n * n : n, smc = D == 3 ? nc * nc : nc;
    constexpr int chunks = NT / sm < n ? NT / sm : n, len = n / chunks;
    const int t = int(threadIdx.x);
    if (sm * chunks == NT || t < sm * chunks) {
        const int z0 = (t / sm) * len, c = z0 * sm + (t & (sm - 1));
        int oi, ni, oj = 0, nj = 0;
        float si, sj = 1.0f;
        pro_axis(t & last, nc, bc, oi, ni, si);
        if (D == 3) pro_axis((t >> LG) & last, nc, bc, oj, nj, sj);
        // a coarse plane's (row's) values at the in-plane neighbours, with the in-plane ghost signs
        constexpr int NP = D == 3 ? 4 : 2;
        auto plane = [&](int K, C (&e)[NP]) {
            float s = 1.0f;
            if (K < 0) { s = bc ? 1.0f : -1.0f; K = bc ? nc - 1 : 0; }
            else if (K >= nc) { s = bc ? 1.0f : -1.0f; K = bc ? 0 : nc - 1; }
#pragma unroll
            for (int b = 0; b < NP / 2; ++b)
#pragma unroll
                for (int a = 0; a < 2; ++a)
                    e[2 * b + a] = C(s * (a ? si : 1.0f) * (b ? sj : 1.0f)) *
                                   E[K * smc + (D == 3 ? (b ? nj : oj) << LC : 0) + (a ? ni : oi)];
        };
        auto mix = [&](const C (&o)[NP], const C (&h)[NP]) -> C {
            C s = C(0);
#pragma unroll
            for (int cz = 0; cz < 2; ++cz)
#pragma unroll
                for (int b = 0; b < NP / 2; ++b)
#pragma unroll
                    for (int a = 0; a < 2; ++a) {
                        // 2D: the marching axis is y, whose weight is the second factor
                        const C w = D == 3 ? C(a ? 0.25 : 0.75) * C(b ? 0.25 : 0.75) * C(cz ? 0.25 : 0.75)
                                           : C(a ? 0.25 : 0.75) * C(cz ? 0.25 : 0.75) * C(1.0);
                        s = np_fma(w, cz ? h[2 * b + a] : o[2 * b + a], s);
                    }
            return s;
        };
        if constexpr (len >= 2) {  // z0 even: coarse planes z0/2 - 1 .. z0/2 + len/2
            C e[len / 2 + 2][NP], x[len];
#pragma unroll
            for (int q = 0; q < len / 2 + 2; ++q) plane((z0 >> 1) - 1 + q, e[q]);
#pragma unroll
            for (int u = 0; u < len; ++u) x[u] = X[c + u * sm];
#pragma unroll
            for (int u = 0; u < len; ++u) X[c + u * sm] = x[u] + mix(e[(u >> 1) + 1], e[(u >> 1) + ((u & 1) ? 2 : 0)]);
        } else {
            C o[NP], h[NP];
            plane(z0 >> 1, o);
            plane((z0 >> 1) + ((z0 & 1) ? 1 : -1), h);
            X[c] = X[c] + mix(o, h);
        }
    }
}

// `cnt` sweeps of a level alternating between X and T; the result ends in X.
template <int D, class C, int NT, int LG, class OP>
__device__ __forceinline__ void tail_sweeps(C *X, const C *F, C *T, int bc, const OP &op, int cnt) {
    for (int it = 0; it + 1 < cnt; it += 2) {
        tail_stage<D, C, NT, LG, kTailSweep>(X, F, T, bc, op);
        tail_sync<NT>();
        tail_stage<D, C, NT, LG, kTailSweep>(T, F, X, bc, op);
        tail_sync<NT>();
    }
    if (cnt & 1) {
        tail_stage<D, C, NT, LG, kTailSweep>(X, F, T, bc, op);
        tail_sync<NT>();
        for (int c = int(threadIdx.x); c < (1 << (D * LG)); c += NT) X[c] = T[c];
        tail_sync<NT>();
    }
}

// The correction of levels LG .. 2 from a zero iterate (LDS arrays xs, fs with every level at
// tail_off; ts: scratch of the finest): nu1 >= 1 pre-sweeps, the coarser levels, nu2 post-sweeps.
// Ms: the coarsest inverse, entry (i, q) at i + q * (4^D + 1).
template <int D, class C, int NT, int LG, class OPS>
__device__ __forceinline__ void tail_down_up(C *xs, C *fs, C *ts, const double *Ms, int bc, const OPS &ops, int nu1,
                                             int nu2);
template <int D, class C, int NT, int LG, class OPS>
__device__ __forceinline__ void tail_zero(C *xs, C *fs, C *ts, const double *Ms, int bc, const OPS &ops, int nu1,
                                          int nu2) {
    constexpr int m = 1 << (D * LG);
    const int tid = int(threadIdx.x);
    if constexpr (m <= 64 && NT > 64) {  // one wavefront from here down
        if (tid < 64) tail_zero<D, C, 64, LG>(xs, fs, ts, Ms, bc, ops, nu1, nu2);
        __syncthreads();
    } else if constexpr (LG == 2) {
        if (tid < m) {
            double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
            for (int q = 0; q < m; q += 4)
#pragma unroll
                for (int u = 0; u < 4; ++u) a[u] += Ms[tid + (q + u) * (m + 1)] * double(fs[q + u]);
            xs[tid] = C((a[0] + a[1]) + (a[2] + a[3]));
        }
        tail_sync<NT>();
    } else {
        C *X = xs + tail_off<D>(LG), *F = fs + tail_off<D>(LG);
        const auto op = ops.template at<LG>();
        if (nu1 >= 2) {
            tail_stage<D, C, NT, LG, kTailZero2>(F, F, X, bc, op);
            tail_sync<NT>();
            if (nu1 > 2) tail_sweeps<D, C, NT, LG>(X, F, ts, bc, op, nu1 - 2);
        } else {
            for (int c = tid; c < m; c += NT) X[c] = op.wd * F[c];
            tail_sync<NT>();
        }
        tail_down_up<D, C, NT, LG>(xs, fs, ts, Ms, bc, ops, nu1, nu2);
    }
}
// The rest of a level's cycle after its pre-sweeps: residual, restriction, the coarser levels,
// prolongation + correction, nu2 post-sweeps.
template <int D, class C, int NT, int LG, class OPS>
__device__ __forceinline__ void tail_down_up(C *xs, C *fs, C *ts, const double *Ms, int bc, const OPS &ops, int nu1,
                                             int nu2) {
    constexpr int n = 1 << LG, LC = LG - 1, nc = n >> 1, mc = 1 << (D * LC);
    C *X = xs + tail_off<D>(LG), *F = fs + tail_off<D>(LG), *Fc = fs + tail_off<D>(LC);
    const auto op = ops.template at<LG>();
    tail_stage<D, C, NT, LG, kTailResid>(X, F, ts, bc, op);
    tail_sync<NT>();
    for (int cc = int(threadIdx.x); cc < mc; cc += NT) {
        const int I = cc & (nc - 1), J = (cc >> LC) & (nc - 1), K = D == 3 ? cc >> (2 * LC) : 0;
        const C *r = ts + ((2 * K) << (2 * LG)) + ((2 * J) << LG) + 2 * I;
        C s = C(0);
#pragma unroll
        for (int kk = 0; kk < (D == 3 ? 2 : 1); ++kk)
#pragma unroll
            for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                for (int ii = 0; ii < 2; ++ii) s += r[(kk << (2 * LG)) + (jj << LG) + ii];
        Fc[cc] = s * C(D == 3 ? 0.125 : 0.25);
    }
    tail_sync<NT>();
    tail_zero<D, C, NT, LC>(xs, fs, ts, Ms, bc, ops, nu1, nu2);
    tail_prolong<D, C, NT, LG>(xs + tail_off<D>(LC), X, bc);
    tail_sync<NT>();
    tail_sweeps<D, C, NT, LG>(X, F, ts, bc, op, nu2);
}

// Calls fn(integral_constant<LG>) with LG = lg in [2, Tail<D>::LG].
template <int D, class Fn> __device__ __forceinline__ void tail_by_level(int lg, Fn &&fn) {
    if (lg == 3) fn(std::integral_constant<int, 3>());
    else if (lg == 4) fn(std::integral_constant<int, 4>());
    else if (D == 2 && lg == 5) fn(std::integral_constant<int, D == 2 ? 5 : 4>());
    else if (D == 2 && lg == 6) fn(std::integral_constant<int, D == 2 ? 6 : 4>());
    else fn(std::integral_constant<int, 2>());
}

// This thread's share of m values of an array (at most MAX) on their way from memory, and their way
// into LDS: the kernel's other round trips to memory run meanwhile.
template <class S, int NT, int MAX> struct TailLoad {
    static constexpr int per = (MAX + NT - 1) / NT;
    typename St<S>::C v[per];
    __device__ __forceinline__ void ask(const S *p, int m) {
#pragma unroll
        for (int u = 0; u < per; ++u) v[u] = St<S>::ld(p + min(int(threadIdx.x) + u * NT, m - 1));
    }
    template <class Put> __device__ __forceinline__ void put(int m, Put &&dst) const {
#pragma unroll
        for (int u = 0; u < per; ++u) {
            const int c = int(threadIdx.x) + u * NT;
            if (c < m) dst(c, v[u]);
        }
    }
};

// The coarsest inverse (row-major Minv, scaled by `sc`) into LDS, transposed with padded rows:
// thread i reading entry (i, q) hits consecutive banks.
template <int D, int NT> __device__ __forceinline__ void tail_minv(double *Ms, const double *Minv, double sc = 1.0) {
    constexpr int m = D == 3 ? 64 : 16;
    for (int g = int(threadIdx.x); g < m * m; g += NT) Ms[(g % m) * (m + 1) + g / m] = Minv[g] * sc;
}

// m values of a field in storage S into LDS: all of this thread's loads first, then the stores
// (one round trip to memory); at most MAX.
template <class S, int NT, int MAX> __device__ __forceinline__ void tail_fetch(typename St<S>::C *d, const S *p, int m) {
    constexpr int per = (MAX + NT - 1) / NT;
    typename St<S>::C v[per];
#pragma unroll
    for (int u = 0; u < per; ++u) {
        const int c = int(threadIdx.x) + u * NT;
        if (c < m) v[u] = St<S>::ld(p + c);
    }
#pragma unroll
    for (int u = 0; u < per; ++u) {
        const int c = int(threadIdx.x) + u * NT;
        if (c < m) d[c] = v[u];
    }
}

// One-workgroup V-cycle from a zero iterate on levels lg_t .. 2.  ctl: first the
// cycle's convergence check on the np partials of the finest level's residual
// norm (the check of k_check), and nothing more if it stops the solve; its operands
// arrive meanwhile (one after the other they took the tail from 8.8 to 11.2 us in 3D BF16
// and from 11.5 to 12.3 in 2D FP64).
template <int D, class S, class OPS>
__global__ __launch_bounds__(Tail<D>::NT) void k_tail(const S *__restrict__ f_t, S *__restrict__ x_t,
                                                      const double *__restrict__ Minv, int lg_t, int bc, OPS ops,
                                                      int nu1, int nu2, const int *stop,
                                                      const double *__restrict__ partial, int np, Ctl *ctl) {
    typedef typename St<S>::C C;
    constexpr int NT = Tail<D>::NT, m = D == 3 ? 64 : 16;
    __shared__ C xs[Tail<D>::levels_sum()];
    __shared__ C fs[Tail<D>::levels_sum()];
    __shared__ C ts[Tail<D>::cells(Tail<D>::LG)];
    __shared__ double Ms[m * (m + 1)];
    const int stopped = stop ? *stop : 0;
    const int o = tail_off<D>(lg_t), mt = 1 << (D * lg_t);
    TailLoad<S, NT, int(Tail<D>::cells(Tail<D>::LG))> tf;
    TailLoad<double, NT, m * m> tm;
    tf.ask(f_t, mt);
    tm.ask(Minv, m * m);
    if (ctl) {  // the operands arrive while the check is made
        __shared__ int halt;
        const int st = check_block<NT>(partial, np, ctl);
        if (threadIdx.x == 0) halt = st;
        __syncthreads();
        if (halt) return;
    }
    landed(tf.v);
    landed(tm.v);
    if (stopped) return;
    tm.put(m * m, [&](int g, double v) { Ms[(g % m) * (m + 1) + g / m] = v; });
    tf.put(mt, [&](int c, C v) { fs[o + c] = v; });
    __syncthreads();
    tail_by_level<D>(lg_t, [&](auto lg) {
        tail_zero<D, C, NT, decltype(lg)::value>(xs, fs, ts, Ms, bc, ops, nu1, nu2);
    });
    for (int c = int(threadIdx.x); c < mt; c += NT) St<S>::st(x_t + c, xs[o + c]);
}

// ------------------------------------------------------------ whole solves
// A solve of a grid that fits one workgroup, from the right-hand side's norm to
// the last cycle, in one launch with every field in LDS.  The multi-launch solve
// spent five to seven launches a cycle on such a grid.  Measured, twelve FP64 cycles: 8^2
// 276 -> 40 us, 64^2 431 -> 112 us, 16^3 479 -> 120 us; a 64^2 solve to 1e-10 529 -> 134 us.
constexpr int kSolve1T = 512;  // threads (1024 in 3D: 128 registers, spilled)
struct Solve1 {
    double tol;
    int nu1, nu2, fixed, maxc;  // as the controller's
    int inner;                  // mixed: V-cycles per refinement step
    int bc, mean;               // mean: remove the right-hand side's and the solution's mean
    int warm, known0;           // x is the starting iterate; the zero iterate's check is known (rr = 1)
};

// v -= its mean; m a power of two.  Never more than four terms are added in a row: four times a value, or sums of
// two equal values, are exact, so that a constant field becomes zero as it does on larger grids (up to 2^20 cells),
// where eight in a row can leave every cell one rounding off.
template <int NT> __device__ __forceinline__ void tail_demean(double *v, int m) {
    constexpr int NW = NT / 64;
    static_assert(NW <= 8, "two runs of four wavefronts");
    __shared__ double mean, wsum[NW];
    const int tid = int(threadIdx.x);
    double a = 0.0, b = 0.0;  // at most 8 cells per thread
    for (int c = tid; c < m; c += 2 * NT) {
        a += v[c];
        if (c + NT < m) b += v[c + NT];
    }
    a += b;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
    if ((tid & 63) == 0) wsum[tid >> 6] = a;
    __syncthreads();
    if (tid == 0) {
        double s[2] = {0.0, 0.0};
#pragma unroll
        for (int w = 0; w < NW; ++w) s[w / 4] += wsum[w];
        mean = (s[0] + s[1]) * (1.0 / double(m));
    }
    __syncthreads();
    for (int c = int(threadIdx.x); c < m; c += NT) v[c] -= mean;
    __syncthreads();
}

// The controller's rule (check_block) on the sum of squares `acc` shared by the workgroup: the stop
// state, 0 while running.
template <int NT>
__device__ __forceinline__ int solve1_check(double acc, double nf, const Solve1 &p, int k, double *hist) {
    __shared__ int halt;
    acc = block_sum_n<NT>(acc);
    if (threadIdx.x == 0) {
        const double rr = sqrt(acc) / nf;
        if (k < 256) hist[k] = rr;
        int st = kRunning;
        if (!(rr <= 1.0e300)) st = kNonFinite;
        else if (p.fixed > 0) { if (k >= p.fixed) st = kFixedDone; }
        else if (rr <= p.tol) st = kConverged;
        else if (k >= p.maxc) st = kMaxCycles;
        else if (k >= 3 && k < 256 && hist[k - 3] < hist[k - 2] && hist[k - 2] < hist[k - 1] && hist[k - 1] < rr)
            st = kDiverged;
        halt = st;
    }
    __syncthreads();
    return halt;
}

// Loads f (and x), takes |f| (of the mean-free f): false when there is nothing to solve -- x is then
// zero (f = 0) or untouched (a non-finite f, out->k = -1) and *out says so.
template <int NT, int MAX>
__device__ __forceinline__ bool solve1_start(const double *f, double *x, double *F, double *X, int m, const Solve1 &p,
                                             double &nf, Ctl *out) {
    __shared__ double norm;
    tail_fetch<double, NT, MAX>(F, f, m);
    if (p.warm) tail_fetch<double, NT, MAX>(X, x, m);
    __syncthreads();
    if (p.mean) tail_demean<NT>(F, m);
    double a = 0.0;
    for (int c = int(threadIdx.x); c < m; c += NT) a += F[c] * F[c];
    a = block_sum_n<NT>(a);
    if (threadIdx.x == 0) norm = sqrt(a);
    __syncthreads();
    nf = norm;
    if (nf > 0.0 && nf <= 1.7976931348623157e308) return true;
    if (nf == 0.0)
        for (int c = int(threadIdx.x); c < m; c += NT) x[c] = 0.0;
    if (threadIdx.x == 0) {
        out->stop = nf == 0.0 ? kConverged : kNonFinite;
        out->k = nf == 0.0 ? 0 : -1;
        out->nhist = 0;
    }
    return false;
}

// The result and the controller's record.
template <int NT>
__device__ __forceinline__ void solve1_end(double *X, double *x, int m, const Solve1 &p, int stop, int k,
                                           const double *hist, Ctl *out) {
    if (p.mean) tail_demean<NT>(X, m);
    for (int c = int(threadIdx.x); c < m; c += NT) x[c] = X[c];
    const int nh = k + 1 < 256 ? k + 1 : 256;
    for (int c = int(threadIdx.x); c < nh; c += NT) out->hist[c] = hist[c];
    if (threadIdx.x == 0) {
        out->stop = stop;
        out->k = k;
        out->nhist = nh;
    }
}

// nu1 pre-sweeps of the finest level from the iterate X and the rest of the cycle.
template <int D, class C, int NT, int LG, class OPS>
__device__ __forceinline__ void solve1_cycle(C *xs, C *fs, C *ts, const double *Ms, int bc, const OPS &ops, int nu1,
                                             int nu2) {
    tail_sweeps<D, C, NT, LG>(xs + tail_off<D>(LG), fs + tail_off<D>(LG), ts, bc, ops.template at<LG>(), nu1);
    tail_down_up<D, C, NT, LG>(xs, fs, ts, Ms, bc, ops, nu1, nu2);
}

// FP64 V(nu1, nu2) cycles, nu1 >= 1, on a grid of 2^lg cells per axis, 3 <= lg <= Tail<D>::LG.
template <int D, class OPS>
__global__ __launch_bounds__(kSolve1T) void k_solve1(const double *__restrict__ f, double *__restrict__ x,
                                                        const double *__restrict__ Minv, int lg, OPS ops, Solve1 p,
                                                        Ctl *__restrict__ out) {
    constexpr int NT = kSolve1T, M = int(Tail<D>::cells(Tail<D>::LG)), mc = D == 3 ? 64 : 16;
    __shared__ double xs[Tail<D>::levels_sum()];
    __shared__ double fs[Tail<D>::levels_sum()];
    __shared__ double ts[M];
    __shared__ double Ms[mc * (mc + 1)];
    __shared__ double hist[256];
    const int o = tail_off<D>(lg), m = 1 << (D * lg);
    double nf;
    tail_minv<D, NT>(Ms, Minv);
    if (!solve1_start<NT, M>(f, x, fs + o, xs + o, m, p, nf, out)) return;
    int stop = kRunning, k = 0;
    tail_by_level<D>(lg, [&](auto l) {
        constexpr int LG = decltype(l)::value;
        if constexpr (LG > 2) {
            double *X = xs + tail_off<D>(LG), *F = fs + tail_off<D>(LG);
            const auto op = ops.template at<LG>();
            if (!p.warm && p.known0) {
                tail_zero<D, double, NT, LG>(xs, fs, ts, Ms, p.bc, ops, p.nu1, p.nu2);
                if (threadIdx.x == 0) hist[0] = 1.0;
                k = 1;
            } else if (!p.warm) {
                for (int c = int(threadIdx.x); c < m; c += NT) X[c] = 0.0;
                __syncthreads();
            }
            for (;; ++k) {
                // the first pre-sweep forms the residual of the iterate, which it leaves in place
                const double acc = tail_stage<D, double, NT, LG, kTailSweep>(X, F, ts, p.bc, op);
                stop = solve1_check<NT>(acc, nf, p, k, hist);
                if (stop) break;
                if (p.nu1 >= 2) {
                    tail_stage<D, double, NT, LG, kTailSweep>(ts, F, X, p.bc, op);
                    __syncthreads();
                    if (p.nu1 > 2) tail_sweeps<D, double, NT, LG>(X, F, ts, p.bc, op, p.nu1 - 2);
                } else {
                    for (int c = int(threadIdx.x); c < m; c += NT) X[c] = ts[c];
                    __syncthreads();
                }
                tail_down_up<D, double, NT, LG>(xs, fs, ts, Ms, p.bc, ops, p.nu1, p.nu2);
            }
        }
    });
    solve1_end<NT>(xs + o, x, m, p, stop, k, hist, out);
}

// Refinement steps with FP32 inner cycles (solve_mixed): r = f - A x in FP64, rounded; `inner` cycles
// from a zero correction in FP32; x += e in FP64.
template <int D>
__global__ __launch_bounds__(kSolve1T) void k_solve1m(const double *__restrict__ f, double *__restrict__ x,
                                                         const double *__restrict__ Minv, int lg, LapTail<D, double> op64,
                                                         LapTail<D, float> ops, Solve1 p, Ctl *__restrict__ out) {
    constexpr int NT = kSolve1T, M = int(Tail<D>::cells(Tail<D>::LG)), mc = D == 3 ? 64 : 16;
    __shared__ double X[M], F[M];
    __shared__ float xs[Tail<D>::levels_sum()];
    __shared__ float fs[Tail<D>::levels_sum()];
    __shared__ float ts[M];
    __shared__ double Ms[mc * (mc + 1)];
    __shared__ double hist[256];
    const int m = 1 << (D * lg);
    double nf;
    tail_minv<D, NT>(Ms, Minv);
    if (!solve1_start<NT, M>(f, x, F, X, m, p, nf, out)) return;
    if (!p.warm)
        for (int c = int(threadIdx.x); c < m; c += NT) X[c] = 0.0;
    __syncthreads();
    int stop = kRunning, k = 0;
    tail_by_level<D>(lg, [&](auto l) {
        constexpr int LG = decltype(l)::value;
        if constexpr (LG > 2) {
            const auto op = op64.template at<LG>();
            for (;; ++k) {
                const double acc = tail_stage<D, double, NT, LG, kTailResid>(X, F, fs + tail_off<D>(LG), p.bc, op);
                stop = solve1_check<NT>(acc, nf, p, k, hist);
                if (stop) break;
                tail_zero<D, float, NT, LG>(xs, fs, ts, Ms, p.bc, ops, p.nu1, p.nu2);
                for (int c = 1; c < p.inner; ++c)
                    solve1_cycle<D, float, NT, LG>(xs, fs, ts, Ms, p.bc, ops, p.nu1, p.nu2);
                for (int c = int(threadIdx.x); c < m; c += NT) X[c] += double(xs[tail_off<D>(LG) + c]);
                __syncthreads();
            }
        }
    });
    solve1_end<NT>(X, x, m, p, stop, k, hist, out);
}

}  // namespace np
