// 2D level kernels on 64 x 16 blocks for the levels above the one-workgroup
// tail (128^2 .. 512^2, and 1024^2 where its fields are not aligned for the wavefront legs),
// where each per-cell kernel costs about a launch:
//  - MODE 0 (down-leg from a zero iterate): the two sweeps from zero (the
//    first, w f, formed per value as k_sweep's zero-start pair forms it), the
//    residual and its restriction;
//  - MODE 1 (down-leg of an iterate): two sweeps, the residual and its
//    restriction; NORM also gives the per-workgroup partial of |f - A x|^2 of
//    the input iterate (the convergence check);
//  - MODE 2 (up-leg): prolongation + correction (formed at every position it
//    is read, rounded to storage, as k_psweep forms it) and the two post-sweeps.
// A workgroup of 1024 threads reads its operands once, with the rings its
// stages need, into LDS (all of them on their way together with the stop flag:
// 4.6 -> 4.4 us per down-leg, 5.1 -> 4.8 per up-leg of 128^2 .. 512^2); each stage is one LDS pass over the block and its
// ring.  Ring values outside the grid follow the boundary rule: periodic grids
// compute them as ordinary cells at the wrapped position, a Dirichlet stage
// takes minus its value at the mirror cell (the 5-point stencil reads such a
// value only next to the wall, where it is minus the cell's own).  Every stage
// does the arithmetic of the per-cell path (k_sweep, k_restrict, k_psweep) in
// the same term order and rounds to storage where that path stores: the
// results equal it bit for bit.
#pragma once

#include "mg_fused3.h"

namespace np {

// The operator a 2D leg applies: the residual at a cell from its neighbours, and the relaxed-Jacobi
// weight.  Lap2: A = -Lap_h (the advection-diffusion operator: Ad2).
template <class C> struct Lap2 {
    C inv_h2, wd;
    __device__ __forceinline__ C resid(C f, C xc, C xm, C xp, C ym, C yp) const {
        const C s = ((xm + xp) + ym) + yp;
        return f - (C(4) * xc - s) * inv_h2;
    }
};

template <class S> struct B2 {
    static constexpr int BX = 64, BY = 16, NT = 1024;
    static constexpr int W(int k) { return BX + 2 * k; }
    static constexpr int H(int k) { return BY + 2 * k; }
    static constexpr int R(int k) { return W(k) * H(k); }
    static constexpr int CW = BX / 2 + 4, CH = BY / 2 + 4;  // coarse cells an up-leg block reads
};

// Position (a, b) relative to the block origin of element e of the region of
// width W with `ring` cells around the block.
__device__ __forceinline__ void region_pos2(int e, int W, int ring, int &a, int &b) {
    a = e % W - ring;
    b = e / W - ring;
}

// Where a stage is evaluated for position (a, b) of a block at (x0, y0):
// periodic: the position itself (sign 1); Dirichlet: the mirror of a position
// outside the grid (sign -1), 0 for a corner outside along both axes (never
// read by a 5-point stage).
__device__ __forceinline__ int eval_pos2(int &a, int &b, int x0, int y0, int n, int bc) {
    if (bc) return 1;
    int sa = 1, sb = 1;
    a = bmap(x0 + a, n, 0, sa) - x0;
    b = bmap(y0 + b, n, 0, sb) - y0;
    const int outs = (sa < 0) + (sb < 0);
    return outs == 0 ? 1 : (outs == 1 ? -1 : 0);
}

template <class S, class OP, int MODE, bool NORM>
__global__ __launch_bounds__(B2<S>::NT) void k_lvl2_b(const S *__restrict__ ec, const S *__restrict__ f,
                                                      const S *__restrict__ xin, S *__restrict__ xout,
                                                      S *__restrict__ fc, double *__restrict__ partial, int lg,
                                                      int bc, OP op, const int *stop) {
    typedef typename St<S>::C C;
    typedef B2<S> G;
    constexpr int BX = G::BX, BY = G::BY, NT = G::NT;
    // region widths: input x on ring 3 (MODE 1) / 2 (MODE 2), f on ring 2 (down) / 1 (up)
    constexpr int WA = MODE == 1 ? G::W(3) : G::W(2), RA = MODE == 1 ? G::R(3) : G::R(2);
    constexpr int RING_A = MODE == 1 ? 3 : 2;
    constexpr int WF = MODE == 2 ? G::W(1) : G::W(2), RF = MODE == 2 ? G::R(1) : G::R(2);
    constexpr int RING_F = MODE == 2 ? 1 : 2;
    constexpr int W2 = G::W(2), W1 = G::W(1);
    // A: the input (x, or x' in the up-leg); S1: first sweep (ring 2 down, ring 1 up); S2: second
    // sweep (ring 1, down only); the block's residuals reuse A
    __shared__ C A[MODE == 0 ? 1 : (RA > BX * BY ? RA : BX * BY)];
    __shared__ C Raw[MODE == 2 ? G::R(2) : 1];
    __shared__ C Fs[RF];
    __shared__ C S1[MODE == 2 ? G::R(1) : (MODE == 1 ? G::R(2) : 1)];
    __shared__ C S2[MODE == 2 ? 1 : G::R(1)];
    __shared__ C Rr0[MODE == 0 ? BX * BY : 1];
    __shared__ C E[MODE == 2 ? G::CW * G::CH : 1];
    const int halt = stop ? *stop : 0;
    const int n = 1 << lg, t = int(threadIdx.x);
    const int nbx = n / BX, blk = int(xcd_block(blockIdx.x, gridDim.x));
    const int x0 = (blk % nbx) * BX, y0 = (blk / nbx) * BY;
    // flat index of block position (a, b) by the boundary rule, its sign into s
    auto gidx = [&](int a, int b, int &s) -> int64_t {
        const int gi = bmap(x0 + a, n, bc, s), gj = bmap(y0 + b, n, bc, s);
        return (int64_t(gj) << lg) + gi;
    };
    // ------------------------------------------------------------------ loads
    constexpr int PF = (RF + NT - 1) / NT, NX = MODE == 1 ? RA : G::R(2), PX = MODE == 0 ? 1 : (NX + NT - 1) / NT;
    C fv[PF], xv[PX], ev[1];
#pragma unroll
    for (int u = 0; u < PF; ++u) {
        int a, b, s = 1;
        region_pos2(min(t + u * NT, RF - 1), WF, RING_F, a, b);
        const int64_t g = gidx(a, b, s);
        fv[u] = C(s) * St<S>::ld(f + g);
    }
    if constexpr (MODE != 0) {
#pragma unroll
        for (int u = 0; u < PX; ++u) {
            int a, b, s = 1;
            region_pos2(min(t + u * NT, NX - 1), MODE == 1 ? WA : W2, MODE == 1 ? RING_A : 2, a, b);
            const int64_t g = gidx(a, b, s);
            xv[u] = C(s) * St<S>::ld(xin + g);
        }
    }
    if constexpr (MODE == 2) {
        const int nc = n >> 1, lgc = lg - 1, X0 = x0 >> 1, Y0 = y0 >> 1;
        static_assert(G::CW * G::CH <= NT, "one coarse cell per thread");
        int a, b, s = 1;
        region_pos2(min(t, G::CW * G::CH - 1), G::CW, 2, a, b);
        const int gi = bmap(X0 + a, nc, bc, s), gj = bmap(Y0 + b, nc, bc, s);
        ev[0] = C(s) * St<S>::ld(ec + (int64_t(gj) << lgc) + gi);
    }
    landed(fv);
    if constexpr (MODE != 0) landed(xv);
    if constexpr (MODE == 2) landed(ev);
    if (halt) return;
#pragma unroll
    for (int u = 0; u < PF; ++u)
        if (t + u * NT < RF) Fs[t + u * NT] = fv[u];
    if constexpr (MODE != 0) {
#pragma unroll
        for (int u = 0; u < PX; ++u)
            if (t + u * NT < NX) (MODE == 1 ? A : Raw)[t + u * NT] = xv[u];
    }
    if constexpr (MODE == 2) {
        if (t < G::CW * G::CH) E[t] = ev[0];
    }
    __syncthreads();
    // -------------------------------------------------- up-leg: x' = x + P ec
    if constexpr (MODE == 2) {
        const int X0 = x0 >> 1, Y0 = y0 >> 1;
        for (int e = t; e < G::R(2); e += NT) {
            int a, b;
            region_pos2(e, W2, 2, a, b);
            const int sgn = eval_pos2(a, b, x0, y0, n, bc);
            C v = C(0);
            if (sgn != 0) {
                // own coarse cell and the neighbour on the fine cell's side, per axis, in the coarse
                // tile (ghosts already carry the boundary rule); terms and order of pro_cell
                const int fx = x0 + a, fy = y0 + b;
                const int oi = (fx >> 1) - X0 + 2, ni = oi + ((fx & 1) ? 1 : -1);
                const int oj = (fy >> 1) - Y0 + 2, nj = oj + ((fy & 1) ? 1 : -1);
                C p = C(0);
#pragma unroll
                for (int bb = 0; bb < 2; ++bb)
#pragma unroll
                    for (int aa = 0; aa < 2; ++aa) {
                        const C w = C(aa ? 0.25 : 0.75) * C(bb ? 0.25 : 0.75) * C(1.0);
                        p = np_fma(w, E[(bb ? nj : oj) * G::CW + (aa ? ni : oi)], p);
                    }
                v = C(sgn) * st_round<S>(Raw[(b + 2) * W2 + a + 2] + p);
            }
            A[e] = v;
        }
        __syncthreads();
    }
    // ------------------------------------------------------- first sweep (S1)
    // down (MODE 1): on ring 2 from the input; up: on ring 1 from x'.  From zero (MODE 0) the
    // first sweep, w f, is formed where the second reads it.
    double acc = 0.0;
    if constexpr (MODE != 0) {
        constexpr int RS = MODE == 2 ? 1 : 2, WS = G::W(RS), NS = G::R(RS);
        for (int e = t; e < NS; e += NT) {
            int a, b;
            region_pos2(e, WS, RS, a, b);
            const bool own = a >= 0 && a < BX && b >= 0 && b < BY;
            const int sgn = eval_pos2(a, b, x0, y0, n, bc);
            C v = C(0);
            if (sgn != 0) {
                const C fv = Fs[(b + RING_F) * WF + a + RING_F];
                const int q = (b + RING_A) * WA + a + RING_A;
                const C xc = A[q];
                const C r = op.resid(fv, xc, A[q - 1], A[q + 1], A[q - WA], A[q + WA]);
                if (NORM && own) acc += double(r) * double(r);
                v = C(sgn) * st_round<S>(xc + op.wd * r);
            }
            S1[e] = v;
        }
        __syncthreads();
    }
    // ------------------------------------------------------ second sweep
    if constexpr (MODE == 2) {
        // on the block from S1 (ring 1), stored
        for (int e = t; e < BX * BY; e += NT) {
            const int a = e % BX, b = e / BX;
            const int q = (b + 1) * W1 + a + 1;
            const C xc = S1[q];
            const C r = op.resid(Fs[q], xc, S1[q - 1], S1[q + 1], S1[q - W1], S1[q + W1]);
            St<S>::st(xout + (int64_t(y0 + b) << lg) + x0 + a, xc + op.wd * r);
        }
    } else {
        // on ring 1 from S1 (ring 2); MODE 0 forms each neighbour's w f as its own product, as
        // k_sweep's zero-start pair does
        for (int e = t; e < G::R(1); e += NT) {
            int a, b;
            region_pos2(e, W1, 1, a, b);
            const bool own = a >= 0 && a < BX && b >= 0 && b < BY;
            const int sgn = eval_pos2(a, b, x0, y0, n, bc);
            C v = C(0);
            if (sgn != 0) {
                const int q = (b + 2) * W2 + a + 2;
                const C fv = Fs[q];
                C xc, r;
                if constexpr (MODE == 0) {
                    xc = op.wd * fv;
                    const C xm = op.wd * Fs[q - 1];
                    const C xp = op.wd * Fs[q + 1];
                    const C ym = op.wd * Fs[q - W2];
                    const C yp = op.wd * Fs[q + W2];
                    r = op.resid(fv, xc, xm, xp, ym, yp);
                } else {
                    xc = S1[q];
                    r = op.resid(fv, xc, S1[q - 1], S1[q + 1], S1[q - W2], S1[q + W2]);
                }
                v = C(sgn) * st_round<S>(xc + op.wd * r);
            }
            S2[e] = v;
            if (own && sgn != 0) St<S>::st(xout + (int64_t(y0 + b) << lg) + x0 + a, v);
        }
        __syncthreads();
        // residual of the second sweep on the block, then its restriction (k_restrict's order:
        // the y-pair outer, the x-pair inner, from zero)
        C *Rr = MODE == 0 ? Rr0 : A;
        for (int e = t; e < BX * BY; e += NT) {
            const int a = e % BX, b = e / BX;
            const int q = (b + 1) * W1 + a + 1;
            const C xc = S2[q];
            Rr[e] = op.resid(Fs[(b + 2) * W2 + a + 2], xc, S2[q - 1], S2[q + 1], S2[q - W1], S2[q + W1]);
        }
        __syncthreads();
        if (t < (BX / 2) * (BY / 2)) {
            const int I = t % (BX / 2), J = t / (BX / 2), nc = n >> 1;
            C r = C(0);
#pragma unroll
            for (int cy = 0; cy < 2; ++cy)
#pragma unroll
                for (int cx = 0; cx < 2; ++cx) r += Rr[(2 * J + cy) * BX + 2 * I + cx];
            St<S>::st(fc + (int64_t((y0 >> 1) + J) * nc + (x0 >> 1) + I), r * C(0.25));
        }
        if constexpr (NORM) {
            acc = block_sum_n<NT>(acc);
            if (threadIdx.x == 0) partial[blockIdx.x] = acc;
        }
    }
}

// Both levels above the tail in one kernel per leg (256^2 and 128^2 under a finer grid), where a leg of
// one level is little more than a launch: 2.5 of its 4.1 (down) and 4.5 us (up).  A workgroup owns
// 32 x 16 cells of the finer level and computes the rings that the coarser one's stages need itself:
// 2.4 times its own cells at the first stage, still one or two LDS passes of 1024 threads a stage.
// Arithmetic, term order and rounding of k_lvl2_b: the same bits.  4.4 us down and 5.1 up for both levels
// (4.1 to 4.4 and 4.5 to 4.8 for each before); a 512^2 FP64 solve 673 -> 577 us, a 1024^2 projection step
// 1.10 -> 0.99 ms.
template <class S> struct P2 {
    static constexpr int BX = 32, BY = 16, ND = 1024, NU = 768;  // cells; threads of the down- and the up-leg
    static constexpr int CX = BX / 2, CY = BY / 2;               // the block on the coarser level
    // a region of `ring` cells around a W x H block
    static constexpr int w(int W, int ring) { return W + 2 * ring; }
};

// The cell a stage is evaluated at for position (a, b), by the boundary rule, and the sign of its value
// there (a corner outside along both axes: the cell itself, as a field read from memory has it).
__device__ __forceinline__ int mirror_pos2(int &a, int &b, int x0, int y0, int n, int bc) {
    if (bc) return 1;
    int s = 1;
    a = bmap(x0 + a, n, 0, s) - x0;
    b = bmap(y0 + b, n, 0, s) - y0;
    return s;
}

// Two sweeps from zero at (a, b) from f (LDS, width W, `ring` cells around the block).
template <class S, class OP, class C>
__device__ __forceinline__ C pair_zero2(const C *F, int W, int ring, int a, int b, const OP &op) {
    const int q = (b + ring) * W + a + ring;
    const C fv = F[q];
    const C xc = op.wd * fv;
    const C xm = op.wd * F[q - 1];
    const C xp = op.wd * F[q + 1];
    const C ym = op.wd * F[q - W];
    const C yp = op.wd * F[q + W];
    const C r = op.resid(fv, xc, xm, xp, ym, yp);
    return st_round<S>(xc + op.wd * r);
}

// Down-legs from zero of a level (n = 2^lg, operator oa) and the next (ob): xa, fb, xb and fc.
template <class S, class OP>
__global__ __launch_bounds__(P2<S>::ND) void k_pair_down(const S *__restrict__ fa, S *__restrict__ xa,
                                                         S *__restrict__ fb, S *__restrict__ xb, S *__restrict__ fc,
                                                         int lg, int bc, OP oa, OP ob, const int *stop) {
    typedef typename St<S>::C C;
    typedef P2<S> G;
    constexpr int BX = G::BX, BY = G::BY, CX = G::CX, CY = G::CY, NT = G::ND;
    constexpr int WF = G::w(BX, 6), WX = G::w(BX, 5), WR = G::w(BX, 4), WG = G::w(CX, 2), WY = G::w(CX, 1);
    constexpr int RF = WF * G::w(BY, 6), RX = WX * G::w(BY, 5), RR = WR * G::w(BY, 4), RG = WG * G::w(CY, 2),
                  RY = WY * G::w(CY, 1);
    __shared__ C F[RF], X[RX], Rr[RR], Gf[RG], Y[RY], Rb[CX * CY];
    const int halt = stop ? *stop : 0;
    const int n = 1 << lg, nb = n >> 1, t = int(threadIdx.x);
    const int nbx = n / BX, blk = int(xcd_block(blockIdx.x, gridDim.x));
    const int x0 = (blk % nbx) * BX, y0 = (blk / nbx) * BY, X0 = x0 >> 1, Y0 = y0 >> 1;
    constexpr int PF = (RF + NT - 1) / NT;
    C fv[PF];
#pragma unroll
    for (int u = 0; u < PF; ++u) {
        int a, b, s = 1;
        region_pos2(min(t + u * NT, RF - 1), WF, 6, a, b);
        const int gi = bmap(x0 + a, n, bc, s), gj = bmap(y0 + b, n, bc, s);
        fv[u] = C(s) * St<S>::ld(fa + (int64_t(gj) << lg) + gi);
    }
    landed(fv);
    if (halt) return;
#pragma unroll
    for (int u = 0; u < PF; ++u)
        if (t + u * NT < RF) F[t + u * NT] = fv[u];
    __syncthreads();
    for (int e = t; e < RX; e += NT) {
        int a, b;
        region_pos2(e, WX, 5, a, b);
        const bool own = a >= 0 && a < BX && b >= 0 && b < BY;
        const int sgn = mirror_pos2(a, b, x0, y0, n, bc);
        const C v = C(sgn) * pair_zero2<S>(F, WF, 6, a, b, oa);
        X[e] = v;
        if (own) St<S>::st(xa + (int64_t(y0 + b) << lg) + x0 + a, v);
    }
    __syncthreads();
    for (int e = t; e < RR; e += NT) {
        int a, b;
        region_pos2(e, WR, 4, a, b);
        const int q = (b + 5) * WX + a + 5;
        Rr[e] = oa.resid(F[(b + 6) * WF + a + 6], X[q], X[q - 1], X[q + 1], X[q - WX], X[q + WX]);
    }
    __syncthreads();
    if (t < RG) {
        int a, b;
        region_pos2(t, WG, 2, a, b);
        const bool own = a >= 0 && a < CX && b >= 0 && b < CY;
        const int sgn = mirror_pos2(a, b, X0, Y0, nb, bc);
        C r = C(0);
#pragma unroll
        for (int cy = 0; cy < 2; ++cy)
#pragma unroll
            for (int cx = 0; cx < 2; ++cx) r += Rr[(2 * b + cy + 4) * WR + 2 * a + cx + 4];
        const C v = st_round<S>(r * C(0.25));
        Gf[t] = C(sgn) * v;
        if (own) St<S>::st(fb + (int64_t(Y0 + b) << (lg - 1)) + X0 + a, v);
    }
    __syncthreads();
    if (t < RY) {
        int a, b;
        region_pos2(t, WY, 1, a, b);
        const bool own = a >= 0 && a < CX && b >= 0 && b < CY;
        const int sgn = mirror_pos2(a, b, X0, Y0, nb, bc);
        const C v = C(sgn) * pair_zero2<S>(Gf, WG, 2, a, b, ob);
        Y[t] = v;
        if (own) St<S>::st(xb + (int64_t(Y0 + b) << (lg - 1)) + X0 + a, v);
    }
    __syncthreads();
    if (t < CX * CY) {
        const int a = t % CX, b = t / CX, q = (b + 1) * WY + a + 1;
        Rb[t] = ob.resid(Gf[(b + 2) * WG + a + 2], Y[q], Y[q - 1], Y[q + 1], Y[q - WY], Y[q + WY]);
    }
    __syncthreads();
    if (t < CX * CY / 4) {
        const int I = t % (CX / 2), J = t / (CX / 2);
        C r = C(0);
#pragma unroll
        for (int cy = 0; cy < 2; ++cy)
#pragma unroll
            for (int cx = 0; cx < 2; ++cx) r += Rb[(2 * J + cy) * CX + 2 * I + cx];
        St<S>::st(fc + (int64_t((Y0 >> 1) + J) << (lg - 2)) + (X0 >> 1) + I, r * C(0.25));
    }
}

// x + P e at (a, b) of a block at (x0, y0): terms and order of pro_cell; E has its block's origin at (ring, ring).
template <class S, class C>
__device__ __forceinline__ C pair_corr(C x, const C *E, int W, int ring, int a, int b, int x0, int y0) {
    const int fx = x0 + a, fy = y0 + b;
    const int oi = (fx >> 1) - (x0 >> 1) + ring, ni = oi + ((fx & 1) ? 1 : -1);
    const int oj = (fy >> 1) - (y0 >> 1) + ring, nj = oj + ((fy & 1) ? 1 : -1);
    C p = C(0);
#pragma unroll
    for (int bb = 0; bb < 2; ++bb)
#pragma unroll
        for (int aa = 0; aa < 2; ++aa) {
            const C w = C(aa ? 0.25 : 0.75) * C(bb ? 0.25 : 0.75) * C(1.0);
            p = np_fma(w, E[(bb ? nj : oj) * W + (aa ? ni : oi)], p);
        }
    return st_round<S>(x + p);
}

// Up-legs of both levels from the correction ec of the level below them; xo: the finer level's result.
template <class S, class OP>
__global__ __launch_bounds__(P2<S>::NU) void k_pair_up(const S *__restrict__ ec, const S *__restrict__ fb,
                                                       const S *__restrict__ xb, const S *__restrict__ fa,
                                                       const S *__restrict__ xa, S *__restrict__ xo, int lg, int bc,
                                                       OP oa, OP ob, const int *stop) {
    typedef typename St<S>::C C;
    typedef P2<S> G;
    constexpr int BX = G::BX, BY = G::BY, CX = G::CX, CY = G::CY, NT = G::NU;
    constexpr int WE = G::w(CX / 2, 3), W4 = G::w(CX, 4), W3 = G::w(CX, 3), W2c = G::w(CX, 2), V2 = G::w(BX, 2),
                  V1 = G::w(BX, 1);
    constexpr int RE = WE * G::w(CY / 2, 3), R4 = W4 * G::w(CY, 4), R3 = W3 * G::w(CY, 3), R2 = W2c * G::w(CY, 2),
                  Q2 = V2 * G::w(BY, 2), Q1 = V1 * G::w(BY, 1);
    static_assert(Q2 <= NT && R4 <= NT, "a cell of a region per thread");
    __shared__ C E[RE], Xb[R4], Gf[R3], S1[R3], S2[R2], Xa[Q2], F[Q1], A1[Q1];
    const int halt = stop ? *stop : 0;
    const int n = 1 << lg, nb = n >> 1, nc = n >> 2, t = int(threadIdx.x);
    const int nbx = n / BX, blk = int(xcd_block(blockIdx.x, gridDim.x));
    const int x0 = (blk % nbx) * BX, y0 = (blk / nbx) * BY, X0 = x0 >> 1, Y0 = y0 >> 1;
    // this thread's cell of a field on a region (clamped past its end)
    auto load = [&](const S *p, int l, int m, int rw, int W, int ring, int bx, int by) -> C {
        int a, b, s = 1;
        region_pos2(min(t, rw - 1), W, ring, a, b);
        const int gi = bmap(bx + a, m, bc, s), gj = bmap(by + b, m, bc, s);
        return C(s) * St<S>::ld(p + (int64_t(gj) << l) + gi);
    };
    C v[5] = {load(ec, lg - 2, nc, RE, WE, 3, X0 >> 1, Y0 >> 1), load(xb, lg - 1, nb, R4, W4, 4, X0, Y0),
              load(fb, lg - 1, nb, R3, W3, 3, X0, Y0), load(xa, lg, n, Q2, V2, 2, x0, y0),
              load(fa, lg, n, Q1, V1, 1, x0, y0)};
    landed(v);
    if (halt) return;
    if (t < RE) E[t] = v[0];
    if (t < R4) Xb[t] = v[1];
    if (t < R3) Gf[t] = v[2];
    if (t < Q2) Xa[t] = v[3];
    if (t < Q1) F[t] = v[4];
    __syncthreads();
    // the coarser level: x' on four rings (each thread's own cell, through a register as mirrors read others)
    C c = C(0);
    int a = 0, b = 0, sgn = 1;
    if (t < R4) {
        region_pos2(t, W4, 4, a, b);
        sgn = mirror_pos2(a, b, X0, Y0, nb, bc);
        c = C(sgn) * pair_corr<S>(Xb[(b + 4) * W4 + a + 4], E, WE, 3, a, b, X0, Y0);
    }
    __syncthreads();
    if (t < R4) Xb[t] = c;
    __syncthreads();
    if (t < R3) {
        region_pos2(t, W3, 3, a, b);
        sgn = mirror_pos2(a, b, X0, Y0, nb, bc);
        const int q = (b + 4) * W4 + a + 4;
        const C xc = Xb[q];
        const C r = ob.resid(Gf[(b + 3) * W3 + a + 3], xc, Xb[q - 1], Xb[q + 1], Xb[q - W4], Xb[q + W4]);
        S1[t] = C(sgn) * st_round<S>(xc + ob.wd * r);
    }
    __syncthreads();
    if (t < R2) {
        region_pos2(t, W2c, 2, a, b);
        sgn = mirror_pos2(a, b, X0, Y0, nb, bc);
        const int q = (b + 3) * W3 + a + 3;
        const C xc = S1[q];
        const C r = ob.resid(Gf[q], xc, S1[q - 1], S1[q + 1], S1[q - W3], S1[q + W3]);
        S2[t] = C(sgn) * st_round<S>(xc + ob.wd * r);
    }
    __syncthreads();
    // the finer level
    if (t < Q2) {
        region_pos2(t, V2, 2, a, b);
        sgn = mirror_pos2(a, b, x0, y0, n, bc);
        c = C(sgn) * pair_corr<S>(Xa[(b + 2) * V2 + a + 2], S2, W2c, 2, a, b, x0, y0);
    }
    __syncthreads();
    if (t < Q2) Xa[t] = c;
    __syncthreads();
    if (t < Q1) {
        region_pos2(t, V1, 1, a, b);
        sgn = mirror_pos2(a, b, x0, y0, n, bc);
        const int q = (b + 2) * V2 + a + 2;
        const C xc = Xa[q];
        const C r = oa.resid(F[(b + 1) * V1 + a + 1], xc, Xa[q - 1], Xa[q + 1], Xa[q - V2], Xa[q + V2]);
        A1[t] = C(sgn) * st_round<S>(xc + oa.wd * r);
    }
    __syncthreads();
    if (t < BX * BY) {
        const int ax = t % BX, by = t / BX, q = (by + 1) * V1 + ax + 1;
        const C xc = A1[q];
        const C r = oa.resid(F[q], xc, A1[q - 1], A1[q + 1], A1[q - V1], A1[q + V1]);
        St<S>::st(xo + (int64_t(y0 + by) << lg) + x0 + ax, xc + oa.wd * r);
    }
}

}  // namespace np
