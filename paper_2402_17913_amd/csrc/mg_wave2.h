// One-pass legs of a large 2D level on row-marching wavefronts.  A wavefront
// owns 64 CPL consecutive columns (CPL cells per lane, one 16-byte access per
// row in FP64 and FP32, 8 bytes in BF16) and marches a chunk of rows on its
// own: every stage of the leg is a register pipeline one row behind the stage
// it reads, column neighbours come from the adjacent lanes (DPP wavefront
// shifts), and nothing goes through LDS or waits at a barrier.  The outermost
// lanes are ghosts: each stage is exact on one cell less per side than the
// stage before it, and only the inner lanes store.
//  - MODE 0 (down-leg from a zero iterate): two sweeps from zero (the first,
//    w f, formed where the second reads it), the residual and its restriction;
//  - MODE 1 (down-leg of an iterate): two sweeps, the residual and its
//    restriction; NORM also sums |f - A x|^2 of the input iterate;
//  - MODE 2 (up-leg): prolongation + correction, formed where the first sweep
//    reads it and rounded to storage, and both post-sweeps;
//  - MODE 3: MODE 2 of one cycle and MODE 1 of the next in one pass, for the
//    finest level of consecutive cycles.
// What bounds it: memory.  A leg reads its operands once (ghost lanes 3 or 6%,
// four to six rows per chunk again) against three or more passes of the
// per-stage kernels, and keeps four rows of every operand in flight per wave.
// Measured, whole solves against the per-stage kernels: 2048^2 Poisson FP64 3.03
// -> 1.76 ms, 4096^2 twelve FP64 cycles 9.83 -> 4.06 ms, 4096^2 advection-diffusion
// 11.9 -> 5.83 ms; at 1024^2 against blocks a projection step 1.33 -> 1.26 ms.
// MODE 3 for MODE 2 and MODE 1: twelve FP64 cycles at 4096^2 3.93 -> 3.36 ms.
// A value outside the grid is minus the cell's own value of that stage
// (Dirichlet; selected next to the wall, never computed) or the wrapped cell's
// (periodic: wrapped lanes and rows are computed like any other).  Terms, their
// order and the points of rounding are those of k_lvl2_b (Poisson) and of
// ad_ax (advection-diffusion).
#pragma once

#include "mg_block2.h"

namespace np {

// The value of the lane below / above (lane 0's and lane 63's are not used: they are ghosts).
__device__ __forceinline__ uint32_t lane_dn(uint32_t v) {
    return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x138, 0xf, 0xf, true));  // wave_shr:1
}
__device__ __forceinline__ uint32_t lane_up(uint32_t v) {
    return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x130, 0xf, 0xf, true));  // wave_shl:1
}
__device__ __forceinline__ float lane_dn(float v) { return __uint_as_float(lane_dn(__float_as_uint(v))); }
__device__ __forceinline__ float lane_up(float v) { return __uint_as_float(lane_up(__float_as_uint(v))); }
__device__ __forceinline__ double lane_dn(double v) {
    return __hiloint2double(int(lane_dn(uint32_t(__double2hiint(v)))), int(lane_dn(uint32_t(__double2loint(v)))));
}
__device__ __forceinline__ double lane_up(double v) {
    return __hiloint2double(int(lane_up(uint32_t(__double2hiint(v)))), int(lane_up(uint32_t(__double2loint(v)))));
}

// N adjacent values of a field in storage S at an index that is a multiple of N.
template <class S, int N> struct Run {
    typedef typename St<S>::C C;
    static __device__ __forceinline__ void ld(const S *p, C (&v)[N]) {
        if constexpr (N == 1) {
            v[0] = St<S>::ld(p);
        } else if constexpr (N == 2) {
            Pair<S>::ld(p, v[0], v[1]);
        } else if constexpr (sizeof(S) == 4) {
            const float4 q = *reinterpret_cast<const float4 *>(p);
            v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
        } else {
            const uint2 q = *reinterpret_cast<const uint2 *>(p);
            v[0] = __uint_as_float(q.x << 16);
            v[1] = __uint_as_float(q.x & 0xffff0000u);
            v[2] = __uint_as_float(q.y << 16);
            v[3] = __uint_as_float(q.y & 0xffff0000u);
        }
    }
    static __device__ __forceinline__ void st(S *p, const C (&v)[N]) {
        if constexpr (N == 1) {
            St<S>::st(p, v[0]);
        } else if constexpr (N == 2) {
            Pair<S>::st(p, v[0], v[1]);
        } else if constexpr (sizeof(S) == 4) {
            *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
        } else {
            *reinterpret_cast<uint2 *>(p) = make_uint2(float2_to_bf16x2(v[0], v[1]), float2_to_bf16x2(v[2], v[3]));
        }
    }
};

// Columns: CPL cells per lane (16 bytes in FP64 and FP32); GL ghost lanes per
// side.  MODE 0 reads two cells beyond its own, MODE 1 three, MODE 2 two,
// whose outer one takes the coarse value of the lane beyond when CPL is 2, and
// MODE 3 five.
template <class S, int MODE> struct W2 {
    static constexpr int CPL = sizeof(S) == 8 ? 2 : 4;
    static constexpr int GL = MODE == 3 ? (CPL == 2 ? 3 : 2) : (MODE != 0 && CPL == 2 ? 2 : 1);
};
template <int I> using Row = std::integral_constant<int, I>;  // a step of an unrolled row loop
constexpr int kW2T = 256;  // threads per workgroup: four wavefronts on adjacent strips

// Strips of an n x n level: `gl` ghost lanes per side, none where one wavefront
// spans the level from wall to wall.
struct W2Strips {
    int gl, cols, count;  // ghost lanes per side, columns a strip stores, strips
};
template <class S, int MODE> __host__ __device__ __forceinline__ W2Strips w2_strips(int n, int bc) {
    typedef W2<S, MODE> G;
    const int gl = !bc && n <= 64 * G::CPL ? 0 : G::GL, cols = (64 - 2 * gl) * G::CPL;
    return W2Strips{gl, cols, (n + cols - 1) / cols};
}

// One wavefront's chunk of a leg: the columns from c0 on (gl ghost lanes per side),
// rows [j0, j1), both even, of an n x n level (n = 2^lg); returns its share of
// |f - A x|^2 (NORM).
template <class S, class OP, int MODE, bool NORM>
__device__ __forceinline__ double wave2_leg(const S *__restrict__ ec, const S *__restrict__ f,
                                            const S *__restrict__ xin, S *__restrict__ xout, S *__restrict__ fc,
                                            int lg, int bc, int c0, int gl, int j0, int j1,
                                            const OP &op, S *__restrict__ xmid = nullptr) {
    typedef typename St<S>::C C;
    typedef W2<S, MODE> G;
    constexpr int N = G::CPL, NC = N / 2;
    typedef Run<S, N> V;
    const int n = 1 << lg, last = n - 1, lane = int(threadIdx.x) & 63;
    const int col = c0 + (lane - gl) * N;  // first column of this lane
    const bool own = lane >= gl && lane < 64 - gl && col < n;
    // periodic: ghost columns wrap; Dirichlet: columns outside are loaded from the nearest cells, unused
    const int lc = bc ? (col & last) : min(max(col, 0), n - N);
    const bool west = !bc && col == 0, east = !bc && col + N == n;
    auto rowp = [&](int r) -> uint32_t {  // offset of row r (mapped as the columns are)
        const int q = bc ? (r & last) : min(max(r, 0), last);
        return (uint32_t(q) << lg) + uint32_t(lc);
    };
    // the residual of one row of a stage: own values v, rows below and above (ghost rows at the walls)
    auto resid = [&](const C (&v)[N], const C (&vm)[N], const C (&vp)[N], const C (&fv)[N], bool south, bool north,
                     C (&r)[N]) {
        const C l = lane_dn(v[N - 1]), u = lane_up(v[0]);
        const C xl = west ? -v[0] : l, xr = east ? -v[N - 1] : u;
#pragma unroll
        for (int c = 0; c < N; ++c) {
            const C xm = c > 0 ? v[c > 0 ? c - 1 : 0] : xl, xp = c < N - 1 ? v[c < N - 1 ? c + 1 : 0] : xr;
            const C ym = south ? -v[c] : vm[c], yp = north ? -v[c] : vp[c];
            r[c] = op.resid(fv[c], v[c], xm, xp, ym, yp);
        }
    };
    const bool dir = !bc;
    double acc = 0.0;
    // residual sums of an even row's column pairs; two scalars, as an array that the lambda keeps goes to
    // scratch in FP32, and waiting for it waits for every row on its way
    // (2048^2 FP32 solve 1490 -> 1453 us)
    C pa0 = C(0), pa1 = C(0);
    auto restrict_row = [&](int r, const C (&rv)[N]) {  // row r of the residual, in order
        if (r < j0 || r >= j1) return;
        if (!(r & 1)) {
            pa0 = rv[0] + rv[1];
            if constexpr (NC == 2) pa1 = rv[2] + rv[3];
        } else {
            C o[NC];
            o[0] = ((pa0 + rv[0]) + rv[1]) * C(0.25);
            if constexpr (NC == 2) o[1] = ((pa1 + rv[2]) + rv[3]) * C(0.25);
            if (own) Run<S, NC>::st(fc + ((uint32_t(r >> 1) << (lg - 1)) + uint32_t(col >> 1)), o);
        }
    };
    C F[MODE == 3 ? 12 : 6][N];
    // the correction of modes 2 and 3: coarse values in E, x' = x + P ec of row q into x, where eo and en are
    // the coarse rows of q and its neighbour
    [[maybe_unused]] const int lgc = lg - 1, nc = n >> 1, lastc = nc - 1, colc = col >> 1;  // col: a multiple of N
    [[maybe_unused]] const int lcc = bc ? (colc & lastc) : min(max(colc, 0), nc - NC);
    auto rowc = [&](int r) -> uint32_t {
        const int q = bc ? (r & lastc) : min(max(r, 0), lastc);
        return (uint32_t(q) << lgc) + uint32_t(lcc);
    };
    typedef Run<S, NC> VC;
    auto correct = [&](int q, const C (&eo)[NC], const C (&en)[NC], C (&x)[N]) {
        const C w00 = C(0.75) * C(0.75) * C(1.0), w01 = C(0.25) * C(0.75) * C(1.0);
        const C w10 = C(0.75) * C(0.25) * C(1.0), w11 = C(0.25) * C(0.25) * C(1.0);
        const bool g = dir && (q == 0 || q == last);  // neighbour row outside: minus the own row
        C e[NC], h[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            e[c] = eo[c];
            h[c] = g ? -eo[c] : en[c];
        }
        const C el = lane_dn(e[NC - 1]), er = lane_up(e[0]), hl = lane_dn(h[NC - 1]), hr = lane_up(h[0]);
#pragma unroll
        for (int c = 0; c < N; ++c) {
            const int k = c >> 1;
            C a, b;  // the neighbour coarse column's values
            if (!(c & 1)) {
                a = k > 0 ? e[k > 0 ? k - 1 : 0] : (west ? -e[0] : el);
                b = k > 0 ? h[k > 0 ? k - 1 : 0] : (west ? -h[0] : hl);
            } else {
                a = k < NC - 1 ? e[k < NC - 1 ? k + 1 : 0] : (east ? -e[NC - 1] : er);
                b = k < NC - 1 ? h[k < NC - 1 ? k + 1 : 0] : (east ? -h[NC - 1] : hr);
            }
            C p = np_fma(w00, e[k], C(0));
            p = np_fma(w01, a, p);
            p = np_fma(w10, h[k], p);
            p = np_fma(w11, b, p);
            x[c] = st_round<S>(x[c] + p);
        }
    };
    if constexpr (MODE == 0) {
        // step z: second sweep of row z from w f of rows z - 1 .. z + 1, residual of row z - 1
        C B[3][N];
        const int z0 = j0 - 1, z1 = j1 + 1;
#pragma unroll
        for (int q = 0; q < 6; ++q) V::ld(f + rowp(z0 - 1 + q), F[q]);
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int c = 0; c < N; ++c) B[q][c] = C(0);
        for (int zz = z0; zz < z1; zz += 6) {
#pragma unroll
            for (int u = 0; u < 6; ++u) {
                const int z = zz + u;
                if (z >= z1) break;
                C xm[N], xc[N], xp[N], r[N];
#pragma unroll
                for (int c = 0; c < N; ++c) {
                    xm[c] = op.wd * F[u][c];
                    xc[c] = op.wd * F[(u + 1) % 6][c];
                    xp[c] = op.wd * F[(u + 2) % 6][c];
                }
                resid(xc, xm, xp, F[(u + 1) % 6], dir && z == 0, dir && z == last, r);
                C(&b)[N] = B[u % 3];
#pragma unroll
                for (int c = 0; c < N; ++c) b[c] = st_round<S>(xc[c] + op.wd * r[c]);
                if (own && z >= j0 && z < j1) V::st(xout + ((uint32_t(z) << lg) + uint32_t(col)), b);
                if (z > j0) {
                    resid(B[(u + 2) % 3], B[(u + 1) % 3], b, F[u], dir && z == 1, dir && z == n, r);
                    restrict_row(z - 1, r);
                }
                V::ld(f + rowp(min(z + 5, j1 + 1)), F[u]);
            }
        }
    } else if constexpr (MODE == 1) {
        // step z: first sweep of row z, second of row z - 1, residual of row z - 2
        C X[6][N], A[3][N], B[3][N];
        const int z0 = j0 - 2, z1 = j1 + 2;
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            V::ld(xin + rowp(z0 - 1 + q), X[q]);
            V::ld(f + rowp(z0 - 2 + q), F[q]);
        }
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int c = 0; c < N; ++c) A[q][c] = B[q][c] = C(0);
        for (int zz = z0; zz < z1; zz += 6) {
#pragma unroll
            for (int u = 0; u < 6; ++u) {
                const int z = zz + u;
                if (z >= z1) break;
                C r[N];
                resid(X[(u + 1) % 6], X[u], X[(u + 2) % 6], F[(u + 2) % 6], dir && z == 0, dir && z == last, r);
                if (NORM && own && z >= j0 && z < j1) {
#pragma unroll
                    for (int c = 0; c < N; ++c) acc += double(r[c]) * double(r[c]);
                }
                C(&a)[N] = A[u % 3];
#pragma unroll
                for (int c = 0; c < N; ++c) a[c] = st_round<S>(X[(u + 1) % 6][c] + op.wd * r[c]);
                V::ld(xin + rowp(min(z + 5, j1 + 2)), X[u]);
                if (z >= j0) {
                    const C(&am)[N] = A[(u + 2) % 3];  // first sweep of row z - 1
                    resid(am, A[(u + 1) % 3], a, F[(u + 1) % 6], dir && z == 1, dir && z == n, r);
                    C(&b)[N] = B[u % 3];
#pragma unroll
                    for (int c = 0; c < N; ++c) b[c] = st_round<S>(am[c] + op.wd * r[c]);
                    if (own && z > j0 && z <= j1) V::st(xout + ((uint32_t(z - 1) << lg) + uint32_t(col)), b);
                    if (z > j0 + 1) {
                        resid(B[(u + 2) % 3], B[(u + 1) % 3], b, F[u], dir && z == 2, dir && z == n + 1, r);
                        restrict_row(z - 2, r);
                    }
                }
                V::ld(f + rowp(min(z + 4, j1 + 1)), F[u]);
            }
        }
    } else if constexpr (MODE == 2) {
        // step z: x' of row z + 1, first sweep of row z, second of row z - 1 (stored)
        C X[6][N], A[3][N];
        const int z0 = j0 - 3, z1 = j1 + 1;
        C E[3][NC];
        const int K0 = (j0 - 2) >> 1;
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            V::ld(xin + rowp(z0 - 1 + q), X[q]);
            V::ld(f + rowp(z0 - 1 + q), F[q]);
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) VC::ld(ec + rowc(K0 - 1 + q), E[q]);
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int c = 0; c < N; ++c) A[q][c] = C(0);
        for (int zz = z0; zz < z1; zz += 6) {
#pragma unroll
            for (int u = 0; u < 6; ++u) {
                const int z = zz + u;
                if (z >= z1) break;
                // x' of row q = z + 1 (q even at even u): coarse rows K = q / 2 and its neighbour
                {
                    constexpr int dn[6] = {0, 2, 1, 0, 2, 1};  // slot of the neighbour row
                    const int q = z + 1;
                    correct(q, E[((u >> 1) + 1) % 3], E[dn[u]], X[(u + 2) % 6]);
                    if (u & 1) VC::ld(ec + rowc(min((q >> 1) + 2, (j1 >> 1) + 1)), E[(u >> 1) % 3]);
                }
                if (z >= j0 - 1) {
                    C r[N];
                    resid(X[(u + 1) % 6], X[u], X[(u + 2) % 6], F[(u + 1) % 6], dir && z == 0, dir && z == last, r);
                    C(&a)[N] = A[u % 3];
#pragma unroll
                    for (int c = 0; c < N; ++c) a[c] = st_round<S>(X[(u + 1) % 6][c] + op.wd * r[c]);
                    if (z > j0) {
                        const C(&am)[N] = A[(u + 2) % 3];
                        resid(am, A[(u + 1) % 3], a, F[u], dir && z == 1, dir && z == n, r);
                        C o[N];
#pragma unroll
                        for (int c = 0; c < N; ++c) o[c] = am[c] + op.wd * r[c];
                        if (own) V::st(xout + ((uint32_t(z - 1) << lg) + uint32_t(col)), o);
                    }
                }
                V::ld(xin + rowp(min(z + 5, j1 + 1)), X[u]);
                V::ld(f + rowp(min(z + 5, j1)), F[u]);
            }
        }
    } else {
        // the up-leg of one cycle and the down-leg of the next.  Step z: x' of row z + 1; post-sweeps of rows z and
        // z - 1 (the cycle's iterate, to xmid where that is asked for); its residual norm and the first pre-sweep of
        // row z - 2; the second of row z - 3 (stored); the residual of row z - 4
        C X[6][N], A[3][N], B[3][N], P[3][N], Q[3][N], E[3][NC];
        const int z0 = j0 - 7, z1 = j1 + 4, K0 = (j0 - 6) >> 1;
#pragma unroll
        for (int q = 0; q < 6; ++q) V::ld(xin + rowp(z0 - 1 + q), X[q]);
#pragma unroll
        for (int q = 0; q < 7; ++q) V::ld(f + rowp(z0 + q), F[q]);
#pragma unroll
        for (int q = 0; q < 3; ++q) VC::ld(ec + rowc(K0 - 1 + q), E[q]);
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int c = 0; c < N; ++c) A[q][c] = B[q][c] = P[q][c] = Q[q][c] = C(0);
#pragma unroll
        for (int q = 7; q < 12; ++q)
#pragma unroll
            for (int c = 0; c < N; ++c) F[q][c] = C(0);
        auto step = [&](int z, auto uc) __attribute__((always_inline)) {
            constexpr int u = decltype(uc)::value;
            constexpr int dn[6] = {0, 2, 1, 0, 2, 1};  // slot of the neighbour coarse row
            const int q = z + 1;
            correct(q, E[((u >> 1) + 1) % 3], E[dn[u % 6]], X[(u + 2) % 6]);
            if (u & 1) VC::ld(ec + rowc(min((q >> 1) + 2, (j1 >> 1) + 3)), E[(u >> 1) % 3]);
            if (z >= j0 - 5) {
                C r[N];
                // row z - d of a stage is row z - d + 1 of the one before it, at its middle; f of row z - d is
                // F[(u - d) mod 12]
                resid(X[(u + 1) % 6], X[u % 6], X[(u + 2) % 6], F[u], dir && z == 0, dir && z == last, r);
                C(&a)[N] = A[u % 3];
#pragma unroll
                for (int c = 0; c < N; ++c) a[c] = st_round<S>(X[(u + 1) % 6][c] + op.wd * r[c]);
                const C(&am)[N] = A[(u + 2) % 3];
                resid(am, A[(u + 1) % 3], a, F[(u + 11) % 12], dir && z == 1, dir && z == n, r);
                C(&b)[N] = B[u % 3];
#pragma unroll
                for (int c = 0; c < N; ++c) b[c] = st_round<S>(am[c] + op.wd * r[c]);
                if (xmid && own && z > j0 && z <= j1) V::st(xmid + ((uint32_t(z - 1) << lg) + uint32_t(col)), b);
                if (z >= j0) {
                    const C(&bm)[N] = B[(u + 2) % 3];
                    resid(bm, B[(u + 1) % 3], b, F[(u + 10) % 12], dir && z == 2, dir && z == n + 1, r);
                    if (NORM && own && z >= j0 + 2 && z < j1 + 2) {
#pragma unroll
                        for (int c = 0; c < N; ++c) acc += double(r[c]) * double(r[c]);
                    }
                    C(&p)[N] = P[u % 3];
#pragma unroll
                    for (int c = 0; c < N; ++c) p[c] = st_round<S>(bm[c] + op.wd * r[c]);
                    const C(&pm)[N] = P[(u + 2) % 3];
                    resid(pm, P[(u + 1) % 3], p, F[(u + 9) % 12], dir && z == 3, dir && z == n + 2, r);
                    C(&s)[N] = Q[u % 3];
#pragma unroll
                    for (int c = 0; c < N; ++c) s[c] = st_round<S>(pm[c] + op.wd * r[c]);
                    if (own && z >= j0 + 3 && z < j1 + 3) V::st(xout + ((uint32_t(z - 3) << lg) + uint32_t(col)), s);
                    if (z >= j0 + 4) {
                        resid(Q[(u + 2) % 3], Q[(u + 1) % 3], s, F[(u + 8) % 12], dir && z == 4, dir && z == n + 3,
                              r);
                        restrict_row(z - 4, r);
                    }
                }
            }
            V::ld(xin + rowp(min(z + 5, j1 + 4)), X[u % 6]);
            V::ld(f + rowp(min(z + 7, j1 + 3)), F[(u + 7) % 12]);
        };
        auto steps = [&](int zz, auto... uc) __attribute__((always_inline)) {
            ((zz + uc.value < z1 ? step(zz + uc.value, uc) : void()), ...);
        };
        for (int zz = z0; zz < z1; zz += 12)
            steps(zz, Row<0>{}, Row<1>{}, Row<2>{}, Row<3>{}, Row<4>{}, Row<5>{}, Row<6>{}, Row<7>{}, Row<8>{}, Row<9>{},
                  Row<10>{}, Row<11>{});
    }
    return acc;
}

// Rows per chunk: even, for about `waves` wavefronts over the level, at least `least` (a chunk computes
// two to four rows beyond its own): 8, or 4 in BF16, whose rows carry half the bytes (four BF16
// refinement steps at 1024^2 750 -> 724 us; FP32 and FP64 the same or slower).
inline int wave2_rows(int n, int64_t strips, int waves, int least = 8) {
    int64_t ry = (int64_t(n) * strips + waves - 1) / waves;
    ry = (ry + 1) & ~int64_t(1);
    return int(ry < least ? (n < least ? n : least) : (ry > n ? n : ry));
}

// A leg of one n x n level; ry rows per wavefront.  Wavefront w takes strip
// w mod strips of chunk w / strips, so the four of a workgroup share the lines
// at their strips' edges.
template <class S, class OP, int MODE, bool NORM>
__global__ __launch_bounds__(kW2T) void k_wave2(const S *__restrict__ ec, const S *__restrict__ f,
                                                const S *__restrict__ xin, S *__restrict__ xout, S *__restrict__ fc,
                                                double *__restrict__ partial, int lg, int bc, int ry, OP op,
                                                const int *stop, S *__restrict__ xmid) {
    if (stop && *stop) return;
    const int n = 1 << lg;
    const W2Strips t = w2_strips<S, MODE>(n, bc);
    const int w = __builtin_amdgcn_readfirstlane(int(xcd_block(blockIdx.x, gridDim.x)) * (kW2T / 64) +
                                                 (int(threadIdx.x) >> 6));
    const int c0 = (w % t.count) * t.cols, j0 = (w / t.count) * ry;
    double acc = 0.0;
    if (j0 < n) acc = wave2_leg<S, OP, MODE, NORM>(ec, f, xin, xout, fc, lg, bc, c0, t.gl, j0, min(j0 + ry, n), op,
                                                 xmid);
    if constexpr (NORM) {
        acc = block_sum_n<kW2T>(acc);
        if (threadIdx.x == 0) partial[blockIdx.x] = acc;
    }
}

}  // namespace np
