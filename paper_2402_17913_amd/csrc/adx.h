// The explicit advection-diffusion step with the paper's filter families: the
// filters, the per-cell predictor and corrector, and the whole step in one pass
// (2D: row-marching wavefronts; 3D: z-marching tiles).  Included by ns.hip.
#pragma once

#include "mg_wave2.h"
#include "np_internal.h"

namespace np {
namespace {

struct APtrs {
    const double *a[3];
    int has;
};

// ------------------------------------- explicit step, filter families
// The filters of Section 2.1 and Appendix A on any n >= 3 (all axes equal):
// scheme 0 central (3-point first differences, 5-/7-point diffusion), 1
// first-order upwind advection (the upstream value: backward difference for a
// positive velocity component) with the same diffusion, 2 the finite-element
// (bilinear / trilinear) filters: first derivatives averaged across the other
// axes with weights (1, 4, 1)/6, diffusion 16 delta - (1,2,1)x(1,2,1) over
// 4 h^2 (2D) or 88 / -6 / -3 / -2 on the centre, faces, edges and corners over
// 26 h^2 (3D).  Boundary rule bc: 0 Dirichlet-0 (ghost = -value), 1 periodic,
// 2 zero normal derivative (ghost = value, the copy padding of Section 2.4).

// The filters' constants at spacing h and diffusivity nu (products, not quotients, per cell).
struct AdxK {
    double nu, i2h, ih, ih2, c12, c72, d4, d26;  // 1/2h, 1/h, 1/h^2, 1/12h, 1/72h, 1/4h^2, 1/26h^2
};
inline AdxK adx_consts(double nu, double h) {
    return AdxK{nu, 0.5 / h, 1.0 / h, 1.0 / (h * h), 1.0 / (12.0 * h), 1.0 / (72.0 * h), 1.0 / (4.0 * h * h),
                1.0 / (26.0 * h * h)};
}

// Index along one axis of the cell q (at most one cell outside [0, n)) and the
// sign its value takes.
__device__ __forceinline__ int adx_res(int q, int n, int bc, double &sg) {
    sg = 1.0;
    if (q < 0) {
        if (bc == 1) return n - 1;
        if (bc == 0) sg = -1.0;
        return 0;
    }
    if (q >= n) {
        if (bc == 1) return 0;
        if (bc == 0) sg = -1.0;
        return n - 1;
    }
    return q;
}

constexpr int kAdxX = 64, kAdxY = 4;  // workgroup: 64 cells along x, 4 rows

// The 3^d neighbourhood v[dz + 1][dy + 1][dx + 1] of cell (i, j, k) of F
// (HALF: of (F + G)/2) with the boundary rule; the 5/7-point families load
// the face neighbours only (the other entries stay zero).
template <int D, int SCHEME, bool HALF>
__device__ __forceinline__ void adx_gather(const double *__restrict__ F, const double *__restrict__ G, int i, int j,
                                           int k, int n, int bc, double (&v)[3][3][3]) {
    const int64_t nn = n;
    int ix[3];
    double sx[3];
    for (int o = 0; o < 3; ++o) ix[o] = adx_res(i + o - 1, n, bc, sx[o]);
#pragma unroll
    for (int dz = -1; dz <= 1; ++dz) {
        if (D == 2 && dz != 0) continue;
        double sz = 1.0;
        const int kk = D == 3 ? adx_res(k + dz, n, bc, sz) : 0;
#pragma unroll
        for (int dy = -1; dy <= 1; ++dy) {
            double sy;
            const int jj = adx_res(j + dy, n, bc, sy);
            const int64_t row = (int64_t(kk) * nn + jj) * nn;
#pragma unroll
            for (int dx = -1; dx <= 1; ++dx) {
                if (SCHEME != 2 && (dx != 0) + (dy != 0) + (dz != 0) > 1) continue;  // 5/7-point only
                const int64_t q = row + ix[dx + 1];
                const double t = HALF ? 0.5 * (G[q] + F[q]) : F[q];
                v[dz + 1][dy + 1][dx + 1] = sx[dx + 1] * sy * sz * t;
            }
        }
    }
}

// What a 3D filter takes from one plane of a cell's neighbourhood, so that a kernel marching along z
// forms it once per plane.  Finite elements: the x and y differences averaged across (weights 1, 4, 1),
// the average itself, and the diffusion sums of a middle and of an outer plane; the 7-point families:
// the face neighbours.
template <int SCHEME> struct AdxPlane {
    double c, q[5];
    __device__ __forceinline__ AdxPlane() {}
    __device__ __forceinline__ explicit AdxPlane(const double (&v)[3][3]) {
        c = v[1][1];
        if (SCHEME == 2) {
            double rs[3], rd[3];
#pragma unroll
            for (int y = 0; y < 3; ++y) {
                rs[y] = (v[y][0] + v[y][2]) + 4.0 * v[y][1];
                rd[y] = v[y][2] - v[y][0];
            }
            q[0] = (rd[0] + rd[2]) + 4.0 * rd[1];
            q[1] = rs[2] - rs[0];
            q[2] = (rs[0] + rs[2]) + 4.0 * rs[1];
            const double face = (v[1][0] + v[1][2]) + (v[0][1] + v[2][1]);
            const double corner = (v[0][0] + v[0][2]) + (v[2][0] + v[2][2]);
            q[3] = 88.0 * c - 6.0 * face - 3.0 * corner;
            q[4] = -6.0 * c - 3.0 * face - 2.0 * corner;
        } else {
            q[0] = v[1][0];
            q[1] = v[1][2];
            q[2] = v[0][1];
            q[3] = v[2][1];
            q[4] = 0.0;
        }
    }
    // the same plane with every value multiplied by sg (1 or -1)
    __device__ __forceinline__ AdxPlane signed_by(double sg) const {
        AdxPlane p;
        p.c = sg * c;
#pragma unroll
        for (int i = 0; i < 5; ++i) p.q[i] = sg * q[i];
        return p;
    }
};

// First derivative along axis e from the planes below, at and above the cell.
template <int SCHEME>
__device__ __forceinline__ double adx_deriv3(const AdxPlane<SCHEME> &l, const AdxPlane<SCHEME> &m,
                                             const AdxPlane<SCHEME> &u, int e, const AdxK &K) {
    if (SCHEME == 2) {
        if (e == 2) return (u.q[2] - l.q[2]) * K.c72;
        return ((l.q[e] + u.q[e]) + 4.0 * m.q[e]) * K.c72;
    }
    if (e == 2) return (u.c - l.c) * K.i2h;
    return (m.q[2 * e + 1] - m.q[2 * e]) * K.i2h;
}

// Advection + diffusion of a 5-/7-point family from the face neighbours.
template <int D, int SCHEME>
__device__ __forceinline__ double adx_rate_faces(double v0, const double (&xm)[3], const double (&xp)[3],
                                                 const double (&a)[3], bool has_a, const AdxK &K) {
    double adv = 0.0, lap = 0.0;
#pragma unroll
    for (int e = 0; e < D; ++e) {
        lap += (v0 - xm[e]) + (v0 - xp[e]);
        if (!has_a) continue;
        if (SCHEME == 0) adv += a[e] * ((xp[e] - xm[e]) * K.i2h);
        else adv += a[e] * ((a[e] >= 0.0 ? v0 - xm[e] : xp[e] - v0) * K.ih);
    }
    return adv + K.nu * (lap * K.ih2);
}

template <int SCHEME>
__device__ __forceinline__ double adx_rate3(const AdxPlane<SCHEME> &l, const AdxPlane<SCHEME> &m,
                                            const AdxPlane<SCHEME> &u, const double (&a)[3], bool has_a,
                                            const AdxK &K) {
    if constexpr (SCHEME == 2) {
        const double dif = ((l.q[4] + u.q[4]) + m.q[3]) * K.d26;
        double adv = 0.0;
        if (has_a)
#pragma unroll
            for (int e = 0; e < 3; ++e) adv += a[e] * adx_deriv3<2>(l, m, u, e, K);
        return adv + K.nu * dif;
    } else {
        const double xm[3] = {m.q[0], m.q[2], l.c}, xp[3] = {m.q[1], m.q[3], u.c};
        return adx_rate_faces<3, SCHEME>(m.c, xm, xp, a, has_a, K);
    }
}

// First derivative along axis e of the gathered field: the finite-element
// filter (scheme 2) or the central difference.
template <int D, int SCHEME>
__device__ __forceinline__ double adx_deriv(const double (&v)[3][3][3], int e, const AdxK &K) {
    if constexpr (D == 3) {
        return adx_deriv3<SCHEME>(AdxPlane<SCHEME>(v[0]), AdxPlane<SCHEME>(v[1]), AdxPlane<SCHEME>(v[2]), e, K);
    } else if constexpr (SCHEME == 2) {
        const double w[3] = {1.0, 4.0, 1.0};
        double g = 0.0;
#pragma unroll
        for (int p = 0; p < 3; ++p) g += w[p] * (e == 0 ? v[1][p][2] - v[1][p][0] : v[1][2][p] - v[1][0][p]);
        return g * K.c12;
    } else {
        return (e == 0 ? v[1][1][2] - v[1][1][0] : v[1][2][1] - v[1][0][1]) * K.i2h;
    }
}

// Advection + diffusion rate of the gathered field, a the velocity at the
// cell (used when has_a).
template <int D, int SCHEME>
__device__ __forceinline__ double adx_rate_at(const double (&v)[3][3][3], const double (&a)[3], bool has_a,
                                              const AdxK &K) {
    if constexpr (D == 3) {
        return adx_rate3<SCHEME>(AdxPlane<SCHEME>(v[0]), AdxPlane<SCHEME>(v[1]), AdxPlane<SCHEME>(v[2]), a, has_a, K);
    } else if constexpr (SCHEME == 2) {
        const double b[3] = {1.0, 2.0, 1.0};
        double sm = 0.0, adv = 0.0;
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int q = 0; q < 3; ++q) sm += b[p] * b[q] * v[1][p][q];
        const double dif = (16.0 * v[1][1][1] - sm) * K.d4;
        if (has_a)
#pragma unroll
            for (int e = 0; e < 2; ++e) adv += a[e] * adx_deriv<2, 2>(v, e, K);
        return adv + K.nu * dif;
    } else {
        const double xm[3] = {v[1][1][0], v[1][0][1], 0.0}, xp[3] = {v[1][1][2], v[1][2][1], 0.0};
        return adx_rate_faces<2, SCHEME>(v[1][1][1], xm, xp, a, has_a, K);
    }
}

// STAGE 0: out = (T~ + T)/2, T~ = T - dt R(T); STAGE 1: out = T - dt R(H), H =
// (T~ + T)/2 from stage 0 (out may be T: it is read at the own cell only).  One
// thread per cell; the 3^d neighbourhood is gathered with the boundary rule,
// then every filter of the family reads it.
template <int D, int SCHEME, int STAGE>
__global__ __launch_bounds__(kAdxX * kAdxY) void k_adx_stage(const double *T, const double *__restrict__ H, double *out,
                                                             APtrs ap, int n, int bc, double dt, AdxK K) {
    const int i = int(blockIdx.x) * kAdxX + int(threadIdx.x), j = int(blockIdx.y) * kAdxY + int(threadIdx.y);
    const int k = D == 3 ? int(blockIdx.z) : 0;
    if (i >= n || j >= n) return;
    double v[3][3][3] = {};
    adx_gather<D, SCHEME, false>(STAGE == 1 ? H : T, nullptr, i, j, k, n, bc, v);
    const int64_t c = (int64_t(k) * n + j) * n + i;
    double a[3] = {0.0, 0.0, 0.0};
    if (ap.has)
#pragma unroll
        for (int e = 0; e < D; ++e) a[e] = ap.a[e][c];
    const double t = STAGE == 1 ? T[c] : v[1][1][1];
    const double o = t - dt * adx_rate_at<D, SCHEME>(v, a, ap.has != 0, K);
    out[c] = STAGE == 0 ? 0.5 * (o + t) : o;
}

// ------------------------------------------------- the whole step in one pass
// T <- T - dt R((T~ + T)/2), T~ = T - dt R(T), reading T and the velocity once and
// writing T once: the half-step average H is formed where the corrector reads it
// and never stored.  A tile reads T up to two cells beyond its own, which its
// neighbours overwrite, so those cells come from a copy `scr` made before.

// 2D: a wavefront owns 124 columns (two per lane, a ghost lane
// per side) and marches a chunk of rows, predictor and corrector one row apart in
// registers, column neighbours from adjacent lanes.  Only the cells that another
// wavefront reads are copied: two rows and two columns along each edge of a chunk
// (k_adx_shell2), 15 % of the field at 4096^2.  Bound by memory: 32 bytes
// per cell against 80 for two stages that also copied T.  Measured, a call (central /
// finite element): 4096^2 299 / 299 -> 152 / 150 us (the two kernels 127 / 127 and 17 us; 4.8 TB/s of
// traffic, of which 0.88 is those 32 bytes), 2048^2 74 / 74 -> 56 / 59; from 1280^2 on
// (at 1024^2 34.2 / 35.6 against 31.5 / 35.4 for two launches of one cell per thread).  VEC: n even and 16-byte aligned fields,
// pairs loaded at once.
constexpr int kStep2Min = 1280, kStep2Cols = 124;

// Rows per chunk: about 4096 wavefronts, at least 8.
inline int step2_rows(int n) {
    const int64_t strips = (n + kStep2Cols - 1) / kStep2Cols;
    const int64_t ry = (n * strips + 4095) / 4096;
    return int(ry < 8 ? 8 : ry);
}

__global__ __launch_bounds__(kBlock) void k_adx_shell2(const double *__restrict__ T, double *__restrict__ scr, int n,
                                                       int ry, int strips, int chunks) {
    const int64_t id = int64_t(blockIdx.x) * kBlock + threadIdx.x, rows = int64_t(chunks) * 4 * n;
    int i, j;
    if (id < rows) {
        const int q = int(id / n), ch = q >> 2, r = q & 3, j0 = ch * ry, j1 = min(j0 + ry, n);
        i = int(id % n);
        j = r < 2 ? min(j0 + r, n - 1) : max(j1 + 1 - r, 0);
    } else {
        const int64_t e = id - rows;
        j = int(e / (4 * strips));
        if (j >= n) return;
        const int q = int(e % (4 * strips)), c0 = (q >> 2) * kStep2Cols, c1 = min(c0 + kStep2Cols, n), r = q & 3;
        i = r < 2 ? min(c0 + r, n - 1) : max(c1 + 1 - r, 0);
    }
    const int64_t c = int64_t(j) * n + i;
    scr[c] = T[c];
}

template <int SCHEME, bool VEC>
__global__ __launch_bounds__(kBlock) void k_adx_step2(double *T, const double *__restrict__ scr, APtrs ap, int n, int bc,
                                                      int ry, int strips, double dt, AdxK K) {
    const int lane = int(threadIdx.x) & 63;
    const int w = __builtin_amdgcn_readfirstlane(int(xcd_block(blockIdx.x, gridDim.x)) * (kBlock / 64) +
                                                 (int(threadIdx.x) >> 6));
    const int j0 = (w / strips) * ry, j1 = min(j0 + ry, n);
    if (j0 >= n) return;
    const int col = (w % strips) * kStep2Cols + (lane - 1) * 2, last = n - 1;
    const bool per = bc == 1, lane_own = lane >= 1 && lane < 63, has = ap.has != 0;
    const double gs = bc == 0 ? -1.0 : 1.0;  // a wall's ghost value: gs times the cell's own
    bool own[2], east[2];
    int cc[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int i = col + c;
        own[c] = lane_own && i < n;
        east[c] = !per && i == last;
        cc[c] = per ? (i < 0 ? i + n : (i >= n ? i - n : i)) : min(max(i, 0), last);
    }
    if (VEC) cc[0] = min(cc[0], n - 2);
    const bool west = !per && col == 0;
    const double *src[2] = {own[0] ? (const double *)T : scr, own[1] ? (const double *)T : scr};
    auto rowp = [&](int r) -> int64_t { return int64_t(per ? (r < 0 ? r + n : (r >= n ? r - n : r)) : min(max(r, 0), last)) * n; };
    auto load_t = [&](int r, double (&x)[2]) {
        const int64_t o = rowp(r);
        const bool in = r >= j0 && r < j1;  // the chunk's own rows; another chunk's come from the copy
        if constexpr (VEC) {
            Pair<double>::ld((in ? src[0] : scr) + o + cc[0], x[0], x[1]);
        } else {
            x[0] = (in ? src[0] : scr)[o + cc[0]];
            x[1] = (in ? src[1] : scr)[o + cc[1]];
        }
    };
    auto load_a = [&](int r, double (&x)[2][2]) {
        if (!has) return;
        const int64_t o = rowp(r);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            if constexpr (VEC) {
                Pair<double>::ld(ap.a[e] + o + cc[0], x[e][0], x[e][1]);
            } else {
                x[e][0] = ap.a[e][o + cc[0]];
                x[e][1] = ap.a[e][o + cc[1]];
            }
        }
    };
    // a row of a stage: cell c's left, own and right values at [c][0..2]
    struct Row {
        double v[2][3];
    };
    auto row_of = [&](const double (&x)[2]) -> Row {
        const double l = lane_dn(x[1]), u = lane_up(x[0]);
        Row r;
        r.v[0][0] = west ? gs * x[0] : l;
        r.v[0][1] = x[0];
        r.v[0][2] = !VEC && east[0] ? gs * x[0] : x[1];
        r.v[1][0] = x[0];
        r.v[1][1] = x[1];
        r.v[1][2] = east[1] ? gs * x[1] : u;
        return r;
    };
    // x - dt R at the cells of the row `m` with the rows `l` and `u` around it (ghost rows at the walls)
    auto stage = [&](const Row &l, const Row &m, const Row &u, bool south, bool north, const double (&t)[2],
                     const double (&a)[2][2], double (&o)[2]) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            double v[3][3][3] = {};
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                v[1][0][q] = south ? gs * m.v[c][q] : l.v[c][q];
                v[1][1][q] = m.v[c][q];
                v[1][2][q] = north ? gs * m.v[c][q] : u.v[c][q];
            }
            const double ac[3] = {a[0][c], a[1][c], 0.0};
            o[c] = t[c] - dt * adx_rate_at<2, SCHEME>(v, ac, has, K);
        }
    };
    double X[6][2], A[6][2][2] = {};  // rows z - 2 .. z + 3 of T and of the velocity, slot by slot
    Row R[3], H[3];
    const int z0 = j0 - 2, z1 = j1 + 2;
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        load_t(max(z0 - 2 + q, j0 - 2), X[q]);
        load_a(max(z0 - 2 + q, j0 - 1), A[q]);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) R[q] = H[q] = Row{};
    for (int zz = z0; zz < z1; zz += 6) {
#pragma unroll
        for (int u = 0; u < 6; ++u) {
            const int z = zz + u;
            if (z >= z1) break;
            R[u % 3] = row_of(X[(u + 2) % 6]);
            Row hn = H[u % 3];
            if (z >= j0) {  // predictor of row z - 1
                double o[2], hv[2];
                const double(&t)[2] = X[(u + 1) % 6];
                stage(R[(u + 1) % 3], R[(u + 2) % 3], R[u % 3], !per && z == 1, !per && z == n, t, A[(u + 1) % 6], o);
#pragma unroll
                for (int c = 0; c < 2; ++c) hv[c] = 0.5 * (o[c] + t[c]);
                hn = row_of(hv);
            }
            if (z >= j0 + 2) {  // corrector of row z - 2: H of rows z - 3, z - 2, z - 1
                double o[2];
                stage(H[(u + 1) % 3], H[(u + 2) % 3], hn, !per && z == 2, !per && z == n + 1, X[u], A[u], o);
                double *d = T + int64_t(z - 2) * n + col;
                if constexpr (VEC) {
                    if (own[0]) Pair<double>::st(d, o[0], o[1]);
                } else {
                    if (own[0]) d[0] = o[0];
                    if (own[1]) d[1] = o[1];
                }
            }
            H[u % 3] = hn;
            load_t(min(z + 4, j1 + 1), X[u]);
            load_a(min(z + 4, j1), A[u]);
        }
    }
}

// 3D: a workgroup of kSt threads owns a kSx x kSy column tile and zc planes, one
// plane of T per step: the plane, with a two-cell ring, goes to LDS; each thread
// forms what the filter takes from it (AdxPlane) at one cell of the tile or of
// the one-cell ring around it, and from the last three planes the predictor's H
// of the plane before, which goes to LDS; the threads of the tile's own cells
// run the corrector two planes behind on the same sums of H.  So a plane's nine
// values are read from LDS once per stage, where a gathered neighbourhood
// reads 27.  One barrier per step (two slots per LDS plane).  One cell per thread and 64 x 13
// tiles (66 x 15 with the ring: 990 of 1024 threads) keep 16 waves on a CU; two
// cells on the first waves of a 64 x 8 tile took 176 registers, 8 waves and 316 us a call at
// 256^3.  Measured, a call (central / finite element), the copy included: 256^3 350 / 389 ->
// 234 / 254 us, 192^3 161 / 192 -> 117 / 127.  A ring cell outside the grid is formed at the cell it mirrors,
// which the tile and its ring hold.
constexpr int kSx = 64, kSy = 13, kSt = 1024;

// How a 3D step runs: two launches of one cell per thread (k_adx_stage), two launches on z-marching tiles
// (k_adx_stage3z), or one pass.  Cells are best while a stage is little more than a launch, for the 27-point family
// only up to 64^3, which fills its rows of 64 cells.  One pass moves 32 bytes per cell and 8 per velocity component
// where two launches move 40 and 16, but computes rings and waits at a barrier per plane; it pays where the fields
// leave the caches.  Measured, us a call (cells / tiles / one pass; periodic, central or finite element):
//   with a velocity, central: 96^3 36 / 40 / 44, 128^3 54 / 50 / 53, 160^3 77 / 76 / 85, 192^3 130 / 120 / 122,
//     256^3 315 / 307 / 241, 512^3 2353 / 2317 / 1727
//   with a velocity, finite element: 64^3 30 / 30 / 41, 72^3 47 / 35 / 42, 128^3 80 / 56 / 59, 160^3 154 / 94 / 100,
//     192^3 248 / 150 / 134, 256^3 621 / 331 / 264, 512^3 4854 / 2458 / 1873
//   without, central: 96^3 33 / 34 / 41, 128^3 41 / 40 / 50, 192^3 84 / 78 / 96, 256^3 164 / 126 / 185,
//     512^3 1586 / 1110 / 1429
//   without, finite element: 72^3 42 / 32 / 37, 128^3 73 / 48 / 54, 256^3 420 / 186 / 209, 288^3 774 / 391 / 351,
//     512^3 3886 / 1736 / 1597
enum Step3 { kStepCells, kStepTiles, kStepOnePass };
inline Step3 step3_route(int n, int scheme, bool has_a) {
    if (n < (scheme == 2 ? 65 : 128)) return kStepCells;
    if (has_a) return n < 192 ? kStepTiles : kStepOnePass;
    return scheme == 2 && n >= 288 ? kStepOnePass : kStepTiles;
}

// Planes per workgroup: a workgroup fills a CU and computes five planes more than it writes, so the chunks (of
// at least four planes) for which the rounds of 256 workgroups take the fewest plane steps.  512^3, with a velocity:
// 1727 us on four chunks of its 320 tiles, 2358 on one (a second round of 64 workgroups).
inline int step3_planes(int n) {
    const int64_t tiles = int64_t((n + kSx - 1) / kSx) * ((n + kSy - 1) / kSy);
    int64_t least = INT64_MAX;
    int best = n;
    for (int chunks = 1; chunks <= n / 4; ++chunks) {
        const int zc = (n + chunks - 1) / chunks;
        const int64_t steps = (tiles * ((n + zc - 1) / zc) + 255) / 256 * (zc + 5);
        if (steps < least) {
            least = steps;
            best = zc;
        }
    }
    return best;
}

// b = a.
__global__ __launch_bounds__(kBlock) void k_adx_copy(const double *__restrict__ a, double *__restrict__ b, int64_t m) {
    const int64_t base = int64_t(blockIdx.x) * 4 * kBlock + threadIdx.x;
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (base + u * kBlock < m) b[base + u * kBlock] = a[base + u * kBlock];
}

template <int SCHEME>
__global__ __launch_bounds__(kSt) void k_adx_step3(const double *__restrict__ T, double *__restrict__ out, APtrs ap,
                                                   int n, int bc, int zc, double dt, AdxK K) {
    constexpr int WT = kSx + 4, NTP = WT * (kSy + 4), WH = kSx + 2, NH = WH * (kSy + 2);
    constexpr int PER = (NTP + kSt - 1) / kSt;
    static_assert(NH <= kSt && PER <= 2, "a thread per cell of the tile and its ring");
    typedef AdxPlane<SCHEME> P;
    __shared__ double Tp[2][NTP];
    __shared__ double Hp[2][kSt];
    const int ntx = (n + kSx - 1) / kSx, nty = (n + kSy - 1) / kSy, blk = int(xcd_block(blockIdx.x, gridDim.x));
    const int t = int(threadIdx.x), last = n - 1;
    const int x0 = (blk % ntx) * kSx, y0 = ((blk / ntx) % nty) * kSy, z0 = (blk / (ntx * nty)) * zc, z1 = min(z0 + zc, n);
    const bool per = bc == 1, has = ap.has != 0;
    const double gs = bc == 0 ? -1.0 : 1.0;
    const int64_t pl = int64_t(n) * n;
    // cell q of an axis by the boundary rule (walls: the nearest cell) and the sign of its value
    auto axis = [&](int q, double &sg) -> int {
        if (per) return ((q % n) + n) % n;
        if (q >= 0 && q < n) return q;
        sg *= gs;
        return q < 0 ? 0 : last;
    };
    int toff[PER];
    double tsg[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int s = min(t + r * kSt, NTP - 1);
        tsg[r] = 1.0;
        const int gi = axis(x0 + s % WT - 2, tsg[r]), gj = axis(y0 + s / WT - 2, tsg[r]);
        toff[r] = gj * n + gi;
    }
    // the thread's cell (a, b): `ev` the LDS cell whose neighbourhood gives its value, `sg` the sign it
    // takes, `g` its in-plane index; threads past the ring repeat its last cell into spare entries
    const int s = min(t, NH - 1), a = s % WH - 1, b = s / WH - 1;
    double sg = 1.0;
    const int gi = axis(x0 + a, sg), gj = axis(y0 + b, sg), g = gj * n + gi;
    const int ev = ((per ? b : gj - y0) + 2) * WT + (per ? a : gi - x0) + 2;
    const bool inner = a >= 0 && a < kSx && b >= 0 && b < kSy && t < NH;
    const bool mine = inner && x0 + a < n && y0 + b < n;
    const int hc = inner ? t : WH + 1;  // where the corrector reads (a spare centre for the others)
    auto plane = [&](int q, double &sz) -> int64_t { return int64_t(axis(q, sz)) * pl; };
    double tn[PER];
    auto load_t = [&](int z) {
        double sz = 1.0;
        const int64_t o = plane(min(z, z1 + 1), sz);
#pragma unroll
        for (int r = 0; r < PER; ++r) tn[r] = sz * tsg[r] * T[o + toff[r]];
    };
    double an[3] = {}, ac[3] = {}, a2[3] = {}, a3[3] = {};  // velocity in flight, of planes z - 1, z - 2, z - 3
    auto load_a = [&](int p) {
        if (!has) return;
        double sz = 1.0;
        const int64_t o = plane(min(p, z1), sz);
#pragma unroll
        for (int e = 0; e < 3; ++e) an[e] = ap.a[e][o + g];
    };
    auto sums = [&](const double *L, int c, int w) -> P {
        double v[3][3];
#pragma unroll
        for (int y = 0; y < 3; ++y)
#pragma unroll
            for (int x = 0; x < 3; ++x) v[y][x] = SCHEME == 2 || x == 1 || y == 1 ? L[c + (y - 1) * w + x - 1] : 0.0;
        return P(v);
    };
    const double zero[3][3] = {};
    P ta(zero), tb(zero), ha(zero), hb(zero);  // T: planes z - 2, z - 1; H: planes z - 4, z - 3
    double t2 = 0.0, t3 = 0.0;                 // T of the cell at z - 2, z - 3
    load_t(z0 - 2);
    load_a(z0 - 1);
    for (int z = z0 - 2; z < z1 + 3; ++z) {
        double *L = Tp[z & 1];
#pragma unroll
        for (int r = 0; r < PER; ++r)
            if (t + r * kSt < NTP) L[t + r * kSt] = tn[r];
        load_t(z + 1);
        __syncthreads();
        const P tz = sums(L, ev, WT);
        if (z >= z0) {  // predictor of plane z - 1
            const double o = tb.c - dt * adx_rate3<SCHEME>(ta, tb, tz, ac, has, K);
            Hp[(z - 1) & 1][t] = sg * (0.5 * (o + tb.c));
        }
        P hz = hb;
        if (z >= z0 + 1) {  // corrector of plane z - 3 from H of planes z - 4, z - 3, z - 2
            hz = sums(Hp[(z - 2) & 1], hc, WH);
            const int q = z - 3;
            if (q >= z0) {
                const P l = !per && q == 0 ? hb.signed_by(gs) : ha, u = !per && q == last ? hb.signed_by(gs) : hz;
                const double o = t3 - dt * adx_rate3<SCHEME>(l, hb, u, a3, has, K);
                if (mine) out[int64_t(q) * pl + int64_t(y0 + b) * n + x0 + a] = o;
            }
        }
        ha = hb;
        hb = hz;
        t3 = t2;
        t2 = tb.c;
        ta = tb;
        tb = tz;
        if (z >= z0 - 1) {
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                a3[e] = a2[e];
                a2[e] = ac[e];
                ac[e] = an[e];
            }
            load_a(z + 1);
        }
    }
}

}  // namespace
}  // namespace np
