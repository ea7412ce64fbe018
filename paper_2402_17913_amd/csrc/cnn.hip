// Learned warm start: a small periodic 3D U-Net (16 channels, BF16 storage,
// FP32 accumulation) with its own forward, backward and Adam kernels.
//
// Activations are channels-last BF16 tensors [z][y][x][16].  A 3x3x3
// convolution is an implicit GEMM per 16-voxel row segment: output channel
// (M = 16) x voxel (N = 16) x (tap, input channel) (K = 27 x 16, two taps
// per 16x16x32 MFMA step, 14 steps).  The workgroup stages its input halo
// tile (x: row + 2, y: 4 rows + 2, z: 3 planes) and the weights in LDS.
// The data gradient is the same kernel on the flipped, transposed filter; the
// weight gradient is an FP32 reduction over voxels.
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <random>
#include <string>
#include <vector>

#include "mg_kernels.h"
#include "np_internal.h"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));  // kept in registers over a barrier, where uint4 arrays go to scratch

namespace np {
namespace {

constexpr int kC = 16;                 // channels
constexpr int kTaps = 27;
constexpr int kWsz = kTaps * kC * kC;  // weights per conv ([tap][out][in])
constexpr int kPsz = kWsz + kC;        // + bias
constexpr int kWgBlocks = 768;         // workgroups of a weight-gradient reduction (three per CU)
}  // namespace
int g_wgrad_mfma = 1;  // tuning knob "wgrad_mfma": weight gradients on the matrix cores
int g_conv3z = 1;  // tuning knob "conv3z": z-marching convolution tiles (0 off, 1 automatic, else planes)
namespace {

__device__ __forceinline__ float b2f(uint16_t u) { return __uint_as_float(uint32_t(u) << 16); }
__device__ __forceinline__ uint16_t f2b(float f) { return float_to_bf16(f); }

__device__ __forceinline__ int wrapi(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// ------------------------------------------------------------------ conv
// Where a field of the network has one channel (its input, the prediction's gradient), it is stored as
// such, and the kernels that read it as 16 channels set the others to zero as they load it (ONE): at 128^3
// writing it takes 6 and 9 us instead of 17 and 20, and its weight gradients 42 us instead of 44.
// 8 channels of a voxel: index i is 2 * voxel + half.
template <bool ONE> __device__ __forceinline__ u32x4 ld_half(const uint16_t *__restrict__ X, int64_t i) {
    if constexpr (ONE) return u32x4{(i & 1) ? 0u : uint32_t(X[i >> 1]), 0u, 0u, 0u};
    else return reinterpret_cast<const u32x4 *>(X)[i];
}

// What a convolution writes: BF16 after ReLU (forward); FP32; BF16 where the activation `act` is
// positive and zero elsewhere (a data gradient already masked for the layer below it, so that the
// FP32 gradient is never stored); FP32 of channel 0 alone (the prediction).
enum ConvOut { kOutRelu, kOutF32, kOutMask, kOutOne };

// Output channels 4 grp .. 4 grp + 3: the lane's bias (zero for data gradients)
__device__ __forceinline__ f32x4 conv_bias(const float *__restrict__ bias, int grp) {
    return bias ? f32x4{bias[4 * grp], bias[4 * grp + 1], bias[4 * grp + 2], bias[4 * grp + 3]} : f32x4{0.f, 0.f, 0.f, 0.f};
}
// The activations of these channels of voxel v that mask them
template <ConvOut OUT> __device__ __forceinline__ uint2 conv_act(const uint16_t *__restrict__ act, int64_t v, int grp) {
    if constexpr (OUT == kOutMask) return *reinterpret_cast<const uint2 *>(act + v * kC + 4 * grp);
    else return make_uint2(0, 0);
}
// Stores these channels of voxel v.
template <ConvOut OUT>
__device__ __forceinline__ void conv_store(const f32x4 &acc, const f32x4 &bias, const uint2 &act, void *__restrict__ Y,
                                           int64_t v, int grp) {
    float o[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float t = acc[r] + bias[r];
        if (OUT == kOutRelu) t = t > 0.f ? t : 0.f;
        o[r] = t;
    }
    if constexpr (OUT == kOutF32) {
        *reinterpret_cast<float4 *>(reinterpret_cast<float *>(Y) + v * kC + 4 * grp) = make_float4(o[0], o[1], o[2], o[3]);
    } else if constexpr (OUT == kOutOne) {
        if (grp == 0) reinterpret_cast<float *>(Y)[v] = o[0];
    } else {
        if constexpr (OUT == kOutMask) {
            const uint32_t aw[2] = {act.x, act.y};
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (!(b2f(uint16_t(aw[r >> 1] >> (16 * (r & 1)))) > 0.f)) o[r] = 0.f;
        }
        uint2 pk;
        pk.x = float2_to_bf16x2(o[0], o[1]);
        pk.y = float2_to_bf16x2(o[2], o[3]);
        *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(Y) + v * kC + 4 * grp) = pk;
    }
}

// Y = conv(X, W) (+ bias, ReLU) on an n^3 periodic grid, n = 2^lg >= 16.
// Workgroup: TXV = min(64, n) voxels along x, 4 rows along y, one plane.
template <ConvOut OUT, bool ONE>
__global__ __launch_bounds__(256) void k_conv(const uint16_t *__restrict__ X, const uint16_t *__restrict__ W,
                                              const float *__restrict__ bias, const uint16_t *__restrict__ act,
                                              void *__restrict__ Y, int lg) {
    __shared__ uint4 xs[(64 + 2) * 6 * 3 * 2];  // halo voxels x 32 B
    __shared__ uint4 ws[kTaps * kC * 2];         // 27 x 16 rows x 32 B
    const int n = 1 << lg, txv = n < 64 ? n : 64, hx = txv + 2;
    const int tiles_x = n / txv;
    const int b = blockIdx.x;
    const int tx = b % tiles_x, y4 = (b / tiles_x) % (n / 4), z = b / (tiles_x * (n / 4));
    const int x0 = tx * txv, y0 = 4 * y4, tid = threadIdx.x;
    const uint4 *W4 = reinterpret_cast<const uint4 *>(W);
    for (int q = tid; q < kTaps * kC * 2; q += 256) ws[q] = W4[q];
    const int nh = hx * 6 * 3;
    for (int q = tid; q < nh * 2; q += 256) {
        const int v = q >> 1, half = q & 1;
        const int lx = v % hx, ly = (v / hx) % 6, lz = v / (hx * 6);
        const int gx = wrapi(x0 + lx - 1, n), gy = wrapi(y0 + ly - 1, n), gz = wrapi(z + lz - 1, n);
        reinterpret_cast<u32x4 *>(xs)[q] = ld_half<ONE>(X, ((((int64_t(gz) << lg) + gy) << lg) + gx) * 2 + half);
    }
    __syncthreads();
    const int w = tid >> 6, l = tid & 63;
    const int col = l & 15, grp = l >> 4;
    const int tsel = grp >> 1, cb = grp & 1;
    const f32x4 bv4 = conv_bias(bias, grp);
    for (int tt = 0; tt < txv / 16; ++tt) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 14; ++s) {
            const int tap = 2 * s + tsel;
            bf16x8 av, bv;
            if (tap < kTaps) {
                const int dz = tap / 9 - 1, dy = (tap / 3) % 3 - 1, dx = tap % 3 - 1;
                const uint4 a4 = ws[(tap * kC + col) * 2 + cb];
                const int hv = ((1 + dz) * 6 + (w + 1 + dy)) * hx + (tt * 16 + col + 1 + dx);
                const uint4 b4 = xs[hv * 2 + cb];
                av = *reinterpret_cast<const bf16x8 *>(&a4);
                bv = *reinterpret_cast<const bf16x8 *>(&b4);
            } else {
                const uint4 zz = make_uint4(0, 0, 0, 0);
                av = *reinterpret_cast<const bf16x8 *>(&zz);
                bv = av;
            }
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, acc, 0, 0, 0);
        }
        // lane holds output channels 4*grp .. +3 of voxel `col`
        const int gx = x0 + tt * 16 + col, gy = y0 + w;
        const int64_t v = (((int64_t(z) << lg) + gy) << lg) + gx;
        conv_store<OUT>(acc, bv4, conv_act<OUT>(act, v, grp), Y, v, grp);
    }
}

// Z-marching form of the same convolution (same MFMA sequence per output, so the same bits).  A workgroup
// owns a column of 256 voxels (TXV = min(64, n) along x by 256 / TXV rows) and zc planes of it; a wave owns
// 16 voxels along x by four rows.  Input planes arrive one by one in a ring of three LDS buffers, through
// registers a plane ahead, and each is used for all three output planes it reaches, whose sums a lane holds:
// of an output's 14 steps (pairs of taps, in order) 0 .. 3 read the plane below it, 4 the plane below and its
// own, 5 .. 8 its own, 9 .. 13 the plane above.  Neighbouring outputs share most operands of a plane: with
// row operands A (dx -1, 0), B (dx 0, 1), C (dx 1, then -1 of the next row), D (dx 1 of the row above in the
// plane below, then -1 of the row below) and E (dx 1, then nothing), four rows and three planes take 26 LDS
// reads where one output row at a time takes 56.  At 128^3 a forward convolution takes 39 us against 67 us
// of a kernel that read all operands per output row, both in a training gradient (its floor, 64 MB read and 64 MB
// written: 28 us).
constexpr int kCzT = 256, kCzRows = 4;
constexpr int kCzSlots = (64 + 2) * (kCzRows + 2) * 2;  // uint4 per plane buffer (halo tile, two per voxel)

template <ConvOut OUT, bool ONE>
__global__ __launch_bounds__(kCzT) void k_conv3z(const uint16_t *__restrict__ X, const uint16_t *__restrict__ W,
                                                 const float *__restrict__ bias, const uint16_t *__restrict__ act,
                                                 void *__restrict__ Y, int lg, int zc) {
    __shared__ uint4 xs[3][kCzSlots];
    const int n = 1 << lg, lt = lg < 6 ? lg : 6, txv = 1 << lt, rows = kCzT >> lt, hx = txv + 2;
    const int tiles_x = n / txv, ncol = tiles_x * (n / rows);
    const int b = int(xcd_block(blockIdx.x, gridDim.x));
    const int x0 = (b % tiles_x) * txv, y0 = ((b % ncol) / tiles_x) * rows, z0 = (b / ncol) * zc, z1 = z0 + zc;
    const int tid = threadIdx.x;
    const uint4 *W4 = reinterpret_cast<const uint4 *>(W);
    // this thread's share of a plane: slot q holds half (q & 1) of voxel (q >> 1) of the halo tile (slots
    // beyond the tile repeat the last one)
    constexpr int NF = (kCzSlots + kCzT - 1) / kCzT;
    const int nslot = hx * (rows + 2) * 2;
    int off[NF], at_q[NF];
    u32x4 pf[NF];
#pragma unroll
    for (int u = 0; u < NF; ++u) {
        const int q = tid + u * kCzT < nslot ? tid + u * kCzT : nslot - 1, v = q >> 1;
        off[u] = ((wrapi(y0 + v / hx - 1, n) << lg) + wrapi(x0 + v % hx - 1, n)) * 2 + (q & 1);
        at_q[u] = q;
    }
    auto fetch = [&](int z) {
        const int64_t p = int64_t(wrapi(z, n)) << (2 * lg + 1);
#pragma unroll
        for (int u = 0; u < NF; ++u) pf[u] = ld_half<ONE>(X, p + off[u]);
    };
    auto place = [&](int slot) {
#pragma unroll
        for (int u = 0; u < NF; ++u) reinterpret_cast<u32x4 *>(xs[slot])[at_q[u]] = pf[u];
    };
    fetch(z0 - 1);
    const int w = tid >> 6, l = tid & 63;
    const int col = l & 15, grp = l >> 4;
    const int tsel = grp >> 1, cb = grp & 1;
    // the lane's weight operands of the 14 steps depend on the lane only: held in registers
    // (the 28th tap does not exist: its operands are zero)
    bf16x8 wa[14];
#pragma unroll
    for (int s = 0; s < 14; ++s) {
        const bool live = 2 * s + tsel < kTaps;
        const uint4 a4 = W4[((live ? 2 * s + tsel : kTaps - 1) * kC + col) * 2 + cb];
        wa[s] = __builtin_bit_cast(bf16x8, live ? a4 : make_uint4(0, 0, 0, 0));
    }
    place(0);
    fetch(z0);
    const int wx = (w << 4) & (txv - 1), wy = ((w << 4) >> lt) * kCzRows;  // the wave's voxels in the tile
    // LDS index of this lane's part of an operand at the wave's row 0
    const int at = ((wy + 1) * hx + wx + col + 1) * 2 + cb;
    const int ia = at + (tsel ? 0 : -2), ib = at + (tsel ? 2 : 0), ic = at + (tsel ? 2 * hx - 2 : 2),
              id = at + (tsel ? -2 * hx - 2 : 2 * hx + 2), ie = at + 2;
    const int hr = 2 * hx;
    const int64_t v0 = (int64_t(y0 + wy) << lg) + x0 + wx + col;
    const f32x4 bv4 = conv_bias(bias, grp);
    f32x4 top[kCzRows], mid[kCzRows], low[kCzRows];  // sums of the output planes z + 1, z, z - 1 at input plane z
#pragma unroll
    for (int y = 0; y < kCzRows; ++y) mid[y] = low[y] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto mac = [&](int s, const uint4 &x, const f32x4 &c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[s], __builtin_bit_cast(bf16x8, x), c, 0, 0, 0);
    };
    // one input plane; T, M, L: it reaches the output planes z + 1, z, z - 1 of this chunk
    auto plane = [&](auto T, auto M, auto L, const uint4 *cur, const uint4 *prev) {
#pragma unroll
        for (int y = 0; y < kCzRows; ++y) {
            f32x4 t = f32x4{0.f, 0.f, 0.f, 0.f};
            const uint4 am = cur[ia + (y - 1) * hr], ap = cur[ia + (y + 1) * hr], cm = cur[ic + (y - 1) * hr],
                        b0 = cur[ib + y * hr];
            if constexpr (T.value) {
                t = mac(0, am, t);
                t = mac(1, cm, t);
                t = mac(2, b0, t);
                t = mac(3, ap, t);
            }
            if constexpr (M.value) {
                f32x4 m = mac(4, (tsel ? cur : prev)[id + y * hr], mid[y]);
                m = mac(5, cur[ib + (y - 1) * hr], m);
                m = mac(6, cur[ia + y * hr], m);
                m = mac(7, cur[ic + y * hr], m);
                mid[y] = mac(8, cur[ib + (y + 1) * hr], m);
            }
            if constexpr (L.value) {
                f32x4 o = mac(9, am, low[y]);
                o = mac(10, cm, o);
                o = mac(11, b0, o);
                o = mac(12, ap, o);
                const uint4 e = cur[ie + (y + 1) * hr];
                low[y] = mac(13, tsel ? make_uint4(0, 0, 0, 0) : e, o);
            }
            top[y] = t;
        }
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    int cs = 0;  // ring slot of plane z
    for (int z = z0 - 1; z <= z1; ++z) {
        const int ns = cs == 2 ? 0 : cs + 1, ps = cs == 0 ? 2 : cs - 1;
        __syncthreads();  // plane z is in LDS, and plane z - 2, whose buffer takes z + 1, is read
        if (z < z1) place(ns);
        uint2 ya[kCzRows] = {};  // asked for before the next plane, so that waiting for them does not wait for it
        if (z > z0)
#pragma unroll
            for (int y = 0; y < kCzRows; ++y)
                ya[y] = conv_act<OUT>(act, (int64_t(z - 1) << (2 * lg)) + v0 + (int64_t(y) << lg), grp);
        if (z + 1 < z1) fetch(z + 2);
        const uint4 *cur = xs[cs], *prev = xs[ps];
        if (z == z0 - 1) plane(yes, no, no, cur, prev);
        else if (z == z1) plane(no, no, yes, cur, prev);
        else if (zc == 1) plane(no, yes, no, cur, prev);
        else if (z == z0) plane(yes, yes, no, cur, prev);
        else if (z == z1 - 1) plane(no, yes, yes, cur, prev);
        else plane(yes, yes, yes, cur, prev);
        if (z > z0) {
            const int64_t v = (int64_t(z - 1) << (2 * lg)) + v0;
#pragma unroll
            for (int y = 0; y < kCzRows; ++y) conv_store<OUT>(low[y], bv4, ya[y], Y, v + (int64_t(y) << lg), grp);
        }
#pragma unroll
        for (int y = 0; y < kCzRows; ++y) {
            low[y] = mid[y];
            mid[y] = top[y];
        }
        cs = ns;
    }
}

// Weight gradient partials: P[blk][tap*256 + o*16 + c] = sum over the
// workgroup's voxels of dZ[v][o] * X[v + tap][c]; P[blk][6912 + o] = sum dZ[v][o].
// Tiles of the forward shape, grid-strided over a capped number of workgroups.
template <bool ONEX, bool ONEZ>
__global__ __launch_bounds__(256) void k_wgrad(const uint16_t *__restrict__ X, const uint16_t *__restrict__ dZ,
                                               float *__restrict__ P, int lg) {
    __shared__ __align__(16) uint16_t xs[(64 + 2) * 6 * 3 * kC];
    __shared__ __align__(16) uint16_t zs[64 * 4 * kC];
    const int n = 1 << lg, txv = n < 64 ? n : 64, hx = txv + 2;
    const int tiles_x = n / txv, ntile = tiles_x * (n / 4) * n;
    const int tid = threadIdx.x, o = tid >> 4, c = tid & 15;
    float acc[kTaps];
#pragma unroll
    for (int t = 0; t < kTaps; ++t) acc[t] = 0.f;
    float bacc = 0.f;
    for (int b = blockIdx.x; b < ntile; b += gridDim.x) {
        const int tx = b % tiles_x, y4 = (b / tiles_x) % (n / 4), z = b / (tiles_x * (n / 4));
        const int x0 = tx * txv, y0 = 4 * y4;
        __syncthreads();
        const int nh = hx * 6 * 3;
        for (int q = tid; q < nh * 2; q += 256) {
            const int v = q >> 1, half = q & 1;
            const int lx = v % hx, ly = (v / hx) % 6, lz = v / (hx * 6);
            const int gx = wrapi(x0 + lx - 1, n), gy = wrapi(y0 + ly - 1, n), gz = wrapi(z + lz - 1, n);
            reinterpret_cast<u32x4 *>(xs)[q] = ld_half<ONEX>(X, ((((int64_t(gz) << lg) + gy) << lg) + gx) * 2 + half);
        }
        for (int q = tid; q < txv * 4 * 2; q += 256) {
            const int v = q >> 1, half = q & 1;
            const int lx = v % txv, ly = v / txv;
            reinterpret_cast<u32x4 *>(zs)[q] =
                ld_half<ONEZ>(dZ, ((((int64_t(z) << lg) + y0 + ly) << lg) + x0 + lx) * 2 + half);
        }
        __syncthreads();
        for (int ly = 0; ly < 4; ++ly)
            for (int lx = 0; lx < txv; ++lx) {
                const float g = b2f(zs[(ly * txv + lx) * kC + o]);
                bacc += g;
                if (g == 0.f) continue;
#pragma unroll
                for (int t = 0; t < kTaps; ++t) {
                    const int dz = t / 9 - 1, dy = (t / 3) % 3 - 1, dx = t % 3 - 1;
                    const int hv = ((1 + dz) * 6 + (ly + 1 + dy)) * hx + (lx + 1 + dx);
                    acc[t] += g * b2f(xs[hv * kC + c]);
                }
            }
    }
    float *Pb = P + int64_t(blockIdx.x) * kPsz;
#pragma unroll
    for (int t = 0; t < kTaps; ++t) Pb[t * 256 + o * 16 + c] = acc[t];
    if (c == 0) Pb[kWsz + o] = bacc;
}

// The same partials on the matrix cores: per tap t, dW_t[o][c] = sum over voxels v of dZ[v][o] X[v + t][c]
// is a 16 x 16 product with the voxels as the contraction (v_mfma_f32_16x16x32_bf16, 32 voxels per step);
// the bias gradient is one more product with X = 1.  A workgroup marches through a chunk of planes of a
// column of TXV x 4 voxels: a ring of four X planes with their halo and two dZ planes lie in LDS, three and
// one of them in use while the next of each arrives through registers, so that a plane costs one barrier.
// Both are staged channel-major, two voxels of a
// channel per dword, so that a lane's operand (8 consecutive voxels of one channel) is one 16-byte read for
// dZ and, for X, one 16-byte and one 4-byte read that serve the three taps of a (dz, dy) row, funnel-shifted
// by 0, 2 or 4 bytes.  The channel pitches put the 16 channels of a read on different banks.  A wave owns
// every fourth step of 32 voxels and all 28 products, and the waves' sums are added in order at the end.
// At 128^3 it takes 44 us, against 125 us when every plane of a tile staged
// a three-plane halo of its own with 2-byte LDS writes and each wave read all of dZ for its share of the taps.
// The two operands read once would take 28 us; what is left is one barrier and a full load latency per plane
// at two workgroups per CU, which the 28 accumulators of a lane allow.
constexpr int kWmT = 256, kWmAim = 512;
constexpr int kWmRow = 72;                    // halo row of up to 66 voxels, a multiple of 8
constexpr int kWmCh = 4 * 6 * kWmRow + 8;     // channel pitch of X (868 dwords: 36 modulo the 64 banks)
constexpr int kWmZCh = 64 * 4 + 8;            // channel pitch of dZ (132 dwords: 4 modulo 64)

__device__ __forceinline__ uint32_t wm_shift(uint32_t lo, uint32_t hi, int bytes) {
    return bytes == 0 ? lo : __builtin_amdgcn_alignbyte(hi, lo, bytes);
}

// Eight channels of two neighbouring voxels a, b to the channel-major rows dst, dst + pitch, ... (dwords)
__device__ __forceinline__ void wm_put(uint32_t *dst, int pitch, const u32x4 &a, const u32x4 &b) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
        dst[e * pitch] = __builtin_amdgcn_perm(b[e >> 1], a[e >> 1], (e & 1) ? 0x07060302u : 0x05040100u);
}

template <bool ONEX, bool ONEZ>
__global__ __launch_bounds__(kWmT) void k_wgrad_mfma(const uint16_t *__restrict__ X, const uint16_t *__restrict__ dZ,
                                                     float *__restrict__ P, int lg, int nch) {
    __shared__ __align__(16) uint16_t xt[kC * kWmCh];   // [c][ring slot][row][x]
    __shared__ __align__(16) uint16_t zt[2][kC * kWmZCh];  // [plane & 1][o][voxel]
    static_assert(sizeof(xt) >= 4 * 7 * 256 * sizeof(float), "the sum over waves takes the place of X");
    const int n = 1 << lg, lt = lg < 6 ? lg : 6, txv = 1 << lt, hp = (txv + 2) / 2;
    const int tiles_x = n / txv, ncol = tiles_x * (n / 4);
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
    const int ch = l & 15, g = l >> 4;  // operand channel (o for dZ, c for X); voxel run within 32
    uint32_t *xd = reinterpret_cast<uint32_t *>(xt);
    f32x4 acc[kTaps + 1];
#pragma unroll
    for (int u = 0; u <= kTaps; ++u) acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
    const uint32_t one2 = 0x3f803f80u;  // two BF16 ones
    const uint4 ones = make_uint4(one2, one2, one2, one2);
    // this thread's staging slots: pairs of voxels x half a voxel's channels (those beyond the tile repeat
    // the last one)
    const int nxs = hp * 6 * 2, nzs = txv * 4;
    int xp[2], xr[2], xl[2];  // a slot's pair in its row, the row, and its place in LDS
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int q = std::min(tid + u * kWmT, nxs - 1), v = q >> 1;
        xp[u] = v % hp;
        xr[u] = v / hp;
        xl[u] = 8 * (q & 1) * (kWmCh / 2) + xr[u] * (kWmRow / 2) + xp[u];
    }
    const int zq = std::min(tid, nzs - 1), zp = (zq >> 1) & (txv / 2 - 1), zy = (zq >> 1) >> (lt - 1);
    const int zl = 8 * (zq & 1) * (kWmZCh / 2) + zy * (txv / 2) + zp;
    for (int b = int(xcd_block(blockIdx.x, gridDim.x)); b < ncol * nch; b += gridDim.x) {
        const int col = b % ncol, x0 = (col % tiles_x) * txv, y0 = (col / tiles_x) * 4;
        const int z0 = int(int64_t(n) * (b / ncol) / nch), z1 = int(int64_t(n) * (b / ncol + 1) / nch);
        int xa[2], xb[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int row = wrapi(y0 + xr[u] - 1, n) << lg, gx = x0 + 2 * xp[u], half = (tid + u * kWmT < nxs ? tid : nxs - 1) & 1;
            xa[u] = (row + wrapi(gx - 1, n)) * 2 + half;
            xb[u] = (row + wrapi(gx, n)) * 2 + half;
        }
        const int za = (((y0 + zy) << lg) + x0 + 2 * zp) * 2 + (zq & 1);
        u32x4 xv[3][2][2], zv[2];  // planes on their way (three at the start of a column, then one)
        auto fetch_x = [&](int z, u32x4 (&t)[2][2]) {
            const int64_t p = int64_t(wrapi(z, n)) << (2 * lg + 1);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                t[u][0] = ld_half<ONEX>(X, p + xa[u]);
                t[u][1] = ld_half<ONEX>(X, p + xb[u]);
            }
        };
        auto store_x = [&](int slot, const u32x4 (&t)[2][2]) {
#pragma unroll
            for (int u = 0; u < 2; ++u) wm_put(xd + xl[u] + slot * (6 * kWmRow / 2), kWmCh / 2, t[u][0], t[u][1]);
        };
        auto fetch_z = [&](int z) {
            const int64_t p = (int64_t(z) << (2 * lg + 1)) + za;
            zv[0] = ld_half<ONEZ>(dZ, p);
            zv[1] = ld_half<ONEZ>(dZ, p + 2);
        };
        auto store_z = [&](int z) {
            wm_put(reinterpret_cast<uint32_t *>(zt[z & 1]) + zl, kWmZCh / 2, zv[0], zv[1]);
        };
        __syncthreads();  // the previous column's operands are read
        fetch_z(z0);
#pragma unroll
        for (int t = 0; t < 3; ++t) fetch_x(z0 - 1 + t, xv[t]);
        store_z(z0);
#pragma unroll
        for (int t = 0; t < 3; ++t) store_x((z0 - 1 + t) & 3, xv[t]);
        for (int z = z0; z < z1; ++z) {
            __syncthreads();  // planes z - 1 .. z + 1 and dZ's z are in LDS; z - 2 and dZ's z - 1 are read
            if (z + 1 < z1) {
                fetch_x(z + 2, xv[0]);
                fetch_z(z + 1);
            }
            for (int kb = w; kb < txv * 4 / 32; kb += 4) {
                const int v0 = kb * 32 + 8 * g, ly = v0 >> lt, lx0 = v0 & (txv - 1);  // 8 voxels of one row
                const bf16x8 av =
                    __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(&zt[z & 1][ch * kWmZCh + v0]));
#pragma unroll
                for (int G = 0; G < 9; ++G) {  // (dz, dy): its three taps share one X row
                    const uint16_t *row = &xt[ch * kWmCh + (((z + G / 3 - 1) & 3) * 6 + ly + G % 3) * kWmRow + lx0];
                    const uint4 lo = *reinterpret_cast<const uint4 *>(row);
                    const uint32_t d[5] = {lo.x, lo.y, lo.z, lo.w, *reinterpret_cast<const uint32_t *>(row + 8)};
#pragma unroll
                    for (int t = 0; t < 3; ++t) {  // dx = t - 1: the run starts t voxels in
                        const int wsh = t >> 1, bsh = 2 * (t & 1);
                        uint4 b4;
                        b4.x = wm_shift(d[wsh + 0], d[bsh ? 1 : wsh], bsh);
                        b4.y = wm_shift(d[wsh + 1], d[bsh ? 2 : wsh + 1], bsh);
                        b4.z = wm_shift(d[wsh + 2], d[bsh ? 3 : wsh + 2], bsh);
                        b4.w = wm_shift(d[wsh + 3], d[bsh ? 4 : wsh + 3], bsh);
                        acc[3 * G + t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, b4),
                                                                                 acc[3 * G + t], 0, 0, 0);
                    }
                }
                acc[kTaps] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, ones), acc[kTaps], 0,
                                                                     0, 0);
            }
            if (z + 1 < z1) {
                store_x((z + 2) & 3, xv[0]);
                store_z(z + 1);
            }
        }
    }
    // lane holds C[o = 4 g + r][c = ch] of each product; the waves' sums are added in order, seven products
    // at a time
    float *sum = reinterpret_cast<float *>(xt), *Pb = P + int64_t(blockIdx.x) * kPsz;
#pragma unroll
    for (int t0 = 0; t0 <= kTaps; t0 += 7) {
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 7; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) sum[(w * 7 + t) * 256 + (4 * g + r) * 16 + ch] = acc[t0 + t][r];
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 7; ++t) {
            const float v = ((sum[t * 256 + tid] + sum[(7 + t) * 256 + tid]) + sum[(14 + t) * 256 + tid]) +
                            sum[(21 + t) * 256 + tid];
            if (t0 + t < kTaps) Pb[(t0 + t) * 256 + tid] = v;
            else if ((tid & 15) == 0) Pb[kWsz + (tid >> 4)] = v;
        }
    }
}

// G[i] += sum over workgroups of P[blk][i] (fixed order): a workgroup owns 32
// consecutive entries; its kRedSl slices of 8 threads (four entries each) sum every
// kRedSl-th partial, then the slices are added in order through LDS.  Bound by the
// latency of a slice's loads: 8 slices of 32 threads (96 loads in a row) took 21 us, 32
// slices 6.1, with 16-byte loads, eight of them in flight, 5.2 (average over the levels).
constexpr int kRedSl = 32;
__global__ __launch_bounds__(8 * kRedSl) void k_wgrad_reduce(const float *__restrict__ P, int nblk,
                                                             float *__restrict__ G) {
    static_assert(kPsz % 4 == 0, "rows of whole float4");
    __shared__ f32x4 part[kRedSl][8];
    const int li = threadIdx.x & 7, sl = threadIdx.x >> 3, i = blockIdx.x * 8 + li;  // i: four entries
    const f32x4 *P4 = reinterpret_cast<const f32x4 *>(P) + (i < kPsz / 4 ? i : 0);
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    int b = sl;
    for (; b + 7 * kRedSl < nblk; b += 8 * kRedSl) {
        f32x4 t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = P4[int64_t(b + u * kRedSl) * (kPsz / 4)];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += t[u];
    }
    for (; b < nblk; b += kRedSl) s += P4[int64_t(b) * (kPsz / 4)];
    part[sl][li] = s;
    __syncthreads();
    if (sl == 0 && i < kPsz / 4) {
        f32x4 t = part[0][li];
#pragma unroll
        for (int q = 1; q < kRedSl; ++q) t += part[q][li];
        reinterpret_cast<f32x4 *>(G)[i] += t;
    }
}

// Flipped, transposed filter for the data gradient: Wt[26 - t][c][o] = W[t][o][c].
__global__ __launch_bounds__(256) void k_wflip(const uint16_t *__restrict__ W, uint16_t *__restrict__ Wt) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= kWsz) return;
    const int t = i / 256, o = (i / 16) % 16, c = i % 16;
    Wt[(26 - t) * 256 + c * 16 + o] = W[i];
}

// The elementwise kernels below are bound by memory: a thread takes eight channels of a voxel (one
// 16-byte BF16 access), and the backward ones write BF16 gradients masked for the next layer.
struct Ch8 {
    float v[8];
};
__device__ __forceinline__ Ch8 ld8(const uint16_t *__restrict__ p) {
    const uint4 d = *reinterpret_cast<const uint4 *>(p);
    const uint32_t w[4] = {d.x, d.y, d.z, d.w};
    Ch8 r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r.v[e] = b2f(uint16_t(w[e >> 1] >> (16 * (e & 1))));
    return r;
}
__device__ __forceinline__ Ch8 ld8(const float *__restrict__ p) {
    const float4 a = reinterpret_cast<const float4 *>(p)[0], b = reinterpret_cast<const float4 *>(p)[1];
    return Ch8{{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w}};
}
__device__ __forceinline__ void st8(uint16_t *__restrict__ p, const Ch8 &r) {
    uint4 d;
    d.x = float2_to_bf16x2(r.v[0], r.v[1]);
    d.y = float2_to_bf16x2(r.v[2], r.v[3]);
    d.z = float2_to_bf16x2(r.v[4], r.v[5]);
    d.w = float2_to_bf16x2(r.v[6], r.v[7]);
    *reinterpret_cast<uint4 *>(p) = d;
}
// g where the activation is positive, else zero
__device__ __forceinline__ void mask8(Ch8 &g, const uint16_t *__restrict__ act) {
    const Ch8 a = ld8(act);
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (!(a.v[e] > 0.f)) g.v[e] = 0.f;
}

// 2x2x2 average (n fine -> n/2), bf16.
__global__ __launch_bounds__(256) void k_pool(const uint16_t *__restrict__ X, uint16_t *__restrict__ Y, int lgc) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x, v = i >> 1;
    const int nc = 1 << lgc, lg = lgc + 1, c8 = int(i & 1) * 8;
    if (v >= (int64_t(1) << (3 * lgc))) return;
    const int x = int(v & (nc - 1)), y = int((v >> lgc) & (nc - 1)), z = int(v >> (2 * lgc));
    Ch8 s{};
    for (int dz = 0; dz < 2; ++dz)
        for (int dy = 0; dy < 2; ++dy)
            for (int dx = 0; dx < 2; ++dx) {
                const Ch8 t = ld8(X + (((((int64_t(2 * z + dz) << lg) + 2 * y + dy) << lg) + 2 * x + dx) << 4) + c8);
#pragma unroll
                for (int e = 0; e < 8; ++e) s.v[e] += t.v[e];
            }
#pragma unroll
    for (int e = 0; e < 8; ++e) s.v[e] *= 0.125f;
    st8(Y + (v << 4) + c8, s);
}

// Gradient of an encoder level's output, masked by it: dY(coarse) / 8 through the pooling plus the
// skip's gradient K (both FP32).
__global__ __launch_bounds__(256) void k_join_back(const float *__restrict__ dY, const float *__restrict__ K,
                                                   const uint16_t *__restrict__ act, uint16_t *__restrict__ Z, int lg) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x, v = i >> 1;
    const int n = 1 << lg, lgc = lg - 1, c8 = int(i & 1) * 8;
    if (v >= (int64_t(1) << (3 * lg))) return;
    const int x = int(v & (n - 1)), y = int((v >> lg) & (n - 1)), z = int(v >> (2 * lg));
    const Ch8 t = ld8(dY + (((((int64_t(z >> 1) << lgc) + (y >> 1)) << lgc) + (x >> 1)) << 4) + c8);
    Ch8 g = ld8(K + (v << 4) + c8);
#pragma unroll
    for (int e = 0; e < 8; ++e) g.v[e] = t.v[e] * 0.125f + g.v[e];
    mask8(g, act + (v << 4) + c8);
    st8(Z + (v << 4) + c8, g);
}

// Y(fine) = up(Xc) + S, periodic cell-centred trilinear, bf16.
__global__ __launch_bounds__(256) void k_up_add(const uint16_t *__restrict__ Xc, const uint16_t *__restrict__ S,
                                                uint16_t *__restrict__ Y, int lg) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x, v = i >> 1;
    const int n = 1 << lg, lgc = lg - 1, nc = n >> 1, c8 = int(i & 1) * 8;
    if (v >= (int64_t(1) << (3 * lg))) return;
    const int x = int(v & (n - 1)), y = int((v >> lg) & (n - 1)), z = int(v >> (2 * lg));
    const int ox = x >> 1, oy = y >> 1, oz = z >> 1;
    const int nx = wrapi((x & 1) ? ox + 1 : ox - 1, nc), ny = wrapi((y & 1) ? oy + 1 : oy - 1, nc),
              nz = wrapi((z & 1) ? oz + 1 : oz - 1, nc);
    Ch8 s{};
    for (int cz = 0; cz < 2; ++cz)
        for (int cy = 0; cy < 2; ++cy)
            for (int cx = 0; cx < 2; ++cx) {
                const float wgt = (cx ? 0.25f : 0.75f) * (cy ? 0.25f : 0.75f) * (cz ? 0.25f : 0.75f);
                const int64_t q = ((((int64_t(cz ? nz : oz) << lgc) + (cy ? ny : oy)) << lgc) + (cx ? nx : ox));
                const Ch8 t = ld8(Xc + (q << 4) + c8);
#pragma unroll
                for (int e = 0; e < 8; ++e) s.v[e] += wgt * t.v[e];
            }
    const Ch8 t = ld8(S + (v << 4) + c8);
#pragma unroll
    for (int e = 0; e < 8; ++e) s.v[e] = s.v[e] + t.v[e];
    st8(Y + (v << 4) + c8, s);
}

// Z(coarse) = up^T dY(fine), masked by act: each coarse cell gathers the 4 fine cells per
// axis that reference it (weights 1/4, 3/4, 3/4, 1/4 at 2I-1 .. 2I+2).  A thread takes four channels
// of two coarse cells along x, which share a third of their fine cells, and has a fine plane's 24
// loads asked for together (64^3 from 128^3: 73 us with eight channels of one cell, four loads at a time, 68
// so; 32^3 and below 10 -> 7.4).
__global__ __launch_bounds__(256) void k_up_back(const float *__restrict__ dY, const uint16_t *__restrict__ act,
                                                 uint16_t *__restrict__ Zc, int lgc) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x, v = i >> 2;  // v: the cell pair
    const int nc = 1 << lgc, lg = lgc + 1, n = nc << 1, c4 = int(i & 3) * 4;
    if (v >= (int64_t(1) << (3 * lgc - 1))) return;
    const int X = int(v & (nc / 2 - 1)) * 2, Yc = int((v >> (lgc - 1)) & (nc - 1)), Z = int(v >> (2 * lgc - 1));
    const float w1[4] = {0.25f, 0.75f, 0.75f, 0.25f};
    int fx[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) fx[c] = wrapi(2 * X - 1 + c, n);
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
    for (int a = 0; a < 4; ++a) {
        const int fz = wrapi(2 * Z - 1 + a, n);
        f32x4 t[4][6];
#pragma unroll
        for (int bb = 0; bb < 4; ++bb)
#pragma unroll
            for (int c = 0; c < 6; ++c)
                t[bb][c] = *reinterpret_cast<const f32x4 *>(
                    dY + (((((int64_t(fz) << lg) + wrapi(2 * Yc - 1 + bb, n)) << lg) + fx[c]) << 4) + c4);
#pragma unroll
        for (int bb = 0; bb < 4; ++bb)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float w = w1[a] * w1[bb] * w1[c];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    s0[e] += w * t[bb][c][e];
                    s1[e] += w * t[bb][c + 2][e];
                }
            }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int64_t at = (((((int64_t(Z) << lgc) + Yc) << lgc) + X + q) << 4) + c4;
        const f32x4 &g = q ? s1 : s0;
        const uint2 m = *reinterpret_cast<const uint2 *>(act + at);
        const uint32_t mw[2] = {m.x, m.y};
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = b2f(uint16_t(mw[e >> 1] >> (16 * (e & 1)))) > 0.f ? g[e] : 0.f;
        *reinterpret_cast<uint2 *>(Zc + at) = make_uint2(float2_to_bf16x2(o[0], o[1]), float2_to_bf16x2(o[2], o[3]));
    }
}

// The input in BF16, one channel.
__global__ __launch_bounds__(256) void k_pack(const float *__restrict__ f, uint16_t *__restrict__ X, int64_t m) {
    const int64_t v = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (v < m) X[v] = f2b(f[v]);
}

// MSE of the prediction y: partials of (y - t)^2 / m per workgroup; Z = bf16(2 (y - t) / m), one channel.
__global__ __launch_bounds__(256) void k_mse(const float *__restrict__ y, const float *__restrict__ t,
                                             uint16_t *__restrict__ Z, double *__restrict__ part, int64_t m) {
    const int64_t v = int64_t(blockIdx.x) * 256 + threadIdx.x;
    double acc = 0.0;
    if (v < m) {
        const float d = y[v] - t[v];
        acc = double(d) * double(d) / double(m);
        Z[v] = f2b(2.f * d / float(m));
    }
    acc = block_sum(acc);
    if (threadIdx.x == 0) part[blockIdx.x] = acc;
}

// Gradient sums and loss to zero.
__global__ __launch_bounds__(256) void k_clear(float *__restrict__ g, int64_t np, double *__restrict__ loss) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i < np) g[i] = 0.f;
    if (i == 0) loss[0] = 0.0;
}

__global__ __launch_bounds__(256) void k_dsum(const double *__restrict__ part, int np, double *__restrict__ out) {
    double a = 0.0;
    int b = threadIdx.x;
    for (; b + 7 * 256 < np; b += 8 * 256) {  // eight loads in flight, summed in order
        double t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = part[b + u * 256];
#pragma unroll
        for (int u = 0; u < 8; ++u) a += t[u];
    }
    for (; b < np; b += 256) a += part[b];
    a = block_sum(a);
    if (threadIdx.x == 0) out[0] += a;
}

// Adam on FP32 master weights (bias-corrected), refreshes the bf16 copies.
__global__ __launch_bounds__(256) void k_adam(float *__restrict__ w, float *__restrict__ m, float *__restrict__ v,
                                              const float *__restrict__ g, uint16_t *__restrict__ wb, int64_t np,
                                              float lr, float b1, float b2, float eps, float c1, float c2, float gs) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i >= np) return;
    const float gi = g[i] * gs;
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    w[i] = wi;
    const int64_t k = i / kPsz, r = i % kPsz;
    if (r < kWsz) wb[k * kWsz + r] = f2b(wi);
}

// bf16 copies of the master weights.
__global__ __launch_bounds__(256) void k_wcast(const float *__restrict__ w, uint16_t *__restrict__ wb, int64_t np) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i >= np) return;
    const int64_t k = i / kPsz, r = i % kPsz;
    if (r < kWsz) wb[k * kWsz + r] = f2b(w[i]);
}

// FP64 field -> FP32 * scale.
__global__ __launch_bounds__(256) void k_to32(const double *__restrict__ a, float *__restrict__ b, double s, int64_t m) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i < m) b[i] = float(a[i] * s);
}

// FP32 * scale -> FP64.
__global__ __launch_bounds__(256) void k_to64(const float *__restrict__ a, double *__restrict__ b, double s, int64_t m) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i < m) b[i] = double(a[i]) * s;
}

// 2^3-cell average, FP64 (no residual).
__global__ __launch_bounds__(256) void k_avg(const double *__restrict__ f, double *__restrict__ fc, int lgc) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i >= (int64_t(1) << (3 * lgc))) return;
    const int nc = 1 << lgc, lg = lgc + 1;
    const int X = int(i & (nc - 1)), Y = int((i >> lgc) & (nc - 1)), Z = int(i >> (2 * lgc));
    double s = 0.0;
    for (int c = 0; c < 2; ++c)
        for (int b = 0; b < 2; ++b)
            for (int a = 0; a < 2; ++a) s += f[(((int64_t(2 * Z + c) << lg) + 2 * Y + b) << lg) + 2 * X + a];
    fc[i] = 0.125 * s;
}

// ----------------------------------------------------------------- network
inline unsigned nb(int64_t m) { return unsigned((m + 255) / 256); }

struct Net {
    int levels = 0, lg0 = 0, nconv = 0;
    int64_t npar = 0;
    float *w = nullptr, *m = nullptr, *v = nullptr, *g = nullptr;  // FP32 master, Adam moments, gradient sums
    uint16_t *wb = nullptr, *wt = nullptr;                            // bf16 weights, flipped for the data gradient
    int64_t step = 0;
    // per level: h (input), a, e (encoder); u, c, d (decoder); Z, Z2 (masked BF16 gradients); FP32
    // gradients: S (of an encoder level's input, levels >= 1), K (of a decoder level's input)
    std::vector<uint16_t *> h, a, e, u, c, d, Z, Z2;
    std::vector<float *> S, K;
    float *out = nullptr, *scr = nullptr;  // FP32: prediction [n^3]; scratch of two such fields
    float *wpart = nullptr;                 // weight-gradient partials
    double *lpart = nullptr, *lsum = nullptr, *hsum = nullptr;
    std::vector<void *> owned;
    std::mutex mu;
};

np_status nalloc(Net *N, void **p, size_t bytes) {
    if (hipMalloc(p, bytes) != hipSuccess) {
        (void)hipGetLastError();
        set_error("hipMalloc of %zu bytes failed", bytes);
        return NP_ENOMEM;
    }
    N->owned.push_back(*p);
    return NP_OK;
}

int64_t vox(int lg) { return int64_t(1) << (3 * lg); }

template <ConvOut OUT, bool ONE = false>
np_status conv(Net *N, int k, const uint16_t *X, const uint16_t *act, void *Y, int lg, bool flip, hipStream_t s) {
    const int n = 1 << lg, txv = n < 64 ? n : 64;
    const uint16_t *W = (flip ? N->wt : N->wb) + int64_t(k) * kWsz;
    const float *bias = flip ? nullptr : N->w + int64_t(k) * kPsz + kWsz;
    // planes per workgroup: n / 8 from n = 128 (three convolutions at 128^3: 160 us with 2 planes, 127 with 8,
    // 122 with 16, 147 with 32; at 256^3 943 with 8, 898 with 32), below it as few as fill the chip (64^3: 49 us
    // with 1 or 2, 63 with 8; 32^3: 34 with 1, 43 with 4, and 36 with the one-plane form)
    const int zc = g_conv3z == 1 ? (n >= 128 ? n / 8 : std::max(1, n / 32)) : std::min(g_conv3z, n);
    if (g_conv3z)
        hipLaunchKernelGGL((k_conv3z<OUT, ONE>), dim3(unsigned((n / txv) * (n * txv / kCzT) * (n / zc))), dim3(kCzT), 0, s, X, W,
                           bias, act, Y, lg, zc);
    else
        hipLaunchKernelGGL((k_conv<OUT, ONE>), dim3(unsigned((n / txv) * (n / 4) * n)), dim3(256), 0, s, X, W, bias, act, Y,
                           lg);
    NP_LAUNCH_CHECK();
    return NP_OK;
}

// Weight and bias gradients of conv k with input `in` from its masked output gradient z (level l).
template <bool ONEX = false, bool ONEZ = false>
np_status wgrad(Net *N, int k, const uint16_t *in, const uint16_t *z, int l, hipStream_t s) {
    const int lg = N->lg0 - l;
    const int n = 1 << lg, txv = n < 64 ? n : 64, ntile = (n / txv) * (n / 4) * n;
    int nblk = ntile < kWgBlocks ? ntile : kWgBlocks;
    if (g_wgrad_mfma) {
        // chunks of planes per column, so that kWmAim workgroups (two per CU) run where there are as many tiles
        const int ncol = ntile / n, nch = std::min(n, std::max(1, kWmAim / ncol));
        nblk = std::min(ncol * nch, kWgBlocks);
        hipLaunchKernelGGL((k_wgrad_mfma<ONEX, ONEZ>), dim3(nblk), dim3(kWmT), 0, s, in, z, N->wpart, lg, nch);
    } else {
        hipLaunchKernelGGL((k_wgrad<ONEX, ONEZ>), dim3(nblk), dim3(256), 0, s, in, z, N->wpart, lg);
    }
    NP_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_wgrad_reduce, dim3(unsigned((kPsz + 31) / 32)), dim3(8 * kRedSl), 0, s, N->wpart, nblk,
                       N->g + int64_t(k) * kPsz);
    NP_LAUNCH_CHECK();
    return NP_OK;
}

// Forward: f (FP32, n^3) -> prediction (FP32, n^3).
np_status forward(Net *N, const float *f, float *pred, hipStream_t s) {
    const int L = N->levels;
    const int64_t m0 = vox(N->lg0);
    hipLaunchKernelGGL(k_pack, dim3(nb(m0)), dim3(256), 0, s, f, N->h[0], m0);
    NP_LAUNCH_CHECK();
    int k = 0;
    for (int l = 0; l < L; ++l) {
        const int lg = N->lg0 - l;
        if (l > 0) {
            hipLaunchKernelGGL(k_pool, dim3(nb(vox(lg) * 2)), dim3(256), 0, s, N->e[l - 1], N->h[l], lg);
            NP_LAUNCH_CHECK();
        }
        if (l == 0) NP_TRY((conv<kOutRelu, true>(N, k++, N->h[0], nullptr, N->a[0], lg, false, s)));
        else NP_TRY(conv<kOutRelu>(N, k++, N->h[l], nullptr, N->a[l], lg, false, s));
        NP_TRY(conv<kOutRelu>(N, k++, N->a[l], nullptr, N->e[l], lg, false, s));
    }
    const uint16_t *dn = N->e[L - 1];
    for (int l = L - 2; l >= 0; --l) {
        const int lg = N->lg0 - l;
        hipLaunchKernelGGL(k_up_add, dim3(nb(vox(lg) * 2)), dim3(256), 0, s, dn, N->e[l], N->u[l], lg);
        NP_LAUNCH_CHECK();
        NP_TRY(conv<kOutRelu>(N, k++, N->u[l], nullptr, N->c[l], lg, false, s));
        NP_TRY(conv<kOutRelu>(N, k++, N->c[l], nullptr, N->d[l], lg, false, s));
        dn = N->d[l];
    }
    NP_TRY(conv<kOutOne>(N, k, dn, nullptr, pred, N->lg0, false, s));
    return NP_OK;
}

// Backward from Z[0] (the prediction's gradient, BF16, one channel); gradient sums accumulate in N->g.
// Every layer's output gradient is masked by its activation where it is formed, alternating between Z
// and Z2 of a level; FP32 gradients are stored only where two are added (K) or crossed by a transfer.
// Two samples of 128^3 with four levels: 5.22 ms with FP32 gradients everywhere, separate mask, add and
// clearing passes and 16-channel FP32 predictions, 3.51 ms so (2.20 with the convolutions, weight gradients
// and one-channel fields as they are now).
np_status backward(Net *N, hipStream_t s) {
    const int L = N->levels;
    const uint16_t *dtop = L >= 2 ? N->d[0] : N->e[0];
    NP_TRY((wgrad<false, true>(N, N->nconv - 1, dtop, N->Z[0], 0, s)));
    NP_TRY((conv<kOutMask, true>(N, N->nconv - 1, N->Z[0], dtop, N->Z2[0], N->lg0, true, s)));
    // decoder levels 0 .. L-2 (conv indices 2L + 2 (L-2-l) .. +1), entered with the gradient in Z2
    for (int l = 0; l <= L - 2; ++l) {
        const int k1 = 2 * L + 2 * (L - 2 - l), k2 = k1 + 1, lg = N->lg0 - l;
        NP_TRY(wgrad(N, k2, N->c[l], N->Z2[l], l, s));
        NP_TRY(conv<kOutMask>(N, k2, N->Z2[l], N->c[l], N->Z[l], lg, true, s));
        NP_TRY(wgrad(N, k1, N->u[l], N->Z[l], l, s));
        NP_TRY(conv<kOutF32>(N, k1, N->Z[l], nullptr, N->K[l], lg, true, s));
        hipLaunchKernelGGL(k_up_back, dim3(nb(vox(lg - 1) * 2)), dim3(256), 0, s, N->K[l],
                           l + 1 <= L - 2 ? N->d[l + 1] : N->e[L - 1], N->Z2[l + 1], lg - 1);
        NP_LAUNCH_CHECK();
    }
    // encoder levels L-1 .. 0, likewise
    for (int l = L - 1; l >= 0; --l) {
        const int lg = N->lg0 - l;
        if (l < L - 1) {
            hipLaunchKernelGGL(k_join_back, dim3(nb(vox(lg) * 2)), dim3(256), 0, s, N->S[l + 1], N->K[l], N->e[l],
                               N->Z2[l], lg);
            NP_LAUNCH_CHECK();
        }
        NP_TRY(wgrad(N, 2 * l + 1, N->a[l], N->Z2[l], l, s));
        NP_TRY(conv<kOutMask>(N, 2 * l + 1, N->Z2[l], N->a[l], N->Z[l], lg, true, s));
        if (l == 0) NP_TRY((wgrad<true, false>(N, 0, N->h[0], N->Z[0], 0, s)));
        else NP_TRY(wgrad(N, 2 * l, N->h[l], N->Z[l], l, s));
        if (l > 0) NP_TRY(conv<kOutF32>(N, 2 * l, N->Z[l], nullptr, N->S[l], lg, true, s));
    }
    return NP_OK;
}

np_status refresh(Net *N, hipStream_t s) {
    hipLaunchKernelGGL(k_wcast, dim3(nb(N->npar)), dim3(256), 0, s, N->w, N->wb, N->npar);
    NP_LAUNCH_CHECK();
    for (int k = 0; k < N->nconv; ++k) {
        hipLaunchKernelGGL(k_wflip, dim3(nb(kWsz)), dim3(256), 0, s, N->wb + int64_t(k) * kWsz,
                           N->wt + int64_t(k) * kWsz);
        NP_LAUNCH_CHECK();
    }
    return NP_OK;
}

np_status loss_grad(Net *N, const float *target, hipStream_t s) {
    const int64_t m = vox(N->lg0);
    hipLaunchKernelGGL(k_mse, dim3(nb(m)), dim3(256), 0, s, N->out, target, N->Z[0], N->lpart, m);
    NP_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_dsum, dim3(1), dim3(256), 0, s, N->lpart, int(nb(m)), N->lsum);
    NP_LAUNCH_CHECK();
    return NP_OK;
}

void free_net(Net *N) {
    for (void *p : N->owned) (void)hipFree(p);
    if (N->hsum) (void)hipHostFree(N->hsum);
    delete N;
}

}  // namespace

// Attached network for warm starts (np_cnn_attach).
static std::mutex g_cnn_mu;
static Net *g_attached = nullptr;

// Warm start used by the solver: x0 (FP64, fine grid of 2^lg cells) from f
// through the attached network at its input resolution, with the fine f
// restricted by averaging and the prediction prolongated back.  tmp buffers:
// fl[l], xl[l] FP64 for levels 1..ell of the hierarchy.  Returns NP_EINVAL
// when no network fits this grid.
np_status cnn_warm_start(int d, int lg, int bc, const double *f, double *x0, const std::vector<void *> &fl,
                         const std::vector<void *> &xl, double *f32buf_bytes_unused, hipStream_t s, bool *used) {
    (void)f32buf_bytes_unused;
    *used = false;
    std::lock_guard<std::mutex> lk(g_cnn_mu);
    Net *N = g_attached;
    if (!N || d != 3 || lg < N->lg0) return NP_OK;
    const int ell = lg - N->lg0;
    if (ell >= int(fl.size())) return NP_OK;
    std::lock_guard<std::mutex> lk2(N->mu);
    // restrict f down to the network's grid
    const double *src = f;
    for (int l = 1; l <= ell; ++l) {
        hipLaunchKernelGGL(k_avg, dim3(nb(vox(lg - l))), dim3(256), 0, s, src, (double *)fl[l], lg - l);
        NP_LAUNCH_CHECK();
        src = (const double *)fl[l];
    }
    const int64_t mc = vox(N->lg0);
    // scale by the rms of the coarse rhs (the map f -> x is linear)
    const unsigned nb2 = std::min<unsigned>(kRedBlocks, unsigned((mc + 255) / 256));
    hipLaunchKernelGGL((k_sum<double>), dim3(nb2), dim3(256), 0, s, src, mc, 1, N->lpart);
    NP_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_finalize, dim3(1), dim3(256), 0, s, N->lpart, int(nb2), N->lsum, 0);
    NP_LAUNCH_CHECK();
    NP_HIP_TRY(hipMemcpyAsync(N->hsum, N->lsum, sizeof(double), hipMemcpyDeviceToHost, s));
    NP_HIP_TRY(hipStreamSynchronize(s));
    const double rms = std::sqrt(N->hsum[0] / double(mc));
    if (!(rms > 0.0) || !std::isfinite(rms)) return NP_OK;
    float *in = N->scr, *pred = N->scr + mc;
    hipLaunchKernelGGL(k_to32, dim3(nb(mc)), dim3(256), 0, s, src, in, 1.0 / rms, mc);
    NP_LAUNCH_CHECK();
    NP_TRY(forward(N, in, pred, s));
    double *xc = ell > 0 ? (double *)xl[ell] : x0;
    hipLaunchKernelGGL(k_to64, dim3(nb(mc)), dim3(256), 0, s, pred, xc, rms, mc);
    NP_LAUNCH_CHECK();
    // prolongate back to the fine grid
    for (int l = ell - 1; l >= 0; --l) {
        double *xf = l > 0 ? (double *)xl[l] : x0;
        const int64_t mf = vox(lg - l);
        hipLaunchKernelGGL((k_zero<double>), dim3(nb(mf)), dim3(256), 0, s, xf, mf, nullptr);
        NP_LAUNCH_CHECK();
        hipLaunchKernelGGL((k_prolong_add<3, double>), dim3(nb(mf)), dim3(256), 0, s, (const double *)xc, xf,
                           lg - l - 1, bc, nullptr);
        NP_LAUNCH_CHECK();
        xc = xf;
    }
    *used = true;
    return NP_OK;
}

// log2 of the attached network's grid size per axis, -1 when none is attached.
int cnn_attached_lg() {
    std::lock_guard<std::mutex> lk(g_cnn_mu);
    return g_attached ? g_attached->lg0 : -1;
}

// Network prediction on a coarse level of the solver's cycle (the learned
// coarse-grid correction): xc = rms * N(fc / rms) on the attached network's own
// grid, fc the level's restricted residual (device FP64, n_in^3 cells, n_in =
// 2^lg), rms its root mean square.  *used = false (xc untouched) when no
// network is attached, its grid is not 2^lg per axis, or fc is zero.  Reads
// the rms on the host (the stream is synchronised).
np_status cnn_coarse_guess(int lg, const double *fc, double *xc, hipStream_t s, bool *used) {
    *used = false;
    std::lock_guard<std::mutex> lk(g_cnn_mu);
    Net *N = g_attached;
    if (!N || N->lg0 != lg) return NP_OK;
    std::lock_guard<std::mutex> lk2(N->mu);
    const int64_t mc = vox(lg);
    const unsigned nb2 = std::min<unsigned>(kRedBlocks, unsigned((mc + 255) / 256));
    hipLaunchKernelGGL((k_sum<double>), dim3(nb2), dim3(256), 0, s, fc, mc, 1, N->lpart);
    NP_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_finalize, dim3(1), dim3(256), 0, s, N->lpart, int(nb2), N->lsum, 0);
    NP_LAUNCH_CHECK();
    NP_HIP_TRY(hipMemcpyAsync(N->hsum, N->lsum, sizeof(double), hipMemcpyDeviceToHost, s));
    NP_HIP_TRY(hipStreamSynchronize(s));
    const double rms = std::sqrt(N->hsum[0] / double(mc));
    if (!(rms > 0.0) || !std::isfinite(rms)) return NP_OK;
    float *in = N->scr, *pred = N->scr + mc;
    hipLaunchKernelGGL(k_to32, dim3(nb(mc)), dim3(256), 0, s, fc, in, 1.0 / rms, mc);
    NP_LAUNCH_CHECK();
    NP_TRY(forward(N, in, pred, s));
    hipLaunchKernelGGL(k_to64, dim3(nb(mc)), dim3(256), 0, s, pred, xc, rms, mc);
    NP_LAUNCH_CHECK();
    *used = true;
    return NP_OK;
}

}  // namespace np

using namespace np;

struct np_cnn {
    Net *net;
};

extern "C" np_status np_cnn_create(int n_in, int levels, np_cnn **out) {
    clear_error();
    if (!out || !is_pow2(n_in) || levels < 1 || levels > 6 || (n_in >> (levels - 1)) < 16 || n_in > 512) {
        set_error("network input must be a power of two >= 16 * 2^(levels-1), <= 512");
        return NP_EINVAL;
    }
    Net *N = new Net;
    N->levels = levels;
    N->lg0 = ilog2(n_in);
    N->nconv = 4 * levels - 1;
    N->npar = int64_t(N->nconv) * kPsz;
    np_status st = NP_OK;
    auto A = [&](void **p, size_t b) {
        if (st == NP_OK) st = nalloc(N, p, b);
        if (st == NP_OK) (void)hipMemset(*p, 0, b);
    };
    A((void **)&N->w, sizeof(float) * N->npar);
    A((void **)&N->m, sizeof(float) * N->npar);
    A((void **)&N->v, sizeof(float) * N->npar);
    A((void **)&N->g, sizeof(float) * N->npar);
    A((void **)&N->wb, sizeof(uint16_t) * N->nconv * kWsz);
    A((void **)&N->wt, sizeof(uint16_t) * N->nconv * kWsz);
    N->h.assign(levels, nullptr); N->a = N->h; N->e = N->h; N->u = N->h; N->c = N->h; N->d = N->h; N->Z = N->h; N->Z2 = N->h;
    N->S.assign(levels, nullptr); N->K = N->S;
    for (int l = 0; l < levels; ++l) {
        const size_t mb = size_t(vox(N->lg0 - l)) * kC;
        A((void **)&N->h[l], 2 * mb);
        A((void **)&N->a[l], 2 * mb);
        A((void **)&N->e[l], 2 * mb);
        A((void **)&N->Z[l], 2 * mb);
        A((void **)&N->Z2[l], 2 * mb);
        if (l > 0) A((void **)&N->S[l], 4 * mb);
        if (l < levels - 1) {
            A((void **)&N->u[l], 2 * mb);
            A((void **)&N->c[l], 2 * mb);
            A((void **)&N->d[l], 2 * mb);
            A((void **)&N->K[l], 4 * mb);
        }
    }
    const size_t m0 = size_t(vox(N->lg0));
    A((void **)&N->out, 4 * m0);
    A((void **)&N->scr, 4 * 2 * m0);
    A((void **)&N->wpart, sizeof(float) * kWgBlocks * kPsz);
    A((void **)&N->lpart, sizeof(double) * std::max<size_t>(kRedBlocks, (m0 + 255) / 256));
    A((void **)&N->lsum, sizeof(double));
    if (st == NP_OK && hipHostMalloc((void **)&N->hsum, sizeof(double), hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        set_error("hipHostMalloc failed");
        st = NP_ENOMEM;
    }
    if (st != NP_OK) {
        free_net(N);
        return st;
    }
    *out = new np_cnn{N};
    return NP_OK;
}

extern "C" void np_cnn_destroy(np_cnn *net) {
    if (!net) return;
    {
        std::lock_guard<std::mutex> lk(g_cnn_mu);
        if (g_attached == net->net) g_attached = nullptr;
    }
    (void)hipDeviceSynchronize();
    free_net(net->net);
    delete net;
}

extern "C" int64_t np_cnn_num_params(const np_cnn *net) { return net ? net->net->npar : -1; }

extern "C" np_status np_cnn_set_params(np_cnn *net, const float *host, int64_t count) {
    clear_error();
    if (!net || !host || count != net->net->npar) { set_error("parameter count mismatch"); return NP_EINVAL; }
    Net *N = net->net;
    std::lock_guard<std::mutex> lk(N->mu);
    NP_HIP_TRY(hipMemcpy(N->w, host, sizeof(float) * count, hipMemcpyHostToDevice));
    NP_HIP_TRY(hipMemset(N->m, 0, sizeof(float) * count));
    NP_HIP_TRY(hipMemset(N->v, 0, sizeof(float) * count));
    N->step = 0;
    NP_TRY(refresh(N, nullptr));
    NP_HIP_TRY(hipDeviceSynchronize());
    return NP_OK;
}

extern "C" np_status np_cnn_get_params(const np_cnn *net, float *host, int64_t count) {
    clear_error();
    if (!net || !host || count != net->net->npar) { set_error("parameter count mismatch"); return NP_EINVAL; }
    NP_HIP_TRY(hipMemcpy(host, net->net->w, sizeof(float) * count, hipMemcpyDeviceToHost));
    return NP_OK;
}

extern "C" np_status np_cnn_get_grads(const np_cnn *net, float *host, int64_t count) {
    clear_error();
    if (!net || !host || count != net->net->npar) { set_error("parameter count mismatch"); return NP_EINVAL; }
    NP_HIP_TRY(hipMemcpy(host, net->net->g, sizeof(float) * count, hipMemcpyDeviceToHost));
    return NP_OK;
}

extern "C" np_status np_cnn_forward(np_cnn *net, const float *in, float *out, void *stream) {
    clear_error();
    if (!net || !in || !out) { set_error("null argument"); return NP_EINVAL; }
    Net *N = net->net;
    std::lock_guard<std::mutex> lk(N->mu);
    hipStream_t s = (hipStream_t)stream;
    NP_TRY(forward(N, in, out, s));
    NP_HIP_TRY(hipStreamSynchronize(s));
    return NP_OK;
}

// Zeroes the gradient sums, then forward + MSE + backward for each pair; the
// gradient sums (not averaged) are left in the network.  *loss: sum of the
// pairs' MSE.
static np_status grads_for(Net *N, int batch, const float *const *in, const float *const *target, double *loss,
                           hipStream_t s) {
    hipLaunchKernelGGL(k_clear, dim3(nb(N->npar)), dim3(256), 0, s, N->g, N->npar, N->lsum);
    NP_LAUNCH_CHECK();
    for (int b = 0; b < batch; ++b) {
        NP_TRY(forward(N, in[b], N->out, s));
        NP_TRY(loss_grad(N, target[b], s));
        NP_TRY(backward(N, s));
    }
    NP_HIP_TRY(hipMemcpyAsync(N->hsum, N->lsum, sizeof(double), hipMemcpyDeviceToHost, s));
    NP_HIP_TRY(hipStreamSynchronize(s));
    if (loss) *loss = N->hsum[0];
    return NP_OK;
}

extern "C" np_status np_cnn_gradients(np_cnn *net, int batch, const float *const *in, const float *const *target,
                                      double *loss, void *stream) {
    clear_error();
    if (!net || batch <= 0 || !in || !target) { set_error("bad argument"); return NP_EINVAL; }
    Net *N = net->net;
    std::lock_guard<std::mutex> lk(N->mu);
    return grads_for(N, batch, in, target, loss, (hipStream_t)stream);
}

// Gradients of the batch, then one Adam step on their mean.
static np_status train_step(Net *N, int batch, const float *const *in, const float *const *target, float lr,
                            double *loss, hipStream_t s) {
    NP_TRY(grads_for(N, batch, in, target, loss, s));
    N->step += 1;
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float c1 = 1.f - std::pow(b1, float(N->step)), c2 = 1.f - std::pow(b2, float(N->step));
    hipLaunchKernelGGL(k_adam, dim3(nb(N->npar)), dim3(256), 0, s, N->w, N->m, N->v, N->g, N->wb, N->npar, lr, b1, b2,
                       eps, c1, c2, 1.f / float(batch));
    NP_LAUNCH_CHECK();
    for (int k = 0; k < N->nconv; ++k) {
        hipLaunchKernelGGL(k_wflip, dim3(nb(kWsz)), dim3(256), 0, s, N->wb + int64_t(k) * kWsz,
                           N->wt + int64_t(k) * kWsz);
        NP_LAUNCH_CHECK();
    }
    NP_HIP_TRY(hipStreamSynchronize(s));
    return NP_OK;
}

extern "C" np_status np_cnn_train_step(np_cnn *net, int batch, const float *const *in, const float *const *target,
                                       float lr, double *loss, void *stream) {
    clear_error();
    if (!net || batch <= 0 || !in || !target || !(lr > 0.f)) { set_error("bad argument"); return NP_EINVAL; }
    Net *N = net->net;
    std::lock_guard<std::mutex> lk(N->mu);
    return train_step(N, batch, in, target, lr, loss, (hipStream_t)stream);
}

// Restricts f (and p) from the fine grid to the network's grid by repeated
// 2^3 averaging, scales both by 1 / rms(restricted f) and writes FP32 copies.
static np_status prepare(Net *N, int lg, const double *f, const double *p, float *in, float *target, double *scale,
                        hipStream_t s) {
    const int ell = lg - N->lg0;
    std::vector<double *> tmp;
    double *fb = nullptr, *pb = nullptr;
    auto chain = [&](const double *src, double **res) -> np_status {
        const double *cur = src;
        for (int l = 1; l <= ell; ++l) {
            double *dst = nullptr;
            if (hipMalloc((void **)&dst, sizeof(double) * vox(lg - l)) != hipSuccess) {
                (void)hipGetLastError();
                set_error("hipMalloc failed");
                return NP_ENOMEM;
            }
            tmp.push_back(dst);
            hipLaunchKernelGGL(k_avg, dim3(nb(vox(lg - l))), dim3(256), 0, s, cur, dst, lg - l);
            NP_LAUNCH_CHECK();
            cur = dst;
        }
        *res = const_cast<double *>(cur);
        return NP_OK;
    };
    np_status st = chain(f, &fb);
    if (st == NP_OK && p) st = chain(p, &pb);
    const int64_t mc = vox(N->lg0);
    double rms = 0.0;
    if (st == NP_OK) {
        const unsigned nb2 = std::min<unsigned>(kRedBlocks, unsigned((mc + 255) / 256));
        hipLaunchKernelGGL((k_sum<double>), dim3(nb2), dim3(256), 0, s, fb, mc, 1, N->lpart);
        hipLaunchKernelGGL(k_finalize, dim3(1), dim3(256), 0, s, N->lpart, int(nb2), N->lsum, 0);
        if (hipMemcpyAsync(N->hsum, N->lsum, sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess) {
            set_error("reduction failed");
            st = NP_EHIP;
        }
        rms = std::sqrt(N->hsum[0] / double(mc));
    }
    if (st == NP_OK) {
        const double sc = rms > 0.0 ? 1.0 / rms : 1.0;
        hipLaunchKernelGGL(k_to32, dim3(nb(mc)), dim3(256), 0, s, fb, in, sc, mc);
        if (p && target) hipLaunchKernelGGL(k_to32, dim3(nb(mc)), dim3(256), 0, s, pb, target, sc, mc);
        if (hipStreamSynchronize(s) != hipSuccess) { set_error("prepare failed"); st = NP_EHIP; }
        if (scale) *scale = rms;
    }
    for (double *q : tmp) (void)hipFree(q);
    return st;
}

extern "C" np_status np_cnn_prepare(np_cnn *net, np_dims dims, const double *f, const double *p, float *in,
                                    float *target, double *scale, void *stream) {
    clear_error();
    const int lg = check_grid(dims);
    if (lg < 0 || dims.ndim != 3 || !net || !f || !in) { set_error("bad argument"); return NP_EINVAL; }
    Net *N = net->net;
    if (lg < N->lg0) { set_error("grid coarser than the network input"); return NP_EINVAL; }
    std::lock_guard<std::mutex> lk(N->mu);
    return prepare(N, lg, f, p, in, target, scale, (hipStream_t)stream);
}

extern "C" np_status np_cnn_attach(np_cnn *net) {
    std::lock_guard<std::mutex> lk(g_cnn_mu);
    g_attached = net ? net->net : nullptr;
    return NP_OK;
}

// File: "NPCNN1\n", int32 levels, int32 n_in, int64 count, count float32 master weights.
extern "C" np_status np_cnn_save(const np_cnn *net, const char *path) {
    clear_error();
    if (!net || !path) { set_error("bad argument"); return NP_EINVAL; }
    const Net *N = net->net;
    std::vector<float> w(N->npar);
    NP_HIP_TRY(hipMemcpy(w.data(), N->w, sizeof(float) * N->npar, hipMemcpyDeviceToHost));
    FILE *fp = std::fopen(path, "wb");
    if (!fp) { set_error("cannot open %s", path); return NP_EINVAL; }
    const int32_t hdr[2] = {N->levels, 1 << N->lg0};
    const int64_t cnt = N->npar;
    const bool ok = std::fwrite("NPCNN1\n", 1, 7, fp) == 7 && std::fwrite(hdr, sizeof hdr, 1, fp) == 1 &&
                    std::fwrite(&cnt, sizeof cnt, 1, fp) == 1 && std::fwrite(w.data(), sizeof(float), cnt, fp) == size_t(cnt);
    std::fclose(fp);
    if (!ok) { set_error("write failed: %s", path); return NP_EINVAL; }
    return NP_OK;
}

extern "C" np_status np_cnn_open(const char *path, np_cnn **out) {
    clear_error();
    if (!path || !out) { set_error("bad argument"); return NP_EINVAL; }
    FILE *fp = std::fopen(path, "rb");
    if (!fp) { set_error("cannot open %s", path); return NP_EINVAL; }
    char magic[7];
    int32_t hdr[2];
    int64_t cnt = 0;
    bool ok = std::fread(magic, 1, 7, fp) == 7 && std::memcmp(magic, "NPCNN1\n", 7) == 0 &&
              std::fread(hdr, sizeof hdr, 1, fp) == 1 && std::fread(&cnt, sizeof cnt, 1, fp) == 1 && cnt > 0 &&
              cnt < (int64_t(1) << 30);
    std::vector<float> w;
    if (ok) {
        w.resize(cnt);
        ok = std::fread(w.data(), sizeof(float), cnt, fp) == size_t(cnt);
    }
    std::fclose(fp);
    if (!ok) { set_error("not a network file: %s", path); return NP_EINVAL; }
    NP_TRY(np_cnn_create(hdr[1], hdr[0], out));
    np_status st = np_cnn_set_params(*out, w.data(), cnt);
    if (st != NP_OK) {
        np_cnn_destroy(*out);
        *out = nullptr;
    }
    return st;
}

// Network owned by the library (np_cnn_load).
static np_cnn *g_owned = nullptr;

extern "C" np_status np_cnn_load(const char *path) {
    clear_error();
    np_cnn *net = nullptr;
    if (path) NP_TRY(np_cnn_open(path, &net));
    np_cnn *old = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_cnn_mu);
        old = g_owned;
        g_owned = net;
        g_attached = net ? net->net : nullptr;
    }
    if (old) np_cnn_destroy(old);
    return NP_OK;
}

// He-normal weights from a seeded host generator: fan-in 27 for the first
// convolution (input channel 0 only), 27 x 16 otherwise; the output
// convolution writes channel 0 only and starts 10x smaller than its fan-in
// scale (the targets' variance is ~1e-2 of the inputs'; a full-scale first
// output makes the early Adam steps shrink every layer until the ReLUs die).
// Biases zero; Adam state reset.
extern "C" np_status np_cnn_init(np_cnn *net, uint64_t seed) {
    clear_error();
    if (!net) { set_error("bad argument"); return NP_EINVAL; }
    Net *N = net->net;
    std::vector<float> w(N->npar, 0.f);
    std::mt19937_64 eng(seed);
    std::normal_distribution<double> nd(0.0, 1.0);
    for (int k = 0; k < N->nconv; ++k) {
        float *W = w.data() + int64_t(k) * kPsz;
        for (int t = 0; t < kTaps; ++t)
            for (int o = 0; o < kC; ++o)
                for (int c = 0; c < kC; ++c) {
                    double sd;
                    if (k == 0) sd = c == 0 ? std::sqrt(2.0 / kTaps) : 0.0;
                    else if (k == N->nconv - 1) sd = o == 0 ? 0.1 * std::sqrt(1.0 / (kTaps * kC)) : 0.0;
                    else sd = std::sqrt(2.0 / (kTaps * kC));
                    W[(t * kC + o) * kC + c] = sd > 0.0 ? float(sd * nd(eng)) : 0.f;
                }
    }
    return np_cnn_set_params(net, w.data(), N->npar);
}

namespace {
// Reads `"key": number` members of a flat JSON object into the named slots;
// any other key or form is an error.
bool parse_cfg(const char *js, const char *const *keys, double *vals, int nkeys, std::string *err) {
    if (!js) return true;
    const char *q = js;
    auto ws = [&]() { while (*q == ' ' || *q == '\t' || *q == '\n' || *q == '\r') ++q; };
    ws();
    if (*q != '{') { *err = "configuration must be a JSON object"; return false; }
    ++q;
    ws();
    if (*q == '}') return true;
    for (;;) {
        ws();
        if (*q != '"') { *err = "expected a quoted key"; return false; }
        const char *k0 = ++q;
        while (*q && *q != '"') ++q;
        if (!*q) { *err = "unterminated key"; return false; }
        const std::string key(k0, q - k0);
        ++q;
        ws();
        if (*q != ':') { *err = "expected ':' after " + key; return false; }
        ++q;
        ws();
        char *end = nullptr;
        const double v = std::strtod(q, &end);
        if (end == q || !std::isfinite(v)) { *err = "value of " + key + " is not a number"; return false; }
        q = end;
        int idx = -1;
        for (int i = 0; i < nkeys; ++i)
            if (key == keys[i]) idx = i;
        if (idx < 0) { *err = "unknown key " + key; return false; }
        vals[idx] = v;
        ws();
        if (*q == ',') { ++q; continue; }
        if (*q == '}') {
            ++q;
            ws();
            if (*q) { *err = "text after the object"; return false; }
            return true;
        }
        *err = "expected ',' or '}'";
        return false;
    }
}
}  // namespace

// Trains a new network on (rhs, p) pairs and writes it to weights_out.
extern "C" np_status np_cnn_train(const np_dims *dims, np_bc bc, int npairs, const double *const *rhs,
                                  const double *const *p, const char *cfg_json, const char *weights_out,
                                  double *epoch_loss) {
    clear_error();
    if (!dims || !rhs || !p || !weights_out || npairs <= 0) { set_error("bad argument"); return NP_EINVAL; }
    if (bc != NP_BC_PERIODIC) { set_error("the network is periodic: bc must be NP_BC_PERIODIC"); return NP_EINVAL; }
    static const char *const keys[] = {"n_in", "levels", "epochs", "batch", "lr", "seed", "verbose"};
    double cfg[7] = {128, 4, 10, 4, 5e-4, 0, 0};
    std::string err;
    if (!parse_cfg(cfg_json, keys, cfg, 7, &err)) { set_error("configuration: %s", err.c_str()); return NP_EINVAL; }
    const bool verbose = cfg[6] != 0.0;
    const int n_in = int(cfg[0]), levels = int(cfg[1]), epochs = int(cfg[2]), batch = int(cfg[3]);
    const float lr = float(cfg[4]);
    const uint64_t seed = uint64_t(cfg[5]);
    if (epochs < 1 || batch < 1 || !(lr > 0.f) || cfg[5] < 0) { set_error("configuration: bad epochs, batch, lr or seed"); return NP_EINVAL; }
    std::vector<int> lgs(npairs);
    for (int i = 0; i < npairs; ++i) {
        lgs[i] = check_grid(dims[i]);
        if (lgs[i] < 0 || dims[i].ndim != 3 || !rhs[i] || !p[i]) { set_error("pair %d: bad grid or pointer", i); return NP_EINVAL; }
        if ((int64_t(1) << lgs[i]) < n_in) { set_error("pair %d: grid coarser than n_in", i); return NP_EINVAL; }
    }
    np_cnn *net = nullptr;
    NP_TRY(np_cnn_create(n_in, levels, &net));
    Net *N = net->net;
    const int64_t mc = vox(N->lg0);
    float *buf = nullptr;
    np_status st = np_cnn_init(net, seed);
    if (st == NP_OK && hipMalloc((void **)&buf, sizeof(float) * mc * 2 * npairs) != hipSuccess) {
        (void)hipGetLastError();
        set_error("hipMalloc of %lld bytes for the prepared pairs failed", (long long)(sizeof(float) * mc * 2 * npairs));
        st = NP_ENOMEM;
    }
    std::vector<const float *> xin(npairs), tgt(npairs);
    {
        std::lock_guard<std::mutex> lk(N->mu);
        for (int i = 0; i < npairs && st == NP_OK; ++i) {
            float *xi = buf + mc * 2 * i, *ti = xi + mc;
            xin[i] = xi;
            tgt[i] = ti;
            st = prepare(N, lgs[i], rhs[i], p[i], xi, ti, nullptr, nullptr);
        }
        const auto t0 = std::chrono::steady_clock::now();
        // seeded Fisher-Yates order per epoch, minibatches of `batch` pairs
        std::mt19937_64 eng(seed ^ 0x9e3779b97f4a7c15ull);
        std::vector<int> order(npairs);
        std::vector<const float *> bx, bt;
        for (int ep = 0; ep < epochs && st == NP_OK; ++ep) {
            for (int i = 0; i < npairs; ++i) order[i] = i;
            for (int i = npairs - 1; i > 0; --i) std::swap(order[i], order[eng() % uint64_t(i + 1)]);
            double tot = 0.0;
            for (int i0 = 0; i0 < npairs && st == NP_OK; i0 += batch) {
                const int nb2 = std::min(batch, npairs - i0);
                bx.assign(nb2, nullptr);
                bt.assign(nb2, nullptr);
                for (int j = 0; j < nb2; ++j) {
                    bx[j] = xin[order[i0 + j]];
                    bt[j] = tgt[order[i0 + j]];
                }
                double l = 0.0;
                st = train_step(N, nb2, bx.data(), bt.data(), lr, &l, nullptr);
                tot += l;
            }
            if (epoch_loss) epoch_loss[ep] = tot / npairs;
            if (verbose && st == NP_OK) {
                const double sec = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
                std::fprintf(stderr, "np_cnn_train: epoch %d/%d mean mse %.4e (%.1f s)\n", ep + 1, epochs,
                             tot / npairs, sec);
                std::fflush(stderr);
            }
        }
    }
    if (buf) (void)hipFree(buf);
    if (st == NP_OK) st = np_cnn_save(net, weights_out);
    np_cnn_destroy(net);
    return st;
}
