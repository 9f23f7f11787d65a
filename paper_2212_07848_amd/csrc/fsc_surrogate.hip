// fsc_surrogate.hip -- learned coarse-grained surrogate of the phase-separating
// lattice: a small periodic convolutional network that maps the block-averaged
// density at time t to the one at t + k lattice steps.  Not part of the paper:
// it is the inference/training path next to the lattice, assessed against the
// lattice's own S(k, t) and L(t).
//
// Network (C = 32 hidden channels, L layers, K = 1 or 2 input channels):
//   x_0 = (rho_t - mean)/in_scale,  x_1 = (rho_t - rho_{t-k})/out_scale (K = 2)
//   a_0 = SiLU(conv(x));  a_l = SiLU(conv(a_{l-1}));  y = conv(a_{L-2})
//   rho_{t+k} = rho_t + out_scale (y - <y>_image)
// The second channel, the last increment, carries the flow that the density
// alone does not determine.
// conv = 3x3 cross-correlation with circular padding.  The C -> C layers run
// as implicit GEMMs on v_mfma_f32_16x16x32_bf16 (BF16 operands, FP32
// accumulation), forward, backward-data and backward-weight.  The C -> 1
// forward runs on the matrix cores too, with its FP32 weights split exactly
// into three BF16 parts; the 1 -> C layer, the other C -> 1 passes and the
// reductions are FP32 vector code.  Parameters are FP32 masters updated by
// Adam; BF16 copies feed the matrix cores.
//
// Activations are NHWC: pixel p = (n H + y) W + x, channel fastest.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <deque>
#include <map>
#include <string>
#include <tuple>
#include <type_traits>
#include <utility>
#include <vector>

#include "../../include/fsc.h"
#include "fsc_internal.h"

namespace fsc {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int SC = 32;          // hidden channels
constexpr int IMG_PARTS = 256;  // segments per image of the per-image FP64 sums

// SiLU and its derivative from the hardware exp2 and reciprocal (about one
// ulp each).  Their results are rounded to bfloat16 (2^-8 relative) or feed
// FP32 sums, so a correctly rounded exp and division would change nothing
// but the cost, which in the matrix-core layers is the epilogue's.
__device__ __forceinline__ float sigmoid(float z) {
    return __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.44269504088896341f * z));
}
__device__ __forceinline__ float silu(float z) { return z * sigmoid(z); }
__device__ __forceinline__ float dsilu(float z) {
    const float s = sigmoid(z);
    return s * (1.f + z * (1.f - s));
}
__device__ __forceinline__ int wrapi(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// ---------------------------------------------------------------------------
// Matrix-core operand layout of v_mfma_f32_16x16x32_bf16 as used here: lane l
// supplies row (l % 16) of A and column (l % 16) of B with the eight K values
// 8 (l / 16) .. 8 (l / 16) + 7; the result element D[4 (l / 16) + r][l % 16] is
// register r of lane l.  (Any K order that is the same for A and B gives the
// same product; the M/N/D placement is checked by fsc_mfma_probe.)
// ---------------------------------------------------------------------------
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// Output channel of row m (0..15) of the A operand in MFMA tile nt (0, 1) of a
// C -> C layer: rows 4j .. 4j + 3 of tile nt hold channels 8j + 4nt .. 8j +
// 4nt + 3.  The result rows 4 (l/16) + r of lane l are then channels
// 8 (l/16) + 4nt + r: over both tiles, the eight consecutive channels
// 8 (l/16) .. 8 (l/16) + 7 of pixel l % 16, and one 16-byte store per lane
// writes whole 64-byte pixel records (a wave's store covers 1 KB).
__device__ __forceinline__ int mid_row_channel(int nt, int m) { return 8 * (m >> 2) + 4 * nt + (m & 3); }

// Epilogue of a C -> C layer tile computed as D = W (32 channels) x A (16
// pixels): lane l holds channels 8 (l/16) + 4nt + r, r = 0..3, of pixel l % 16
// in acc[nt] (mid_row_channel).  The forward pass starts its accumulators at
// the bias, so acc is already z.
//   forward:  z = acc (kept if ZOUT), a = bf16(SiLU(z))
//   backward: a = bf16(acc SiLU'(z_prev))
template <bool BWD, bool ZOUT>
__device__ __forceinline__ void mid_epilogue(const f32x4 (&acc)[2], size_t pix, int g,
                                             float *__restrict__ zout, bf16 *__restrict__ aout,
                                             const f32x4 (&zprev)[2]) {
    const size_t o = pix * SC + 8 * g;
    bf16x8 out;
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        if (!BWD && ZOUT) *reinterpret_cast<f32x4 *>(zout + o + 4 * nt) = acc[nt];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            out[4 * nt + r] = bf16(BWD ? acc[nt][r] * dsilu(zprev[nt][r]) : silu(acc[nt][r]));
    }
    // inference: non-temporal, the next layer reads the records from memory
    // anyway (3% per rollout pass against the default policy).  Training keeps
    // them cached: the launch after this one reads them (an Adam step of the
    // nine-layer network on 32 images of 128^2: 876 against 920 us).
    if (BWD || ZOUT) *reinterpret_cast<bf16x8 *>(aout + o) = out;
    else __builtin_nontemporal_store(out, reinterpret_cast<bf16x8 *>(aout + o));
}
__device__ __forceinline__ void load_z(const float *__restrict__ z, size_t pix, int g, f32x4 (&v)[2]) {
    const f32x4 *p = reinterpret_cast<const f32x4 *>(z + pix * SC + 8 * g);
    v[0] = p[0];
    v[1] = p[1];
}

__global__ void k_mfma_probe(const float *A, const float *B, float *Cm) {
    const int l = threadIdx.x, r16 = l & 15, g = l >> 4;
    bf16x8 a, b;
    for (int e = 0; e < 8; ++e) {
        a[e] = bf16(A[r16 * 32 + 8 * g + e]);
        b[e] = bf16(B[(8 * g + e) * 16 + r16]);
    }
    f32x4 c = {0.f, 0.f, 0.f, 0.f};
    c = mfma16(a, b, c);
    for (int r = 0; r < 4; ++r) Cm[(4 * g + r) * 16 + r16] = c[r];
}

// ---------------------------------------------------------------------------
// Layer 0 (K -> C) forward, FP32: one lane per pixel computes all 32 output
// channels.  The weights and biases are the same for every lane, so they are
// read through the scalar cache and enter the FMAs as scalar operands.  ZOUT
// keeps the FP32 pre-activations for the backward pass (training).  The
// network input is formed from the fields on the fly.  A pixel's 32 BF16
// activations go out as four 16-byte stores.  In training the pre-activations
// are twice as many bytes as those, and lane-strided 16-byte pieces of 128-byte
// records took 44 us at 32 images of 128^2 (100 MB written): there a wave
// passes them through LDS and stores 1 KB of consecutive bytes at a time
// (31.3 us).
// ---------------------------------------------------------------------------
template <int K, bool ZOUT>
__global__ void __launch_bounds__(256) k_first(const float *__restrict__ cur,
                                               const float *__restrict__ prev, float mean, float inv_in,
                                               float inv_out, int B, int H, int W,
                                               const float *__restrict__ w,
                                               const float *__restrict__ b, float *__restrict__ z,
                                               bf16 *__restrict__ a) {
    const int P = B * H * W;
    [[maybe_unused]] const int wave = threadIdx.x >> 6;
    // training: a wave's pre-activations, pieces of four channels, pixel l's at
    // 8 l + (piece ^ (l % 8)), so that neither side meets a bank conflict
    __shared__ __attribute__((aligned(16))) f32x4 zt[ZOUT ? 4 : 1][ZOUT ? 64 * 8 : 1];
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (!ZOUT && p >= P) return;
    const int pc = min(p, P - 1);  // lanes past the end repeat the last pixel
    const int x = pc % W, t = pc / W, y = t % H, n = t / H;
    float xi[K][9];
#pragma unroll
    for (int ky = 0; ky < 3; ++ky)
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
            const size_t q = size_t((n * H + wrapi(y + ky - 1, H)) * W + wrapi(x + kx - 1, W));
            const float c = cur[q];
            xi[0][ky * 3 + kx] = (c - mean) * inv_in;
            if constexpr (K == 2) xi[1][ky * 3 + kx] = (c - prev[q]) * inv_out;
        }
    [[maybe_unused]] const int lane = threadIdx.x & 63;
#pragma unroll
    for (int c8 = 0; c8 < SC / 8; ++c8) {
        bf16x8 out;
        f32x4 zq[2];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int co = c8 * 8 + j;
            float acc = b[co];
#pragma unroll
            for (int ci = 0; ci < K; ++ci)
#pragma unroll
                for (int k = 0; k < 9; ++k) acc += w[(co * K + ci) * 9 + k] * xi[ci][k];
            zq[j >> 2][j & 3] = acc;
            if constexpr (!ZOUT) out[j] = bf16(silu(acc));
        }
        if constexpr (ZOUT) {
            zt[wave][lane * 8 + ((2 * c8) ^ (lane & 7))] = zq[0];
            zt[wave][lane * 8 + ((2 * c8 + 1) ^ (lane & 7))] = zq[1];
        } else {
            *reinterpret_cast<bf16x8 *>(a + size_t(p) * SC + c8 * 8) = out;
        }
    }
    if constexpr (ZOUT) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // a wave reads what its own lanes wrote
        __builtin_amdgcn_wave_barrier();
        const int p0 = p - lane;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int px = i * 8 + (lane >> 3), q = lane & 7;
            if (p0 + px >= P) break;
            const f32x4 v = zt[wave][px * 8 + (q ^ (px & 7))];
            bf16x4 o;
#pragma unroll
            for (int r = 0; r < 4; ++r) o[r] = bf16(silu(v[r]));
            *reinterpret_cast<f32x4 *>(z + size_t(p0 + px) * SC + q * 4) = v;
            *reinterpret_cast<bf16x4 *>(a + size_t(p0 + px) * SC + q * 4) = o;
        }
    }
}

// ---------------------------------------------------------------------------
// C -> C layer on the matrix cores.  A wave computes 16 consecutive pixels of
// one image row for all 32 output channels: 9 taps x 2 tiles of 16x16x32
// MFMA, with the packed weights held in registers.  The weights are the A
// operand (16 output channels by 32 input channels) and the activations the B
// operand (32 input channels by 16 pixels); with the rows ordered by
// mid_row_channel, each lane's results over the two tiles are eight
// consecutive channels of one pixel (mid_epilogue).
//   forward:   out = conv(a_in; W) + bias -> z (FP32), SiLU(z) (BF16)
//   backward:  out = conv(dZ; W') (W' = tap-flipped transpose: the adjoint)
//              -> dZ_prev = out * SiLU'(z_prev) (BF16)
// ---------------------------------------------------------------------------
template <bool BWD, bool ZOUT = true>
__global__ void __launch_bounds__(256) k_mid(const bf16 *__restrict__ ain,
                                             const bf16 *__restrict__ wpk,
                                             const float *__restrict__ bias, int B, int H, int W,
                                             float *__restrict__ zout, bf16 *__restrict__ aout,
                                             const float *__restrict__ zprev) {
    const int lane = threadIdx.x & 63;
    const int wave = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int nwaves = gridDim.x * 4;
    const int r16 = lane & 15, g = lane >> 4;
    bf16x8 bop[9][2];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
            bop[t][nt] = *reinterpret_cast<const bf16x8 *>(
                wpk + (t * SC + mid_row_channel(nt, r16)) * SC + g * 8);
    f32x4 bv[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    if (!BWD) {
        bv[0] = *reinterpret_cast<const f32x4 *>(bias + 8 * g);
        bv[1] = *reinterpret_cast<const f32x4 *>(bias + 8 * g + 4);
    }
    const int tiles = (B * H * W) / 16;
    for (int tile = wave; tile < tiles; tile += nwaves) {
        const int p0 = tile * 16;
        const int x0 = p0 % W, t2 = p0 / W, y = t2 % H, n = t2 / H;
        f32x4 acc[2] = {bv[0], bv[1]};
#pragma unroll
        for (int ky = 0; ky < 3; ++ky) {
            const int rowbase = (n * H + wrapi(y + ky - 1, H)) * W;
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) {
                const int q = rowbase + wrapi(x0 + r16 + kx - 1, W);
                const bf16x8 aop = *reinterpret_cast<const bf16x8 *>(ain + size_t(q) * SC + g * 8);
                acc[0] = mfma16(bop[ky * 3 + kx][0], aop, acc[0]);
                acc[1] = mfma16(bop[ky * 3 + kx][1], aop, acc[1]);
            }
        }
        f32x4 zp[2];
        if (BWD) load_z(zprev, size_t(p0 + r16), g, zp);
        mid_epilogue<BWD, ZOUT>(acc, size_t(p0 + r16), g, zout, aout, zp);
    }
}

// The same layer with the input staged in LDS: a block computes a tile of
// MR rows x MW pixels of one image (MR MW / 16 MFMA tiles of 16 pixels, dealt
// to the 4 waves in order), after loading the tile's (MR+2) x (MW+2) input
// pixels with their 32 channels once (coalesced 16-byte pieces) instead of
// reading each pixel for each of the 9 taps from L2.  Needs H % MR == 0 and
// W % MW == 0.  The tile shape is a build-time choice (FSC_SUR_MR, FSC_SUR_MW).
#ifndef FSC_SUR_MR
#define FSC_SUR_MR 4
#endif
#ifndef FSC_SUR_MW
#define FSC_SUR_MW 64
#endif
constexpr int MR = FSC_SUR_MR, MW = FSC_SUR_MW;
static_assert(MW % 16 == 0 && (MR * MW / 16) % 4 == 0, "whole MFMA tiles, the same count per wave");
template <bool BWD, bool ZOUT>
__global__ void __launch_bounds__(256) k_mid_lds(const bf16 *__restrict__ ain,
                                                 const bf16 *__restrict__ wpk,
                                                 const float *__restrict__ bias, int B, int H, int W,
                                                 float *__restrict__ zout, bf16 *__restrict__ aout,
                                                 const float *__restrict__ zprev) {
    constexpr int LW = MW + 2;
    __shared__ __attribute__((aligned(16))) bf16 tile_in[(MR + 2) * LW * SC];
#ifdef FSC_LDS_POISON
    lds_poison(tile_in, (MR + 2) * LW * SC);
    __syncthreads();
#endif
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    const int txs = W / MW, tys = H / MR;
    const int bx = blockIdx.x % txs, t1 = blockIdx.x / txs;
    const int by = t1 % tys, n = t1 / tys;
    const int x0 = bx * MW, y0 = by * MR;
    // stage the input window: pixel (r, c) of the window is image pixel
    // (y0 - 1 + r, x0 - 1 + c), periodic; 4 pieces of 8 channels per pixel
    for (int k = threadIdx.x; k < (MR + 2) * LW * 4; k += 256) {
        const int piece = k & 3, pc = k >> 2;
        const int r = pc / LW, c = pc % LW;
        const int yy = wrapi(y0 - 1 + r, H), xx = wrapi(x0 - 1 + c, W);
        const size_t q = size_t((n * H + yy) * W + xx);
        *reinterpret_cast<bf16x8 *>(tile_in + pc * SC + piece * 8) =
            *reinterpret_cast<const bf16x8 *>(ain + q * SC + piece * 8);
    }
    bf16x8 bop[9][2];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
            bop[t][nt] = *reinterpret_cast<const bf16x8 *>(
                wpk + (t * SC + mid_row_channel(nt, r16)) * SC + g * 8);
    f32x4 bv[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    if (!BWD) {
        bv[0] = *reinterpret_cast<const f32x4 *>(bias + 8 * g);
        bv[1] = *reinterpret_cast<const f32x4 *>(bias + 8 * g + 4);
    }
    __syncthreads();
    constexpr int TPW = MR * MW / 64;  // MFMA tiles per wave
#pragma unroll
    for (int j = 0; j < TPW; ++j) {
        const int k = wave * TPW + j;
        const int row = k / (MW / 16), tx = k % (MW / 16);
        const int y = y0 + row;
        f32x4 acc[2] = {bv[0], bv[1]};
#pragma unroll
        for (int ky = 0; ky < 3; ++ky)
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) {
                const int pc = (row + ky) * LW + tx * 16 + r16 + kx;
                const bf16x8 aop = *reinterpret_cast<const bf16x8 *>(tile_in + pc * SC + g * 8);
                acc[0] = mfma16(bop[ky * 3 + kx][0], aop, acc[0]);
                acc[1] = mfma16(bop[ky * 3 + kx][1], aop, acc[1]);
            }
        const size_t p0 = size_t((n * H + y) * W + x0 + tx * 16);
        f32x4 zp[2];
        if (BWD) load_z(zprev, p0 + r16, g, zp);
        mid_epilogue<BWD, ZOUT>(acc, p0 + r16, g, zout, aout, zp);
    }
}

// Two consecutive C -> C layers A and B of the forward pass (inference) in
// one launch.  A block stages the 8 x 68-pixel input window of its 4 x 64
// output tile, computes layer A on the 6 x 66-pixel window that layer B reads
// (the tile and a one-pixel ring: 24 row tiles of 16 pixels and one tile of
// the 12 ring pixels in the left and right columns) into LDS, then layer B on
// the tile, stored to memory.  Every activation is the same MFMA sequence on
// the same operands as in two k_mid_lds launches, so the results are bit for
// bit those of the unfused layers, without the round trip of layer A's
// activations through memory and one launch less.  Needs H % 4 == 0 and
// W % 64 == 0; without training (layer A's pre-activations are not kept).
constexpr int F2R = 4, F2W = 64;
constexpr int F2IR = F2R + 4, F2IW = F2W + 4;  // input window
constexpr int F2MR = F2R + 2, F2MW = F2W + 2;  // layer A window
__global__ void __launch_bounds__(256) k_mid2_lds(const bf16 *__restrict__ ain,
                                                  const bf16 *__restrict__ wA,
                                                  const float *__restrict__ bA,
                                                  const bf16 *__restrict__ wB,
                                                  const float *__restrict__ bB, int B, int H, int W,
                                                  bf16 *__restrict__ aout) {
    __shared__ __attribute__((aligned(16))) bf16 win[F2IR * F2IW * SC];
    __shared__ __attribute__((aligned(16))) bf16 mid[F2MR * F2MW * SC];
#ifdef FSC_LDS_POISON
    lds_poison(win, F2IR * F2IW * SC);
    lds_poison(mid, F2MR * F2MW * SC);
    __syncthreads();
#endif
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    const int txs = W / F2W, tys = H / F2R;
    const int bx = blockIdx.x % txs, t1 = blockIdx.x / txs;
    const int by = t1 % tys, n = t1 / tys;
    const int x0 = bx * F2W, y0 = by * F2R;
    // input window: pixel (r, c) is image pixel (y0 - 2 + r, x0 - 2 + c), periodic
    for (int k = threadIdx.x; k < F2IR * F2IW * 4; k += 256) {
        const int piece = k & 3, pc = k >> 2;
        const int r = pc / F2IW, c = pc % F2IW;
        const int yy = ((y0 - 2 + r) % H + H) % H, xx = ((x0 - 2 + c) % W + W) % W;
        const size_t q = size_t((n * H + yy) * W + xx);
        *reinterpret_cast<bf16x8 *>(win + pc * SC + piece * 8) =
            *reinterpret_cast<const bf16x8 *>(ain + q * SC + piece * 8);
    }
    bf16x8 bop[9][2];
    f32x4 bv[2];
    auto load_layer = [&](const bf16 *__restrict__ wpk, const float *__restrict__ bias) {
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
                bop[t][nt] = *reinterpret_cast<const bf16x8 *>(
                    wpk + (t * SC + mid_row_channel(nt, r16)) * SC + g * 8);
        bv[0] = *reinterpret_cast<const f32x4 *>(bias + 8 * g);
        bv[1] = *reinterpret_cast<const f32x4 *>(bias + 8 * g + 4);
    };
    // acc = bias + sum over taps of W_tap x (32 channels of the tap pixel);
    // `src` is the window and (r, c) the window position of tap (0, 0)
    auto tile = [&](const bf16 *src, int sw, int r, int c, f32x4 (&acc)[2]) {
        acc[0] = bv[0];
        acc[1] = bv[1];
#pragma unroll
        for (int ky = 0; ky < 3; ++ky)
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) {
                const bf16x8 aop =
                    *reinterpret_cast<const bf16x8 *>(src + ((r + ky) * sw + c + kx) * SC + g * 8);
                acc[0] = mfma16(bop[ky * 3 + kx][0], aop, acc[0]);
                acc[1] = mfma16(bop[ky * 3 + kx][1], aop, acc[1]);
            }
    };
    load_layer(wA, bA);
    __syncthreads();
    // layer A: window pixel (mr, mc) is image pixel (y0 - 1 + mr, x0 - 1 + mc);
    // its tap (0, 0) is input window pixel (mr, mc)
    for (int t = wave; t < F2MR * (F2W / 16) + 1; t += 4) {  // wave-uniform
        int mr, mc;
        bool keep = true;
        if (t < F2MR * (F2W / 16)) {
            mr = t / (F2W / 16);
            mc = 1 + 16 * (t % (F2W / 16)) + r16;
        } else {  // the ring columns 0 and F2MW - 1 of the F2MR rows; 4 lanes spare
            keep = r16 < 2 * F2MR;
            const int e = keep ? r16 : 0;
            mr = e >> 1;
            mc = (e & 1) ? F2MW - 1 : 0;
        }
        f32x4 acc[2];
        tile(win, F2IW, mr, mc, acc);
        bf16x8 out;
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int r = 0; r < 4; ++r) out[4 * nt + r] = bf16(silu(acc[nt][r]));
        if (keep) *reinterpret_cast<bf16x8 *>(mid + (mr * F2MW + mc) * SC + 8 * g) = out;
    }
    __syncthreads();
    load_layer(wB, bB);
    // layer B: output pixel (y0 + row, x0 + cx), its tap (0, 0) is layer-A
    // window pixel (row, cx)
#pragma unroll
    for (int j = 0; j < F2R * F2W / 64; ++j) {
        const int k = wave * (F2R * F2W / 64) + j;
        const int row = k / (F2W / 16), cx = 16 * (k % (F2W / 16)) + r16;
        f32x4 acc[2];
        tile(mid, F2MW, row, cx, acc);
        const size_t p = size_t((n * H + y0 + row) * W + x0 + cx);
        mid_epilogue<false, false>(acc, p, g, nullptr, aout, bv);
    }
}

// ---------------------------------------------------------------------------
// The same pair for rows of at most 128 pixels, marching down the image.  A
// workgroup takes R rows over the whole width, so that columns wrap inside it.
// Four waves per layer hold that layer's weights in registers; a step takes one
// input row, and the row that this completes goes to the other layer's waves
// through LDS.  A layer's input row j adds to the output rows j, j - 1 and j - 2
// (taps ky = 0, 1, 2), whose accumulators stay in registers: a row is read from
// LDS once per kx instead of once per tap, and two rows of each layer are all that
// is held.  The second layer is three steps behind the first, which computes the
// two rows beyond the strip as well.  Bit for bit the unfused layers.
//
// R gives at most one workgroup per CU; two of them on a CU with half the rows
// each are slower (9-layer passes over 16 images: 98.6 us, 114).  What bounds it
// is the chain of a step (LDS reads, 18 MFMAs per tile, SiLU, barrier), about
// 2800 cycles where a SIMD's MFMAs take 1150.  A pair at 16 images of 128^2: 27.4 us
// as two tiled layers, 17.0 so.  9-layer passes, us, tiled layers / tiled pairs
// (k_mid2_lds) / with the pairs marching / and the single and last layers (k_march,
// k_last_march): 1 image 74 / 62 / 53 / 48, 4 88 / 74 / 65 / 61, 16 130 / 132 / 99 /
// 91, 32 222 / 238 / 154 / 136.  (Three and four layers per launch spill; a SiLU
// that runs a step late, beside the other layer's products, took 19.1 us per pair.)
// LDS: [layer][2][W pixels][4 pieces of 8 channels], a pixel's piece g at slot
// g ^ (pixel / 4 % 4): 16 lanes that read one piece of 16 pixels in a row then
// meet every bank once.
// ---------------------------------------------------------------------------
// element of a pixel's piece of eight channels in a row's LDS buffer
__device__ __forceinline__ int row_slot(int px, int piece) { return px * SC + ((piece ^ ((px >> 2) & 3)) * 8); }
// barrier that orders LDS accesses alone: global loads and stores stay in flight
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
constexpr int CH_W = 128;             // widest row
constexpr int CH_WAVES = 4;           // waves per layer
constexpr int CH_BLOCKS = 256;        // one workgroup per CU

// The loading waves of a marching layer: rows 0 .. nin - 1 of its input (image rows
// y0 - 1 .., periodic) into the two LDS rows, one step ahead of the multiplying
// waves, with which they share every barrier (one, then one per step, steps in
// pairs).
// (`first` .. is their first thread; LW: their number)
template <int LW, int ROW>
__device__ __forceinline__ void march_load(const bf16 *__restrict__ ain, size_t img, int y0, int nin, int steps, int H,
                                           int W, int first, bf16 (&rows)[2][ROW]) {
    constexpr int LOADERS = LW * 64, NP = ROW / 8 / LOADERS;
    const int t = int(threadIdx.x) - first;
    auto fetch = [&](int row, u32x4 (&v)[NP]) {
        const size_t base = (img + size_t(wrap_any(y0 - 1 + min(row, nin - 1), H))) * W;
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const int e = min(t + k * LOADERS, W * 4 - 1);
            v[k] = *reinterpret_cast<const u32x4 *>(ain + (base + (e >> 2)) * SC + (e & 3) * 8);
        }
    };
    auto put = [&](int row, const u32x4 (&v)[NP]) {
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const int e = min(t + k * LOADERS, W * 4 - 1);
            *reinterpret_cast<u32x4 *>(&rows[row & 1][row_slot(e >> 2, e & 3)]) = v[k];
        }
    };
    // row q is asked for two steps before it is put down, and read one step later
    u32x4 va[NP], vb[NP];
    fetch(0, va);
    fetch(1, vb);
    put(0, va);
    fetch(2, va);
    lds_barrier();
    for (int s = 0; s < steps; s += 2) {
        put(s + 1, vb);
        fetch(s + 3, vb);
        lds_barrier();
        put(s + 2, va);
        fetch(s + 4, va);
        lds_barrier();
    }
}

// TPW: tiles of 16 pixels per wave; a row has at most 4 TPW of them.
template <int TPW>
__global__ void __launch_bounds__((2 * CH_WAVES + TPW) * 64) k_chain(const bf16 *__restrict__ ain,
                                                            const bf16 *__restrict__ wA,
                                                            const float *__restrict__ bA,
                                                            const bf16 *__restrict__ wB,
                                                            const float *__restrict__ bB, int R, int strips,
                                                            int H, int W, bf16 *__restrict__ aout) {
    constexpr int ROW = CH_WAVES * TPW * 16 * SC;
    __shared__ __attribute__((aligned(16))) bf16 rows[2][2][ROW];
#ifdef FSC_LDS_POISON
    lds_poison(&rows[0][0][0], 4 * ROW);
    __syncthreads();
#endif
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, g = lane >> 4;
    const int layer = wave / CH_WAVES, wl = wave % CH_WAVES;
    const int n = blockIdx.x / strips, y0 = (blockIdx.x % strips) * R;
    const int Rr = min(R, H - y0), tiles = W / 16;
    const size_t img = size_t(n) * H;
    const int nin = Rr + 4, steps = Rr + 5;  // rows that the first layer reads
    if (layer == 2) return march_load<TPW>(ain, img, y0 - 1, nin, steps, H, W, 2 * CH_WAVES * 64, rows[0]);
    const bf16 *wpk = layer == 0 ? wA : wB;
    const float *bias = layer == 0 ? bA : bB;
    bf16x8 bop[9][2];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
            bop[t][nt] = *reinterpret_cast<const bf16x8 *>(wpk + (t * SC + mid_row_channel(nt, r16)) * SC + g * 8);
    const f32x4 bv[2] = {*reinterpret_cast<const f32x4 *>(bias + 8 * g),
                         *reinterpret_cast<const f32x4 *>(bias + 8 * g + 4)};
    __builtin_amdgcn_s_waitcnt(0);  // the weights: here, not in the loops, where it would wait for more
    // this lane's pixels and the LDS offsets of their columns x - 1, x, x + 1
    // (tiles past a narrower row's end repeat its last one: the same values again)
    int at[TPW][3], pix[TPW];
    f32x4 p0[TPW][2], p1[TPW][2];
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
        pix[q] = min(wl + CH_WAVES * q, tiles - 1) * 16 + r16;
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) at[q][kx] = row_slot(wrapi(pix[q] + kx - 1, W), g);
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) p0[q][nt] = p1[q][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    auto step = [&](int s, auto first) {
        const int j = first ? s : s - 3;  // this layer's input row
        if (j < 0 || j >= (first ? nin : nin - 2)) return;
        const bf16 *src = rows[first ? 0 : 1][(first ? s : s - 1) & 1];
        bf16x8 x[TPW][3];
#pragma unroll
        for (int q = 0; q < TPW; ++q)
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) x[q][kx] = *reinterpret_cast<const bf16x8 *>(src + at[q][kx]);
        f32x4 done[TPW][2];
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                done[q][nt] = p1[q][nt];
                p1[q][nt] = p0[q][nt];
                p0[q][nt] = bv[nt];
            }
#pragma unroll
            for (int kx = 0; kx < 3; ++kx)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) {
                    done[q][nt] = mfma16(bop[6 + kx][nt], x[q][kx], done[q][nt]);
                    p1[q][nt] = mfma16(bop[3 + kx][nt], x[q][kx], p1[q][nt]);
                    p0[q][nt] = mfma16(bop[kx][nt], x[q][kx], p0[q][nt]);
                }
        }
        if (j < 2) return;  // no output row is complete
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
            if constexpr (!first) {
                mid_epilogue<false, false>(done[q], (img + size_t(y0 + j - 2)) * W + pix[q], g, nullptr, aout, bv);
            } else {
                bf16x8 o;
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) o[4 * nt + r] = bf16(silu(done[q][nt][r]));
                *reinterpret_cast<bf16x8 *>(&rows[1][s & 1][row_slot(pix[q], g)]) = o;
            }
        }
    };
    auto march = [&](auto first) {
        lds_barrier();
        for (int s = 0; s < steps; s += 2) {
            step(s, first);
            lds_barrier();
            step(s + 1, first);  // (past the last step: nothing to do)
            lds_barrier();
        }
    };
    if (layer == 0) march(std::true_type{});
    else march(std::false_type{});
}

// One C -> C layer in the same form, forward or backward (training, and the odd
// layer of an inference pass): CW waves multiply, a tile of 16 pixels each, and CW/4
// more load the rows, so that the multiplying waves have only stores in flight,
// which nothing waits for; backward they load their next row's pre-activations a
// step ahead.  Per layer at 32 images of 128^2, tiles and marching, us: forward with
// pre-activations 32.4 and 26.0 (134 MB, 5.2 TB/s), backward 35.6 and 30.4, inference
// at 16 images 13.6 and 11.7; 6 images of 90 x 96 (no tiles divide them) 11.1 and
// 9.3, 15.0 and 9.7.
template <int CW, bool BWD, bool ZOUT>
__global__ void __launch_bounds__((CW + CW / 4) * 64) k_march(const bf16 *__restrict__ ain,
                                                              const bf16 *__restrict__ wpk,
                                                              const float *__restrict__ bias, int R, int strips,
                                                              int H, int W, float *__restrict__ zout,
                                                              bf16 *__restrict__ aout,
                                                              const float *__restrict__ zprev) {
    constexpr int ROW = CW * 16 * SC;
    __shared__ __attribute__((aligned(16))) bf16 rows[2][ROW];
#ifdef FSC_LDS_POISON
    lds_poison(&rows[0][0], 2 * ROW);
    __syncthreads();
#endif
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = blockIdx.x / strips, y0 = (blockIdx.x % strips) * R;
    const int Rr = min(R, H - y0), nin = Rr + 2;  // rows written and read
    const size_t img = size_t(n) * H;
    if (wave >= CW) return march_load<CW / 4>(ain, img, y0, nin, nin, H, W, CW * 64, rows);
    const int r16 = lane & 15, g = lane >> 4;
    bf16x8 bop[9][2];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
            bop[t][nt] = *reinterpret_cast<const bf16x8 *>(wpk + (t * SC + mid_row_channel(nt, r16)) * SC + g * 8);
    f32x4 bv[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    if (!BWD) {
        bv[0] = *reinterpret_cast<const f32x4 *>(bias + 8 * g);
        bv[1] = *reinterpret_cast<const f32x4 *>(bias + 8 * g + 4);
    }
    // (waves past a narrower row's end repeat its last tile: the same values again)
    const int px = min(wave, W / 16 - 1) * 16 + r16;
    int at[3];
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) at[kx] = row_slot(wrapi(px + kx - 1, W), g);
    auto pixel = [&](int row) { return (img + size_t(y0 + row)) * W + px; };
    f32x4 p0[2], p1[2], za[2], zb[2];
    p0[0] = p0[1] = p1[0] = p1[1] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (BWD) load_z(zprev, pixel(0), g, za);
    __builtin_amdgcn_s_waitcnt(0);  // the weights: here, not in the loop, where it would wait for more
    auto step = [&](int s, const f32x4 (&z)[2], f32x4 (&znext)[2]) {
        if (BWD) load_z(zprev, pixel(min(max(s - 1, 0), Rr - 1)), g, znext);
        const bf16 *src = rows[s & 1];
        bf16x8 x[3];
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) x[kx] = *reinterpret_cast<const bf16x8 *>(src + at[kx]);
        f32x4 done[2];
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            done[nt] = p1[nt];
            p1[nt] = p0[nt];
            p0[nt] = bv[nt];
        }
#pragma unroll
        for (int kx = 0; kx < 3; ++kx)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                done[nt] = mfma16(bop[6 + kx][nt], x[kx], done[nt]);
                p1[nt] = mfma16(bop[3 + kx][nt], x[kx], p1[nt]);
                p0[nt] = mfma16(bop[kx][nt], x[kx], p0[nt]);
            }
        if (s >= 2 && s < nin) mid_epilogue<BWD, ZOUT>(done, pixel(s - 2), g, zout, aout, z);
        lds_barrier();
    };
    lds_barrier();
    for (int s = 0; s < nin; s += 2) {  // (a step past the last row writes nothing)
        step(s, za, zb);
        step(s + 1, zb, za);
    }
}

// ---------------------------------------------------------------------------
// Last layer (C -> 1) forward on the matrix cores.  Its FP32 weights enter as
// three BF16 parts each, w = hi + mid + lo (k_update; exact for normal FP32
// values), in rows 0..2 of the A operand (rows 3..15 zero); B is 32 channels
// by 16 pixels for one tap, and the 9 taps accumulate.  Lane l < 16 ends with
// the three partial sums of pixel l in acc[0..2]: y = (hi + mid) + lo + bias.
// The products of BF16 activations with BF16 weight parts are exact and the
// sums FP32, so y is the FP32 evaluation of the layer up to the order of the
// sums.  Each wave takes one of the IMG_PARTS segments of an image: its
// pixels in tiles of 16, two tiles' loads in flight at a time (lanes past the
// segment repeat its last pixel), and the segment's FP64 sum of y (a fixed
// lane order).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_last(const bf16 *__restrict__ a, int B, int H, int W,
                                              const bf16 *__restrict__ wl3,
                                              const float *__restrict__ b, float *__restrict__ y,
                                              double *__restrict__ part) {
    const int lane = threadIdx.x & 63;
    const int r16 = lane & 15, g = lane >> 4;
    const int sg = blockIdx.x * 4 + (threadIdx.x >> 6);  // segment over the batch
    bf16x8 wop[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        if (r16 < 3) {
            wop[t] = *reinterpret_cast<const bf16x8 *>(wl3 + (t * 3 + r16) * SC + g * 8);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) wop[t][e] = bf16(0.f);
        }
    }
    const float bias = b[0];
    const int HW = H * W;
    const int img = sg / IMG_PARTS, seg = sg % IMG_PARTS;
    const int len = (HW + IMG_PARTS - 1) / IMG_PARTS;
    const int lo = seg * len, hi = min(HW, lo + len);
    double s = 0.0;
    for (int i0 = lo; i0 < hi; i0 += 32) {  // wave-uniform: whole waves run the MFMAs
        bf16x8 bop[2][9];
        int pix[2];
        bool on[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int i = i0 + 16 * u + r16;
            on[u] = i < hi;
            pix[u] = img * HW + (on[u] ? i : hi - 1);
            const int p = pix[u];
            const int x = p % W, t = p / W, yy = t % H, n = t / H;
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) {
                const int rowbase = (n * H + wrapi(yy + ky - 1, H)) * W;
#pragma unroll
                for (int kx = 0; kx < 3; ++kx) {
                    const int q = rowbase + wrapi(x + kx - 1, W);
                    bop[u][ky * 3 + kx] = *reinterpret_cast<const bf16x8 *>(a + size_t(q) * SC + g * 8);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 9; ++t) acc = mfma16(wop[t], bop[u][t], acc);
            if (g == 0 && on[u]) {
                const float v = (acc[0] + acc[1]) + acc[2] + bias;
                y[pix[u]] = v;
                s += double(v);
            }
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) part[sg] = s;
}

// The last layer in the marching form (rows of at most 128 pixels; see k_march):
// the same MFMA sequence per pixel.  A strip's sum of y goes to entry `strip` of the
// image's segment sums, the entries past the last strip are zero.  Forward pass at
// 16 images of 128^2: 12.4 us as k_last, 8.1 so; 32 images 23.0 and 11.0.
template <int CW>
__global__ void __launch_bounds__((CW + CW / 4) * 64) k_last_march(const bf16 *__restrict__ ain, int R, int strips,
                                                                   int H, int W, const bf16 *__restrict__ wl3,
                                                                   const float *__restrict__ b,
                                                                   float *__restrict__ y,
                                                                   double *__restrict__ part) {
    constexpr int ROW = CW * 16 * SC;
    __shared__ __attribute__((aligned(16))) bf16 rows[2][ROW];
    __shared__ double sums[CW];
#ifdef FSC_LDS_POISON
    lds_poison(&rows[0][0], 2 * ROW);
    __syncthreads();
#endif
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = blockIdx.x / strips, strip = blockIdx.x % strips, y0 = strip * R;
    const int Rr = min(R, H - y0), nin = Rr + 2;  // rows written and read
    const size_t img = size_t(n) * H;
    if (wave >= CW) {
        march_load<CW / 4>(ain, img, y0, nin, nin, H, W, CW * 64, rows);
        __syncthreads();
        return;
    }
    const int r16 = lane & 15, g = lane >> 4;
    bf16x8 wop[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        if (r16 < 3) {
            wop[t] = *reinterpret_cast<const bf16x8 *>(wl3 + (t * 3 + r16) * SC + g * 8);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) wop[t][e] = bf16(0.f);
        }
    }
    const float bias = b[0];
    const int px = min(wave, W / 16 - 1) * 16 + r16;
    const bool on = g == 0 && wave < W / 16;
    int at[3];
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) at[kx] = row_slot(wrapi(px + kx - 1, W), g);
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 p0 = zero, p1 = zero;
    double sum = 0.0;
    __builtin_amdgcn_s_waitcnt(0);  // the weights: here, not in the loop
    lds_barrier();
    for (int s = 0; s < nin + (nin & 1); ++s) {
        const bf16 *src = rows[s & 1];
        f32x4 done = p1;
        p1 = p0;
        p0 = zero;
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
            const bf16x8 x = *reinterpret_cast<const bf16x8 *>(src + at[kx]);
            done = mfma16(wop[6 + kx], x, done);
            p1 = mfma16(wop[3 + kx], x, p1);
            p0 = mfma16(wop[kx], x, p0);
        }
        if (s >= 2 && s < nin && on) {
            const float v = (done[0] + done[1]) + done[2] + bias;
            y[(img + size_t(y0 + s - 2)) * W + px] = v;
            sum += double(v);
        }
        lds_barrier();
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if (lane == 0) sums[wave] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < CW; ++w) t += sums[w];
        part[n * IMG_PARTS + strip] = t;
    }
    for (int k = strip + strips * (1 + int(threadIdx.x)); k < IMG_PARTS; k += strips * CW * 64)
        part[n * IMG_PARTS + k] = 0.0;
}
static_assert(CH_BLOCKS <= IMG_PARTS, "an entry per strip");

// sum of an image's IMG_PARTS segment sums by one wave, in a fixed order
__device__ inline double image_total(const double *__restrict__ part, int img) {
    const int lane = threadIdx.x & 63;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < IMG_PARTS / 64; ++k) s += part[img * IMG_PARTS + k * 64 + lane];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    return s;
}
static_assert(IMG_PARTS % 64 == 0, "a wave sums the segment sums (and k_last's blocks of four)");

// prediction rho_t + out_scale (y - <y>_image); `lanes` per (image, segment), the
// image's mean from its IMG_PARTS segment sums.  A wave per segment, or a workgroup
// where a segment has as many pixels (pred): a few large images are else on 64 CUs
// (three layers on one image of 1024^2: 336 us a pass, 321 so; 4096 x 2048 3013 and 2850).
__global__ void __launch_bounds__(256) k_pred(const float *__restrict__ in,
                                              const float *__restrict__ y,
                                              const double *__restrict__ part, int HW, int lanes,
                                              float out_scale, float *__restrict__ out) {
    const int sg = (int(blockIdx.x) * 256 + int(threadIdx.x)) / lanes, img = sg / IMG_PARTS, seg = sg % IMG_PARTS;
    const float mean = float(image_total(part, img) / HW);
    const int len = (HW + IMG_PARTS - 1) / IMG_PARTS;
    const int lo = seg * len, hi = min(HW, lo + len);
    for (int i = lo + int(threadIdx.x) % lanes; i < hi; i += lanes) {
        const size_t p = size_t(img) * HW + i;
        out[p] = in[p] + out_scale * (y[p] - mean);
    }
}

// Loss terms and dL/dyhat; a wave per (image, segment) as k_pred, the image's mean
// of y from its segment sums.  Every wave leaves the FP64 sums of its segment's
// dL/dyhat and of its squared errors (fixed order, no atomics: 2048 blocks adding
// to one double took 27 us at 32 images of 128^2; a block of 256 per segment, of
// which 64 lanes had a pixel, 14.5 us; like this 6.6).
__global__ void __launch_bounds__(256) k_loss(const float *__restrict__ in,
                                              const float *__restrict__ tgt,
                                              const float *__restrict__ y,
                                              const double *__restrict__ ypart, int HW,
                                              float inv_out_scale, float invM,
                                              float *__restrict__ gout, double *__restrict__ gpart,
                                              double *__restrict__ epart) {
    const int sg = blockIdx.x * 4 + (threadIdx.x >> 6), img = sg / IMG_PARTS, seg = sg % IMG_PARTS;
    const float mean = float(image_total(ypart, img) / HW);
    const int len = (HW + IMG_PARTS - 1) / IMG_PARTS;
    const int lo = seg * len, hi = min(HW, lo + len);
    double gs = 0.0, e2 = 0.0;
    for (int i = lo + int(threadIdx.x & 63); i < hi; i += 64) {
        const size_t p = size_t(img) * HW + i;
        const float e = (y[p] - mean) - (tgt[p] - in[p]) * inv_out_scale;
        const float gv = 2.f * e * invM;
        gout[p] = gv;
        gs += double(gv);
        e2 += double(e) * double(e);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        gs += __shfl_xor(gs, o, 64);
        e2 += __shfl_xor(e2, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        gpart[sg] = gs;
        epart[sg] = e2;
    }
}

// Per-image sums of dL/dyhat (one block each) and, in one more block, the
// loss, from the segment sums in a fixed order.
__global__ void __launch_bounds__(256) k_loss_total(const double *__restrict__ gpart,
                                                    const double *__restrict__ epart, int B,
                                                    double *__restrict__ gsum,
                                                    double *__restrict__ loss) {
    __shared__ double sh[4];
    const bool all = int(blockIdx.x) == B;
    const double *v = all ? epart : gpart + blockIdx.x * IMG_PARTS;
    const int n = all ? B * IMG_PARTS : IMG_PARTS;
    double s = 0.0;
#pragma unroll 8
    for (int k = threadIdx.x; k < n; k += 256) s += v[k];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) (all ? loss[0] : gsum[blockIdx.x]) = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// Last layer backward-data: dZ_{L-2}[p][c] = SiLU'(z) sum_t dy[p - off(t)] W[c][t]
// with dy = g - <g>_image (the mean-free projection's adjoint).  Four lanes per
// pixel, eight channels each: the FP32 pre-activations arrive and the BF16
// gradients leave as whole 16-byte pieces of consecutive lanes (the kernel
// moves 192 B per pixel and little else; one lane per pixel with 2-byte stores
// took 36 us at 32 images of 128^2, this form 20 us).
__global__ void __launch_bounds__(256) k_last_bwd(const float *__restrict__ g,
                                                  const double *__restrict__ gsum, int B, int H,
                                                  int W, const float *__restrict__ w,
                                                  const float *__restrict__ zprev,
                                                  bf16 *__restrict__ dz) {
    __shared__ __attribute__((aligned(16))) float wt[9][SC];
    for (int k = threadIdx.x; k < 9 * SC; k += 256) wt[k % 9][k / 9] = w[k];
    __syncthreads();
    const int P = B * H * W;
    const int o = threadIdx.x & 3;
    const int p = blockIdx.x * 64 + (threadIdx.x >> 2);
    if (p >= P) return;
    const size_t at = size_t(p) * SC + 8 * o;
    const f32x4 zp[2] = {*reinterpret_cast<const f32x4 *>(zprev + at),
                         *reinterpret_cast<const f32x4 *>(zprev + at + 4)};
    const int x = p % W, t = p / W, yy = t % H, n = t / H;
    const float gm = float(gsum[n] / (H * W));
    float da[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ky = 0; ky < 3; ++ky)
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
            const float dy = g[(n * H + wrapi(yy - ky + 1, H)) * W + wrapi(x - kx + 1, W)] - gm;
            const f32x4 w0 = *reinterpret_cast<const f32x4 *>(&wt[ky * 3 + kx][8 * o]);
            const f32x4 w1 = *reinterpret_cast<const f32x4 *>(&wt[ky * 3 + kx][8 * o + 4]);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                da[c] += dy * w0[c];
                da[4 + c] += dy * w1[c];
            }
        }
    bf16x8 out;
#pragma unroll
    for (int c = 0; c < 8; ++c) out[c] = bf16(da[c] * dsilu(zp[c >> 2][c & 3]));
    *reinterpret_cast<bf16x8 *>(dz + at) = out;
}

// ---------------------------------------------------------------------------
// Weight gradients: GEMMs over the pixels on the matrix cores,
//   C -> C layers:  dW[co][ci][t] = sum_p dZ[p][co] a[p + off(t)][ci]
//   first layer:    dW[co][ci][t] = sum_p dZ[p][co] X[p + off(t)][ci]
//   last layer:     dW[c][t]      = sum_q a[q][c] dy[q - off(t)]
// and the biases sum_p dZ[p][co], sum_p dy[p].
//
// The operands have the pixel as the MFMA's K index, so a lane needs one
// channel of eight pixels, while memory holds the channels of a pixel side by
// side.  A tile is staged in LDS as it lies in memory (16-byte pieces).  Lane
// (r, g) = (l % 16, l / 16) then reads the channel pair (2r, 2r + 1) of pixels
// g + 4j, j = 0..7, as eight words: the 64 lanes of one read cover four
// consecutive pixels, 256 contiguous bytes, free of bank conflicts.  The low
// halves of the words are the operand of the even channels and the high halves
// that of the odd ones (v_perm), so row m of operand tile mt is channel 2m + mt;
// any order of K that is the same for both operands gives the same product.
//
// Every block sums its tiles in FP32 accumulators and writes one partial
// result; k_wgrad_sum adds the partials in FP64 in a fixed order, so the
// gradient does not depend on the order in which blocks finish.
// ---------------------------------------------------------------------------
constexpr int WG_TR = 16, WG_TW = 32;  // pixel tile (W is a multiple of 32)
constexpr int WG_AW = WG_TW + 2;       // activations with their one-pixel halo
constexpr int WG_MAX_BLOCKS = 256;     // one per CU
constexpr int WG_EDGE_BLOCKS = 512;    // two per CU
constexpr int WG_LEN = 9 * SC * SC + SC;
constexpr int WG_DZ_PIECES = WG_TR * WG_TW * 4, WG_A_PIECES = (WG_TR + 2) * WG_AW * 4;
// words of LDS: the staged tile, then (reused) the sums of two of four row
// groups, three kernel rows of 56 accumulators per lane each
constexpr int WG_LDS = std::max((WG_DZ_PIECES + WG_A_PIECES) * 4, 2 * 3 * 56 * 64);

__host__ __device__ inline int wg_tiles(int B, int H, int W) {
    return B * ((H + WG_TR - 1) / WG_TR) * (W / WG_TW);
}

// operands of the even and the odd channels from eight channel-pair words
__device__ __forceinline__ void split_pairs(const uint32_t (&d)[8], bf16x8 &even, bf16x8 &odd) {
    u32x4 e, o;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        e[k] = __builtin_amdgcn_perm(d[2 * k + 1], d[2 * k], 0x05040100u);
        o[k] = __builtin_amdgcn_perm(d[2 * k + 1], d[2 * k], 0x07060302u);
    }
    even = __builtin_bit_cast(bf16x8, e);
    odd = __builtin_bit_cast(bf16x8, o);
}

// C -> C layer.  A block of 12 waves marches over tiles of 16 rows x 32
// columns; wave (ky, pg) takes the three taps of kernel row ky over the tile's
// rows 4pg .. 4pg + 3 (12 MFMAs per 32 pixels), which keeps its accumulators at
// 48 registers.  The next tile is on its way in registers while this one is
// multiplied.  Bounds at 32 images of 128^2: 67 MB of operands, 11 us at the
// card's copy rate, and 9.7 GFLOP.  Measured 23.4 us; staging transposed
// copies with 2-byte LDS stores and adding 9216 atomics per block took 527 us.
// element e of a block's partial result: ((t * 4 + 2 mt + nt) * 4 + r) * 64 + lane
// for dW[2 (4g + r) + mt][2 (lane % 16) + nt][t], then the 32 biases.
__global__ void __launch_bounds__(768) k_mid_wgrad(const bf16 *__restrict__ dz,
                                                   const bf16 *__restrict__ ain, int B, int H,
                                                   int W, float *__restrict__ part) {
    __shared__ __attribute__((aligned(16))) uint32_t lds[WG_LDS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    const int ky = wave % 3, pg = wave / 3;
    const int txs = W / WG_TW, tys = (H + WG_TR - 1) / WG_TR;
    const int tiles = wg_tiles(B, H, W);
    constexpr int PRE = (WG_DZ_PIECES + WG_A_PIECES + 767) / 768;
    u32x4 pre[PRE];
    auto fetch = [&](int tile) {
        const int x0 = (tile % txs) * WG_TW, t1 = tile / txs;
        const int y0 = (t1 % tys) * WG_TR, n = t1 / tys;
#pragma unroll
        for (int i = 0; i < PRE; ++i) {
            const int k = tid + i * 768;
            pre[i] = u32x4{0u, 0u, 0u, 0u};
            if (k < WG_DZ_PIECES) {
                const int px = k >> 2, y = y0 + px / WG_TW, x = x0 + px % WG_TW;
                if (y < H)
                    pre[i] = *reinterpret_cast<const u32x4 *>(dz + size_t((n * H + y) * W + x) * SC + (k & 3) * 8);
            } else if (k < WG_DZ_PIECES + WG_A_PIECES) {
                const int k2 = k - WG_DZ_PIECES, px = k2 >> 2;
                const int r = px / WG_AW, c = px % WG_AW;
                // rows past the image's end and its halo are not used: any valid row
                const int y = wrapi(min(y0 - 1 + r, H), H), x = wrapi(x0 - 1 + c, W);
                pre[i] = *reinterpret_cast<const u32x4 *>(ain + size_t((n * H + y) * W + x) * SC + (k2 & 3) * 8);
            }
        }
    };
    f32x4 acc[3][2][2], accb[2];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) acc[k][mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    accb[0] = accb[1] = f32x4{0.f, 0.f, 0.f, 0.f};
    const u32x4 one4 = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
    const bf16x8 ones = __builtin_bit_cast(bf16x8, one4);
    fetch(blockIdx.x);
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PRE; ++i) {
            const int k = tid + i * 768;
            if (k < WG_DZ_PIECES + WG_A_PIECES) *reinterpret_cast<u32x4 *>(lds + k * 4) = pre[i];
        }
        __syncthreads();
        if (tile + int(gridDim.x) < tiles) fetch(tile + gridDim.x);
        const int y0 = ((tile / txs) % tys) * WG_TR;
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int row = pg * 4 + rr;
            if (y0 + row >= H) break;  // wave-uniform
            uint32_t d[8];
            bf16x8 aop[2];
            const uint32_t *dp = lds + (row * WG_TW + g) * 16 + r16;
#pragma unroll
            for (int j = 0; j < 8; ++j) d[j] = dp[j * 64];
            split_pairs(d, aop[0], aop[1]);
            if (ky == 0) {
                accb[0] = mfma16(aop[0], ones, accb[0]);
                accb[1] = mfma16(aop[1], ones, accb[1]);
            }
            const uint32_t *ap = lds + WG_DZ_PIECES * 4 + ((row + ky) * WG_AW + g) * 16 + r16;
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) {
                bf16x8 bop[2];
#pragma unroll
                for (int j = 0; j < 8; ++j) d[j] = ap[kx * 16 + j * 64];
                split_pairs(d, bop[0], bop[1]);
#pragma unroll
                for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                    for (int nt = 0; nt < 2; ++nt) acc[kx][mt][nt] = mfma16(aop[mt], bop[nt], acc[kx][mt][nt]);
            }
        }
    }
    // the four row groups of each kernel row: 2, 3 into 0, 1, then 1 into 0
    float *red = reinterpret_cast<float *>(lds);  // [2][3][56][64]
#pragma unroll
    for (int half = 2; half >= 1; half >>= 1) {
        __syncthreads();
        if (pg >= half && pg < 2 * half) {
            float *q = red + ((pg - half) * 3 + ky) * 56 * 64 + lane;
#pragma unroll
            for (int k = 0; k < 12; ++k)
#pragma unroll
                for (int r = 0; r < 4; ++r) q[(k * 4 + r) * 64] = acc[k >> 2][(k >> 1) & 1][k & 1][r];
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) q[(48 + mt * 4 + r) * 64] = accb[mt][r];
        }
        __syncthreads();
        if (pg < half) {
            const float *q = red + (pg * 3 + ky) * 56 * 64 + lane;
#pragma unroll
            for (int k = 0; k < 12; ++k)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[k >> 2][(k >> 1) & 1][k & 1][r] += q[(k * 4 + r) * 64];
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) accb[mt][r] += q[(48 + mt * 4 + r) * 64];
        }
    }
    if (pg != 0) return;
    float *out = part + size_t(blockIdx.x) * WG_LEN;
#pragma unroll
    for (int k = 0; k < 12; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            out[(((ky * 3 + (k >> 2)) * 4 + (k & 3)) * 4 + r) * 64 + lane] = acc[k >> 2][(k >> 1) & 1][k & 1][r];
    if (ky == 0 && r16 == 0) {
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) out[9 * SC * SC + 2 * (4 * g + r) + mt] = accb[mt][r];
    }
}

// First (LAST = false) and last layer: one operand is the BF16 activation
// gradient (activation) of the 32 channels, the other an FP32 field per input
// channel, the network input X formed from the fields (or dy = g - <g>).  Each
// FP32 value enters as three BF16 parts that sum to it exactly, so that the
// products are exact and the sums FP32, as with FP32 factors (split_field): columns
// (part, ci, tap) of the second operand, 27 per input channel, then one of ones
// (sum_p dZ[p][co], the first layer's bias).  Four waves, four rows of the
// tile each.  It reads 64 + 4K B per pixel.  Measured at 32 images of 128^2:
// 21.1 us (first, K = 2) and 14.9 us (last); one lane per channel
// with FP32 FMAs and atomics took 251 and 178 us.
// Element of a block's partial result: (nt * 2 + mt) * 256 + r * 64 + lane for
// channel 2 (4g + r) + mt and column 16 nt + lane % 16, then sum_p of the field.
template <int K>
constexpr int wg_edge_tiles() { return K == 1 ? 2 : 4; }  // columns / 16
template <int K>
constexpr int wg_edge_len() { return wg_edge_tiles<K>() * 512 + 1; }

// v = hi + mid + lo, each the leading 8 bits of what the ones before it leave.  Cut
// off, not rounded: a v beyond the largest BF16 value would round to infinity, and
// parts of one sign overflow to one infinity.  An infinite v is its first part.
__device__ __forceinline__ void split_field(float v, uint16_t (&part)[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const uint32_t bits = __builtin_bit_cast(uint32_t, v) & 0xffff0000u;
        const float lead = __builtin_bit_cast(float, bits);
        part[k] = uint16_t(bits >> 16);
        v = v == lead ? 0.f : v - lead;
    }
}

template <int K, bool LAST>
__global__ void __launch_bounds__(256) k_edge_wgrad(const bf16 *__restrict__ act, const float *__restrict__ cur,
                                                    const float *__restrict__ prev, float mean, float inv_in,
                                                    float inv_out, const double *__restrict__ gsum, int B,
                                                    int H, int W, float *__restrict__ part) {
    static_assert(!LAST || K == 1, "the last layer has one output");
    constexpr int NT = wg_edge_tiles<K>();
    constexpr int PL = (WG_TR + 2) * WG_AW;  // values per part plane
    __shared__ __attribute__((aligned(16))) uint32_t sact[WG_DZ_PIECES * 4];
    __shared__ uint16_t sx[K * 3 * PL + 2];  // planes [ci][part], then 1 and 0
    __shared__ float red[3][NT * 2 * 4 * 64];
    __shared__ double dred[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    const int txs = W / WG_TW, tys = (H + WG_TR - 1) / WG_TR;
    const int tiles = wg_tiles(B, H, W);
    // this lane's columns: offset of pixel (row 0, column g) and the step of four pixels
    int base[NT], hop[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int q = nt * 16 + r16;
        if (q < 27 * K) {
            const int pt = q / (9 * K), ci = (q / 9) % K, tap = q % 9;
            const int ky = LAST ? 2 - tap / 3 : tap / 3, kx = LAST ? 2 - tap % 3 : tap % 3;
            base[nt] = (ci * 3 + pt) * PL + ky * WG_AW + kx + g;
            hop[nt] = 1;
        } else {
            base[nt] = K * 3 * PL + (q == 27 * K ? 0 : 1);
            hop[nt] = 0;
        }
    }
    if (tid == 0) {
        sx[K * 3 * PL] = 0x3F80u;  // 1
        sx[K * 3 * PL + 1] = 0u;
    }
    f32x4 acc[NT][2];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[nt][0] = acc[nt][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    double fsum = 0.0;
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int x0 = (tile % txs) * WG_TW, t1 = tile / txs;
        const int y0 = (t1 % tys) * WG_TR, n = t1 / tys;
        const float gm = LAST ? float(gsum[n] / (H * W)) : 0.f;
        __syncthreads();
        for (int k = tid; k < WG_DZ_PIECES; k += 256) {
            const int px = k >> 2, y = y0 + px / WG_TW, x = x0 + px % WG_TW;
            if (y < H)
                *reinterpret_cast<u32x4 *>(sact + k * 4) =
                    *reinterpret_cast<const u32x4 *>(act + size_t((n * H + y) * W + x) * SC + (k & 3) * 8);
        }
        for (int k = tid; k < PL; k += 256) {
            const int r = k / WG_AW, c = k % WG_AW;
            const int y = wrapi(min(y0 - 1 + r, H), H), x = wrapi(x0 - 1 + c, W);
            const size_t q = size_t(n * H + y) * W + x;
            const float v0 = cur[q];
            float v[2] = {LAST ? v0 - gm : (v0 - mean) * inv_in, 0.f};
            if constexpr (K == 2) v[1] = (v0 - prev[q]) * inv_out;
            if (LAST && r >= 1 && r <= WG_TR && c >= 1 && c <= WG_TW && y0 - 1 + r < H) fsum += double(v[0]);
#pragma unroll
            for (int ci = 0; ci < K; ++ci) {
                uint16_t part[3];
                split_field(v[ci], part);
#pragma unroll
                for (int q = 0; q < 3; ++q) sx[(ci * 3 + q) * PL + k] = part[q];
            }
        }
        __syncthreads();
#pragma unroll
        for (int rr = 0; rr < WG_TR / 4; ++rr) {
            const int row = wave * (WG_TR / 4) + rr;
            if (y0 + row >= H) break;  // wave-uniform
            uint32_t d[8];
            bf16x8 aop[2];
            const uint32_t *dp = sact + (row * WG_TW + g) * 16 + r16;
#pragma unroll
            for (int j = 0; j < 8; ++j) d[j] = dp[j * 64];
            split_pairs(d, aop[0], aop[1]);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const uint16_t *xp = sx + base[nt] + hop[nt] * row * WG_AW;
                u32x4 b4;
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    b4[k] = uint32_t(xp[hop[nt] * 8 * k]) | (uint32_t(xp[hop[nt] * (8 * k + 4)]) << 16);
                const bf16x8 bop = __builtin_bit_cast(bf16x8, b4);
                acc[nt][0] = mfma16(aop[0], bop, acc[nt][0]);
                acc[nt][1] = mfma16(aop[1], bop, acc[nt][1]);
            }
        }
    }
    if (LAST) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) fsum += __shfl_xor(fsum, o, 64);
        if (lane == 0) dred[wave] = fsum;
    }
    if (wave > 0) {
#pragma unroll
        for (int k = 0; k < NT * 2; ++k)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[wave - 1][k * 256 + r * 64 + lane] = acc[k >> 1][k & 1][r];
    }
    __syncthreads();
    if (wave > 0) return;
    float *out = part + size_t(blockIdx.x) * wg_edge_len<K>();
#pragma unroll
    for (int k = 0; k < NT * 2; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int e = k * 256 + r * 64 + lane;
            out[e] = (acc[k >> 1][k & 1][r] + red[0][e]) + (red[1][e] + red[2][e]);
        }
    if (lane == 0) out[NT * 512] = LAST ? float((dred[0] + dred[1]) + (dred[2] + dred[3])) : 0.f;
}

// Sums the blocks' partial results of every layer into the gradient vector
// (each partial once, in FP64, in a fixed order; see k_wgrad_sum).
struct WgradSum {
    int nmid, mid_blocks, edge_blocks, in_ch;
    const float *mid, *first, *last;  // [layer][block][WG_LEN], [block][len]
    int woff0, boff0, woff1, mid_stride, woffl, boffl;  // offsets in the gradient vector
};
constexpr int WG_MID_GROUPS = (WG_LEN + 255) / 256;
static_assert(WG_LEN % 4 == 0, "whole 16-byte pieces");

// A workgroup of k_wgrad_sum is sixteen waves.  C -> C layers (66
// MB at nine layers and 32 images): 256 columns each, a wave reads 1 KB of a partial
// at a time and keeps sixteen such loads in flight.  First and last layers: eight
// columns each, 128 lanes per column; their columns lie apart, a load touches 64
// lines, and with 64 columns per workgroup the fifteen CUs that had them took 44
// us.  Nine-layer network, 32 images: 45 -> 22.6 us; five layers, 6 images of 90 x
// 96: 17.6 -> 5.4.
constexpr int WG_SUM_WAVES = 16;

__device__ inline double to_double(float v) { return double(v); }
typedef double f64x4 __attribute__((ext_vector_type(4)));
__device__ inline f64x4 to_double(f32x4 v) { return f64x4{double(v[0]), double(v[1]), double(v[2]), double(v[3])}; }

// Sum of the partials first, first + step, ..., U at a time; V: float or f32x4,
// len in units of V.
template <int U, class V>
__device__ inline auto wg_column(const V *__restrict__ part, int blocks, int len, int e, int first, int step) {
    const V *p = part + e;
    decltype(to_double(V{})) s{};
    for (int b = first; b < blocks; b += U * step) {
        V v[U];
#pragma unroll
        for (int k = 0; k < U; ++k) v[k] = p[size_t(min(b + step * k, blocks - 1)) * len];
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (b + step * k < blocks) s += to_double(v[k]);
    }
    return s;
}

constexpr int WG_EDGE_COLS = 8, WG_EDGE_STEP = WG_SUM_WAVES * 64 / WG_EDGE_COLS;
__device__ inline double wg_edge_column(const float *__restrict__ part, int blocks, int len, int e) {
    return wg_column<4>(part, blocks, len, e, int(threadIdx.x) / WG_EDGE_COLS, WG_EDGE_STEP);
}

template <int K>
__device__ inline double wg_edge_value(const float *__restrict__ part, int blocks, int ch, int col) {
    const int mt = ch & 1, row = ch >> 1;  // channel 2 (4g + r) + mt
    const int e = ((col >> 4) * 2 + mt) * 256 + (row & 3) * 64 + (row >> 2) * 16 + (col & 15);
    return wg_edge_column(part, blocks, wg_edge_len<K>(), e);
}

__global__ void __launch_bounds__(64 * WG_SUM_WAVES) k_wgrad_sum(WgradSum a, float *__restrict__ grads) {
    __shared__ __attribute__((aligned(32))) double sh[WG_SUM_WAVES][256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int mid_groups = a.nmid * WG_MID_GROUPS;
    auto total = [&](int col) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < WG_SUM_WAVES; ++w) t += sh[w][col];
        return float(t);
    };
    if (int(blockIdx.x) < mid_groups) {
        const int l = blockIdx.x / WG_MID_GROUPS, e0 = (blockIdx.x % WG_MID_GROUPS) * 256;
        if (e0 + lane * 4 < WG_LEN) {
            const f32x4 *part = reinterpret_cast<const f32x4 *>(a.mid + size_t(l) * a.mid_blocks * WG_LEN);
            *reinterpret_cast<f64x4 *>(&sh[wave][lane * 4]) =
                wg_column<16>(part, a.mid_blocks, WG_LEN / 4, e0 / 4 + lane, wave, WG_SUM_WAVES);
        }
        __syncthreads();
        const int e = e0 + int(threadIdx.x);
        if (threadIdx.x >= 256 || e >= WG_LEN) return;
        int dst = a.woff1 + l * a.mid_stride;
        if (e < 9 * SC * SC) {
            const int q = e >> 6, el = e & 63;
            const int r = q & 3, nt = (q >> 2) & 1, mt = (q >> 3) & 1, t = q >> 4;
            const int co = 2 * (4 * (el >> 4) + r) + mt, ci = 2 * (el & 15) + nt;
            dst += (co * SC + ci) * 9 + t;
        } else {
            dst += e;  // the biases follow the weights
        }
        grads[dst] = total(threadIdx.x);
        return;
    }
    double s = 0.0;
    int dst = -1;
    const int e = (int(blockIdx.x) - mid_groups) * WG_EDGE_COLS + lane % WG_EDGE_COLS;
    const int n0 = SC * (9 * a.in_ch + 1), nl = SC * 9 + 1;  // first layer, last layer
    if (e < n0) {
        const int ch = e / (9 * a.in_ch + 1), k = e % (9 * a.in_ch + 1);
        const bool bias = k == 9 * a.in_ch;  // the column of ones
        dst = bias ? a.boff0 + ch : a.woff0 + ch * 9 * a.in_ch + k;
        for (int pt = 0; pt < (bias ? 1 : 3); ++pt) {
            const int col = (bias ? 27 * a.in_ch : pt * 9 * a.in_ch + k);
            s += a.in_ch == 2 ? wg_edge_value<2>(a.first, a.edge_blocks, ch, col)
                              : wg_edge_value<1>(a.first, a.edge_blocks, ch, col);
        }
    } else if (e < n0 + nl) {
        const int k = e - n0;
        if (k < SC * 9) {
            dst = a.woffl + k;
            for (int pt = 0; pt < 3; ++pt)
                s += wg_edge_value<1>(a.last, a.edge_blocks, k / 9, pt * 9 + k % 9);
        } else {
            dst = a.boffl;
            s = wg_edge_column(a.last, a.edge_blocks, wg_edge_len<1>(), wg_edge_len<1>() - 1);
        }
    }
    sh[wave][lane] = s;
    __syncthreads();
    if (int(threadIdx.x) < WG_EDGE_COLS && dst >= 0) {
        double t = 0.0;
        for (int w = 0; w < WG_SUM_WAVES; ++w)
#pragma unroll
            for (int k = 0; k < 64; k += WG_EDGE_COLS) t += sh[w][lane + k];
        grads[dst] = float(t);
    }
}

// Packed copies of the parameters for the matrix cores, one parameter per
// thread, every layer in one launch, after an Adam step (ADAM) or a plain
// change of the parameters:
//   C -> C layers: forward wf[t][co][ci], adjoint wb[t][ci][co] = W[co][ci][8 - t]
//   (tap flip);
//   last layer: its FP32 weights w[c][t] as three BF16 parts wl3[t][part][c]: hi =
//   bf16(w), mid = bf16(w - hi), lo = bf16(w - hi - mid).  Each difference is exact
//   in FP32, and what lo leaves is zero for normal FP32 weights, so hi + mid + lo = w.
struct AdamArgs {
    const float *g;
    float *m, *v;
    float lr, b1, b2, eps, bc1, bc2;
};
template <bool ADAM>
__global__ void __launch_bounds__(256) k_update(float *__restrict__ p, int n, int mid0, int last0, AdamArgs o,
                                                bf16 *__restrict__ wf, bf16 *__restrict__ wb,
                                                bf16 *__restrict__ wl3) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= n) return;
    float w = p[k];
    if constexpr (ADAM) {
        const float gk = o.g[k];
        const float mk = o.b1 * o.m[k] + (1.f - o.b1) * gk;
        const float vk = o.b2 * o.v[k] + (1.f - o.b2) * gk * gk;
        o.m[k] = mk;
        o.v[k] = vk;
        w -= o.lr * (mk / o.bc1) / (sqrtf(vk / o.bc2) + o.eps);
        p[k] = w;
    }
    if (k >= last0) {
        const int e = k - last0, t = e % 9, c = e / 9;
        if (c >= SC) return;  // the bias
        const bf16 hi = bf16(w);
        const float r1 = w - float(hi);
        const bf16 mid = bf16(r1);
        wl3[(t * 3 + 0) * SC + c] = hi;
        wl3[(t * 3 + 1) * SC + c] = mid;
        wl3[(t * 3 + 2) * SC + c] = bf16(r1 - float(mid));
    } else if (k >= mid0) {
        const int l = (k - mid0) / WG_LEN, e = (k - mid0) % WG_LEN;
        if (e >= 9 * SC * SC) return;  // the biases
        const int t = e % 9, ci = (e / 9) % SC, co = e / (9 * SC);
        const size_t off = size_t(l) * 9 * SC * SC;
        wf[off + (t * SC + co) * SC + ci] = bf16(w);
        wb[off + ((8 - t) * SC + ci) * SC + co] = bf16(w);
    }
}

// ---------------------------------------------------------------------------
// Coarse-graining: mean density over f x f blocks of the streamed state.  A
// workgroup takes a strip of one coarse row: lanes run along x (coalesced pulls,
// TX columns), TY = 1, 2 or 4 groups of them share the strip's rows; a lane sums
// its column's density in FP64 and the columns of a cell meet in LDS.  It reads
// 36 B per node: 4096^2 in blocks of 8 takes 115 us (one lane per cell,
// walking f rows of 32-byte pieces, took 478), 128^2 to 512^2 5 (66).
// ---------------------------------------------------------------------------
template <class L, typename real>
__global__ void __launch_bounds__(256) k_coarsen(Geometry g, const real *__restrict__ src,
                                                 double rho0, int f, int TX, int strips,
                                                 float *__restrict__ out) {
    __shared__ double sh[256];
    const int TY = 256 / TX, tx = threadIdx.x % TX, ty = threadIdx.x / TX;
    const int cells = f <= TX ? TX / f : 1, cx = g.nx / f;
    const int Y = int(blockIdx.x) / strips, X0 = (int(blockIdx.x) % strips) * cells;
    const int n = min(cells, cx - X0), width = n * f;
    double s = 0.0;
    for (int c = tx; c < width; c += TX) {
        const int x = X0 * f + c;
        const int xs[3] = {x + 1 == g.nx ? 0 : x + 1, x, x == 0 ? g.nx - 1 : x - 1};  // x - c_x
        for (int dy = ty; dy < f; dy += TY) {
            const int y = Y * f + dy;
            const int ys[3] = {y + 1 == g.ny ? 0 : y + 1, y, y == 0 ? g.ny - 1 : y - 1};
#pragma unroll
            for (int i = 0; i < L::Q; ++i)
                s += double(src[int64_t(i) * g.N + xs[L::c(i, 0) + 1] + int64_t(g.nx) * ys[L::c(i, 1) + 1]]);
        }
    }
    if (f > TX) {  // one cell, all lanes
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
        __syncthreads();
        if (threadIdx.x == 0)
            out[Y * cx + X0] = float(rho0 + ((sh[0] + sh[1]) + (sh[2] + sh[3])) / (double(f) * double(f)));
        return;
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int k = threadIdx.x; k < n; k += 256) {
        double t = 0.0;
        for (int r = 0; r < TY; ++r)
            for (int c = 0; c < f; ++c) t += sh[r * TX + k * f + c];
        out[Y * cx + X0 + k] = float(rho0 + t / (double(f) * double(f)));
    }
}

// One lane per cell: single nodes, where there is nothing to sum, and small cells of
// many narrow rows, which leave most lanes of a strip idle (nx f^3 <= 1300 and more
// than 4096 strips, from the times over 1 to 128 columns, 1200 to 120000 rows and f = 1
// to 8).  us, strips / so: f = 1 1000^2 10.1 / 8.9, 2048^2 32.2 / 29.3, 1 x 100000 94 / 6.2;
// f = 2 64 x 24000 17.1 / 12.5; f = 4 8 x 120000 44 / 38, but 48 x 24000 12.6 / 24.8.
template <class L, typename real>
__global__ void __launch_bounds__(256) k_coarsen_cells(Geometry g, const real *__restrict__ src, double rho0, int f,
                                                       float *__restrict__ out) {
    const int cx = g.nx / f, cells = cx * (g.ny / f);
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= cells) return;
    const int X = (k % cx) * f, Y = (k / cx) * f;
    double s = 0.0;
    for (int y = Y; y < Y + f; ++y) {
        const int ys[3] = {y + 1 == g.ny ? 0 : y + 1, y, y == 0 ? g.ny - 1 : y - 1};
        for (int x = X; x < X + f; ++x) {
            const int xs[3] = {x + 1 == g.nx ? 0 : x + 1, x, x == 0 ? g.nx - 1 : x - 1};
#pragma unroll
            for (int i = 0; i < L::Q; ++i)
                s += double(src[int64_t(i) * g.N + xs[L::c(i, 0) + 1] + int64_t(g.nx) * ys[L::c(i, 1) + 1]]);
        }
    }
    out[k] = float(rho0 + s / (double(f) * double(f)));
}

hipError_t launch_coarsen(const Geometry &g, int precision, const void *buf, double rho0, int f,
                          float *out, hipStream_t s) {
    if (g.D != 2 || f < 1 || g.nx % f || g.ny % f) return hipErrorInvalidValue;
    const int TX = f >= 4 ? 64 : (f >= 2 ? 128 : 256);
    const int cells = f <= TX ? TX / f : 1, strips = (g.nx / f + cells - 1) / cells;
    const int64_t nb = int64_t(strips) * (g.ny / f);
    if (nb > 0x7fffffff) return hipErrorInvalidValue;
    if (f == 1 || (nb > 4096 && f <= 10 && int64_t(g.nx) * f * f * f <= 1300)) {
        const unsigned cb = unsigned((int64_t(g.nx / f) * (g.ny / f) + 255) / 256);
        auto cells = [&](auto kernel, auto p) {
            hipLaunchKernelGGL(kernel, dim3(cb), dim3(256), 0, s, g, p, rho0, f, out);
            return hipGetLastError();
        };
        return precision == 0 ? cells(k_coarsen_cells<D2Q9, float>, static_cast<const float *>(buf))
                              : cells(k_coarsen_cells<D2Q9, double>, static_cast<const double *>(buf));
    }
    auto go = [&](auto kernel, auto p) {
        hipLaunchKernelGGL(kernel, dim3(unsigned(nb)), dim3(256), 0, s, g, p, rho0, f, TX, strips, out);
        return hipGetLastError();
    };
    return precision == 0 ? go(k_coarsen<D2Q9, float>, static_cast<const float *>(buf))
                          : go(k_coarsen<D2Q9, double>, static_cast<const double *>(buf));
}

// ---------------------------------------------------------------------------
// Training batches from a snapshot stack S[K][R][H][W]: image b of the batch
// is snapshot t_b + dt of run r_b, moved by a periodic shift and optionally
// transposed (symmetries of the periodic square lattice):
//   out[b][y][x] = S[t_b + dt][r_b][(Y - sy) mod H][(X - sx) mod W],
//   (Y, X) = (x, y) if transposed, else (y, x).
// ---------------------------------------------------------------------------
constexpr int GATHER_MAX = 64;
struct GatherIdx {
    int t[GATHER_MAX], r[GATHER_MAX];
};

__global__ void __launch_bounds__(256) k_gather(const float *__restrict__ snaps, int R, int H,
                                                int W, GatherIdx idx, int dt, int sy, int sx,
                                                int transpose, float *__restrict__ out) {
    const int b = blockIdx.y;
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= H * W) return;
    const int x = k % W, y = k / W;
    const int Y = transpose ? x : y, X = transpose ? y : x;
    int ys = (Y - sy) % H, xs = (X - sx) % W;
    ys += ys < 0 ? H : 0;
    xs += xs < 0 ? W : 0;
    const size_t img = size_t(idx.t[b] + dt) * R + idx.r[b];
    out[size_t(b) * H * W + k] = snaps[img * H * W + size_t(ys) * W + xs];
}

// Partial FP64 sums over a snapshot stack for the data scales: per block,
// sum (x - c) and (x - c)^2 over snapshots t_first.. K-1 and sum d, d^2 of the
// increments d = S[k+1] - S[k], k >= t_first (c: a centre close to the mean).
__global__ void __launch_bounds__(256) k_stack_moments(const float *__restrict__ S, int K,
                                                       int64_t per, int t_first, double c,
                                                       double *__restrict__ part) {
    __shared__ double sh[4][4];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    const int64_t n = int64_t(K - t_first) * per;
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += int64_t(gridDim.x) * 256) {
        const int64_t j = int64_t(t_first) * per + i;
        const double v = double(S[j]) - c;
        acc[0] += v;
        acc[1] += v * v;
        if (j + per < int64_t(K) * per) {
            const double d = double(S[j + per]) - double(S[j]);
            acc[2] += d;
            acc[3] += d * d;
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) acc[q] += __shfl_xor(acc[q], o, 64);
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6][q] = acc[q];
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int q = threadIdx.x;
        part[blockIdx.x * 4 + q] = sh[0][q] + sh[1][q] + sh[2][q] + sh[3][q];
    }
}

}  // namespace fsc

// ===========================================================================
// Surrogate object and its C ABI.
// ===========================================================================
using namespace fsc;

struct fsc_sur {
    int layers = 5, in_ch = 1, H = 0, W = 0, maxB = 0;
    float mean = 1.f, in_scale = 1.f, out_scale = 1.f;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    int64_t nparams = 0;
    void *arena = nullptr;  // holds every device buffer below
    std::vector<int64_t> woff, boff;  // offsets of each layer's weights / biases
    float *params = nullptr, *grads = nullptr, *m = nullptr, *v = nullptr;
    bf16 *wf = nullptr, *wb = nullptr;  // [mid layer][9][32][32]
    bf16 *wl3 = nullptr;                // last layer, [9][3][32] (see k_update)
    std::vector<float *> z;            // [layers - 1] of P x 32
    std::vector<bf16 *> a;             // [layers - 1] of P x 32
    bf16 *dzA = nullptr, *dzB = nullptr;
    float *y = nullptr, *gbuf = nullptr;
    float *wpart = nullptr;  // blocks' partial weight gradients: C -> C layers, first, last
    int wblocks = 0, eblocks = 0;  // blocks of a weight-gradient launch at max_batch
    double *gsum = nullptr, *loss = nullptr;
    double *part = nullptr;  // [3][maxB][IMG_PARTS] segment sums of y, dL/dy and the squared errors
    Mailbox box;             // the loss on its way to the host
    int64_t adam_t = 0;
    // captured rollouts: (prev, traj, batch, passes) -> graph, replayed on a
    // stream of the surrogate's own that is ordered after and before `stream`
    hipStream_t cap_stream = nullptr;
    hipEvent_t ev_in = nullptr, ev_out = nullptr;
    std::map<std::tuple<const float *, float *, int, int>, hipGraphExec_t> rollouts;
    std::deque<std::tuple<const float *, float *, int, int>> rollout_order;  // oldest first
    int fuse = 2;  // pairs of C -> C layers in one launch: 0 never, 1 always, 2 where it is faster
    std::string err;
};

namespace {

thread_local std::string g_sur_error;

int sur_fail(fsc_sur *s, int code, const std::string &msg) {
    if (s) s->err = msg;
    else g_sur_error = msg;
    return code;
}

#define SCHK(s, expr)                                                                       \
    do {                                                                                    \
        hipError_t _e = (expr);                                                             \
        if (_e != hipSuccess) return sur_fail((s), FSC_E_HIP, std::string(#expr) + ": " +   \
                                                                 hipGetErrorString(_e));    \
    } while (0)

int nmid(const fsc_sur *s) { return s->layers - 2; }

void sur_free(fsc_sur *s) {
    if (!s) return;
    (void)hipStreamSynchronize(s->stream);
    if (s->arena) (void)hipFree(s->arena);
    for (auto &kv : s->rollouts) (void)hipGraphExecDestroy(kv.second);
    if (s->cap_stream) {
        (void)hipStreamSynchronize(s->cap_stream);
        (void)hipStreamDestroy(s->cap_stream);
    }
    if (s->ev_in) (void)hipEventDestroy(s->ev_in);
    if (s->ev_out) (void)hipEventDestroy(s->ev_out);
    if (s->own_stream) (void)hipStreamDestroy(s->stream);
    delete s;
}

// Fused pairs of C -> C layers in images wider than 128 (narrower ones march, see
// k_chain): k_mid2_lds holds 60 KB of LDS per block, so 2 blocks per CU instead of
// 4, and wins while the blocks fit the chip in one round.  9-layer passes, us, single
// layers / pairs: 192^2 88 / 72, 256^2 100 / 86, 2 x 256^2 111 / 96, 3 x 256^2 122 / 133,
// 512^2 174 / 176, 8 x 256^2 225 / 241, 1024^2 624 / 667.  Mode 2 fuses up to
// FUSE_MAX_PIXELS pixels per batch.
constexpr int64_t FUSE_MAX_PIXELS = 8 * 128 * 128;
bool fuse_pairs(const fsc_sur *s, int B) {
    return s->fuse == 1 || (s->fuse == 2 && int64_t(B) * s->H * s->W <= FUSE_MAX_PIXELS);
}

// Destroys the captured rollout graphs (after any replay still running), so
// that the next rollout captures the current settings.
int drop_rollouts(fsc_sur *s) {
    if (s->rollouts.empty()) return FSC_OK;
    if (s->cap_stream) SCHK(s, hipStreamSynchronize(s->cap_stream));
    for (auto &kv : s->rollouts) (void)hipGraphExecDestroy(kv.second);
    s->rollouts.clear();
    s->rollout_order.clear();
    return FSC_OK;
}

// Captured rollouts kept per surrogate; beyond that the oldest capture is
// dropped (a caller that hands over fresh buffers every time would otherwise
// grow the cache without bound).
constexpr size_t ROLLOUT_CACHE_MAX = 8;

// packs the current parameters, after one Adam step on them if `o` is given
int update_params(fsc_sur *s, const AdamArgs *o) {
    const dim3 nb(unsigned((s->nparams + 255) / 256));
    const int n = int(s->nparams), mid0 = int(s->woff[1]), last0 = int(s->woff[s->layers - 1]);
    if (o)
        hipLaunchKernelGGL(k_update<true>, nb, dim3(256), 0, s->stream, s->params, n, mid0, last0, *o, s->wf,
                           s->wb, s->wl3);
    else
        hipLaunchKernelGGL(k_update<false>, nb, dim3(256), 0, s->stream, s->params, n, mid0, last0, AdamArgs{},
                           s->wf, s->wb, s->wl3);
    SCHK(s, hipGetLastError());
    return FSC_OK;
}

// rows per workgroup of the marching kernels, and workgroups per image: at most
// one per CU
void chain_strips(const fsc_sur *s, int B, int &R, int &strips) {
    const int most = std::min(s->H, std::max(1, CH_BLOCKS / B));
    R = (s->H + most - 1) / most;
    strips = (s->H + R - 1) / R;
}

int check_batch(fsc_sur *s, int batch) {
    if (batch < 1 || batch > s->maxB) return sur_fail(s, FSC_E_INVAL, "batch out of range");
    return FSC_OK;
}

// one C -> C layer, marching; rows of at most CH_W pixels
template <bool BWD, bool ZOUT>
void launch_march(const fsc_sur *s, int B, const bf16 *ain, const bf16 *w, const float *bias, float *zout, bf16 *aout,
                  const float *zprev) {
    int R, strips;
    chain_strips(s, B, R, strips);
    auto go = [&](auto kernel, int cw) {
        hipLaunchKernelGGL(kernel, dim3(unsigned(B * strips)), dim3(unsigned((cw + cw / 4) * 64)), 0, s->stream, ain, w,
                           bias, R, strips, s->H, s->W, zout, aout, zprev);
    };
    if (s->W <= CH_W / 2) go(k_march<4, BWD, ZOUT>, 4);
    else go(k_march<8, BWD, ZOUT>, 8);
}

// the LDS-staged C -> C layer applies when its tiles divide the image
bool lds_tiles(const fsc_sur *s) { return s->H % MR == 0 && s->W % MW == 0; }

// forward pass up to y (and its sums over the segments of every image); `train` keeps what the
// backward pass needs (the FP32 pre-activations)
int sur_forward_core(fsc_sur *s, const float *prev, const float *cur, int B, bool train) {
    const int P = B * s->H * s->W;
    const unsigned nb = unsigned((P + 255) / 256);
    const float ii = 1.f / s->in_scale, io = 1.f / s->out_scale;
    const float *w0 = s->params + s->woff[0], *b0 = s->params + s->boff[0];
    auto first = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nb), dim3(256), 0, s->stream, cur, prev, s->mean, ii, io, B, s->H,
                           s->W, w0, b0, s->z[0], s->a[0]);
    };
    if (s->in_ch == 2) train ? first(k_first<2, true>) : first(k_first<2, false>);
    else train ? first(k_first<1, true>) : first(k_first<1, false>);
    SCHK(s, hipGetLastError());
    const int tiles = P / 16;
    const unsigned mb = unsigned(std::min(2048, std::max(1, tiles / 16)));
    for (int l = 1; l <= nmid(s); ++l) {
        const size_t off = size_t(l - 1) * 9 * SC * SC;
        const bf16 *ain = s->a[l - 1], *wl = s->wf + off;
        const float *bl = s->params + s->boff[l];
        if (!train && s->fuse != 0 && s->W <= CH_W && l + 1 <= nmid(s)) {
            // layers l and l + 1 in one launch; a[l] is not written
            int R, strips;
            chain_strips(s, B, R, strips);
            auto chain = [&](auto kernel, int tpw) {
                hipLaunchKernelGGL(kernel, dim3(unsigned(B * strips)), dim3(unsigned((2 * CH_WAVES + tpw) * 64)), 0, s->stream, ain,
                                   wl, bl, wl + size_t(9) * SC * SC, s->params + s->boff[l + 1], R, strips, s->H,
                                   s->W, s->a[l + 1]);
            };
            if (s->W <= CH_W / 2) chain(k_chain<1>, 1);
            else chain(k_chain<2>, 2);
            SCHK(s, hipGetLastError());
            ++l;
            continue;
        }
        if (!train && fuse_pairs(s, B) && l + 1 <= nmid(s) && s->H % F2R == 0 && s->W % F2W == 0) {
            // layers l and l + 1 in one launch; a[l] is not written
            const dim3 g(unsigned(B * (s->H / F2R) * (s->W / F2W)));
            hipLaunchKernelGGL(k_mid2_lds, g, dim3(256), 0, s->stream, ain, wl, bl,
                               s->wf + off + size_t(9) * SC * SC, s->params + s->boff[l + 1], B,
                               s->H, s->W, s->a[l + 1]);
            SCHK(s, hipGetLastError());
            ++l;
            continue;
        }
        if (s->W <= CH_W) {
            if (train) launch_march<false, true>(s, B, ain, wl, bl, s->z[l], s->a[l], nullptr);
            else launch_march<false, false>(s, B, ain, wl, bl, nullptr, s->a[l], nullptr);
        } else if (lds_tiles(s)) {
            const dim3 g(unsigned(B * (s->H / MR) * (s->W / MW)));
            if (train)
                hipLaunchKernelGGL((k_mid_lds<false, true>), g, dim3(256), 0, s->stream, ain, wl, bl, B,
                                   s->H, s->W, s->z[l], s->a[l], nullptr);
            else
                hipLaunchKernelGGL((k_mid_lds<false, false>), g, dim3(256), 0, s->stream, ain, wl, bl, B,
                                   s->H, s->W, s->z[l], s->a[l], nullptr);
        } else if (train) {
            hipLaunchKernelGGL((k_mid<false, true>), dim3(mb), dim3(256), 0, s->stream, ain, wl, bl, B,
                               s->H, s->W, s->z[l], s->a[l], nullptr);
        } else {
            hipLaunchKernelGGL((k_mid<false, false>), dim3(mb), dim3(256), 0, s->stream, ain, wl, bl, B,
                               s->H, s->W, s->z[l], s->a[l], nullptr);
        }
        SCHK(s, hipGetLastError());
    }
    const int last = s->layers - 1;
    if (s->W <= CH_W) {
        int R, strips;
        chain_strips(s, B, R, strips);
        auto go = [&](auto kernel, int cw) {
            hipLaunchKernelGGL(kernel, dim3(unsigned(B * strips)), dim3(unsigned((cw + cw / 4) * 64)), 0, s->stream,
                               s->a[last - 1], R, strips, s->H, s->W, s->wl3, s->params + s->boff[last], s->y,
                               s->part);
        };
        if (s->W <= CH_W / 2) go(k_last_march<4>, 4);
        else go(k_last_march<8>, 8);
    } else {
        hipLaunchKernelGGL(k_last, dim3(unsigned(B * IMG_PARTS / 4)), dim3(256), 0, s->stream, s->a[last - 1], B,
                           s->H, s->W, s->wl3, s->params + s->boff[last], s->y, s->part);
    }
    SCHK(s, hipGetLastError());
    return FSC_OK;
}

void pred(const fsc_sur *s, const float *in, float *out, int B) {
    const int HW = s->H * s->W, lanes = HW >= 256 * IMG_PARTS ? 256 : 64;
    hipLaunchKernelGGL(k_pred, dim3(unsigned(B * IMG_PARTS / (256 / lanes))), dim3(256), 0, s->stream, in, s->y,
                       s->part, HW, lanes, s->out_scale, out);
}

int sur_backward(fsc_sur *s, const float *prev, const float *in, const float *tgt, int B) {
    const int H = s->H, W = s->W, P = B * H * W;
    const float ii = 1.f / s->in_scale, io = 1.f / s->out_scale;
    double *gpart = s->part + size_t(IMG_PARTS) * s->maxB, *epart = gpart + size_t(IMG_PARTS) * s->maxB;
    hipLaunchKernelGGL(k_loss, dim3(unsigned(B * IMG_PARTS / 4)), dim3(256), 0, s->stream, in, tgt, s->y, s->part,
                       H * W, io, 1.f / float(P), s->gbuf, gpart, epart);
    SCHK(s, hipGetLastError());
    hipLaunchKernelGGL(k_loss_total, dim3(unsigned(B + 1)), dim3(256), 0, s->stream, gpart, epart, B, s->gsum,
                       s->loss);
    SCHK(s, hipGetLastError());
    const int last = s->layers - 1;
    const int wtiles = wg_tiles(B, H, W);
    WgradSum ws{};
    ws.nmid = nmid(s);
    ws.in_ch = s->in_ch;
    ws.mid_blocks = std::min(wtiles, WG_MAX_BLOCKS);
    ws.edge_blocks = std::min(wtiles, WG_EDGE_BLOCKS);
    float *pmid = s->wpart, *pfirst = pmid + size_t(nmid(s)) * s->wblocks * WG_LEN;
    float *plast = pfirst + size_t(s->eblocks) * wg_edge_len<2>();
    ws.mid = pmid;
    ws.first = pfirst;
    ws.last = plast;
    ws.woff0 = int(s->woff[0]);
    ws.boff0 = int(s->boff[0]);
    ws.woff1 = int(s->woff[1]);
    ws.mid_stride = WG_LEN;
    ws.woffl = int(s->woff[last]);
    ws.boffl = int(s->boff[last]);
    const dim3 eb(unsigned(ws.edge_blocks));
    hipLaunchKernelGGL((k_edge_wgrad<1, true>), eb, dim3(256), 0, s->stream, s->a[last - 1], s->gbuf, nullptr,
                       0.f, 0.f, 0.f, s->gsum, B, H, W, plast);
    SCHK(s, hipGetLastError());
    bf16 *dz = s->dzA, *dzn = s->dzB;
    hipLaunchKernelGGL(k_last_bwd, dim3(unsigned((P + 63) / 64)), dim3(256), 0, s->stream, s->gbuf, s->gsum, B,
                       H, W, s->params + s->woff[last], s->z[last - 1], dz);
    SCHK(s, hipGetLastError());
    const int tiles = P / 16;
    const unsigned mb = unsigned(std::min(2048, std::max(1, tiles / 16)));
    for (int l = nmid(s); l >= 1; --l) {
        // dz holds dL/dz_l; weight gradient, then dL/dz_{l-1}
        hipLaunchKernelGGL(k_mid_wgrad, dim3(unsigned(ws.mid_blocks)), dim3(768), 0, s->stream, dz, s->a[l - 1],
                           B, H, W, pmid + size_t(l - 1) * ws.mid_blocks * WG_LEN);
        SCHK(s, hipGetLastError());
        const size_t off = size_t(l - 1) * 9 * SC * SC;
        if (s->W <= CH_W)
            launch_march<true, true>(s, B, dz, s->wb + off, nullptr, nullptr, dzn, s->z[l - 1]);
        else if (lds_tiles(s))
            hipLaunchKernelGGL((k_mid_lds<true, true>), dim3(unsigned(B * (H / MR) * (W / MW))), dim3(256),
                               0, s->stream, dz, s->wb + off, nullptr, B, H, W, nullptr, dzn, s->z[l - 1]);
        else
            hipLaunchKernelGGL((k_mid<true, true>), dim3(mb), dim3(256), 0, s->stream, dz, s->wb + off,
                               nullptr, B, H, W, nullptr, dzn, s->z[l - 1]);
        SCHK(s, hipGetLastError());
        std::swap(dz, dzn);
    }
    if (s->in_ch == 2)
        hipLaunchKernelGGL((k_edge_wgrad<2, false>), eb, dim3(256), 0, s->stream, dz, in, prev, s->mean, ii, io,
                           nullptr, B, H, W, pfirst);
    else
        hipLaunchKernelGGL((k_edge_wgrad<1, false>), eb, dim3(256), 0, s->stream, dz, in, prev, s->mean, ii, io,
                           nullptr, B, H, W, pfirst);
    SCHK(s, hipGetLastError());
    const int edge = SC * (9 * s->in_ch + 1) + SC * 9 + 1;
    hipLaunchKernelGGL(k_wgrad_sum,
                       dim3(unsigned(ws.nmid * WG_MID_GROUPS + (edge + WG_EDGE_COLS - 1) / WG_EDGE_COLS)),
                       dim3(64 * WG_SUM_WAVES), 0,
                       s->stream, ws, s->grads);
    SCHK(s, hipGetLastError());
    return FSC_OK;
}

int check_inputs(fsc_sur *s, const float *prev, const float *cur) {
    if (!cur || (s->in_ch == 2 && !prev))
        return sur_fail(s, FSC_E_INVAL, "missing input field (two-channel networks need prev)");
    return FSC_OK;
}

}  // namespace

extern "C" {

int fsc_sur_create(int layers, int in_ch, int H, int W, int max_batch, uint64_t seed,
                   void *stream, fsc_sur **out) {
    if (!out) return FSC_E_INVAL;
    *out = nullptr;
    if (layers < 3 || layers > 16 || (in_ch != 1 && in_ch != 2) || H < 1 || W < 16 || (W % 32) ||
        max_batch < 1 || int64_t(max_batch) * H * W >= (int64_t(1) << 26))
        return sur_fail(nullptr, FSC_E_INVAL,
                        "need 3 <= layers <= 16, in_ch 1 or 2, W a multiple of 32, batch*H*W < 2^26");
    fsc_sur *s = new fsc_sur();
    s->layers = layers;
    s->in_ch = in_ch;
    s->H = H;
    s->W = W;
    s->maxB = max_batch;
    // NULL is the device's default (null) stream, so that calls are ordered
    // with other work on it (torch's default stream is the null stream)
    s->stream = static_cast<hipStream_t>(stream);
    // parameter layout: per layer W[co][ci][3][3] then b[co]
    int64_t o = 0;
    std::vector<float> host;
    uint64_t st = seed * 0x9E3779B97F4A7C15ull + 0x2545F4914F6CDD1Dull;
    auto rnd = [&]() {  // splitmix64 -> uniform in [-1, 1)
        st += 0x9E3779B97F4A7C15ull;
        uint64_t zz = st;
        zz = (zz ^ (zz >> 30)) * 0xBF58476D1CE4E5B9ull;
        zz = (zz ^ (zz >> 27)) * 0x94D049BB133111EBull;
        zz ^= zz >> 31;
        return double(zz >> 11) * (2.0 / 9007199254740992.0) - 1.0;
    };
    for (int l = 0; l < layers; ++l) {
        const int ci = l == 0 ? in_ch : SC, co = l == layers - 1 ? 1 : SC;
        s->woff.push_back(o);
        // uniform in +-1/sqrt(fan_in) for weights and biases: a small initial
        // map keeps the rollouts of early training (used as inputs) tame
        const double bound = 1.0 / std::sqrt(double(ci * 9));
        for (int k = 0; k < co * ci * 9; ++k) host.push_back(float(bound * rnd()));
        o += co * ci * 9;
        s->boff.push_back(o);
        for (int k = 0; k < co; ++k) host.push_back(float(bound * rnd()));
        o += co;
    }
    s->nparams = o;
    const size_t P = size_t(max_batch) * H * W;
    s->wblocks = std::min(wg_tiles(max_batch, H, W), WG_MAX_BLOCKS);
    s->eblocks = std::min(wg_tiles(max_batch, H, W), WG_EDGE_BLOCKS);
    const size_t wlen = size_t(layers - 2) * s->wblocks * WG_LEN +
                        size_t(s->eblocks) * (wg_edge_len<2>() + wg_edge_len<1>());
    // every buffer of the object from one allocation (an allocation takes 30 to
    // 300 us, and there are over thirty)
    const size_t nw = sizeof(bf16) * 9 * SC * SC * std::max(1, layers - 2);
    s->z.assign(size_t(layers - 1), nullptr);
    s->a.assign(size_t(layers - 1), nullptr);
    std::vector<std::pair<void **, size_t>> parts;
    auto want = [&](auto *&p, size_t bytes) { parts.emplace_back(reinterpret_cast<void **>(&p), bytes); };
    for (float **p : {&s->params, &s->grads, &s->m, &s->v}) want(*p, sizeof(float) * size_t(o));
    want(s->wf, nw);
    want(s->wb, nw);
    want(s->wl3, sizeof(bf16) * 9 * 3 * SC);
    want(s->dzA, sizeof(bf16) * P * SC);
    want(s->dzB, sizeof(bf16) * P * SC);
    want(s->y, sizeof(float) * P);
    want(s->gbuf, sizeof(float) * P);
    want(s->wpart, sizeof(float) * wlen);
    want(s->part, sizeof(double) * 3 * IMG_PARTS * size_t(max_batch));
    want(s->gsum, sizeof(double) * size_t(max_batch));
    want(s->loss, sizeof(double));
    for (auto &p : s->z) want(p, sizeof(float) * P * SC);
    for (auto &p : s->a) want(p, sizeof(bf16) * P * SC);
    size_t total = 0;
    for (auto &q : parts) total += (q.second + 255) & ~size_t(255);
    const bool ok = hipMalloc(&s->arena, total) == hipSuccess;
    char *at = static_cast<char *>(s->arena);
    for (auto &q : parts) {
        *q.first = ok ? at : nullptr;
        at += ok ? (q.second + 255) & ~size_t(255) : 0;
    }
    if (!ok) {
        (void)hipGetLastError();
        sur_free(s);
        return sur_fail(nullptr, FSC_E_OOM, "surrogate allocation failed");
    }
    if (hipMemcpy(s->params, host.data(), sizeof(float) * o, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemset(s->m, 0, sizeof(float) * o) != hipSuccess ||
        hipMemset(s->v, 0, sizeof(float) * o) != hipSuccess || update_params(s, nullptr) != FSC_OK ||
        hipStreamSynchronize(s->stream) != hipSuccess) {
        sur_free(s);
        return sur_fail(nullptr, FSC_E_HIP, "surrogate initialisation failed");
    }
    *out = s;
    return FSC_OK;
}

int fsc_sur_destroy(fsc_sur *s) {
    if (!s) return FSC_E_INVAL;
    sur_free(s);
    return FSC_OK;
}

const char *fsc_sur_last_error(const fsc_sur *s) { return s ? s->err.c_str() : g_sur_error.c_str(); }

int fsc_sur_nparams(const fsc_sur *s, int64_t *n) {
    if (!s || !n) return FSC_E_INVAL;
    *n = s->nparams;
    return FSC_OK;
}

int fsc_sur_set_params(fsc_sur *s, const float *host, int64_t n) {
    if (!s || !host || n != s->nparams) return FSC_E_INVAL;
    SCHK(s, hipMemcpyAsync(s->params, host, sizeof(float) * n, hipMemcpyHostToDevice, s->stream));
    int rc = update_params(s, nullptr);
    if (rc) return rc;
    SCHK(s, hipMemsetAsync(s->m, 0, sizeof(float) * n, s->stream));
    SCHK(s, hipMemsetAsync(s->v, 0, sizeof(float) * n, s->stream));
    s->adam_t = 0;
    SCHK(s, hipStreamSynchronize(s->stream));
    return FSC_OK;
}

int fsc_sur_get_params(fsc_sur *s, float *host, int64_t n) {
    if (!s || !host || n != s->nparams) return FSC_E_INVAL;
    SCHK(s, hipMemcpyAsync(host, s->params, sizeof(float) * n, hipMemcpyDeviceToHost, s->stream));
    SCHK(s, hipStreamSynchronize(s->stream));
    return FSC_OK;
}

int fsc_sur_set_norm(fsc_sur *s, float mean, float in_scale, float out_scale) {
    if (!s || !(in_scale > 0.f) || !(out_scale > 0.f)) return FSC_E_INVAL;
    if (mean != s->mean || in_scale != s->in_scale || out_scale != s->out_scale) {
        // the captured rollouts hold the old values as kernel arguments
        int rc = drop_rollouts(s);
        if (rc) return rc;
    }
    s->mean = mean;
    s->in_scale = in_scale;
    s->out_scale = out_scale;
    return FSC_OK;
}

int fsc_sur_set_fusion(fsc_sur *s, int mode) {
    if (!s || mode < 0 || mode > 2) return FSC_E_INVAL;
    if (mode != s->fuse) {
        int rc = drop_rollouts(s);  // captured with another kernel sequence
        if (rc) return rc;
    }
    s->fuse = mode;
    return FSC_OK;
}

int fsc_sur_forward(fsc_sur *s, const float *dev_prev, const float *dev_in, float *dev_out,
                    int batch) {
    TraceRange trace_("fsc sur_forward");
    if (!s || !dev_out) return FSC_E_INVAL;
    int rc = check_inputs(s, dev_prev, dev_in);
    if (rc) return rc;
    rc = check_batch(s, batch);
    if (rc) return rc;
    rc = sur_forward_core(s, dev_prev, dev_in, batch, false);
    if (rc) return rc;
    pred(s, dev_in, dev_out, batch);
    SCHK(s, hipGetLastError());
    return FSC_OK;
}

int fsc_sur_grad(fsc_sur *s, const float *dev_prev, const float *dev_in, const float *dev_target,
                 int batch, float *host_grad, double *loss) {
    if (!s || !dev_target) return FSC_E_INVAL;
    int rc = check_inputs(s, dev_prev, dev_in);
    if (rc) return rc;
    rc = check_batch(s, batch);
    if (rc) return rc;
    rc = sur_forward_core(s, dev_prev, dev_in, batch, true);
    if (rc) return rc;
    rc = sur_backward(s, dev_prev, dev_in, dev_target, batch);
    if (rc) return rc;
    // the loss goes ahead of the copy, not in a second one
    const bool mailed = s->box.make(sizeof(double)) == hipSuccess;
    if (mailed) SCHK(s, launch_mail(s->loss, 1, s->box.next(), s->stream));
    if (host_grad)
        SCHK(s, hipMemcpyAsync(host_grad, s->grads, sizeof(float) * s->nparams,
                               hipMemcpyDeviceToHost, s->stream));
    double l = 0.0;
    if (!mailed) SCHK(s, hipMemcpyAsync(&l, s->loss, sizeof(double), hipMemcpyDeviceToHost, s->stream));
    SCHK(s, hipStreamSynchronize(s->stream));
    if (mailed) {
        SCHK(s, s->box.wait(s->stream));
        l = s->box.data()[0];
    }
    if (loss) *loss = l / double(batch * s->H * s->W);
    return FSC_OK;
}

int fsc_sur_train_step(fsc_sur *s, const float *dev_prev, const float *dev_in,
                       const float *dev_target, int batch, float lr, double *loss) {
    TraceRange trace_("fsc sur_train_step");
    if (!s || !dev_target || !(lr > 0.f)) return FSC_E_INVAL;
    int rc = check_inputs(s, dev_prev, dev_in);
    if (rc) return rc;
    rc = check_batch(s, batch);
    if (rc) return rc;
    rc = sur_forward_core(s, dev_prev, dev_in, batch, true);
    if (rc) return rc;
    rc = sur_backward(s, dev_prev, dev_in, dev_target, batch);
    if (rc) return rc;
    s->adam_t += 1;
    const float b1 = 0.9f, b2 = 0.999f;
    const float bc1 = 1.f - std::pow(b1, float(s->adam_t));
    const float bc2 = 1.f - std::pow(b2, float(s->adam_t));
    const AdamArgs o{s->grads, s->m, s->v, lr, b1, b2, 1e-8f, bc1, bc2};
    rc = update_params(s, &o);
    if (rc) return rc;
    if (loss) {
        double l = 0.0;
        if (s->box.make(sizeof(double)) == hipSuccess) {
            SCHK(s, launch_mail(s->loss, 1, s->box.next(), s->stream));
            SCHK(s, s->box.wait(s->stream));
            l = s->box.data()[0];
        } else {
            SCHK(s, hipMemcpyAsync(&l, s->loss, sizeof(double), hipMemcpyDeviceToHost, s->stream));
            SCHK(s, hipStreamSynchronize(s->stream));
        }
        *loss = l / double(batch * s->H * s->W);
    }
    return FSC_OK;
}

int fsc_sur_rollout(fsc_sur *s, const float *dev_prev, float *dev_traj, int batch, int passes) {
    TraceRange trace_("fsc sur_rollout");
    if (!s || !dev_traj || passes < 1) return FSC_E_INVAL;
    int rc = check_batch(s, batch);
    if (rc) return rc;
    if (s->in_ch == 2 && !dev_prev)
        return sur_fail(s, FSC_E_INVAL, "missing input field (two-channel networks need prev)");
    if (!s->cap_stream) {
        SCHK(s, hipStreamCreateWithFlags(&s->cap_stream, hipStreamNonBlocking));
        SCHK(s, hipEventCreateWithFlags(&s->ev_in, hipEventDisableTiming));
        SCHK(s, hipEventCreateWithFlags(&s->ev_out, hipEventDisableTiming));
    }
    const size_t img = size_t(batch) * s->H * s->W;
    auto key = std::make_tuple(dev_prev, dev_traj, batch, passes);
    auto it = s->rollouts.find(key);
    if (it == s->rollouts.end()) {
        // capture the passes on the private stream: the forward kernels use
        // no memset nodes, only launches
        hipStream_t user = s->stream;
        s->stream = s->cap_stream;
        hipGraph_t graph = nullptr;
        hipError_t ec = hipStreamBeginCapture(s->cap_stream, hipStreamCaptureModeThreadLocal);
        int frc = FSC_OK;
        if (ec == hipSuccess) {
            for (int k = 0; k < passes && frc == FSC_OK; ++k) {
                const float *prev = k == 0 ? dev_prev : dev_traj + (k - 1) * img;
                frc = sur_forward_core(s, prev, dev_traj + k * img, batch, false);
                if (frc == FSC_OK) {
                    pred(s, dev_traj + k * img, dev_traj + (k + 1) * img, batch);
                    if (hipGetLastError() != hipSuccess) frc = FSC_E_HIP;
                }
            }
            hipError_t ee = hipStreamEndCapture(s->cap_stream, &graph);
            if (ec == hipSuccess) ec = ee;
        }
        s->stream = user;
        if (frc != FSC_OK || ec != hipSuccess) {
            if (graph) (void)hipGraphDestroy(graph);
            return frc != FSC_OK ? frc : sur_fail(s, FSC_E_HIP, std::string("rollout capture: ") +
                                                                      hipGetErrorString(ec));
        }
        hipGraphExec_t exec = nullptr;
        ec = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (ec != hipSuccess)
            return sur_fail(s, FSC_E_HIP, std::string("rollout instantiate: ") + hipGetErrorString(ec));
        if (s->rollouts.size() >= ROLLOUT_CACHE_MAX) {
            SCHK(s, hipStreamSynchronize(s->cap_stream));  // no replay of it still running
            auto old = s->rollouts.find(s->rollout_order.front());
            (void)hipGraphExecDestroy(old->second);
            s->rollouts.erase(old);
            s->rollout_order.pop_front();
        }
        it = s->rollouts.emplace(key, exec).first;
        s->rollout_order.push_back(key);
    }
    // ordered after the caller's stream and before its later work
    SCHK(s, hipEventRecord(s->ev_in, s->stream));
    SCHK(s, hipStreamWaitEvent(s->cap_stream, s->ev_in, 0));
    SCHK(s, hipGraphLaunch(it->second, s->cap_stream));
    SCHK(s, hipEventRecord(s->ev_out, s->cap_stream));
    SCHK(s, hipStreamWaitEvent(s->stream, s->ev_out, 0));
    return FSC_OK;
}

int fsc_sur_gather(fsc_sur *s, const float *dev_snaps, int K, int R, const int *host_t,
                   const int *host_r, int batch, int dt, int sy, int sx, int transpose,
                   float *dev_out) {
    if (!s || !dev_snaps || !host_t || !host_r || !dev_out || K < 1 || R < 1) return FSC_E_INVAL;
    if (batch < 1 || batch > GATHER_MAX || batch > s->maxB)
        return sur_fail(s, FSC_E_INVAL, "gather batch out of range");
    if (transpose && s->H != s->W) return sur_fail(s, FSC_E_INVAL, "transpose needs H == W");
    GatherIdx idx{};
    for (int b = 0; b < batch; ++b) {
        if (host_t[b] + dt < 0 || host_t[b] + dt >= K || host_r[b] < 0 || host_r[b] >= R)
            return sur_fail(s, FSC_E_INVAL, "gather index out of the snapshot stack");
        idx.t[b] = host_t[b];
        idx.r[b] = host_r[b];
    }
    const int HW = s->H * s->W;
    const dim3 g(unsigned((HW + 255) / 256), unsigned(batch));
    hipLaunchKernelGGL(k_gather, g, dim3(256), 0, s->stream, dev_snaps, R, s->H, s->W, idx, dt,
                       ((sy % s->H) + s->H) % s->H, ((sx % s->W) + s->W) % s->W, transpose ? 1 : 0,
                       dev_out);
    SCHK(s, hipGetLastError());
    return FSC_OK;
}

int fsc_stack_scales(const float *dev_snaps, int K, int64_t per_snap, int t_first, double centre,
                     double *host_in_std, double *host_out_std, void *stream) {
    if (!dev_snaps || K < 2 || per_snap < 1 || t_first < 0 || t_first > K - 2 || !host_in_std ||
        !host_out_std)
        return FSC_E_INVAL;
    const hipStream_t st = static_cast<hipStream_t>(stream);
    const int nb = 1024;
    double *part = nullptr;
    if (hipMalloc(&part, sizeof(double) * 4 * nb) != hipSuccess) return FSC_E_OOM;
    hipLaunchKernelGGL(k_stack_moments, dim3(nb), dim3(256), 0, st, dev_snaps, K, per_snap, t_first,
                       centre, part);
    std::vector<double> h(4 * nb);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess)
        e = hipMemcpyAsync(h.data(), part, sizeof(double) * 4 * nb, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    (void)hipFree(part);
    if (e != hipSuccess) return FSC_E_HIP;
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    for (int b = 0; b < nb; ++b)
        for (int q = 0; q < 4; ++q) a[q] += h[4 * b + q];
    const double n = double(K - t_first) * double(per_snap);
    const double nd = double(K - 1 - t_first) * double(per_snap);
    *host_in_std = std::sqrt((a[1] - a[0] * a[0] / n) / (n - 1.0));
    *host_out_std = std::sqrt((a[3] - a[2] * a[2] / nd) / (nd - 1.0));
    return FSC_OK;
}

int fsc_mfma_probe(const float *host_a, const float *host_b, float *host_c) {
    if (!host_a || !host_b || !host_c) return FSC_E_INVAL;
    float *d = nullptr;
    if (hipMalloc(&d, sizeof(float) * (16 * 32 + 32 * 16 + 16 * 16)) != hipSuccess) return FSC_E_OOM;
    hipError_t e = hipMemcpy(d, host_a, sizeof(float) * 512, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(d + 512, host_b, sizeof(float) * 512, hipMemcpyHostToDevice);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_mfma_probe, dim3(1), dim3(64), 0, nullptr, d, d + 512, d + 1024);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpy(host_c, d + 1024, sizeof(float) * 256, hipMemcpyDeviceToHost);
    (void)hipFree(d);
    return e == hipSuccess ? FSC_OK : FSC_E_HIP;
}

}  // extern "C"
