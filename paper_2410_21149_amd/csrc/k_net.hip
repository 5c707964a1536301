// Learned pose proposal for submap alignment: a small 3-D convolutional
// network on coarse ESDF summaries, trained and run with hand-written
// kernels.  (Not part of the paper; it proposes the initial pose that the
// correspondence-free ESDF alignment of Sec. III-F then refines.)
//
// Network (input 32^3 x 4 channels, NDHWC):
//   conv 3x3x3, 4 -> 16, stride 1 (32^3), ReLU
//   conv 3x3x3, 16 -> 32, stride 2 (16^3), ReLU
//   conv 3x3x3, 32 -> 64, stride 2 (8^3), ReLU
//   conv 3x3x3, 64 -> 64, stride 2 (4^3), ReLU
//   global mean -> fully connected 64 -> 5 (tx, ty, tz, cos yaw, sin yaw)
// Convolutions (zero padding 1) run as implicit GEMMs on the bf16 matrix
// cores (v_mfma_f32_16x16x32_bf16): bf16 activations and weights, FP32
// accumulation, bias and ReLU in FP32, outputs rounded to bf16 (nearest
// even).  FP32 master weights; the backward pass takes bf16 operands and sums in
// FP32, Adam runs in FP32.
#include "covox_impl.h"

#include <math.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <vector>

namespace covox {

namespace {

typedef float v4f32 __attribute__((ext_vector_type(4)));

// binary32 -> bfloat16, round to nearest even (NaN kept quiet).
__host__ __device__ inline uint16_t f2bf(float f)
{
    uint32_t x;
    memcpy(&x, &f, 4);
    if ((x & 0x7F800000u) == 0x7F800000u && (x & 0x7FFFFFu)) return (uint16_t)((x >> 16) | 0x40);
    const uint32_t lsb = (x >> 16) & 1u;
    x += 0x7FFFu + lsb;
    return (uint16_t)(x >> 16);
}

__host__ __device__ inline float bf2f(uint16_t h)
{
    const uint32_t x = (uint32_t)h << 16;
    float f;
    memcpy(&f, &x, 4);
    return f;
}

struct ConvShape {
    int cin, cout, din, dout, stride;
    constexpr int K() const { return 27 * cin; }
};

constexpr int kLayers = 4;
constexpr ConvShape kShapes[kLayers] = {{4, 16, 32, 32, 1}, {16, 32, 32, 16, 2}, {32, 64, 16, 8, 2}, {64, 64, 8, 4, 2}};
constexpr int kOut = 5;
constexpr int kFeat = 64;

// ------------------------------------------------------------ forward

// Operands of v_mfma_f32_16x16x32_bf16: lane l supplies A[m = l % 16][k = 8 (l /
// 16) + i] and B[k = 8 (l / 16) + i][n = l % 16], i = 0..7, and receives D[m =
// 4 (l / 16) + i][n = l % 16], i = 0..3.  The convolutions put the weights on
// the A side (m = output channel) and the positions on the B side, so that a
// lane ends with four consecutive channels of one position.
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef uint32_t v4u32 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4f32 mfma32(v4u32 a, v4u32 b, v4f32 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}

// Two binary32 values as bf16 (round to nearest even), a in the low half.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    return (uint32_t)f2bf(a) | ((uint32_t)f2bf(b) << 16);
}

// Bias and ReLU of a lane's four channels, to y as bf16.
__device__ __forceinline__ void store_relu(uint16_t *y, v4f32 acc, const float *bias)
{
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = fmaxf(acc[i] + bias[i], 0.0f);
    *(uint2 *)y = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
}

// First layer, 4 -> 16 channels at 32^3.  A workgroup takes 32 x 4 x 4
// positions: their input with one voxel around it is read once as binary32,
// rounded to bf16 and staged in LDS (8 bytes a voxel, zeros outside the grid),
// the weights stay in registers (K = 27 taps x 4 channels, 8 taps to an MFMA,
// the last five empty).  Bound by its traffic, 16 bytes read and 32 written a
// position; a pass that wrote the input as bf16 and a kernel that gathered each
// tap from memory took 15 + 87 us for 64 items, this one 28 us.
constexpr int kInTY = 4, kInTZ = 4;
constexpr int kInHX = 34, kInHY = kInTY + 2, kInHZ = kInTZ + 2, kInVox = kInHX * kInHY * kInHZ;

__global__ __launch_bounds__(256) void k_conv_in(const float *__restrict__ x, const uint16_t *__restrict__ w,
                                                 const float *__restrict__ bias, uint16_t *__restrict__ y)
{
    constexpr int D = 32, K = 108, NY = D / kInTY, NZ = D / kInTZ;
    __shared__ uint2 in[kInVox];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, g = lane >> 4, n = lane & 15;
    const int ty = (int)(blockIdx.x % NY) * kInTY, tz = (int)(blockIdx.x / NY % NZ) * kInTZ;
    const int64_t item = blockIdx.x / (NY * NZ);
    v4u32 wf[4];
    int off[8];  // voxel offset of tap 8 c + 2 g + j at [2 c + j]
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        uint2 t[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int tap = 8 * c + 2 * g + j;
            t[j] = tap < 27 ? *(const uint2 *)(w + n * K + 4 * tap) : make_uint2(0u, 0u);
            off[2 * c + j] = tap < 27 ? ((tap / 9) * kInHY + tap / 3 % 3) * kInHX + tap % 3 : 0;
        }
        wf[c] = (v4u32){t[0].x, t[0].y, t[1].x, t[1].y};
    }
    constexpr int kPer = (kInVox + 255) / 256;
    float v[kPer][4];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int e = tid + 256 * q;
        const int ix = e % kInHX - 1, iy = ty + e / kInHX % kInHY - 1, iz = tz + e / (kInHX * kInHY) - 1;
        const bool ok = e < kInVox && ix >= 0 && iy >= 0 && iz >= 0 && ix < D && iy < D && iz < D;
        const float *src = x + (ok ? 4 * (((item * D + iz) * D + iy) * D + ix) : 0);
        __builtin_memcpy(v[q], src, 16);
#pragma unroll
        for (int k = 0; k < 4; ++k) v[q][k] = ok ? v[q][k] : 0.0f;
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q)
        if (tid + 256 * q < kInVox) in[tid + 256 * q] = make_uint2(pack_bf16(v[q][0], v[q][1]), pack_bf16(v[q][2], v[q][3]));
    __syncthreads();
    float bv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) bv[i] = bias[4 * g + i];
    // 16 rows of 32 positions, four to a wave, two MFMA tiles to a row
#pragma unroll 2
    for (int t = 0; t < 2 * kInTY * kInTZ / 4; ++t) {
        const int r = wid * (kInTY * kInTZ / 4) + (t >> 1), ry = r % kInTY, rz = r / kInTY, ox = 16 * (t & 1) + n;
        const uint2 *p = in + (rz * kInHY + ry) * kInHX + ox;
        v4f32 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            uint2 a = p[off[2 * c]], b = p[off[2 * c + 1]];
            if (c == 3) {  // taps 27..31 do not exist
                a = g < 2 ? a : make_uint2(0u, 0u);
                b = g < 1 ? b : make_uint2(0u, 0u);
            }
            acc = mfma32(wf[c], (v4u32){a.x, a.y, b.x, b.y}, acc);
        }
        store_relu(y + (((item * D + tz + rz) * D + ty + ry) * D + ox) * 16 + 4 * g, acc, bv);
    }
}

// The stride-2 layers.  A workgroup copies the weights of its 16 CT output
// channels to LDS once, in operand order (conflict-free 16-byte reads), and its
// waves take tiles of 16 positions: the activations of all 27 taps come straight
// from memory, 16 bytes (8 channels of one tap) a lane, every read in flight
// before the first MFMA.  K chunks of 32 are summed in order.  Bound by reading
// the activations once (16 -> 32 channels: 67 MB for 64 items), then by latency.
// With 8-byte reads of both operands for every chunk of 16 the three layers took
// 77 + 38 + 30 us for 64 items, with each wave's weights in registers and its
// activations read by four waves 22 + 29 + 13, now 25 + 13 + 13.
template <int CIN, int COUT, int DIN, int DOUT, int CT, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(1, CIN == 16 ? 4 : (NT + 255) / 256))) void k_conv_fwd(
    const uint16_t *__restrict__ x, const uint16_t *__restrict__ w, const float *__restrict__ bias,
    uint16_t *__restrict__ y, int64_t n_tiles)
{
    constexpr int K = 27 * CIN, NC = (K + 31) / 32;
    static_assert(DOUT * DOUT * DOUT % 16 == 0, "a tile lies in one item");
    __shared__ v4u32 wl[NC * CT * 64];  // [chunk][channel tile][lane]
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, g = lane >> 4, n = lane & 15;
    const int co0 = 16 * CT * blockIdx.y;
    // chunk c of lane group q: tap and first channel
    auto tap_of = [](int c, int q) { return CIN == 16 ? 2 * c + (q >> 1) : (CIN == 32 ? c : c >> 1); };
    auto ch_of = [](int c, int q) { return CIN == 16 ? 8 * (q & 1) : (CIN == 64 ? 32 * (c & 1) : 0) + 8 * q; };
    constexpr int kBatch = 7;  // reads in flight a lane
    for (int e0 = tid; e0 < NC * CT * 64; e0 += kBatch * NT) {
        v4u32 v[kBatch];
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            const int e = min(e0 + b * NT, NC * CT * 64 - 1);
            const int c = e / (64 * CT), t = e / 64 % CT, q = (e >> 4) & 3, m = e & 15;
            const int tap = tap_of(c, q);
            v[b] = *(const v4u32 *)(w + (int64_t)(co0 + 16 * t + m) * K + (tap < 27 ? tap * CIN + ch_of(c, q) : 0));
            if (tap >= 27) v[b] = (v4u32){0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int b = 0; b < kBatch; ++b)
            if (e0 + b * NT < NC * CT * 64) wl[e0 + b * NT] = v[b];
    }
    bool staged = false;
    for (int64_t tile = (int64_t)blockIdx.x * (NT / 64) + wid; !staged || tile < n_tiles;
         tile += (int64_t)gridDim.x * (NT / 64)) {
        constexpr int kTiles = DOUT * DOUT * DOUT / 16;
        const int64_t tt = min(tile, n_tiles - 1);
        const int64_t item = tt / kTiles;
        const int p = (int)(tt % kTiles) * 16 + n;
        const int ox = p % DOUT, oy = p / DOUT % DOUT, oz = p / (DOUT * DOUT);
        const uint16_t *xi = x + item * (DIN * DIN * DIN * CIN);
        // input position of tap (0, 0, 0): below the grid only at the low faces
        const int base = (((2 * oz - 1) * DIN + 2 * oy - 1) * DIN + 2 * ox - 1) * CIN;
        v4u32 v[NC];
        bool in[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int tap = tap_of(c, g), kd = tap / 9, kh = tap / 3 % 3, kw = tap % 3;
            in[c] = tap < 27 && (kd > 0 || oz > 0) && (kh > 0 || oy > 0) && (kw > 0 || ox > 0);
            v[c] = *(const v4u32 *)(xi + (in[c] ? base + ((kd * DIN + kh) * DIN + kw) * CIN + ch_of(c, g) : 0));
        }
        if (!staged) {  // the first tile's reads overlap the copy of the weights
            __syncthreads();
            staged = true;
            if (tile >= n_tiles) break;
        }
        asm volatile("" ::: "memory");  // keeps the weights in LDS: they do not fit beside the reads in flight
        v4f32 acc[CT];
#pragma unroll
        for (int t = 0; t < CT; ++t) acc[t] = (v4f32){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NC; ++c) {
#pragma unroll
            for (int k = 0; k < 4; ++k) v[c][k] = in[c] ? v[c][k] : 0u;
#pragma unroll
            for (int t = 0; t < CT; ++t) acc[t] = mfma32(wl[(c * CT + t) * 64 + lane], v[c], acc[t]);
        }
#pragma unroll
        for (int t = 0; t < CT; ++t) {
            const int co = co0 + 16 * t + 4 * g;
            store_relu(y + (item * (DOUT * DOUT * DOUT) + p) * COUT + co, acc[t], bias + co);
        }
    }
}

// Global mean over the 4^3 positions and the fully connected head.
__global__ void k_pool_fc(const uint16_t *__restrict__ a4, const float *__restrict__ wfc,
                          const float *__restrict__ bfc, float *__restrict__ pooled, float *__restrict__ out, int n)
{
    const int b = blockIdx.x, c = threadIdx.x;  // 64 threads
    if (b >= n) return;
    __shared__ float f[kFeat];
    float s = 0.f;
    for (int p = 0; p < 64; ++p) s += bf2f(a4[((int64_t)b * 64 + p) * kFeat + c]);
    s *= (1.0f / 64.0f);
    f[c] = s;
    pooled[b * kFeat + c] = s;
    __syncthreads();
    if (c < kOut) {
        float o = bfc[c];
        for (int k = 0; k < kFeat; ++k) o += wfc[c * kFeat + k] * f[k];
        out[b * kOut + c] = o;
    }
}

// ------------------------------------------------------------ backward

// Loss: sum over the batch of (|t - t*|^2 / s_t^2 + |(c, s) - (c*, s*)|^2),
// divided by n, summed by one workgroup in a fixed order.  d_out = its gradient.
__global__ __launch_bounds__(256) void k_loss(const float *__restrict__ out, const float *__restrict__ y,
                                              float *__restrict__ dout, float *__restrict__ loss, int n, float inv_st2)
{
    __shared__ float red[4];
    float s = 0.f;
    for (int i = threadIdx.x; i < n * kOut; i += 256) {
        const float wgt = i % kOut < 3 ? inv_st2 : 1.0f;
        const float d = out[i] - y[i];
        dout[i] = 2.0f * wgt * d / (float)n;
        s += wgt * d * d / (float)n;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) *loss = (red[0] + red[1]) + (red[2] + red[3]);
}

// FC backward: gradients of the head, then d a4 = (d pooled / 64) masked by
// ReLU (a4 > 0).  Workgroup n + o (64 threads) sums output o of the head's
// gradients over the batch, eight items' reads in flight (one workgroup for all
// five outputs, an item at a time, took 32 us for 64 items); workgroup b < n
// writes d a4 of item b.
__global__ __launch_bounds__(64) void k_fc_bwd(const float *__restrict__ dout, const float *__restrict__ pooled,
                                               const float *__restrict__ wfc, const uint16_t *__restrict__ a4,
                                               float *__restrict__ gwfc, float *__restrict__ gbfc,
                                               float *__restrict__ da4, int n)
{
    const int t = threadIdx.x, b = blockIdx.x;
    if (b >= n) {
        const int o = b - n;
        float g = 0.f, gb = 0.f;
#pragma unroll 8
        for (int bb = 0; bb < n; ++bb) {
            g += dout[bb * kOut + o] * pooled[bb * kFeat + t];
            gb += dout[bb * kOut + o];
        }
        gwfc[o * kFeat + t] = g;
        if (t == 0) gbfc[o] = gb;
        return;
    }
    float dp = 0.f;
    for (int o = 0; o < kOut; ++o) dp += dout[b * kOut + o] * wfc[o * kFeat + t];
    dp *= (1.0f / 64.0f);
#pragma unroll 16
    for (int p = 0; p < 64; ++p) {
        const int64_t q = ((int64_t)b * 64 + p) * kFeat + t;
        da4[q] = bf2f(a4[q]) > 0.f ? dp : 0.f;
    }
}

// Weight gradients on the matrix cores: gw[co][tap][ci] = sum over the output
// positions p of dy[p][co] x[2 p + tap - 1][ci] (x zero outside the grid), the
// positions being the reduction (32 to an MFMA, A side dy, B side x), and a
// column of ones for the bias.  Memory has channels fastest while an operand
// lane holds eight consecutive positions of one channel, so a tile of positions
// is transposed on its way into LDS: dy as [co][position], x as [kw][ci][z][y]
// [ox] with ox the output position that tap kw maps the voxel to (odd voxels
// serve taps 0 and 2, even ones tap 1).  Every operand is then one aligned LDS
// read.  Plane strides are odd in 16-byte units, so that the 16 channels of an
// operand lie in different banks.  A workgroup takes 16 input channels (one
// MFMA column tile a tap) and walks tiles with the sums in registers, its four
// waves seven taps each; k_wgrad_sum adds the workgroups' sums in a fixed order.
// Bound by the transposition (LDS writes of two bytes).  Gathering the operands
// from memory two bytes a lane, with atomics for the sums, took 391 + 203 + 53
// us for the three layers and 64 items; now 37 + 23 + 14 and 6 each for the sums.
template <int L>
struct WgradShape {
    static constexpr int kCin = kShapes[L].cin, kCout = kShapes[L].cout, kDin = kShapes[L].din, kDout = kShapes[L].dout;
    static constexpr int kTY = L == 1 ? 4 : kDout, kTZ = L == 1 ? 2 : (L == 2 ? 1 : 4);  // positions of a tile
    static constexpr int kTiles = kDout / kTY * (kDout / kTZ);                           // tiles of an item
    static constexpr int kPos = kTZ * kTY * kDout;
    static constexpr int kIY = 2 * kTY + 1, kIZ = 2 * kTZ + 1;
    static constexpr int kRow = kDout * 2;  // bytes
    // planes of x: odd in 16-byte units (8-byte ones in the last layer, whose rows are 8 bytes)
    static constexpr int kPlane = L == 1 ? kIZ * kIY * kRow + 16 : kIZ * kIY * kRow;
    static_assert(L == 3 ? kPlane / 8 % 2 == 1 : kPlane / 16 % 2 == 1 && kPlane % 16 == 0, "bank spread");
    static constexpr int kDyRow = kPos * 2 + 16;
    static constexpr int kCT = kCout / 16;
    static constexpr int kPart = 28 * kCT * 256;  // floats of one workgroup's sums
    static constexpr int kSplits = L == 1 ? 512 : (L == 2 ? 128 : 32);
};

template <int L>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 2))) void k_conv_wgrad(
    const uint16_t *__restrict__ x, const float *__restrict__ dy, float *__restrict__ part, int64_t n_tiles)
{
    using G = WgradShape<L>;
    constexpr int DIN = G::kDin, DOUT = G::kDout;
    __shared__ __align__(16) uint8_t xs[48 * G::kPlane];
    __shared__ __align__(16) uint8_t ds[G::kCout * G::kDyRow];
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, n = lane & 15;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c0 = 16 * blockIdx.y;
    v4f32 acc[7][G::kCT];
#pragma unroll
    for (int j = 0; j < 7; ++j)
#pragma unroll
        for (int t = 0; t < G::kCT; ++t) acc[j][t] = (v4f32){0.f, 0.f, 0.f, 0.f};
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const int64_t item = tile / G::kTiles;
        const int q = (int)(tile % G::kTiles);
        const int oy0 = q % (DOUT / G::kTY) * G::kTY, oz0 = q / (DOUT / G::kTY) * G::kTZ;
        // x: eight channels of one voxel a lane, ix fastest
        constexpr int kX = G::kIZ * G::kIY * DIN * 2, kXPer = (kX + 255) / 256;
        v4u32 xv[kXPer];
#pragma unroll
        for (int b = 0; b < kXPer; ++b) {
            const int e = min(tid + 256 * b, kX - 1);
            const int ix = e % DIN, h = e / DIN & 1, r = e / (2 * DIN);
            const int iy = 2 * oy0 - 1 + r % G::kIY, iz = 2 * oz0 - 1 + r / G::kIY;
            const bool ok = iy >= 0 && iz >= 0;
            xv[b] = *(const v4u32 *)(x + (ok ? (((item * DIN + iz) * DIN + iy) * DIN + ix) * G::kCin + c0 + 8 * h : 0));
#pragma unroll
            for (int k = 0; k < 4; ++k) xv[b][k] = ok ? xv[b][k] : 0u;
        }
        // dy: four channels of one position a lane, channels fastest
        constexpr int kD = G::kPos * G::kCout / 4, kDPer = kD / 256;
        static_assert(kD % 256 == 0, "whole rounds");
        float4 dv[kDPer];
#pragma unroll
        for (int b = 0; b < kDPer; ++b) {
            const int e = tid + 256 * b, co = 4 * (e % (G::kCout / 4)), p = e / (G::kCout / 4);
            const int ox = p % DOUT, oy = oy0 + p / DOUT % G::kTY, oz = oz0 + p / (DOUT * G::kTY);
            dv[b] = *(const float4 *)(dy + (((item * DOUT + oz) * DOUT + oy) * DOUT + ox) * G::kCout + co);
        }
        __syncthreads();  // the operands of the last tile are read
#pragma unroll
        for (int b = 0; b < kXPer; ++b) {
            const int e = tid + 256 * b;
            if (e < kX) {
                const int ix = e % DIN, h = e / DIN & 1, r = e / (2 * DIN);
                uint8_t *p = xs + 8 * h * G::kPlane + r * G::kRow;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const uint16_t v = (uint16_t)(xv[b][k >> 1] >> (16 * (k & 1)));
                    uint8_t *pk = p + k * G::kPlane;
                    if (ix & 1) {
                        // tap 0 of the next position (the last voxel's slot holds what lies below the grid)
                        const bool last = ix == DIN - 1;
                        *(uint16_t *)(pk + (last ? 0 : ix + 1)) = last ? (uint16_t)0 : v;
                        *(uint16_t *)(pk + 32 * G::kPlane + ix - 1) = v;
                    } else {
                        *(uint16_t *)(pk + 16 * G::kPlane + ix) = v;
                    }
                }
            }
        }
#pragma unroll
        for (int b = 0; b < kDPer; ++b) {
            const int e = tid + 256 * b, co = 4 * (e % (G::kCout / 4)), p = e / (G::kCout / 4);
            const float v[4] = {dv[b].x, dv[b].y, dv[b].z, dv[b].w};
#pragma unroll
            for (int k = 0; k < 4; ++k) *(uint16_t *)(ds + (co + k) * G::kDyRow + 2 * p) = f2bf(v[k]);
        }
        __syncthreads();
#pragma unroll 1
        for (int s = 0; s < G::kPos / 32; ++s) {
            // this lane's eight positions: the first one's row and place in it
            const int p = 32 * s + 8 * g, ox = p % DOUT, oy = p / DOUT % G::kTY, oz = p / (DOUT * G::kTY);
            const uint8_t *xb = xs + n * G::kPlane + (2 * oz * G::kIY + 2 * oy) * G::kRow + 2 * ox;
            v4u32 a[G::kCT];
#pragma unroll
            for (int t = 0; t < G::kCT; ++t) a[t] = *(const v4u32 *)(ds + (16 * t + n) * G::kDyRow + 2 * p);
#pragma unroll
            for (int j = 0; j < 7; ++j) {
                const int tap = 7 * wid + j;  // 27: the bias column
                v4u32 b = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
                if (tap < 27) {  // uniform
                    const uint8_t *src = xb + 16 * (tap % 3) * G::kPlane + (tap / 9 * G::kIY + tap / 3 % 3) * G::kRow;
                    if constexpr (L == 3) {  // rows of four positions: the eight are two rows of y
                        const uint2 u = *(const uint2 *)src, v = *(const uint2 *)(src + 2 * G::kRow);
                        b = (v4u32){u.x, u.y, v.x, v.y};
                    } else {
                        b = *(const v4u32 *)src;
                    }
                }
#pragma unroll
                for (int t = 0; t < G::kCT; ++t) acc[j][t] = mfma32(a[t], b, acc[j][t]);
            }
        }
    }
    float *out = part + ((int64_t)blockIdx.x * gridDim.y + blockIdx.y) * G::kPart + wid * (7 * G::kCT * 256) + 4 * lane;
#pragma unroll
    for (int j = 0; j < 7; ++j)
#pragma unroll
        for (int t = 0; t < G::kCT; ++t) *(v4f32 *)(out + (j * G::kCT + t) * 256) = acc[j][t];
}

// First layer: positions of a tile, its sums ([column tile][lane][4], columns
// tap 4 + ci, then the bias) and the workgroups of a launch.
constexpr int kInTiles = 32, kInCols = 7, kInPart = kInCols * 256, kInSplits = 512;

constexpr int64_t kPartFloats =
    std::max({(int64_t)WgradShape<1>::kSplits * WgradShape<1>::kPart, (int64_t)WgradShape<2>::kSplits * 2 * WgradShape<2>::kPart,
              (int64_t)WgradShape<3>::kSplits * 4 * WgradShape<3>::kPart, (int64_t)kInSplits * kInPart});

// Adds the workgroups' sums (64 values a workgroup, its 16 waves every 16th
// split, then the waves in order) and puts each where the parameters have it.
template <int L>
__global__ __launch_bounds__(1024) void k_wgrad_sum(const float *__restrict__ part, int splits, float *__restrict__ gw,
                                                    float *__restrict__ gb)
{
    __shared__ float red[16][64];
    constexpr int CIN = kShapes[L].cin, K = 27 * CIN;
    constexpr int kLen = L == 0 ? kInPart : WgradShape<L == 0 ? 1 : L>::kPart * (CIN / 16);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int r = blockIdx.x * 64 + lane;
    float s = 0.f;
#pragma unroll 4
    for (int q = wid; q < splits; q += 16) s += part[(int64_t)q * kLen + r];
    red[wid][lane] = s;
    __syncthreads();
    if (wid) return;
    s = red[0][lane];
    for (int w = 1; w < 16; ++w) s += red[w][lane];
    const int i = r & 3, l = r >> 2 & 63, col = l & 15, row = 4 * (l >> 4) + i;
    if constexpr (L == 0) {
        const int kk = 16 * (r >> 8) + col;
        if (kk < K) gw[row * K + kk] = s;
        else if (kk == K) gb[row] = s;
    } else {
        using G = WgradShape<L>;
        const int cig = r / G::kPart, at = r % G::kPart >> 8, t = at % G::kCT, tap = at / G::kCT;
        const int co = 16 * t + row;
        if (tap < 27) gw[co * K + tap * CIN + 16 * cig + col] = s;
        else if (cig == 0 && col == 0) gb[co] = s;
    }
}

// Input gradient of a stride-2 layer, masked by the ReLU of the layer that
// produced x (x > 0): dx[q][ci] = sum over (tap, co) dy[o][co] w[co][tap][ci], o
// the output position that tap maps onto input position q.  Per axis an even q =
// 2 o has tap 1 of o alone, an odd q = 2 o + 1 has taps 0 of o + 1 and 2 of o: so
// the input positions of one parity class share their taps (1, 2, 4 or 8 of
// them), and the products are 16 positions o of the class x 16 channels ci, no
// tap wasted.  A workgroup stages its positions' dy and their upper neighbours
// as bf16 in LDS ([position][co], strides odd in 16-byte units) and takes 32
// input channels; its waves share the classes out by taps (8, 8, 8 and 3).
// Bound by latency and by writing dx.  Looking for each tile's taps position by
// position took 136 + 63 us for the two layers and 64 items; now 22 + 17.
template <int L>
struct DgradShape {
    static constexpr int kTZ = L == 2 ? 1 : 4;                    // z planes of a tile: 64 positions
    static constexpr int kTiles = kShapes[L].dout / kTZ;
    static_assert(kTZ * kShapes[L].dout * kShapes[L].dout == 64, "four MFMA tiles");
};

template <int L, int PZ, int PY, int PX>
__device__ __forceinline__ void dgrad_class(const uint8_t *ds, const uint16_t *__restrict__ wt,
                                            const uint16_t *__restrict__ x, float *__restrict__ dx, int64_t item, int oz0)
{
    constexpr int CIN = kShapes[L].cin, COUT = kShapes[L].cout, DIN = kShapes[L].din, DOUT = kShapes[L].dout;
    constexpr int NCH = COUT / 32, H = DOUT + 1, kStride = 2 * COUT + 16;
    const int lane = threadIdx.x & 63, g = lane >> 4, n = lane & 15;
    const int t0 = 2 * blockIdx.y;
    int at[4];  // the lane's position of each MFMA tile
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const int p = 16 * m + n;
        at[m] = ((p / (DOUT * DOUT)) * H + p / DOUT % DOUT) * H + p % DOUT;
    }
    v4f32 acc[4][2];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[m][t] = (v4f32){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < (1 << (PZ + PY + PX)); ++k) {
        // the bits of k go to the odd axes: set, tap 2 of o; clear, tap 0 of o + 1
        const int bz = PZ ? k & 1 : 0, by = PY ? k >> PZ & 1 : 0, bx = PX ? k >> (PZ + PY) & 1 : 0;
        const int tap = (PZ ? 2 * bz : 1) * 9 + (PY ? 2 * by : 1) * 3 + (PX ? 2 * bx : 1);
        const int shift = ((PZ & !bz) * H + (PY & !by)) * H + (PX & !bx);
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            v4u32 w[2];
#pragma unroll
            for (int t = 0; t < 2; ++t)
                w[t] = *(const v4u32 *)(wt + (((tap * NCH + c) * (CIN / 16) + t0 + t) * 64 + lane) * 8);
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const v4u32 v = *(const v4u32 *)(ds + (at[m] + shift) * kStride + 64 * c + 16 * g);
#pragma unroll
                for (int t = 0; t < 2; ++t) acc[m][t] = mfma32(w[t], v, acc[m][t]);
            }
        }
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const int p = 16 * m + n;
        const int iz = 2 * (oz0 + p / (DOUT * DOUT)) + PZ, iy = 2 * (p / DOUT % DOUT) + PY, ix = 2 * (p % DOUT) + PX;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int64_t id = (((item * DIN + iz) * DIN + iy) * DIN + ix) * CIN + 16 * (t0 + t) + 4 * g;
            const uint2 xm = *(const uint2 *)(x + id);
            float4 o;
            o.x = (int16_t)xm.x > 0 ? acc[m][t][0] : 0.f;
            o.y = (int32_t)xm.x >> 16 > 0 ? acc[m][t][1] : 0.f;
            o.z = (int16_t)xm.y > 0 ? acc[m][t][2] : 0.f;
            o.w = (int32_t)xm.y >> 16 > 0 ? acc[m][t][3] : 0.f;
            *(float4 *)(dx + id) = o;
        }
    }
}

template <int L>
__global__ __launch_bounds__(256) void k_conv_dgrad(const uint16_t *__restrict__ x, const float *__restrict__ dy,
                                                    const uint16_t *__restrict__ wt, float *__restrict__ dx)
{
    constexpr int COUT = kShapes[L].cout, DOUT = kShapes[L].dout, TZ = DgradShape<L>::kTZ;
    constexpr int H = DOUT + 1, kHalo = (TZ + 1) * H * H, kStride = 2 * COUT + 16;
    __shared__ __align__(16) uint8_t ds[kHalo * kStride];
    const int tid = threadIdx.x;
    const int64_t item = blockIdx.x / DgradShape<L>::kTiles;
    const int oz0 = (int)(blockIdx.x % DgradShape<L>::kTiles) * TZ;
    constexpr int kD = kHalo * COUT / 4, kPer = (kD + 255) / 256;
    float4 v[kPer];
#pragma unroll
    for (int b = 0; b < kPer; ++b) {
        const int e = min(tid + 256 * b, kD - 1), co = 4 * (e % (COUT / 4)), p = e / (COUT / 4);
        const int ox = p % H, oy = p / H % H, oz = oz0 + p / (H * H);
        const bool ok = ox < DOUT && oy < DOUT && oz < DOUT;
        v[b] = *(const float4 *)(dy + (ok ? (((item * DOUT + oz) * DOUT + oy) * DOUT + ox) * COUT + co : 0));
        if (!ok) v[b] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int b = 0; b < kPer; ++b) {
        const int e = tid + 256 * b;
        if (e < kD)
            *(uint2 *)(ds + e / (COUT / 4) * kStride + 8 * (e % (COUT / 4))) =
                make_uint2(pack_bf16(v[b].x, v[b].y), pack_bf16(v[b].z, v[b].w));
    }
    __syncthreads();
    switch (__builtin_amdgcn_readfirstlane(tid >> 6)) {
    case 0:
        dgrad_class<L, 1, 1, 1>(ds, wt, x, dx, item, oz0);
        break;
    case 1:
        dgrad_class<L, 1, 1, 0>(ds, wt, x, dx, item, oz0);
        dgrad_class<L, 1, 0, 1>(ds, wt, x, dx, item, oz0);
        break;
    case 2:
        dgrad_class<L, 0, 1, 1>(ds, wt, x, dx, item, oz0);
        dgrad_class<L, 1, 0, 0>(ds, wt, x, dx, item, oz0);
        dgrad_class<L, 0, 1, 0>(ds, wt, x, dx, item, oz0);
        break;
    default:
        dgrad_class<L, 0, 0, 1>(ds, wt, x, dx, item, oz0);
        dgrad_class<L, 0, 0, 0>(ds, wt, x, dx, item, oz0);
        break;
    }
}

// Input gradient of the second layer and weight gradients of the first in one
// kernel: the gradient of the first layer's output (134 MB for 64 items) has no
// other reader, so it goes to LDS, rounded to bf16 as the weight gradients take
// it, and never to memory.  A workgroup takes 16 x 4 x 2 positions of the second
// layer, that is 32 x 8 x 4 of the first: each wave makes the eight parity
// classes of two rows of 16 (27 taps in registers, dy from memory), masks them by
// the first layer's ReLU, and then sums eight rows of 32 positions over 7 column
// tiles (tap 4 + ci, the bias at 108).  x is staged transposed as in k_conv_wgrad
// with a copy for each kw.  Bound by reading the first layer's output and dy and
// by the LDS writes; the three separate steps (dx 324, gathered weight gradients
// 405, the bf16 input 16 us for 64 items) became 92.
constexpr int kInPlane = 6 * 10 * 64 + 16, kInDsRow = 1024 * 2 + 16;

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_bwd_in(
    const float *__restrict__ x, const uint16_t *__restrict__ a0, const float *__restrict__ d1,
    const uint16_t *__restrict__ wt, float *__restrict__ part, int64_t n_tiles)
{
    __shared__ __align__(16) uint8_t lds[12 * kInPlane + 16 * kInDsRow];
    uint8_t *xs = lds, *ds = lds + 12 * kInPlane;  // [kw][ci][z][y][ox], [co][position]
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, g = lane >> 4, n = lane & 15;
    v4u32 wf[27];
#pragma unroll
    for (int k = 0; k < 27; ++k) wf[k] = *(const v4u32 *)(wt + (k * 64 + lane) * 8);
    int boff[kInCols];  // column 16 t + n: where its first position lies in xs
#pragma unroll
    for (int t = 0; t < kInCols; ++t) {
        const int kk = min(16 * t + n, 107), tap = kk >> 2, ci = kk & 3;
        boff[t] = (4 * (tap % 3) + ci) * kInPlane + (tap / 9 * 10 + tap / 3 % 3) * 64 + 16 * g;
    }
    v4f32 acc[kInCols];
#pragma unroll
    for (int t = 0; t < kInCols; ++t) acc[t] = (v4f32){0.f, 0.f, 0.f, 0.f};
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const int64_t item = tile / kInTiles;
        const int oy0 = (int)(tile % 4) * 4, oz0 = (int)(tile / 4 % 8) * 2;
        __syncthreads();  // the operands of the last tile are read
        // x: the four channels of one voxel a lane
        float xv[8][4];
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const int e = min(tid + 256 * b, 1919), ix = e & 31, iy = 2 * oy0 - 1 + e / 32 % 10, iz = 2 * oz0 - 1 + e / 320;
            const bool ok = iy >= 0 && iz >= 0 && iy < 32 && iz < 32;
            __builtin_memcpy(xv[b], x + (ok ? 4 * (((item * 32 + iz) * 32 + iy) * 32 + ix) : 0), 16);
#pragma unroll
            for (int k = 0; k < 4; ++k) xv[b][k] = ok ? xv[b][k] : 0.0f;
        }
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const int e = tid + 256 * b, ix = e & 31;
            if (e < 1920) {
                uint8_t *p = xs + (e >> 5) * 64;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint16_t v = f2bf(xv[b][k]);
                    uint8_t *pk = p + k * kInPlane;
                    // voxel ix is tap kw of position ix + 1 - kw; the ends' free slots are outside the grid
                    *(uint16_t *)(pk + (ix == 31 ? 0 : 2 * ix + 2)) = ix == 31 ? (uint16_t)0 : v;
                    *(uint16_t *)(pk + 4 * kInPlane + 2 * ix) = v;
                    *(uint16_t *)(pk + 8 * kInPlane + (ix == 0 ? 62 : 2 * ix - 2)) = ix == 0 ? (uint16_t)0 : v;
                }
            }
        }
#pragma unroll 1
        for (int m = 0; m < 2; ++m) {
            const int row = 2 * wid + m, oyl = row & 3, ozl = row >> 2, oy = oy0 + oyl, oz = oz0 + ozl;
            // dy of the row's positions and their upper neighbours (shift 4 z + 2 y + x)
            v4u32 f[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                if (s == 4) __builtin_amdgcn_sched_barrier(0);
                const int z = oz + (s >> 2), yy = oy + (s >> 1 & 1), xx = n + (s & 1);
                const bool ok = z < 16 && yy < 16 && xx < 16;
                const float *src = d1 + (ok ? (((item * 16 + z) * 16 + yy) * 16 + xx) * 32 + 8 * g : 0);
                const float4 u = *(const float4 *)src, v = *(const float4 *)(src + 4);
                f[s] = (v4u32){pack_bf16(u.x, u.y), pack_bf16(u.z, u.w), pack_bf16(v.x, v.y), pack_bf16(v.z, v.w)};
#pragma unroll
                for (int k = 0; k < 4; ++k) f[s][k] = ok ? f[s][k] : 0u;
            }
            __builtin_amdgcn_sched_barrier(0);  // the raw reads give their registers back
            uint2 mask[8];
#pragma unroll
            for (int c = 0; c < 8; ++c)
                mask[c] = *(const uint2 *)(a0 + (((item * 32 + 2 * oz + (c >> 2)) * 32 + 2 * oy + (c >> 1 & 1)) * 32 +
                                                 2 * n + (c & 1)) * 16 + 4 * g);
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int pz = c >> 2, py = c >> 1 & 1, px = c & 1;
                v4f32 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < (1 << (pz + py + px)); ++k) {
                    const int bz = pz ? k & 1 : 0, by = py ? k >> pz & 1 : 0, bx = px ? k >> (pz + py) & 1 : 0;
                    const int tap = (pz ? 2 * bz : 1) * 9 + (py ? 2 * by : 1) * 3 + (px ? 2 * bx : 1);
                    d = mfma32(wf[tap], f[4 * (pz & !bz) + 2 * (py & !by) + (px & !bx)], d);
                }
                const bool on[4] = {(int16_t)mask[c].x > 0, (int32_t)mask[c].x >> 16 > 0, (int16_t)mask[c].y > 0,
                                    (int32_t)mask[c].y >> 16 > 0};
                uint8_t *p = ds + 4 * g * kInDsRow + 2 * (((2 * ozl + pz) * 8 + 2 * oyl + py) * 32 + 2 * n + px);
#pragma unroll
                for (int i = 0; i < 4; ++i) *(uint16_t *)(p + i * kInDsRow) = on[i] ? f2bf(d[i]) : (uint16_t)0;
            }
        }
        __syncthreads();
#pragma unroll 2
        for (int q = 0; q < 8; ++q) {
            const int r = 8 * wid + q;  // row (z = r / 8, y = r % 8)
            const v4u32 a = *(const v4u32 *)(ds + n * kInDsRow + 64 * r + 16 * g);
            const uint8_t *xb = xs + ((r >> 3) * 10 + (r & 7)) * 64;
#pragma unroll
            for (int t = 0; t < kInCols; ++t) {
                v4u32 b = *(const v4u32 *)(xb + boff[t]);
                if (t == kInCols - 1) {  // columns 96..107, then the ones of the bias
                    const uint32_t one = n == 12 ? 0x3F803F80u : 0u;
#pragma unroll
                    for (int k = 0; k < 4; ++k) b[k] = n < 12 ? b[k] : one;
                }
                acc[t] = mfma32(a, b, acc[t]);
            }
        }
    }
    // the four waves' sums, in order
    __syncthreads();
    float *red = (float *)lds;
#pragma unroll
    for (int t = 0; t < kInCols; ++t) *(v4f32 *)(red + wid * kInPart + t * 256 + 4 * lane) = acc[t];
    __syncthreads();
    for (int e = tid; e < kInPart; e += 256)
        part[(int64_t)blockIdx.x * kInPart + e] = ((red[e] + red[kInPart + e]) + red[2 * kInPart + e]) + red[3 * kInPart + e];
}

// Adam (Kingma and Ba, 2015) on the FP32 master weights; refreshes the bf16
// copies of the convolution weights.
__global__ void k_adam(float *__restrict__ w, const float *__restrict__ g, float *__restrict__ m, float *__restrict__ v,
                       int64_t n, float lr, float b1, float b2, float eps, float c1, float c2)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// The bf16 copies of a convolution's weights: wb as the masters lie, and wt (from
// the second layer on) in the operand order of the input gradient: [tap][32
// output channels][16 input channels][lane], eight output channels a lane.
template <int CIN, int COUT>
__global__ void k_refresh_bf16(const float *__restrict__ w, uint16_t *__restrict__ wb, uint16_t *__restrict__ wt)
{
    constexpr int K = 27 * CIN;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= COUT * K) return;
    const uint16_t v = f2bf(w[i]);
    wb[i] = v;
    if constexpr (CIN >= 16) {
        const int co = i / K, tap = i % K / CIN, ci = i % K % CIN;
        wt[(((tap * (COUT / 32) + co / 32) * (CIN / 16) + ci / 16) * 64 + co % 32 / 8 * 16 + ci % 16) * 8 + co % 8] = v;
    }
}

unsigned blocks_for(int64_t n, int t) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + t - 1) / t, 1 << 20)); }

}  // namespace

// Parameter layout (FP32 master, in order): for each convolution w[cout][27
// cin], b[cout]; then fc w[5][64], b[5].
struct NetParams {
    int64_t off_w[kLayers], off_b[kLayers], off_fcw, off_fcb, total;
    NetParams()
    {
        int64_t o = 0;
        for (int l = 0; l < kLayers; ++l) {
            off_w[l] = o;
            o += (int64_t)kShapes[l].cout * kShapes[l].K();
            off_b[l] = o;
            o += kShapes[l].cout;
        }
        off_fcw = o;
        o += kOut * kFeat;
        off_fcb = o;
        o += kOut;
        total = o;
    }
};

}  // namespace covox

struct covox_net {
    covox_ctx *ctx = nullptr;
    covox::NetParams P;
    float *w = nullptr, *g = nullptr, *m = nullptr, *v = nullptr;  // FP32 master, grad, Adam moments
    uint16_t *wb[covox::kLayers] = {nullptr, nullptr, nullptr, nullptr};
    uint16_t *wt[covox::kLayers] = {nullptr, nullptr, nullptr, nullptr};
    int64_t step = 0;
    // activations for the current batch capacity
    int batch_cap = 0;
    uint16_t *a[covox::kLayers] = {nullptr, nullptr, nullptr, nullptr};
    float *pooled = nullptr, *out = nullptr, *dout = nullptr, *loss = nullptr;
    // training: gradients of the layer outputs (the first layer's stays on chip),
    // for d_cap items, and the weight gradients' partial sums
    int d_cap = 0;
    float *d[covox::kLayers] = {nullptr, nullptr, nullptr, nullptr};
    float *part = nullptr;
};

namespace covox {

static int64_t act_elems(int l, int n)
{
    const ConvShape &s = kShapes[l];
    return (int64_t)n * s.dout * s.dout * s.dout * s.cout;
}

static int net_reserve(covox_net *net, int n)
{
    if (n <= net->batch_cap) return COVOX_OK;
    covox_ctx *ctx = net->ctx;
    int rc = hip_check(ctx, hipStreamSynchronize(ctx->stream), "net reserve sync");  // readers of the old buffers
    if (rc) return rc;
    auto fr = [](void *p) { if (p) (void)hipFree(p); };
    for (float **p : {&net->pooled, &net->out, &net->dout, &net->loss}) { fr(*p); *p = nullptr; }
    for (int l = 0; l < kLayers; ++l) { fr(net->a[l]); net->a[l] = nullptr; }
    hipError_t e = hipSuccess;
    for (int l = 0; l < kLayers && e == hipSuccess; ++l)
        e = hipMalloc((void **)&net->a[l], sizeof(uint16_t) * act_elems(l, n));
    if (e == hipSuccess) e = hipMalloc((void **)&net->pooled, sizeof(float) * n * kFeat);
    if (e == hipSuccess) e = hipMalloc((void **)&net->out, sizeof(float) * n * kOut);
    if (e == hipSuccess) e = hipMalloc((void **)&net->dout, sizeof(float) * n * kOut);
    if (e == hipSuccess) e = hipMalloc((void **)&net->loss, sizeof(float));
    if (e != hipSuccess) {
        net->batch_cap = 0;
        return fail(ctx, COVOX_EHIP, std::string("net buffers: ") + hipGetErrorString(e));
    }
    net->batch_cap = n;
    return COVOX_OK;
}

// Buffers of a training step of n items.
static int net_reserve_train(covox_net *net, int n)
{
    if (n <= net->d_cap && net->part) return COVOX_OK;
    covox_ctx *ctx = net->ctx;
    int rc = hip_check(ctx, hipStreamSynchronize(ctx->stream), "net reserve sync");
    if (rc) return rc;
    hipError_t e = hipSuccess;
    for (int l = 1; l < kLayers; ++l) {
        if (net->d[l]) (void)hipFree(net->d[l]);
        net->d[l] = nullptr;
        if (e == hipSuccess) e = hipMalloc((void **)&net->d[l], sizeof(float) * act_elems(l, n));
    }
    if (e == hipSuccess && !net->part) e = hipMalloc((void **)&net->part, sizeof(float) * kPartFloats);
    if (e != hipSuccess) {
        net->d_cap = 0;
        return fail(ctx, COVOX_EHIP, std::string("net training buffers: ") + hipGetErrorString(e));
    }
    net->d_cap = n;
    return COVOX_OK;
}

template <int L>
static void launch_conv_fwd(covox_net *net, const uint16_t *x, uint16_t *y, int n)
{
    constexpr ConvShape s = kShapes[L];
    // Channels of a workgroup: all, but half of the last layer's (its weights
    // are 221 KB); waves of a workgroup: enough to fill the CU beside the LDS
    // that the weights take; grid: what the chip holds at once.
    constexpr int CT = L == 1 ? 2 : (L == 2 ? 4 : 2), NT = L == 2 ? 512 : (L == 3 ? 128 : 256), kPerCu = L == 1 ? 4 : 1;
    const int64_t tiles = (int64_t)n * s.dout * s.dout * s.dout / 16;
    const unsigned gy = s.cout / (16 * CT);
    const unsigned gx = (unsigned)std::min<int64_t>((tiles + NT / 64 - 1) / (NT / 64), 256 * kPerCu / gy);
    hipLaunchKernelGGL((k_conv_fwd<s.cin, s.cout, s.din, s.dout, CT, NT>), dim3(gx, gy), dim3(NT), 0,
                       net->ctx->stream, x, net->wb[L], net->w + net->P.off_b[L], y, tiles);
}

// Buffers of one forward pass: the four bf16 layer outputs, the pooled features
// and the network outputs.
struct FwdBuffers {
    uint16_t *a[kLayers];
    float *pooled, *out;
};

// The forward pass's launches on the context stream, into the given buffers
// (every element of each buffer is written before it is read).
static void forward_launches(covox_net *net, const float *x_dev, int n, const FwdBuffers &b)
{
    covox_ctx *ctx = net->ctx;
    hipLaunchKernelGGL(k_conv_in, dim3((unsigned)n * (32 / kInTY) * (32 / kInTZ)), dim3(256), 0, ctx->stream, x_dev,
                       net->wb[0], net->w + net->P.off_b[0], b.a[0]);
    launch_conv_fwd<1>(net, b.a[0], b.a[1], n);
    launch_conv_fwd<2>(net, b.a[1], b.a[2], n);
    launch_conv_fwd<3>(net, b.a[2], b.a[3], n);
    hipLaunchKernelGGL(k_pool_fc, dim3(n), dim3(64), 0, ctx->stream, b.a[3], net->w + net->P.off_fcw,
                       net->w + net->P.off_fcb, b.pooled, b.out, n);
}

// out: n x 5, or null for the network's own buffer (which net_reserve may move).
static int net_forward(covox_net *net, const float *x_dev, int n, float *out)
{
    covox_ctx *ctx = net->ctx;
    int rc = net_reserve(net, n);
    if (rc) return rc;
    {
        TimedLaunch tl(ctx, COVOX_K_NET);
        forward_launches(net, x_dev, n, FwdBuffers{{net->a[0], net->a[1], net->a[2], net->a[3]}, net->pooled, out ? out : net->out});
    }
    return hip_check(ctx, hipGetLastError(), "net forward");
}

// Weight and bias gradients of a stride-2 layer.
template <int L>
static void launch_wgrad(covox_net *net, const uint16_t *x, int n)
{
    using G = WgradShape<L>;
    constexpr ConvShape s = kShapes[L];
    hipStream_t st = net->ctx->stream;
    const int64_t tiles = (int64_t)n * G::kTiles;
    const int splits = (int)std::min<int64_t>(tiles, G::kSplits);
    hipLaunchKernelGGL(k_conv_wgrad<L>, dim3(splits, s.cin / 16), dim3(256), 0, st, x, net->d[L], net->part, tiles);
    hipLaunchKernelGGL(k_wgrad_sum<L>, dim3(G::kPart * (s.cin / 16) / 64), dim3(1024), 0, st, net->part, splits,
                       net->g + net->P.off_w[L], net->g + net->P.off_b[L]);
}

template <int L>
static void launch_dgrad(covox_net *net, const uint16_t *x, int n)
{
    constexpr ConvShape s = kShapes[L];
    hipLaunchKernelGGL(k_conv_dgrad<L>, dim3((unsigned)n * DgradShape<L>::kTiles, s.cin / 32), dim3(256), 0,
                       net->ctx->stream, x, net->d[L], net->wt[L], net->d[L - 1]);
}

static int net_backward(covox_net *net, const float *x_dev, int n)
{
    covox_ctx *ctx = net->ctx;
    hipLaunchKernelGGL(k_fc_bwd, dim3(n + kOut), dim3(64), 0, ctx->stream, net->dout, net->pooled,
                       net->w + net->P.off_fcw, net->a[3], net->g + net->P.off_fcw, net->g + net->P.off_fcb, net->d[3],
                       n);
    launch_wgrad<3>(net, net->a[2], n);
    launch_dgrad<3>(net, net->a[2], n);
    launch_wgrad<2>(net, net->a[1], n);
    launch_dgrad<2>(net, net->a[1], n);
    launch_wgrad<1>(net, net->a[0], n);
    const int64_t tiles = (int64_t)n * kInTiles;
    const int splits = (int)std::min<int64_t>(tiles, kInSplits);
    hipLaunchKernelGGL(k_bwd_in, dim3(splits), dim3(256), 0, ctx->stream, x_dev, net->a[0], net->d[1], net->wt[1],
                       net->part, tiles);
    hipLaunchKernelGGL(k_wgrad_sum<0>, dim3(kInPart / 64), dim3(1024), 0, ctx->stream, net->part, splits,
                       net->g + net->P.off_w[0], net->g + net->P.off_b[0]);
    return hip_check(ctx, hipGetLastError(), "net backward");
}

template <int L>
static void refresh_layer(covox_net *net)
{
    constexpr ConvShape s = kShapes[L];
    hipLaunchKernelGGL((k_refresh_bf16<s.cin, s.cout>), dim3(blocks_for((int64_t)s.cout * s.K(), 256)), dim3(256), 0,
                       net->ctx->stream, net->w + net->P.off_w[L], net->wb[L], net->wt[L]);
}

static void refresh_bf16(covox_net *net)
{
    refresh_layer<0>(net);
    refresh_layer<1>(net);
    refresh_layer<2>(net);
    refresh_layer<3>(net);
}

int net_forward_api(covox_net *net, const float *x_dev, int n, float *out_dev)
{
    return net_forward(net, x_dev, n, out_dev);
}

const float *net_loss_dev(const covox_net *net) { return net->loss; }

// ------------------------------------------------- forward without allocation
//
// Activations of at most COVOX_NET_NOALLOC_MAX_PAIRS pairs in a file-scope
// device array.  Its address on each device comes from hipGetSymbolAddress,
// taken once per device when a context is created there; host code never
// uses the array's name as a device address.

constexpr int64_t noalloc_act(int l)
{
    return (int64_t)COVOX_NET_NOALLOC_MAX_PAIRS * kShapes[l].dout * kShapes[l].dout * kShapes[l].dout *
           kShapes[l].cout;
}
constexpr int64_t kNoAllocBytes =
    2 * (noalloc_act(0) + noalloc_act(1) + noalloc_act(2) + noalloc_act(3)) +
    4 * (int64_t)COVOX_NET_NOALLOC_MAX_PAIRS * kFeat;
static_assert(kNoAllocBytes % 256 == 0, "scratch regions stay 256-byte aligned");

}  // namespace covox

static __device__ __align__(256) unsigned char scratch[covox::kNoAllocBytes];

namespace covox {

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

int noalloc_scratch_init(covox_ctx *ctx)
{
    const int dev = ctx->device;
    if (dev < 0 || dev >= kMaxDevices) return fail(ctx, COVOX_EHIP, "no-alloc scratch: device index out of range");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_ptr[dev]) return COVOX_OK;
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e == hipSuccess && cur != dev) e = hipSetDevice(dev);
    void *ptr = nullptr;
    if (e == hipSuccess) e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (cur >= 0 && cur != dev) (void)hipSetDevice(cur);
    if (e != hipSuccess || !ptr)
        return fail(ctx, COVOX_EHIP, std::string("no-alloc scratch address: ") + hipGetErrorString(e));
    g_scratch_ptr[dev] = ptr;
    return COVOX_OK;
}

int net_forward_noalloc(covox_net *net, const float *x_dev, int n, float *out_dev)
{
    covox_ctx *ctx = net->ctx;
    if (n > COVOX_NET_NOALLOC_MAX_PAIRS)
        return fail(ctx, COVOX_EINVAL, "net_forward_noalloc: more than COVOX_NET_NOALLOC_MAX_PAIRS pairs");
    unsigned char *base = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        if (ctx->device >= 0 && ctx->device < kMaxDevices) base = (unsigned char *)g_scratch_ptr[ctx->device];
    }
    if (!base) return fail(ctx, COVOX_EHIP, "net_forward_noalloc: scratch address not set up on this device");
    // Regions sized for the maximum batch; n pairs use the front of each.
    FwdBuffers b;
    for (int l = 0; l < kLayers; ++l) {
        b.a[l] = (uint16_t *)base;
        base += 2 * noalloc_act(l);
    }
    b.pooled = (float *)base;
    b.out = out_dev;
    forward_launches(net, x_dev, n, b);
    return hip_check(ctx, hipGetLastError(), "net forward (no allocation)");
}

int net_train_step(covox_net *net, const float *x_dev, const float *y_dev, int n, float lr, float trans_scale,
                   float *loss_host)
{
    int rc = net_train_async(net, x_dev, y_dev, n, lr, trans_scale);
    if (rc) return rc;
    if (loss_host) {
        covox_ctx *ctx = net->ctx;
        if ((rc = hip_check(ctx, hipMemcpyAsync(loss_host, net->loss, sizeof(float), hipMemcpyDeviceToHost, ctx->stream),
                            "loss copy")))
            return rc;
        return hip_check(ctx, hipStreamSynchronize(ctx->stream), "train sync");
    }
    return COVOX_OK;
}

int net_train_async(covox_net *net, const float *x_dev, const float *y_dev, int n, float lr, float trans_scale)
{
    covox_ctx *ctx = net->ctx;
    int rc = net_reserve_train(net, n);
    if (!rc) rc = net_forward(net, x_dev, n, nullptr);
    if (rc) return rc;
    hipLaunchKernelGGL(k_loss, dim3(1), dim3(256), 0, ctx->stream, net->out, y_dev, net->dout, net->loss, n,
                       1.0f / (trans_scale * trans_scale));
    {
        TimedLaunch tl(ctx, COVOX_K_NET);
        if ((rc = net_backward(net, x_dev, n))) return rc;
    }
    net->step += 1;
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = 1.f - powf(b1, (float)net->step), c2 = 1.f - powf(b2, (float)net->step);
    hipLaunchKernelGGL(k_adam, dim3(blocks_for(net->P.total, 256)), dim3(256), 0, ctx->stream, net->w, net->g, net->m,
                       net->v, net->P.total, lr, b1, b2, 1e-8f, c1, c2);
    refresh_bf16(net);
    return hip_check(ctx, hipGetLastError(), "net train step");
}

int net_grads(covox_net *net, const float *x_dev, const float *y_dev, int n, float trans_scale, float *grad_host,
              float *loss_host)
{
    covox_ctx *ctx = net->ctx;
    int rc = net_reserve_train(net, n);
    if (!rc) rc = net_forward(net, x_dev, n, nullptr);
    if (rc) return rc;
    hipLaunchKernelGGL(k_loss, dim3(1), dim3(256), 0, ctx->stream, net->out, y_dev, net->dout, net->loss, n,
                       1.0f / (trans_scale * trans_scale));
    if ((rc = net_backward(net, x_dev, n))) return rc;
    if ((rc = hip_check(ctx, hipMemcpyAsync(grad_host, net->g, sizeof(float) * net->P.total, hipMemcpyDeviceToHost,
                                            ctx->stream), "grad copy")))
        return rc;
    if (loss_host &&
        (rc = hip_check(ctx, hipMemcpyAsync(loss_host, net->loss, sizeof(float), hipMemcpyDeviceToHost, ctx->stream),
                        "loss copy")))
        return rc;
    return hip_check(ctx, hipStreamSynchronize(ctx->stream), "grad sync");
}

int net_create(covox_ctx *ctx, uint64_t seed, covox_net **out)
{
    covox_net *net = new covox_net();
    net->ctx = ctx;
    const int64_t np = net->P.total;
    hipError_t e = hipSuccess;
    for (float **p : {&net->w, &net->g, &net->m, &net->v})
        if (e == hipSuccess) e = hipMalloc((void **)p, sizeof(float) * np);
    for (int l = 0; l < kLayers && e == hipSuccess; ++l)
        for (uint16_t **p : {&net->wb[l], &net->wt[l]})
            if (e == hipSuccess) e = hipMalloc((void **)p, sizeof(uint16_t) * (int64_t)kShapes[l].cout * kShapes[l].K());
    if (e != hipSuccess) {
        net_destroy(net);
        return fail(ctx, COVOX_EHIP, std::string("net_create: ") + hipGetErrorString(e));
    }
    // He-uniform initialisation from SplitMix64 (zero biases)
    std::vector<float> h(np, 0.f);
    uint64_t state = seed;
    auto uni = [&]() {
        state += 0x9e3779b97f4a7c15ull;
        return (double)(mix64(state) >> 11) * (1.0 / 9007199254740992.0);
    };
    for (int l = 0; l < kLayers; ++l) {
        const double lim = sqrt(6.0 / (double)kShapes[l].K());
        for (int64_t i = 0; i < (int64_t)kShapes[l].cout * kShapes[l].K(); ++i)
            h[net->P.off_w[l] + i] = (float)((2.0 * uni() - 1.0) * lim);
    }
    const double lim = sqrt(6.0 / (double)kFeat);
    for (int i = 0; i < kOut * kFeat; ++i) h[net->P.off_fcw + i] = (float)((2.0 * uni() - 1.0) * lim) * 0.1f;
    std::vector<float> zeros(np, 0.f);
    e = hipMemcpy(net->w, h.data(), sizeof(float) * np, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(net->m, zeros.data(), sizeof(float) * np, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(net->v, zeros.data(), sizeof(float) * np, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        net_destroy(net);
        return fail(ctx, COVOX_EHIP, std::string("net_create upload: ") + hipGetErrorString(e));
    }
    refresh_bf16(net);
    int rc = hip_check(ctx, hipGetLastError(), "net init");
    if (rc) {
        net_destroy(net);
        return rc;
    }
    ctx->nets.push_back(net);
    *out = net;
    return COVOX_OK;
}

static void net_free_device(covox_net *net)
{
    for (float **p : {&net->w, &net->g, &net->m, &net->v, &net->pooled, &net->out, &net->dout, &net->loss, &net->part}) {
        if (*p) (void)hipFree(*p);
        *p = nullptr;
    }
    for (int l = 0; l < kLayers; ++l) {
        for (void **p : {(void **)&net->wb[l], (void **)&net->wt[l], (void **)&net->a[l], (void **)&net->d[l]}) {
            if (*p) (void)hipFree(*p);
            *p = nullptr;
        }
    }
    net->batch_cap = net->d_cap = 0;
}

void net_detach(covox_net *net)
{
    if (!net) return;
    net_free_device(net);
    net->ctx = nullptr;
}

void net_destroy(covox_net *net)
{
    if (!net) return;
    if (covox_ctx *ctx = net->ctx) {
        (void)hipStreamSynchronize(ctx->stream);
        ctx->nets.erase(std::remove(ctx->nets.begin(), ctx->nets.end(), net), ctx->nets.end());
    }
    net_free_device(net);
    delete net;
}

int64_t net_num_params(const covox_net *net) { return net->P.total; }

covox_ctx *net_ctx(const covox_net *net) { return net->ctx; }

int net_get_params(covox_net *net, float *host, int64_t n)
{
    if (n != net->P.total) return fail(net->ctx, COVOX_EINVAL, "net params: wrong count");
    int rc = hip_check(net->ctx, hipStreamSynchronize(net->ctx->stream), "params sync");  // pending training steps
    if (rc) return rc;
    return hip_check(net->ctx, hipMemcpy(host, net->w, sizeof(float) * n, hipMemcpyDeviceToHost), "params copy");
}

int net_set_params(covox_net *net, const float *host, int64_t n)
{
    if (n != net->P.total) return fail(net->ctx, COVOX_EINVAL, "net params: wrong count");
    int rc = hip_check(net->ctx, hipStreamSynchronize(net->ctx->stream), "params sync");  // readers in flight
    if (rc) return rc;
    rc = hip_check(net->ctx, hipMemcpy(net->w, host, sizeof(float) * n, hipMemcpyHostToDevice), "params upload");
    if (rc) return rc;
    refresh_bf16(net);
    return hip_check(net->ctx, hipStreamSynchronize(net->ctx->stream), "params sync");
}

}  // namespace covox
