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
// even).  FP32 master weights; the backward pass and Adam run in FP32.
#include "covox_impl.h"

#include <math.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <vector>

namespace covox {

namespace {

typedef short v4i16 __attribute__((ext_vector_type(4)));
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

__global__ void k_to_bf16(const float *__restrict__ x, uint16_t *__restrict__ y, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        y[i] = f2bf(x[i]);
}

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

// ------------------------------------------------------------ backward (FP32)

// Loss: sum over the batch of (|t - t*|^2 / s_t^2 + |(c, s) - (c*, s*)|^2),
// divided by n.  d_out = its gradient.
__global__ void k_loss(const float *__restrict__ out, const float *__restrict__ y, float *__restrict__ dout,
                       float *__restrict__ loss, int n, float inv_st2)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * kOut) return;
    const int k = i % kOut;
    const float wgt = k < 3 ? inv_st2 : 1.0f;
    const float d = out[i] - y[i];
    dout[i] = 2.0f * wgt * d / (float)n;
    atomicAdd(loss, wgt * d * d / (float)n);
}

// FC backward: gradients of the head, then d a4 = (d pooled / 64) masked by
// ReLU (a4 > 0).  Workgroup n (64 threads) sums the head's gradients over the
// batch; workgroup b < n writes d a4 of item b.
__global__ void k_fc_bwd(const float *__restrict__ dout, const float *__restrict__ pooled,
                         const float *__restrict__ wfc, const uint16_t *__restrict__ a4, float *__restrict__ gwfc,
                         float *__restrict__ gbfc, float *__restrict__ da4, int n)
{
    const int t = threadIdx.x, b = blockIdx.x;
    if (b == n) {
        // weight and bias gradients (each thread one feature column)
        for (int o = 0; o < kOut; ++o) {
            float g = 0.f, gb = 0.f;
            for (int bb = 0; bb < n; ++bb) {
                g += dout[bb * kOut + o] * pooled[bb * kFeat + t];
                gb += dout[bb * kOut + o];
            }
            gwfc[o * kFeat + t] += g;
            if (t == 0) gbfc[o] += gb;
        }
        return;
    }
    float dp = 0.f;
    for (int o = 0; o < kOut; ++o) dp += dout[b * kOut + o] * wfc[o * kFeat + t];
    dp *= (1.0f / 64.0f);
    for (int p = 0; p < 64; ++p) {
        const int64_t q = ((int64_t)b * 64 + p) * kFeat + t;
        da4[q] = bf2f(a4[q]) > 0.f ? dp : 0.f;
    }
}

// Weight and bias gradients on the matrix cores (MFMA 16x16x16 bf16, FP32
// accumulation): gw[co][kk] = sum_p dy[p][co] xcol[p][kk], kk = tap CIN +
// ci, xcol the input activation under tap kk of output position p (zero
// outside the grid); column kk = K of xcol is 1, which gives the bias
// gradient sum_p dy[p][co].  One wave per 16 output channels, G tiles of 16
// columns and chunk of positions (16 per MFMA, the reduction dimension):
// dy is read and rounded to bf16 once per step for the G tiles (the
// activations are bf16 already), and each position's coordinates are
// computed once for them; one atomic add per output and chunk.
template <int CIN, int COUT, int DIN, int DOUT, int STRIDE, int G>
__global__ __launch_bounds__(256) void k_conv_wgrad(const uint16_t *__restrict__ x, const float *__restrict__ dy,
                                                    float *__restrict__ gw, float *__restrict__ gb, int64_t n_pos,
                                                    int64_t chunk)
{
    constexpr int K = 27 * CIN;
    constexpr int NCT = COUT / 16;
    constexpr int NKT = (K + 1 + 15) / 16;  // column tiles, the bias column included
    constexpr int NKG = (NKT + G - 1) / G;  // groups of G tiles
    const int lane = threadIdx.x & 63;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t tile = wave % (NCT * NKG), part = wave / (NCT * NKG);
    const int64_t p0 = part * chunk;
    if (p0 >= n_pos) return;  // uniform across the wave
    const int64_t p1 = min(n_pos, p0 + chunk);
    const int ct = (int)(tile % NCT), kg = (int)(tile / NCT);
    const int co = ct * 16 + (lane & 15);  // this lane's A row
    const int q4 = 4 * (lane >> 4);         // its 4 positions of a step
    int tap[G], ci[G];                      // this lane's B column of each tile: tap and channel
    bool is_w[G], is_b[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int kk = (kg * G + g) * 16 + (lane & 15);
        is_w[g] = kk < K;
        is_b[g] = kk == K;
        tap[g] = is_w[g] ? kk / CIN : 0;
        ci[g] = is_w[g] ? kk % CIN : 0;
    }
    v4f32 acc[G];
#pragma unroll
    for (int g = 0; g < G; ++g) acc[g] = (v4f32){0.f, 0.f, 0.f, 0.f};
    for (int64_t pb = p0; pb < p1; pb += 16) {
        v4i16 av = {0, 0, 0, 0};
        int oxs[4], oys[4], ozs[4];
        int64_t nbs[4];
        bool pin[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t p = pb + q4 + i;
            pin[i] = p < p1;
            const int64_t pp = pin[i] ? p : p0;
            av[i] = pin[i] ? (short)f2bf(dy[pp * COUT + co]) : (short)0;
            oxs[i] = (int)(pp % DOUT);
            oys[i] = (int)((pp / DOUT) % DOUT);
            ozs[i] = (int)((pp / (DOUT * DOUT)) % DOUT);
            nbs[i] = pp / ((int64_t)DOUT * DOUT * DOUT);
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (kg * G + g >= NKT) break;  // uniform
            const int kd = tap[g] / 9, kh = (tap[g] / 3) % 3, kw = tap[g] % 3;
            v4i16 bv = {0, 0, 0, 0};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (!pin[i]) continue;
                if (is_b[g]) {
                    bv[i] = (short)0x3F80;  // bf16 1.0
                } else if (is_w[g]) {
                    const int iz = ozs[i] * STRIDE + kd - 1, iy = oys[i] * STRIDE + kh - 1, ix = oxs[i] * STRIDE + kw - 1;
                    if (iz >= 0 && iy >= 0 && ix >= 0 && iz < DIN && iy < DIN && ix < DIN)
                        bv[i] = (short)x[(((nbs[i] * DIN + iz) * DIN + iy) * DIN + ix) * CIN + ci[g]];
                }
            }
            acc[g] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av, bv, acc[g], 0, 0, 0);
        }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
        if (kg * G + g >= NKT) break;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int co_o = ct * 16 + q4 + i, kk_o = (kg * G + g) * 16 + (lane & 15);
            if (kk_o < K) atomicAdd(&gw[(int64_t)co_o * K + kk_o], acc[g][i]);
            else if (kk_o == K) atomicAdd(&gb[co_o], acc[g][i]);
        }
    }
}

// Input gradient through the convolution on the matrix cores, masked by the
// ReLU of the layer that produced x (x > 0): dx[p][ci] = sum over (tap, co)
// dy[o][co] w[co][tap CIN + ci], o the output position that tap maps onto
// input position p (none where the stride skips it).  One wave per tile of
// 16 input positions x 16 input channels; the reduction runs over the taps
// that map some position of the tile onto an output and, per tap, over the
// output channels 16 at a time; dy is rounded to bf16 and the bf16 copy of
// the weights is used.
template <int CIN, int COUT, int DIN, int DOUT, int STRIDE>
__global__ __launch_bounds__(256) void k_conv_dgrad(const uint16_t *__restrict__ x, const float *__restrict__ dy,
                                                    const uint16_t *__restrict__ wb, float *__restrict__ dx,
                                                    int64_t n_in)
{
    constexpr int K = 27 * CIN;
    constexpr int NCI = CIN / 16;
    static_assert(CIN % 16 == 0 && COUT % 16 == 0, "channel counts in multiples of 16");
    const int lane = threadIdx.x & 63;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (wave >= ((n_in + 15) / 16) * NCI) return;  // uniform across the wave
    const int cit = (int)(wave % NCI);
    const int64_t pt = wave / NCI;
    const int64_t pm = pt * 16 + (lane & 15);  // this lane's A row: an input position
    const bool pin = pm < n_in;
    const int64_t pp = pin ? pm : 0;
    const int ix = (int)(pp % DIN), iy = (int)((pp / DIN) % DIN), iz = (int)((pp / (DIN * DIN)) % DIN);
    const int64_t nb = pp / ((int64_t)DIN * DIN * DIN);
    const int cib = cit * 16 + (lane & 15);  // this lane's B column: an input channel
    const int q4 = 4 * (lane >> 4);
    v4f32 acc = {0.f, 0.f, 0.f, 0.f};
    for (int tap = 0; tap < 27; ++tap) {
        const int kd = tap / 9, kh = (tap / 3) % 3, kw = tap % 3;
        const int tz = iz + 1 - kd, ty = iy + 1 - kh, tx = ix + 1 - kw;
        const bool ok = pin && tz >= 0 && ty >= 0 && tx >= 0 && tz % STRIDE == 0 && ty % STRIDE == 0 &&
                        tx % STRIDE == 0 && tz / STRIDE < DOUT && ty / STRIDE < DOUT && tx / STRIDE < DOUT;
        // a tap that maps no position of the tile onto an output adds only
        // zeros (with stride 2, most taps for a row of input positions)
        if (__ballot(ok) == 0) continue;  // uniform
        const int64_t o = ok ? ((nb * DOUT + tz / STRIDE) * DOUT + ty / STRIDE) * DOUT + tx / STRIDE : 0;
#pragma unroll
        for (int c0 = 0; c0 < COUT; c0 += 16) {
            v4i16 av = {0, 0, 0, 0}, bv;
            if (ok) {
                const float4 g = *(const float4 *)(dy + o * COUT + c0 + q4);
                av[0] = (short)f2bf(g.x);
                av[1] = (short)f2bf(g.y);
                av[2] = (short)f2bf(g.z);
                av[3] = (short)f2bf(g.w);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) bv[i] = (short)wb[(int64_t)(c0 + q4 + i) * K + tap * CIN + cib];
            acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av, bv, acc, 0, 0, 0);
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t p = pt * 16 + q4 + i;
        if (p < n_in) {
            const int64_t id = p * CIN + cit * 16 + (lane & 15);
            dx[id] = bf2f(x[id]) > 0.f ? acc[i] : 0.f;
        }
    }
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

__global__ void k_refresh_bf16(const float *__restrict__ w, uint16_t *__restrict__ wb, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) wb[i] = f2bf(w[i]);
}

__global__ void k_zero(float *p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.f;
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
    int64_t step = 0;
    // activations for the current batch capacity
    int batch_cap = 0;
    uint16_t *x0 = nullptr, *a[covox::kLayers] = {nullptr, nullptr, nullptr, nullptr};
    float *pooled = nullptr, *out = nullptr, *dout = nullptr, *loss = nullptr;
    float *d[covox::kLayers] = {nullptr, nullptr, nullptr, nullptr};  // gradients of the layer outputs
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
    fr(net->x0); fr(net->pooled); fr(net->out); fr(net->dout); fr(net->loss);
    for (int l = 0; l < kLayers; ++l) { fr(net->a[l]); fr(net->d[l]); net->a[l] = nullptr; net->d[l] = nullptr; }
    hipError_t e = hipSuccess;
    if (e == hipSuccess) e = hipMalloc((void **)&net->x0, sizeof(uint16_t) * (int64_t)n * 32768 * 4);
    for (int l = 0; l < kLayers && e == hipSuccess; ++l) {
        e = hipMalloc((void **)&net->a[l], sizeof(uint16_t) * act_elems(l, n));
        if (e == hipSuccess) e = hipMalloc((void **)&net->d[l], sizeof(float) * act_elems(l, n));
    }
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

template <int L>
static void launch_wgrad(covox_net *net, const uint16_t *x, int n)
{
    constexpr ConvShape s = kShapes[L];
    // One column tile per wave: sharing dy over 4 tiles (fewer, longer waves)
    // measured slower on every layer.
    constexpr int G = 1;
    constexpr int64_t tiles = (int64_t)(s.cout / 16) * (((s.K() + 1 + 15) / 16 + G - 1) / G);
    const int64_t npos = (int64_t)n * s.dout * s.dout * s.dout;
    // positions per wave (a multiple of 16): at most 1024, fewer where the
    // layer has few positions, so that a launch has about 12 k waves
    const int64_t chunk = std::max<int64_t>(64, std::min<int64_t>(1024, npos * tiles / 12288 / 16 * 16));
    const int64_t waves = tiles * ((npos + chunk - 1) / chunk);
    hipLaunchKernelGGL((k_conv_wgrad<s.cin, s.cout, s.din, s.dout, s.stride, G>), dim3(blocks_for(waves * 64, 256)),
                       dim3(256), 0, net->ctx->stream, x, net->d[L], net->g + net->P.off_w[L],
                       net->g + net->P.off_b[L], npos, chunk);
}

template <int L>
static void launch_dgrad(covox_net *net, const uint16_t *x, float *dx, int n)
{
    constexpr ConvShape s = kShapes[L];
    const int64_t nin = (int64_t)n * s.din * s.din * s.din;
    const int64_t waves = ((nin + 15) / 16) * (s.cin / 16);
    hipLaunchKernelGGL((k_conv_dgrad<s.cin, s.cout, s.din, s.dout, s.stride>), dim3(blocks_for(waves * 64, 256)),
                       dim3(256), 0, net->ctx->stream, x, net->d[L], net->wb[L], dx, nin);
}

static int net_backward(covox_net *net, const float *x_dev, int n)
{
    covox_ctx *ctx = net->ctx;
    const int64_t nx = (int64_t)n * 32768 * 4;
    hipLaunchKernelGGL(k_to_bf16, dim3(blocks_for(nx, 256)), dim3(256), 0, ctx->stream, x_dev, net->x0, nx);
    const int64_t np = net->P.total;
    hipLaunchKernelGGL(k_zero, dim3(blocks_for(np, 256)), dim3(256), 0, ctx->stream, net->g, np);
    hipLaunchKernelGGL(k_fc_bwd, dim3(n + 1), dim3(64), 0, ctx->stream, net->dout, net->pooled, net->w + net->P.off_fcw,
                       net->a[3], net->g + net->P.off_fcw, net->g + net->P.off_fcb, net->d[3], n);
    launch_wgrad<3>(net, net->a[2], n);
    launch_dgrad<3>(net, net->a[2], net->d[2], n);
    launch_wgrad<2>(net, net->a[1], n);
    launch_dgrad<2>(net, net->a[1], net->d[1], n);
    launch_wgrad<1>(net, net->a[0], n);
    launch_dgrad<1>(net, net->a[0], net->d[0], n);
    launch_wgrad<0>(net, net->x0, n);
    return hip_check(ctx, hipGetLastError(), "net backward");
}

static void refresh_bf16(covox_net *net)
{
    for (int l = 0; l < kLayers; ++l) {
        const int64_t nw = (int64_t)kShapes[l].cout * kShapes[l].K();
        hipLaunchKernelGGL(k_refresh_bf16, dim3(blocks_for(nw, 256)), dim3(256), 0, net->ctx->stream,
                           net->w + net->P.off_w[l], net->wb[l], nw);
    }
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
    int rc = net_forward(net, x_dev, n, nullptr);
    if (rc) return rc;
    hipLaunchKernelGGL(k_zero, dim3(1), dim3(64), 0, ctx->stream, net->loss, (int64_t)1);
    hipLaunchKernelGGL(k_loss, dim3(blocks_for((int64_t)n * kOut, 64)), dim3(64), 0, ctx->stream, net->out, y_dev,
                       net->dout, net->loss, n, 1.0f / (trans_scale * trans_scale));
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
    int rc = net_forward(net, x_dev, n, nullptr);
    if (rc) return rc;
    hipLaunchKernelGGL(k_zero, dim3(1), dim3(64), 0, ctx->stream, net->loss, (int64_t)1);
    hipLaunchKernelGGL(k_loss, dim3(blocks_for((int64_t)n * kOut, 64)), dim3(64), 0, ctx->stream, net->out, y_dev,
                       net->dout, net->loss, n, 1.0f / (trans_scale * trans_scale));
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
        e = hipMalloc((void **)&net->wb[l], sizeof(uint16_t) * (int64_t)kShapes[l].cout * kShapes[l].K());
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
    for (float **p : {&net->w, &net->g, &net->m, &net->v, &net->pooled, &net->out, &net->dout, &net->loss}) {
        if (*p) (void)hipFree(*p);
        *p = nullptr;
    }
    if (net->x0) (void)hipFree(net->x0);
    net->x0 = nullptr;
    for (int l = 0; l < kLayers; ++l) {
        for (void **p : {(void **)&net->wb[l], (void **)&net->a[l], (void **)&net->d[l]}) {
            if (*p) (void)hipFree(*p);
            *p = nullptr;
        }
    }
    net->batch_cap = 0;
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
