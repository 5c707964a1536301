// Incremental ESDF by wavefront propagation (paper Sec. III-E: voxels that
// become occupied or free seed work in per-block queues, a wave processes a
// block, every axis of the block is swept, block faces hand better
// distances to the neighbours, repeated until nothing changes).
//
// Each voxel of an allocated block keeps its nearest known site (a packed
// offset) and the squared distance k to it in voxels^2, k <= R^2.  One
// update:
//   k_page_sites  (k_esdf.hip) the page, and site masks (observed, |D| <= vs) by
//                 dense block of the box: none for a block that is not allocated;
//   k_wf_seed     one wave per block: blocks allocated since the last update
//                 start empty, sites take themselves (k = 0), voxels whose
//                 parent is no longer a site lose it; changed blocks are
//                 queued;
//   rounds, until the queue is empty (a launch each):
//     k_wf_round  one wave per queued block: the six faces take the parents of
//                 the neighbours' face voxels from the previous round's state,
//                 then forward and backward sweeps along x, y, z (one lane per
//                 line); the block is written to its other buffer and, if it
//                 changed, it and its six neighbours are flagged for the next
//                 round;
//   k_wf_phi      one wave per block: phi as for the exact EDT, from k, and the
//                 state back into the first buffer.
// Rounds read only the previous round's state (every block has two buffers, and
// which holds its state is noted a round apart too), so the result does not depend
// on scheduling; all of it is integer arithmetic.
#include "covox_impl.h"

#include <math.h>

#include <algorithm>

namespace covox {

namespace {

constexpr int32_t kWfInf = INT32_MAX;
constexpr int32_t kWfNone = -1;

__device__ __forceinline__ int32_t wf_pack(int dx, int dy, int dz)
{
    return (dx + 128) | ((dy + 128) << 8) | ((dz + 128) << 16);
}

// v takes the parent of its neighbour u (k_u, p_u; e = u - v) when nearer
// and within R.
__device__ __forceinline__ void wf_offer(int32_t &kv, int32_t &pv, int32_t ku, int32_t pu, int ex, int ey, int ez,
                                         int R2)
{
    if (ku == kWfInf) return;
    const int ox = (pu & 255) - 128 + ex, oy = ((pu >> 8) & 255) - 128 + ey, oz = ((pu >> 16) & 255) - 128 + ez;
    const int k = ox * ox + oy * oy + oz * oz;
    if (k > R2 || k >= kv) return;
    kv = k;
    pv = wf_pack(ox, oy, oz);
}

template <typename S> __device__ __forceinline__ float ldw(const S *p);
template <> __device__ __forceinline__ float ldw<float>(const float *p) { return *p; }
template <> __device__ __forceinline__ float ldw<__half>(const __half *p) { return __half2float(*p); }

// Number of a block in the page's domain, the box of all allocated blocks; -1 outside.
__device__ __forceinline__ int64_t dense_block(const SubmapMeta *meta, int bx, int by, int bz)
{
    const int x = bx - meta->dom_min[0], y = by - meta->dom_min[1], z = bz - meta->dom_min[2];
    const bool in = x >= 0 && x < meta->dom_dim[0] && y >= 0 && y < meta->dom_dim[1] && z >= 0 && z < meta->dom_dim[2];
    return in ? ((int64_t)z * meta->dom_dim[1] + y) * meta->dom_dim[0] + x : -1;
}

// Buffer index of an allocated block by the page, -1 for any other.
__device__ __forceinline__ int32_t page_block(const SubmapMeta *meta, const int32_t *page, int bx, int by, int bz)
{
    const int64_t g = dense_block(meta, bx, by, bz);
    const int32_t v = page[g >= 0 ? g : 0];
    return g >= 0 ? v : -1;
}

// The look-ups of a lane's eight voxels are in flight together, each one read of the
// dense masks (6 us in a room of 1.4 k blocks; by the hash table and masks by buffer
// index, one after the other, 12, and 3 for those masks).
__global__ __launch_bounds__(256) void k_wf_seed(const SubmapMeta *__restrict__ meta, const int64_t *__restrict__ wn,
                                                 const uint64_t *__restrict__ keys,
                                                 const uint64_t *__restrict__ sites, int32_t *__restrict__ wk,
                                                 int32_t *__restrict__ wp, uint32_t *__restrict__ flag)
{
    const int64_t j = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (j >= meta->n_blocks) return;  // uniform across the wave
    const bool fresh = j >= *wn;
    int bx, by, bz;
    unpack_key(keys[j], bx, by, bz);
    const int64_t g = dense_block(meta, bx, by, bz);  // (an allocated block is in the domain)
    const int x = 8 * bx + (lane & 7), y = 8 * by + (lane >> 3);
    bool dirty = fresh;
    int32_t k[8], p[8];
    int64_t sg[8];
    uint64_t own[8], at[8];
    int sl[8];
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        const int64_t o = j * 512 + lane + 64 * z;
        k[z] = wk[o];
        p[z] = wp[o];
        own[z] = sites[g * 8 + z];
        if (fresh) {
            k[z] = kWfInf;
            p[z] = kWfNone;
        }
    }
#pragma unroll
    for (int z = 0; z < 8; ++z) {  // the parent's block and bit
        const bool has = k[z] != kWfInf;
        const int sx = x + (has ? (p[z] & 255) - 128 : 0), sy = y + (has ? ((p[z] >> 8) & 255) - 128 : 0);
        const int sz = 8 * bz + z + (has ? ((p[z] >> 16) & 255) - 128 : 0);
        sg[z] = dense_block(meta, sx >> 3, sy >> 3, sz >> 3);
        sl[z] = (sx & 7) + 8 * (sy & 7) + 64 * (sz & 7);
    }
#pragma unroll
    for (int z = 0; z < 8; ++z) at[z] = sites[(sg[z] >= 0 ? sg[z] : g) * 8 + (sl[z] >> 6)];
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        const int64_t o = j * 512 + lane + 64 * z;
        if ((own[z] >> lane) & 1ull) {
            if (k[z] != 0) { k[z] = 0; p[z] = wf_pack(0, 0, 0); dirty = true; }
        } else if (k[z] != kWfInf) {
            if (sg[z] < 0 || !((at[z] >> (sl[z] & 63)) & 1ull)) {
                k[z] = kWfInf;
                p[z] = kWfNone;
                dirty = true;
            }
        }
        wk[o] = k[z];
        wp[o] = p[z];
    }
    if (__ballot(dirty) && lane == 0) flag[j] = 1u;
}

// A round's counters: the blocks queued in it, in a ring of slots, and the sum over
// the rounds before.
constexpr int kWfSlots = 64;
struct WfCounts {
    int64_t total;
    int32_t queued[kWfSlots];
};
constexpr int kWfCountWords = (int)(sizeof(WfCounts) / sizeof(uint32_t));

// A line of eight voxels along axis a: forward, then backward.
template <int A>
__device__ __forceinline__ void wf_sweep(int32_t k[8], int32_t p[8], int R2)
{
#pragma unroll
    for (int q = 1; q < 8; ++q) wf_offer(k[q], p[q], k[q - 1], p[q - 1], A == 0 ? -1 : 0, A == 1 ? -1 : 0, A == 2 ? -1 : 0, R2);
#pragma unroll
    for (int q = 6; q >= 0; --q) wf_offer(k[q], p[q], k[q + 1], p[q + 1], A == 0 ? 1 : 0, A == 1 ? 1 : 0, A == 2 ? 1 : 0, R2);
}

// LDS word of a voxel: 8 words more a z plane, so that the lines of every axis spread
// over the banks.
__device__ __forceinline__ int wf_word(int x, int y, int z) { return x + 8 * y + 72 * z; }
constexpr int kWfWords = 72 * 8;

// Bound by latency: a wave has one block, and one chain of reads and sweeps.  The six
// neighbours' faces are read together before any is used, and a sweep has its line in
// registers (each of its 14 steps was two LDS reads); a block without work only
// carries on which buffer holds its state.  Room, 1.4 k blocks, a round of some 300:
// 3 + 10 + 3 us as queue, round and copy back, 7 now.
__global__ __launch_bounds__(256) void k_wf_round(const SubmapMeta *__restrict__ meta, const int32_t *__restrict__ page,
                                                  const uint64_t *__restrict__ keys, int32_t *k0, int32_t *p0,
                                                  int32_t *k1, int32_t *p1, uint32_t *__restrict__ flag,
                                                  uint32_t *__restrict__ flag_next, const uint32_t *__restrict__ cur,
                                                  uint32_t *__restrict__ cur_next, WfCounts *counts, int round, int R2)
{
    __shared__ __align__(16) int32_t sk[4][kWfWords], sp[4][kWfWords];
    const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (round > 0) counts->total += counts->queued[(round - 1) % kWfSlots];
        counts->queued[(round + kWfSlots / 2) % kWfSlots] = 0;
    }
    const int64_t j = (int64_t)blockIdx.x * 4 + wid;
    if (j >= meta->n_blocks) return;  // uniform across the wave (the waves share no barrier)
    const uint32_t c = cur[j], queued = flag[j];
    if (!queued) {  // uniform
        if (lane == 0) cur_next[j] = c;
        return;
    }
    const int32_t *wk = c ? k1 : k0, *wp = c ? p1 : p0;
    int32_t ok[8], op[8];
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        ok[z] = wk[j * 512 + lane + 64 * z];
        op[z] = wp[j * 512 + lane + 64 * z];
    }
    int32_t nb = -1;  // lane d < 6 holds the neighbour in direction d
    uint32_t nc = 0;  // and the buffer of its state
    if (lane < 6) {
        int b[3];
        unpack_key(keys[j], b[0], b[1], b[2]);
        const int e = (lane & 1) ? 1 : -1, a = lane >> 1;
        nb = page_block(meta, page, b[0] + (a == 0 ? e : 0), b[1] + (a == 1 ? e : 0), b[2] + (a == 2 ? e : 0));
        if (nb >= 0) nc = cur[nb];
    }
    // faces -x, +x, -y, +y, -z, +z; lane = (u1, u2) on the face
    const int u1 = lane & 7, u2 = lane >> 3;
    int32_t fk[6], fp[6];
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        const int32_t n = __builtin_amdgcn_readlane(nb, d);
        const uint32_t m = (uint32_t)__builtin_amdgcn_readlane((int)nc, d);
        const int a = d >> 1, far = (d & 1) ? 0 : 7;
        const int lu = a == 0 ? far + 8 * u1 + 64 * u2 : a == 1 ? u1 + 8 * far + 64 * u2 : u1 + 8 * u2 + 64 * far;
        const int64_t o = (n >= 0 ? (int64_t)n : j) * 512 + lu;
        fk[d] = (m ? k1 : k0)[o];
        fp[d] = (m ? p1 : p0)[o];
        if (n < 0) fk[d] = kWfInf;  // offers nothing
    }
    int32_t *K = sk[wid], *P = sp[wid];
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        K[wf_word(u1, u2, z)] = ok[z];
        P[wf_word(u1, u2, z)] = op[z];
    }
    wave_sync();
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        const int a = d >> 1, side = (d & 1) ? 7 : 0, e = (d & 1) ? 1 : -1;
        const int lv = a == 0 ? wf_word(side, u1, u2) : a == 1 ? wf_word(u1, side, u2) : wf_word(u1, u2, side);
        int32_t kv = K[lv], pv = P[lv];
        wf_offer(kv, pv, fk[d], fp[d], a == 0 ? e : 0, a == 1 ? e : 0, a == 2 ? e : 0, R2);
        K[lv] = kv;
        P[lv] = pv;
        wave_sync();
    }
    int32_t k[8], p[8];
    {
        int4 *K4 = (int4 *)(K + wf_word(0, u1, u2)), *P4 = (int4 *)(P + wf_word(0, u1, u2));
        const int4 a = K4[0], b = K4[1], g = P4[0], h = P4[1];
        k[0] = a.x; k[1] = a.y; k[2] = a.z; k[3] = a.w; k[4] = b.x; k[5] = b.y; k[6] = b.z; k[7] = b.w;
        p[0] = g.x; p[1] = g.y; p[2] = g.z; p[3] = g.w; p[4] = h.x; p[5] = h.y; p[6] = h.z; p[7] = h.w;
        wf_sweep<0>(k, p, R2);
        K4[0] = make_int4(k[0], k[1], k[2], k[3]);
        K4[1] = make_int4(k[4], k[5], k[6], k[7]);
        P4[0] = make_int4(p[0], p[1], p[2], p[3]);
        P4[1] = make_int4(p[4], p[5], p[6], p[7]);
    }
    wave_sync();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        k[q] = K[wf_word(u1, q, u2)];
        p[q] = P[wf_word(u1, q, u2)];
    }
    wf_sweep<1>(k, p, R2);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        K[wf_word(u1, q, u2)] = k[q];
        P[wf_word(u1, q, u2)] = p[q];
    }
    wave_sync();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        k[q] = K[wf_word(u1, u2, q)];
        p[q] = P[wf_word(u1, u2, q)];
    }
    wf_sweep<2>(k, p, R2);
    int32_t *nk = c ? k0 : k1, *np = c ? p0 : p1;
    bool ch = false;
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        ch = ch || k[z] != ok[z] || p[z] != op[z];
        nk[j * 512 + lane + 64 * z] = k[z];
        np[j * 512 + lane + 64 * z] = p[z];
    }
    const bool changed = __ballot(ch) != 0;
    if (lane < 6 && nb >= 0 && changed) flag_next[nb] = 1u;
    if (lane == 0) {
        flag[j] = 0u;
        cur_next[j] = 1u - c;
        if (changed) flag_next[j] = 1u;
        atomicAdd(&counts->queued[round % kWfSlots], 1);
    }
}

template <typename S>
__global__ __launch_bounds__(256) void k_wf_phi(SubmapMeta *__restrict__ meta, const S *__restrict__ D,
                                                const S *__restrict__ W, int32_t *__restrict__ wk,
                                                int32_t *__restrict__ wp, const int32_t *__restrict__ k1,
                                                const int32_t *__restrict__ p1, const uint32_t *__restrict__ cur,
                                                float vs, float tau, float dmax, float *__restrict__ phi,
                                                int64_t *__restrict__ wn)
{
    const int64_t j = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    const int64_t n = meta->n_blocks;
    if (j == 0 && lane == 0) *wn = n;
    if (j >= n) return;
    const bool second = cur[j] != 0;  // uniform across the wave
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        const int64_t o = j * 512 + lane + 64 * z;
        const float Dv = ldw(D + o), Wv = ldw(W + o);
        const int32_t k = second ? k1[o] : wk[o];
        if (second) {
            wk[o] = k;
            wp[o] = p1[o];
        }
        float out;
        if (!(Wv > 0.0f)) out = __builtin_nanf("");
        else if (fabsf(Dv) < tau) out = Dv;
        else {
            const float sg = Dv > 0.0f ? 1.0f : -1.0f;
            out = k == kWfInf ? sg * dmax : sg * fminf(dmax, vs * sqrtf((float)k));
        }
        phi[o] = out;
    }
}

__global__ void k_wf_zero(int64_t *p) { *p = 0; }

}  // namespace

int wavefront_reset(covox_ctx *ctx, covox_submap *s)
{
    if (!s->wf_wn) return COVOX_OK;
    hipLaunchKernelGGL(k_wf_zero, dim3(1), dim3(1), 0, ctx->stream, s->wf_wn);
    return hip_check(ctx, hipGetLastError(), "wavefront reset");
}

int update_esdf_wavefront(covox_ctx *ctx, covox_submap *s)
{
    if (ctx->capturing) return fail(ctx, COVOX_EINVAL, "update_esdf: the wavefront ESDF cannot be captured");
    const covox_params &p = ctx->p;
    int rc;
    const int64_t cap = s->cap;
    if (!s->wf_k) {
        if ((rc = hip_check(ctx, hipMalloc((void **)&s->wf_k, sizeof(int32_t) * 512 * cap), "wavefront state")) ||
            (rc = hip_check(ctx, hipMalloc((void **)&s->wf_p, sizeof(int32_t) * 512 * cap), "wavefront state")) ||
            (rc = hip_check(ctx, hipMalloc((void **)&s->wf_wn, sizeof(int64_t)), "wavefront state")))
            return rc;
        hipLaunchKernelGGL(k_wf_zero, dim3(1), dim3(1), 0, ctx->stream, s->wf_wn);
    }
    if ((rc = ensure_buffer(ctx, (void **)&ctx->wf_nk, &ctx->wf_nk_cap, 512 * cap, sizeof(int32_t), "wavefront")) ||
        (rc = ensure_buffer(ctx, (void **)&ctx->wf_np, &ctx->wf_np_cap, 512 * cap, sizeof(int32_t), "wavefront")) ||
        (rc = ensure_buffer(ctx, (void **)&ctx->wf_flag, &ctx->wf_flag_cap, 4 * cap + kWfCountWords, sizeof(uint32_t),
                            "wavefront")))
        return rc;
    if (!ctx->wf_pin) {
        if ((rc = hip_check(ctx, hipHostMalloc((void **)&ctx->wf_pin, sizeof(WfCounts), hipHostMallocDefault),
                            "wavefront counter")))
            return rc;
    }
    // the page (dense block index) serves the alignment and the summaries too
    if ((rc = build_page_and_sites(ctx, s))) return rc;
    const uint64_t *sites = ctx->sites[ctx->esdf_slot];
    const int R = (int)std::llround(p.d_max / p.voxel_size);
    const int64_t nbu = std::max<int64_t>(std::min(s->nb_upper, cap), 1);
    const unsigned gw = (unsigned)((nbu + 3) / 4);
    const float vs = (float)p.voxel_size;
    // the counters, then queue flags and state buffers for rounds of even and odd numbers
    WfCounts *counts = (WfCounts *)ctx->wf_flag;
    const WfCounts *seen = (const WfCounts *)ctx->wf_pin;
    uint32_t *at = ctx->wf_flag + kWfCountWords;
    uint32_t *flag[2] = {at, at + nbu}, *cur[2] = {at + 2 * nbu, at + 3 * nbu};
    fill_u32(ctx->stream, ctx->wf_flag, 0u, 4 * nbu + kWfCountWords);
    {
        TimedLaunch tl(ctx, COVOX_K_WAVEFRONT);
        hipLaunchKernelGGL(k_wf_seed, dim3(gw), dim3(256), 0, ctx->stream, s->meta, s->wf_wn, s->keys, sites, s->wf_k,
                           s->wf_p, flag[0]);
    }
    if ((rc = hip_check(ctx, hipGetLastError(), "wavefront seed"))) return rc;
    // rounds in groups between reads of the queue size: a wait costs as much as four
    // rounds without work, and a frame's changes take some eight to twelve to settle
    int64_t rounds = 0;
    for (;;) {
        const int group = rounds == 0 ? 8 : 4;
        for (int r = 0; r < group; ++r) {
            TimedLaunch tl(ctx, COVOX_K_WAVEFRONT);
            const int e = (int)(rounds & 1);
            hipLaunchKernelGGL(k_wf_round, dim3(gw), dim3(256), 0, ctx->stream, s->meta, s->page, s->keys, s->wf_k,
                               s->wf_p, ctx->wf_nk, ctx->wf_np, flag[e], flag[1 - e], cur[e], cur[1 - e], counts,
                               (int)rounds, R * R);
            ++rounds;
        }
        if ((rc = hip_check(ctx, hipGetLastError(), "wavefront round"))) return rc;
        // the queue size of the last round: zero means that it did nothing
        if ((rc = hip_check(ctx, hipMemcpyAsync(ctx->wf_pin, counts, sizeof(WfCounts), hipMemcpyDeviceToHost,
                                                ctx->stream), "wavefront count")) ||
            (rc = hip_check(ctx, hipStreamSynchronize(ctx->stream), "wavefront sync")))
            return rc;
        if (seen->queued[(rounds - 1) % kWfSlots] == 0) break;
        if (rounds > 4 * (cap + 8)) return fail(ctx, COVOX_EHIP, "update_esdf: the wavefront did not settle");
    }
    ctx->wf_last_block_rounds = seen->total;
    {
        TimedLaunch tl(ctx, COVOX_K_WAVEFRONT);
        const float tau = (float)band_limit(p), dmax = (float)p.d_max;
        if (p.precision == COVOX_FP16)
            hipLaunchKernelGGL(k_wf_phi<__half>, dim3(gw), dim3(256), 0, ctx->stream, s->meta, (const __half *)s->D,
                               (const __half *)s->W, s->wf_k, s->wf_p, ctx->wf_nk, ctx->wf_np, cur[rounds & 1], vs, tau, dmax,
                               s->phi, s->wf_wn);
        else
            hipLaunchKernelGGL(k_wf_phi<float>, dim3(gw), dim3(256), 0, ctx->stream, s->meta, (const float *)s->D,
                               (const float *)s->W, s->wf_k, s->wf_p, ctx->wf_nk, ctx->wf_np, cur[rounds & 1], vs, tau, dmax,
                               s->phi, s->wf_wn);
    }
    if ((rc = hip_check(ctx, hipGetLastError(), "wavefront phi"))) return rc;
    s->esdf_version = s->version;
    s->esdf_exact = false;  // phi is the wavefront's, not the exact transform
    return COVOX_OK;
}

}  // namespace covox
