// Projective TSDF integration (paper Sec. III-C projection mapping; the
// count / allocate / update phases of Sec. III-D).
//
// One frame is two launches on the context stream where the host's bound on the
// block count leaves room for the whole frustum (nearly always):
//   k_probe          one wave64 per block of the frustum's block box: the 512
//                    voxels are tested for validity (lane = (x, y), z in
//                    registers), a ballot gives "any valid", lane 0 looks the
//                    key up in the hash table; a block that exists is updated at
//                    once, a new one leaves a flag byte;
//   k_integrate_new  one wave64 per new block, which finds its place among the
//                    flags: box order is ascending packed-key order, so new
//                    blocks receive n_blocks + rank deterministically; it
//                    activates them (key store + hash insert) and applies the
//                    running-average update; one workgroup takes the counts.  It
//                    refuses them all when they do not fit after all.
// and three where it does not:
//   k_probe          as above, but every block's buffer index, or NEW, is stored;
//   k_scan           one 1024-lane workgroup compacts them in box order and
//                    checks capacity before anything is committed;
//   k_integrate      one wave64 per touched block: activation and update.
// A batch of up to 64 frames is five launches (see "frame batches" below):
// k_batch_tiles, k_probe_batch, k_batch_rank, k_batch_activate, k_integrate_batch.
// Parity-relevant arithmetic is binary32 in a fixed operation order (the
// library is built with -ffp-contract=off; division is correctly rounded).
#include "covox_impl.h"
#include "edt_columns.h"

#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

namespace covox {

namespace {

constexpr uint32_t kNew = 0xFFFFFFFFu;

template <typename S> __device__ __forceinline__ float ld(const S *p);
template <> __device__ __forceinline__ float ld<float>(const float *p) { return *p; }
template <> __device__ __forceinline__ float ld<__half>(const __half *p) { return __half2float(*p); }
template <typename S> __device__ __forceinline__ void st(S *p, float v);
template <> __device__ __forceinline__ void st<float>(float *p, float v) { *p = v; }
template <> __device__ __forceinline__ void st<__half>(__half *p, float v) { *p = __float2half_rn(v); }

// Validity of the 8 voxels (ix, iy, iz0 + z), z = 0..7, of one lane under
// the frame's projection: the voxel centre lies in front of the camera, its
// nearest pixel is inside the image, the pixel's depth d is in (0, max
// range], and the signed distance sdf = d - (voxel depth) is at least -tau.
// Sets sdf and the observation weight w (1, or 1 / d^2) of each valid voxel
// and returns the mask of valid voxels.  The steps run in three passes (the
// pixel of every voxel, the 8 depth reads, the tests) so that the reads are
// in flight together; the arithmetic of each voxel is unchanged.
__device__ __forceinline__ uint32_t proj_column(const FrameArgs &f, float vs, float tau, float maxr, int ix, int iy,
                                                int iz0, float sdf[8], float w[8])
{
    const float cx = ((float)ix + 0.5f) * vs;
    const float cy = ((float)iy + 0.5f) * vs;
    float pzv[8];
    int64_t pix[8];
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        const float cz = ((float)(iz0 + z) + 0.5f) * vs;
        const float px = ((f.R[0] * cx + f.R[1] * cy) + f.R[2] * cz) + f.t[0];
        const float py = ((f.R[3] * cx + f.R[4] * cy) + f.R[5] * cz) + f.t[1];
        const float pz = ((f.R[6] * cx + f.R[7] * cy) + f.R[8] * cz) + f.t[2];
        pzv[z] = pz;
        pix[z] = -1;
        if (pz > 0.0f) {
            const float u = ((f.K[0] * px) / pz) + f.K[2];
            const float v = ((f.K[1] * py) / pz) + f.K[3];
            const float uf = floorf(u + 0.5f);
            const float vf = floorf(v + 0.5f);
            if (uf >= 0.0f && uf < (float)f.W && vf >= 0.0f && vf < (float)f.H)
                pix[z] = (int64_t)(int)vf * f.W + (int)uf;
        }
    }
    float d[8];
#pragma unroll
    for (int z = 0; z < 8; ++z) d[z] = f.depth[pix[z] >= 0 ? pix[z] : 0];  // pixel 0 stands in, unused
    uint32_t okm = 0;
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        sdf[z] = 0.0f;
        w[z] = 0.0f;
        if (pix[z] < 0 || !(d[z] > 0.0f && d[z] <= maxr)) continue;
        sdf[z] = d[z] - pzv[z];
        w[z] = f.weight_mode == COVOX_WEIGHT_INV_DEPTH2 ? 1.0f / (d[z] * d[z]) : 1.0f;
        okm |= (uint32_t)(sdf[z] >= -tau) << z;
    }
    return okm;
}

// The nearest pixel of the voxel centre (cx, cy, cz) and its camera depth
// pz, by the arithmetic of proj_column (kept written out there, where the
// compiler schedules the eight voxels of a lane together); -1 when the
// centre is behind the camera or projects outside the image.
__device__ __forceinline__ int64_t proj_pixel(const FrameArgs &f, float cx, float cy, float cz, float &pz)
{
    const float px = ((f.R[0] * cx + f.R[1] * cy) + f.R[2] * cz) + f.t[0];
    const float py = ((f.R[3] * cx + f.R[4] * cy) + f.R[5] * cz) + f.t[1];
    pz = ((f.R[6] * cx + f.R[7] * cy) + f.R[8] * cz) + f.t[2];
    if (pz > 0.0f) {
        const float u = ((f.K[0] * px) / pz) + f.K[2];
        const float v = ((f.K[1] * py) / pz) + f.K[3];
        const float uf = floorf(u + 0.5f);
        const float vf = floorf(v + 0.5f);
        if (uf >= 0.0f && uf < (float)f.W && vf >= 0.0f && vf < (float)f.H) return (int64_t)(int)vf * f.W + (int)uf;
    }
    return -1;
}

// Whether some voxel (ix, iy, iz0 + z), Z0 <= z < Z1, of the lane passes the
// validity test of proj_column (same arithmetic; the weights are not needed).
template <int Z0, int Z1>
__device__ __forceinline__ bool proj_any(const FrameArgs &f, float vs, float tau, float maxr, int ix, int iy, int iz0)
{
    const float cx = ((float)ix + 0.5f) * vs;
    const float cy = ((float)iy + 0.5f) * vs;
    float pzv[Z1 - Z0];
    int64_t pix[Z1 - Z0];
#pragma unroll
    for (int z = Z0; z < Z1; ++z) pix[z - Z0] = proj_pixel(f, cx, cy, ((float)(iz0 + z) + 0.5f) * vs, pzv[z - Z0]);
    float d[Z1 - Z0];
#pragma unroll
    for (int k = 0; k < Z1 - Z0; ++k) d[k] = f.depth[pix[k] >= 0 ? pix[k] : 0];  // pixel 0 stands in, unused
    bool any = false;
#pragma unroll
    for (int k = 0; k < Z1 - Z0; ++k) any |= pix[k] >= 0 && d[k] > 0.0f && d[k] <= maxr && d[k] - pzv[k] >= -tau;
    return any;
}

// False only if no voxel centre of block (bx, by, bz) can pass the validity
// test in this frame: the sphere holding the centres lies behind the
// camera, beyond the far limit, or outside a side plane of the image.
__device__ __forceinline__ bool block_may_be_visible(const FrameArgs &f, float vs, int bx, int by, int bz)
{
    const float cx = (float)(8 * bx + 4) * vs, cy = (float)(8 * by + 4) * vs, cz = (float)(8 * bz + 4) * vs;
    const float px = ((f.R[0] * cx + f.R[1] * cy) + f.R[2] * cz) + f.t[0];
    const float py = ((f.R[3] * cx + f.R[4] * cy) + f.R[5] * cz) + f.t[1];
    const float pz = ((f.R[6] * cx + f.R[7] * cy) + f.R[8] * cz) + f.t[2];
    const float r = f.cull_r;
    if (pz < -r || pz > f.zfar + r) return false;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (f.plane[k][0] * px + f.plane[k][1] * py + f.plane[k][2] * pz < -r) return false;
    return true;
}

// (64-bit divisions are some 130 instructions each, 32-bit ones 20.)
__device__ __forceinline__ void box_block(const FrameArgs &f, int64_t j, int &bx, int &by, int &bz)
{
    if (((int64_t)f.bdim[0] * f.bdim[1] * f.bdim[2]) >> 31 == 0) {  // uniform
        const uint32_t q = (uint32_t)j / (uint32_t)f.bdim[2], r = q / (uint32_t)f.bdim[1];
        bz = f.blo[2] + (int)((uint32_t)j - q * (uint32_t)f.bdim[2]);
        by = f.blo[1] + (int)(q - r * (uint32_t)f.bdim[1]);
        bx = f.blo[0] + (int)r;
        return;
    }
    const int64_t nz = f.bdim[2], ny = f.bdim[1];
    bz = f.blo[2] + (int)(j % nz);
    by = f.blo[1] + (int)((j / nz) % ny);
    bx = f.blo[0] + (int)(j / (nz * ny));
}

// The running-average update of one voxel column (8 z values of a lane) of
// an allocated block; returns the number of updated voxels of the wave.
template <typename S>
__device__ __forceinline__ int update_column(S *Db, S *Wb, const float sdf[8], const float wt[8], uint32_t okm, float tau,
                                             bool is_new)
{
    // Every read is issued in straight-line code, so that the eight are in
    // flight together (a conditional read would make the compiler wait for
    // each one in turn), but a voxel that is not updated reads its lane's
    // z = 0 voxel instead: rows of the block that no lane updates are not
    // fetched.  Only updated voxels are written, and every voxel of a new
    // block (zero where not updated).
    float Dp[8], Wp[8];
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        const int o = ((okm >> z) & 1u) ? 64 * z : 0;
        Dp[z] = ld(Db + o);
        Wp[z] = ld(Wb + o);
    }
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        Dp[z] = is_new ? 0.0f : Dp[z];
        Wp[z] = is_new ? 0.0f : Wp[z];
    }
    int n_ok = 0;
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        const bool ok = (okm >> z) & 1u;
        n_ok += __popcll(__ballot(ok));
        const float tr = fminf(sdf[z], tau);
        const float Wn = Wp[z] + wt[z];
        const float Dn = ((Dp[z] * Wp[z]) + (tr * wt[z])) / Wn;
        Dp[z] = ok ? Dn : Dp[z];
        Wp[z] = ok ? Wn : Wp[z];
    }
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        if (((okm >> z) & 1u) || is_new) {
            st(Db + 64 * z, Dp[z]);
            st(Wb + 64 * z, Wp[z]);
        }
    }
    return n_ok;
}

// Work item of workgroup w in a grid of n_wg = 8 C workgroups: with XCD
// order, item (w mod 8) C + floor(w / 8), so that the workgroups the
// dispatcher deals to one XCD cover one contiguous eighth of the items;
// otherwise w.
__device__ __forceinline__ int64_t work_item(int64_t w, int64_t n_wg, bool xcd)
{
    return xcd ? (w & 7) * (n_wg >> 3) + (w >> 3) : w;
}

// FUSED: blocks that already exist are updated here (their buffer index is
// known), so only new blocks are left, a flag byte each, to k_integrate_new.
// Used only when the host bound proves that this frame cannot overflow the pool
// or the table, so that no capacity failure can follow a partial update.
template <typename S, bool FUSED, typename E>
__global__ __launch_bounds__(256) void k_probe(const E edt, FrameArgs f, float vs, float tau, float maxr,
                                               const uint64_t *__restrict__ tkeys,
                                               const uint32_t *__restrict__ tvals, uint64_t tmask,
                                               uint32_t *__restrict__ cand, int64_t n_box, S *D, S *W,
                                               SubmapMeta *meta, uint8_t *__restrict__ dirty, int xcd)
{
    int64_t wg = blockIdx.x, n_wg = gridDim.x;
    if constexpr (E::rides) {
        __shared__ EdtXyLds<1> elds;
        extern __shared__ __align__(16) uint32_t colw[];
        if (wg < edt.grid_y) {
            edt.run_xy(elds, colw);
            return;
        }
        wg -= edt.grid_y;
        n_wg -= edt.grid_y;
    }
    uint8_t *fresh = (uint8_t *)cand;
    if (FUSED && wg == 0 && threadIdx.x == 0) meta->batch_n0 = meta->n_blocks;
    const int64_t j = work_item(wg, n_wg, xcd) * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (j >= n_box) return;  // uniform across the wave
    int bx, by, bz;
    box_block(f, j, bx, by, bz);
    if (!block_may_be_visible(f, vs, bx, by, bz)) {  // uniform across the wave
        if (lane == 0) {
            if (FUSED) fresh[j] = 0;
            else cand[j] = 0;
        }
        return;
    }
    // the home slot of the block's key is read before the validity test, so
    // that its latency overlaps the depth reads
    // (every lane reads the same slot: one request, no branch)
    const uint64_t key = pack_key(bx, by, bz);
    const HashProbe hp = hash_first(tkeys, tvals, tmask, key);
    const int ix = 8 * bx + (lane & 7);
    const int iy = 8 * by + (lane >> 3);
    float sdf[8], wt[8];
    const uint32_t okm = proj_column(f, vs, tau, maxr, ix, iy, 8 * bz, sdf, wt);
    const uint64_t m = __ballot(okm != 0);
    uint32_t out = 0;
    if (m) {
        int64_t idx = -1;
        if (lane == 0) idx = hash_resolve(hp, tkeys, tvals, tmask, key);
        idx = __shfl(idx, 0, 64);
        out = idx >= 0 ? (uint32_t)idx + 1u : kNew;
        if (FUSED && idx >= 0) {
            const int n_ok = update_column(D + idx * 512 + lane, W + idx * 512 + lane, sdf, wt, okm, tau, false);
            if (lane == 0) {
                atomicAdd(&meta->n_updates, (unsigned long long)n_ok);
                dirty[idx] = 1;
            }
        }
    }
    if (lane == 0) {
        if (FUSED) fresh[j] = out == kNew;
        else cand[j] = out;
    }
}

// Exclusive scan of one int64 per thread over a 1024-thread workgroup.
__device__ int64_t block_exclusive_scan(int64_t v, int64_t *lds, int64_t *total)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    int64_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        int64_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) lds[wid] = x;
    __syncthreads();
    if (wid == 0) {
        int64_t w = lane < nw ? lds[lane] : 0;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            int64_t y = __shfl_up(w, o, 64);
            if (lane >= o) w += y;
        }
        if (lane < nw) lds[lane] = w;  // inclusive wave totals
    }
    __syncthreads();
    const int64_t before = (wid > 0 ? lds[wid - 1] : 0) + x - v;
    *total = lds[nw - 1];
    __syncthreads();
    return before;
}

// Block count and call sequence for the host's bound (pinned host memory).
__device__ __forceinline__ void publish_count(uint64_t *host_nb, uint64_t seq, int64_t n_blocks)
{
    *(volatile uint64_t *)host_nb = ((seq & 0xFFFFFFull) << 40) | (uint64_t)n_blocks;
}

__global__ void k_publish(const SubmapMeta *meta, uint64_t *host_nb, uint64_t seq)
{
    publish_count(host_nb, seq, meta->n_blocks);
}

__global__ __launch_bounds__(1024) void k_scan(const uint32_t *__restrict__ cand, int64_t n_box, FrameArgs f,
                                               SubmapMeta *meta, int64_t cap, int64_t table_limit,
                                               uint64_t *__restrict__ t_key, uint32_t *__restrict__ t_idx,
                                               uint64_t *host_nb, uint64_t seq)
{
    __shared__ int64_t lds[16];
    __shared__ int32_t red[6][16];
    const int tid = threadIdx.x;
    const int64_t C = (n_box + blockDim.x - 1) / blockDim.x;
    const int64_t beg = std::min<int64_t>((int64_t)tid * C, n_box);
    const int64_t end = std::min<int64_t>(beg + C, n_box);
    // the first kCache entries of the thread's range stay in registers for
    // the second pass; their reads are issued together
    constexpr int kCache = 8;
    uint32_t cv[kCache];
#pragma unroll
    for (int q = 0; q < kCache; ++q) cv[q] = beg + q < end ? cand[beg + q] : 0u;
    int64_t nt = 0, nn = 0;
#pragma unroll
    for (int q = 0; q < kCache; ++q) {
        nt += cv[q] != 0;
        nn += cv[q] == kNew;
    }
    for (int64_t j = beg + kCache; j < end; ++j) {
        const uint32_t v = cand[j];
        nt += v != 0;
        nn += v == kNew;
    }
    // one scan of both counts (touched in the low, new in the high 32 bits:
    // each is at most n_box < 2^32, so the fields never carry into each other)
    int64_t tot;
    const int64_t off = block_exclusive_scan(nt | (nn << 32), lds, &tot);
    int64_t off_t = off & 0xFFFFFFFFll, off_n = off >> 32;
    const int64_t tot_t = tot & 0xFFFFFFFFll, tot_n = tot >> 32;
    const int64_t n0 = meta->n_blocks;
    __syncthreads();  // every thread has read n_blocks before it changes
    const bool pool_full = n0 + tot_n > cap;
    const bool table_full = n0 + tot_n > table_limit;
    if (pool_full || table_full) {
        if (tid == 0) {
            meta->status = pool_full ? COVOX_EPOOL_FULL : COVOX_ETABLE_FULL;
            meta->n_new = 0;
            meta->n_touched = 0;
            publish_count(host_nb, seq, n0);
        }
        return;
    }
    int32_t lo[3] = {INT32_MAX, INT32_MAX, INT32_MAX}, hi[3] = {INT32_MIN, INT32_MIN, INT32_MIN};
    auto emit = [&](int64_t j, uint32_t v) {
        if (!v) return;
        int bx, by, bz;
        box_block(f, j, bx, by, bz);
        uint32_t idx;
        if (v == kNew) {
            idx = (uint32_t)(n0 + off_n++) | 0x80000000u;
            lo[0] = min(lo[0], bx); lo[1] = min(lo[1], by); lo[2] = min(lo[2], bz);
            hi[0] = max(hi[0], bx); hi[1] = max(hi[1], by); hi[2] = max(hi[2], bz);
        } else {
            idx = v - 1u;
        }
        t_key[off_t] = pack_key(bx, by, bz);
        t_idx[off_t] = idx;
        ++off_t;
    };
#pragma unroll
    for (int q = 0; q < kCache; ++q)
        if (beg + q < end) emit(beg + q, cv[q]);
    for (int64_t j = beg + kCache; j < end; ++j) emit(j, cand[j]);
    // box of the new blocks: wave reduction, then across waves
    const int lane = tid & 63, wid = tid >> 6, nw = blockDim.x >> 6;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        for (int o = 32; o > 0; o >>= 1) {
            lo[a] = min(lo[a], __shfl_xor(lo[a], o, 64));
            hi[a] = max(hi[a], __shfl_xor(hi[a], o, 64));
        }
        if (lane == 0) { red[a][wid] = lo[a]; red[3 + a][wid] = hi[a]; }
    }
    __syncthreads();
    if (tid == 0) {
        int32_t L[3], Hh[3];
        for (int a = 0; a < 3; ++a) {
            L[a] = INT32_MAX; Hh[a] = INT32_MIN;
            for (int w = 0; w < nw; ++w) { L[a] = min(L[a], red[a][w]); Hh[a] = max(Hh[a], red[3 + a][w]); }
        }
        if (tot_n > 0) {
            for (int a = 0; a < 3; ++a) {
                if (n0 == 0) { meta->bmin[a] = L[a]; meta->bmax[a] = Hh[a]; }
                else { meta->bmin[a] = min(meta->bmin[a], L[a]); meta->bmax[a] = max(meta->bmax[a], Hh[a]); }
            }
        }
        meta->n_blocks = n0 + tot_n;
        meta->n_new = (int32_t)tot_n;
        meta->n_touched = (int32_t)tot_t;
        publish_count(host_nb, seq, n0 + tot_n);
    }
}

// One wave per touched block, after the scan of a frame that might overflow.
template <typename S, typename E>
__global__ __launch_bounds__(256) void k_integrate(const E edt, FrameArgs f, float vs, float tau, float maxr,
                                                   SubmapMeta *__restrict__ meta,
                                                   const uint64_t *__restrict__ t_key,
                                                   const uint32_t *__restrict__ t_idx, uint64_t *keys, S *D, S *W,
                                                   uint64_t *tkeys, uint32_t *tvals, uint64_t tmask,
                                                   uint8_t *__restrict__ dirty)
{
    int64_t wg = blockIdx.x, n_wg = gridDim.x;
    if constexpr (E::rides) {
        __shared__ EdtZLds<1> elds;
        extern __shared__ __align__(16) uint32_t colw[];
        if (wg < edt.grid_z) {
            edt.run_z(elds, colw);
            return;
        }
        wg -= edt.grid_z;
        n_wg -= edt.grid_z;
    }
    const int64_t wave = (wg * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = (n_wg * blockDim.x) >> 6;
    const int lane = threadIdx.x & 63;
    const int64_t n_t = (int64_t)meta->n_touched;
    for (int64_t t = wave; t < n_t; t += nwaves) {
        const uint32_t v = t_idx[t];
        const bool is_new = (v >> 31) != 0;
        const uint64_t key = t_key[t];
        const int64_t idx = v & 0x7FFFFFFFu;
        int bx, by, bz;
        unpack_key(key, bx, by, bz);
        if (is_new && lane == 0) {
            keys[idx] = key;
            hash_insert(tkeys, tvals, tmask, key, (uint32_t)idx);
        }
        const int ix = 8 * bx + (lane & 7);
        const int iy = 8 * by + (lane >> 3);
        float sdf[8], wt[8];
        const uint32_t okm = proj_column(f, vs, tau, maxr, ix, iy, 8 * bz, sdf, wt);
        const int n_ok = update_column(D + idx * 512 + lane, W + idx * 512 + lane, sdf, wt, okm, tau, is_new);
        if (lane == 0) {
            atomicAdd(&meta->n_updates, (unsigned long long)n_ok);
            dirty[idx] = 1;
        }
    }
}

// The flag bytes (0 or 1) of blocks 64 g .. 64 g + 63 of the box as bits, in one go.
__device__ __forceinline__ uint64_t flags64(const uint8_t *fresh, int64_t n_box, int64_t g)
{
    const ulonglong2 *p = (const ulonglong2 *)fresh;
    const int64_t last = (n_box - 1) >> 4;  // the last 16 bytes that hold a flag
    ulonglong2 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = p[min(4 * g + k, last)];
    uint64_t m = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        // byte i of eight goes to bit i of the product's top byte, without a carry
        // (bytes beyond the box can hold anything)
        const uint64_t x = v[k].x & 0x0101010101010101ull, y = v[k].y & 0x0101010101010101ull;
        m |= ((x * 0x0102040810204080ull) >> 56) << (16 * k);
        m |= ((y * 0x0102040810204080ull) >> 56) << (16 * k + 8);
    }
    const int64_t left = n_box - 64 * g;
    return left >= 64 ? m : left <= 0 ? 0 : m & ((1ull << left) - 1ull);
}

// The new blocks of a fused probe, in box order (= key order): keys, table entries,
// first update, and by the last workgroup the counts.  A frame adds a few of them,
// and what it costs is latency: a kernel of one workgroup that ordered them first
// took 8 us of a 25 us frame, and its launch 5 us of the host's time.  Here every
// wave reads all flags (64 blocks a lane, 4096 at once) and finds
// the position of its own new blocks by ballots; the block count of before the
// frame was put aside by the probe, so nothing waits for anything: 8 us in place of 6 + 8 and a launch.
template <typename S, typename E>
__global__ __launch_bounds__(256) void k_integrate_new(const E edt, FrameArgs f, float vs, float tau, float maxr, SubmapMeta *meta,
                                                       const uint8_t *__restrict__ fresh, int64_t n_box,
                                                       uint64_t *keys, S *D, S *W, uint64_t *tkeys, uint32_t *tvals,
                                                       uint64_t tmask, uint8_t *__restrict__ dirty, int64_t cap,
                                                       int64_t table_limit, uint64_t *host_nb, uint64_t seq)
{
    int64_t wg = blockIdx.x, n_wg = gridDim.x;
    if constexpr (E::rides) {
        __shared__ EdtZLds<1> elds;
        extern __shared__ __align__(16) uint32_t colw[];
        if (wg < edt.grid_z) {
            edt.run_z(elds, colw);
            return;
        }
        wg -= edt.grid_z;
        n_wg -= edt.grid_z;
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int64_t n0 = meta->batch_n0, groups = (n_box + 63) >> 6;
    if (wg == n_wg - 1) {
        __shared__ int32_t s_box[4][6];
        __shared__ int64_t s_cnt[4];
        int64_t cnt = 0;
        int32_t b[6] = {INT32_MAX, INT32_MAX, INT32_MAX, INT32_MIN, INT32_MIN, INT32_MIN};
        for (int64_t g = threadIdx.x; g < groups; g += 256) {
            uint64_t m = flags64(fresh, n_box, g);
            if (!m) continue;
            cnt += __popcll(m);
            int p[3];
            box_block(f, 64 * g, p[0], p[1], p[2]);
            for (; m; m >>= 1) {
                if (m & 1)
                    for (int a = 0; a < 3; ++a) {
                        b[a] = min(b[a], p[a]);
                        b[3 + a] = max(b[3 + a], p[a]);
                    }
                if (++p[2] == f.blo[2] + f.bdim[2]) {
                    p[2] = f.blo[2];
                    if (++p[1] == f.blo[1] + f.bdim[1]) {
                        p[1] = f.blo[1];
                        ++p[0];
                    }
                }
            }
        }
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            cnt += __shfl_xor(cnt, o, 64);
#pragma unroll
            for (int a = 0; a < 6; ++a) {
                const int32_t y = __shfl_xor(b[a], o, 64);
                b[a] = a < 3 ? min(b[a], y) : max(b[a], y);
            }
        }
        if (lane == 0) {
            s_cnt[wid] = cnt;
#pragma unroll
            for (int a = 0; a < 6; ++a) s_box[wid][a] = b[a];
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < 4; ++w) {
                cnt += s_cnt[w];
                for (int a = 0; a < 6; ++a) b[a] = a < 3 ? min(b[a], s_box[w][a]) : max(b[a], s_box[w][a]);
            }
            if (n0 + cnt > cap || n0 + cnt > table_limit) {  // none of them is entered
                meta->status = n0 + cnt > cap ? COVOX_EPOOL_FULL : COVOX_ETABLE_FULL;
                cnt = 0;
            }
            if (cnt > 0)
                for (int a = 0; a < 3; ++a) {
                    meta->bmin[a] = n0 == 0 ? b[a] : min(meta->bmin[a], b[a]);
                    meta->bmax[a] = n0 == 0 ? b[3 + a] : max(meta->bmax[a], b[3 + a]);
                }
            meta->n_blocks = n0 + cnt;
            meta->n_new = (int32_t)cnt;
            meta->n_touched = 0;
            publish_count(host_nb, seq, n0 + cnt);
        }
        return;
    }
    // The host's bound on the block count says that the whole box fits.  Should it not,
    // the new blocks are counted before any is entered, as k_scan does.
    if (n0 + n_box > min(cap, table_limit)) {  // uniform
        int64_t cnt = 0;
        for (int64_t g = lane; g < groups; g += 64) cnt += __popcll(flags64(fresh, n_box, g));
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) cnt += __shfl_xor(cnt, o, 64);
        if (n0 + cnt > min(cap, table_limit)) return;
    }
    int64_t t = wg * 4 + __builtin_amdgcn_readfirstlane(wid);  // this wave's next new block
    const int64_t nwaves = (n_wg - 1) * 4;
    int64_t base = 0;  // new blocks before the flags looked at
    for (int64_t g0 = 0; g0 < groups; g0 += 64) {  // uniform
        const uint64_t m = flags64(fresh, n_box, g0 + lane);
        const int n = __popcll(m);
        if (__ballot(n != 0) == 0) continue;
        int incl = n;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        const int tot = __builtin_amdgcn_readlane(incl, 63);
        for (; t < base + tot; t += nwaves) {  // uniform
            const int q = (int)(t - base);
            // the last lane with at most q new blocks before it holds this one
            const int src = 63 - __builtin_clzll(__ballot(incl - n <= q));
            uint64_t bits = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(m >> 32), src) << 32) |
                            (uint32_t)__builtin_amdgcn_readlane((int)m, src);
            for (int nth = q - __builtin_amdgcn_readlane(incl - n, src); nth > 0; --nth) bits &= bits - 1;
            const int64_t j = 64 * (g0 + src) + __builtin_ctzll(bits), idx = n0 + t;
            int bx, by, bz;
            box_block(f, j, bx, by, bz);
            if (lane == 0) {
                const uint64_t key = pack_key(bx, by, bz);
                keys[idx] = key;
                hash_insert(tkeys, tvals, tmask, key, (uint32_t)idx);
            }
            const int ix = 8 * bx + (lane & 7);
            const int iy = 8 * by + (lane >> 3);
            float sdf[8], wt[8];
            const uint32_t okm = proj_column(f, vs, tau, maxr, ix, iy, 8 * bz, sdf, wt);
            const int n_ok = update_column(D + idx * 512 + lane, W + idx * 512 + lane, sdf, wt, okm, tau, true);
            if (lane == 0) {
                atomicAdd(&meta->n_updates, (unsigned long long)n_ok);
                dirty[idx] = 1;
            }
        }
        base += tot;
    }
}

// ------------------------------------------------------- frame batches
// k_probe_batch tests every frame's box blocks against the table as it was
// before the batch; the allocation below numbers the new blocks, lists the
// others that some frame touches and collects the frames that touch a block in a
// 64-bit mask; k_integrate_batch gives each of them one workgroup that applies
// those frames in order in registers and writes D and W once.
//
// The allocation equals per-frame calls: a block is new in the first frame of the
// batch that touches it and not before the batch; new blocks take n_blocks + rank
// in (first frame, key) order; the frames up to the first one that would overflow
// the pool or the table are committed, the rest dropped.
//   k_batch_tiles     clears the first-frame table; depth maxima for the probe
//   k_probe_batch     candidates; first frame of every new key (min, in the table)
//   k_batch_rank      one workgroup a frame: the frame's first-time new blocks
//                     ranked in box order (= key order); the last workgroup to end
//                     sums the frames, checks the capacity and sets the counts
//   k_batch_activate  keys, table entries, touched masks, the list

// A candidate: 0 none, index + 1 of a block that existed before the batch, or
// kCandNew | slot of its key in the first-frame table.
constexpr uint32_t kCandNew = 0x80000000u;

// fcount: new blocks per frame, first new index per frame, the workgroups of
// k_batch_rank that have ended, and per frame the box of its new blocks.
constexpr int kCountOff = kMaxBatch, kCountTicket = 2 * kMaxBatch, kCountBox = 2 * kMaxBatch + 1;
constexpr int kCountWords = kCountBox + 3 * kMaxBatch;

// The largest valid depth of every 8 x 8, 16 x 16, 32 x 32 and 64 x 64 pixel tile
// (-inf: none valid), one workgroup a 64 x 64 region, regions padded beyond the
// image.  level l of a frame starts at tile_level(l) * regions.
constexpr int kTileLevels = 4, kTilesPerRegion = 64 + 16 + 4 + 1;
__device__ __forceinline__ int tile_level(int l) { return l == 0 ? 0 : l == 1 ? 64 : l == 2 ? 80 : 84; }

// Bound by the reading of the depth images: 15 us for 64 of 640 x 480 (79 MB).
__global__ __launch_bounds__(256) void k_batch_tiles(const FrameArgs *__restrict__ frames, int rx, float maxr,
                                                     float *__restrict__ tiles, uint64_t *__restrict__ fkeys,
                                                     uint2 *__restrict__ finfo, int64_t fslots, int64_t *fcount)
{
    __shared__ float s_16[4][4];
    const int64_t wg = (int64_t)blockIdx.y * gridDim.x + blockIdx.x, threads = (int64_t)gridDim.x * gridDim.y * 256;
    for (int64_t i = wg * 256 + threadIdx.x; i < fslots; i += threads) {
        fkeys[i] = kEmpty;
        finfo[i] = make_uint2(0xFFFFFFFFu, 0u);
    }
    if (wg == 0 && threadIdx.x == 0) fcount[kCountTicket] = 0;

    const FrameArgs &f = frames[blockIdx.y];
    const int regions = gridDim.x, ty = blockIdx.x / rx, tx = blockIdx.x % rx;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    // a lane's column of 16 rows; beyond the image the edge pixel stands in, which
    // belongs to the same tile or to none that is read
    const int x = min(64 * tx + lane, f.W - 1);
    float d[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) d[r] = f.depth[(int64_t)min(64 * ty + 16 * wid + r, f.H - 1) * f.W + x];
    float a[2] = {-INFINITY, -INFINITY};
#pragma unroll
    for (int r = 0; r < 16; ++r) a[r >> 3] = fmaxf(a[r >> 3], d[r] > 0.0f && d[r] <= maxr ? d[r] : -INFINITY);
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) {
        a[0] = fmaxf(a[0], __shfl_xor(a[0], o, 64));
        a[1] = fmaxf(a[1], __shfl_xor(a[1], o, 64));
    }
    float *out = tiles + (int64_t)blockIdx.y * regions * kTilesPerRegion;
    if ((lane & 7) == 0) {
        float *o = out + (int64_t)(8 * ty + 2 * wid) * (8 * rx) + 8 * tx + (lane >> 3);
        o[0] = a[0];
        o[8 * rx] = a[1];
    }
    float b = fmaxf(a[0], a[1]);
    b = fmaxf(b, __shfl_xor(b, 8, 64));
    if ((lane & 15) == 0) {
        out[(int64_t)tile_level(1) * regions + (int64_t)(4 * ty + wid) * (4 * rx) + 4 * tx + (lane >> 4)] = b;
        s_16[wid][lane >> 4] = b;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int qx = threadIdx.x & 1, qy = threadIdx.x >> 1;
        float c = fmaxf(fmaxf(s_16[2 * qy][2 * qx], s_16[2 * qy][2 * qx + 1]),
                        fmaxf(s_16[2 * qy + 1][2 * qx], s_16[2 * qy + 1][2 * qx + 1]));
        out[(int64_t)tile_level(2) * regions + (int64_t)(2 * ty + qy) * (2 * rx) + 2 * tx + qx] = c;
        c = fmaxf(c, __shfl_xor(c, 1, 64));
        c = fmaxf(c, __shfl_xor(c, 2, 64));
        if (threadIdx.x == 0) out[(int64_t)tile_level(3) * regions + (int64_t)ty * rx + tx] = c;
    }
}

// What a block's voxel centres can see of a frame: the tiles of level `level` that
// hold their pixels, at most 8 x 8, and the depth below which none is valid.
struct BlockView {
    int tx0, tx1, ty0, ty1, level;
    float reach;
};

// False only if no voxel centre of the block can pass the validity test, from the
// box along the camera's axes that holds the centres (a sphere drops a tenth fewer);
// else its view.  The box is widened by the rounding of the camera coordinates and
// the pixels by two, so that the decision is safe; a block that reaches the camera
// or covers more than 384 pixels is left undecided (reach -inf).
__device__ __forceinline__ bool view_block(const FrameArgs &f, float vs, float tau, int bx, int by, int bz,
                                           BlockView &w)
{
    if (!block_may_be_visible(f, vs, bx, by, bz)) return false;
    const float cx = (float)(8 * bx + 4) * vs, cy = (float)(8 * by + 4) * vs, cz = (float)(8 * bz + 4) * vs;
    const float px = ((f.R[0] * cx + f.R[1] * cy) + f.R[2] * cz) + f.t[0];
    const float py = ((f.R[3] * cx + f.R[4] * cy) + f.R[5] * cz) + f.t[1];
    const float pz = ((f.R[6] * cx + f.R[7] * cy) + f.R[8] * cz) + f.t[2];
    const float slack = 1e-6f * (((fabsf(cx) + fabsf(cy)) + fabsf(cz)) +
                                 ((fabsf(f.t[0]) + fabsf(f.t[1])) + fabsf(f.t[2])));
    const float ex = f.cull_e[0] + slack, ey = f.cull_e[1] + slack, ez = f.cull_e[2] + slack;
    w.tx0 = w.tx1 = w.ty0 = w.ty1 = 0;
    w.level = kTileLevels - 1;
    w.reach = -INFINITY;
    const float zn = pz - ez, zf = pz + ez;
    if (!(zn > 0.5f * f.cull_r)) return true;
    const float in = 1.0f / zn, far = 1.0f / zf;
    const float xl = px - ex, xh = px + ex, yl = py - ey, yh = py + ey;
    const float u0 = f.K[0] * (xl * (xl < 0.0f ? in : far)) + f.K[2] - 2.0f;
    const float u1 = f.K[0] * (xh * (xh < 0.0f ? far : in)) + f.K[2] + 2.0f;
    const float v0 = f.K[1] * (yl * (yl < 0.0f ? in : far)) + f.K[3] - 2.0f;
    const float v1 = f.K[1] * (yh * (yh < 0.0f ? far : in)) + f.K[3] + 2.0f;
    const float um = (float)(f.W - 1), vm = (float)(f.H - 1);
    if (u1 < 0.0f || u0 > um || v1 < 0.0f || v0 > vm) return false;
    const int iu0 = (int)fminf(fmaxf(u0, 0.0f), um), iu1 = (int)fminf(fmaxf(u1, 0.0f), um);
    const int iv0 = (int)fminf(fmaxf(v0, 0.0f), vm), iv1 = (int)fminf(fmaxf(v1, 0.0f), vm);
    const int ext = max(iu1 - iu0, iv1 - iv0);
    int l = 0;
    while (l < kTileLevels - 1 && ext > (48 << l)) ++l;
    if (ext > (48 << l)) return true;
    w.level = l;
    w.tx0 = iu0 >> (3 + l);
    w.tx1 = iu1 >> (3 + l);
    w.ty0 = iv0 >> (3 + l);
    w.ty1 = iv1 >> (3 + l);
    w.reach = zn * 0.999999f - tau;
    return true;
}

// Bound by arithmetic: a block without a valid voxel costs the exact test of all its
// 512, two divisions each, and of an outdoor frame's 7500 box blocks 2400 meet the
// frustum but 700 hold a valid voxel.  One wave a block took 179 us for 64 such
// frames.  Now the frustum test takes a lane a block, not a wave; those that pass
// are laid side by side in LDS, and a wave drops half of the hidden ones by reading
// the depth maxima of the up to 8 x 8 tiles that a block covers, a tile a lane;
// what is left takes the exact test, the bottom row of voxels first, which decides
// most blocks that hold a valid one; the table look-ups take a lane a block again.
// 75 us.  A workgroup's blocks are spread over the box in runs of eight, so that
// each has its share of the frustum.
template <typename E>
__global__ __launch_bounds__(256) void k_probe_batch(const E edt, const FrameArgs *__restrict__ frames, float vs, float tau,
                                                     float maxr, const uint64_t *__restrict__ tkeys,
                                                     const uint32_t *__restrict__ tvals, uint64_t tmask,
                                                     const float *__restrict__ tiles, int rx, int regions,
                                                     uint64_t *fkeys, uint2 *finfo, uint64_t fmask,
                                                     uint32_t *__restrict__ cand, int64_t stride, int per,
                                                     int64_t n_share, int F, int xcd)
{
    int64_t wg = blockIdx.x, n_wg = gridDim.x;
    if constexpr (E::rides) {
        __shared__ EdtXyLds<1> elds;
        extern __shared__ __align__(16) uint32_t colw[];
        if (wg < edt.grid_y) {
            edt.run_xy(elds, colw);
            return;
        }
        wg -= edt.grid_y;
        n_wg -= edt.grid_y;
    }
    __shared__ int64_t s_j[256];
    __shared__ uint64_t s_key[256];
    __shared__ int s_x[256], s_y[256], s_l[256];
    __shared__ float s_reach[256];
    __shared__ int s_hit[256];
    __shared__ int s_n;
    // work items: (frame, share of its blocks), frame-major, in a grid stride;
    // with XCD order the workgroups on XCD r (w mod 8 = r) stride over the r-th
    // eighth of the items
    const int64_t n_items = n_share * F;
    int64_t first, end, step;
    if (xcd) {
        const int64_t part = (n_items + 7) / 8, r = wg & 7;
        first = r * part + (wg >> 3);
        end = min(n_items, (r + 1) * part);
        step = n_wg >> 3;
    } else {
        first = wg;
        end = n_items;
        step = n_wg;
    }
    const int lane = threadIdx.x & 63, tid = threadIdx.x;
    for (int64_t item = first; item < end; item += step) {  // uniform
        const int fi = (int)(item / n_share);
        const FrameArgs &f = frames[fi];
        const float *ft = tiles + (int64_t)fi * regions * kTilesPerRegion;
        const int64_t n_box = (int64_t)f.bdim[0] * f.bdim[1] * f.bdim[2];
        if (tid == 0) s_n = 0;
        __syncthreads();
        {
            const int64_t j = ((tid >> 3) * n_share + item % n_share) * 8 + (tid & 7);
            BlockView w;
            bool in = false;
            int bx = 0, by = 0, bz = 0;
            if (tid < per && j < n_box) {
                box_block(f, j, bx, by, bz);
                in = view_block(f, vs, tau, bx, by, bz, w);
                if (!in) cand[(int64_t)fi * stride + j] = 0;
            }
            const uint64_t m = __ballot(in);
            int at = 0;
            if (lane == 0 && m) at = atomicAdd(&s_n, __popcll(m));
            at = __shfl(at, 0, 64) + __popcll(m & ((1ull << lane) - 1ull));
            if (in) {
                s_j[at] = j;
                s_key[at] = pack_key(bx, by, bz);
                s_x[at] = w.tx0 | (w.tx1 - w.tx0) << 28;
                s_y[at] = w.ty0 | (w.ty1 - w.ty0) << 28;
                s_l[at] = w.level;
                s_reach[at] = w.reach;
            }
        }
        __syncthreads();
        const int n = __builtin_amdgcn_readfirstlane(s_n);
        // A wave takes every fourth block.  (Not the next one by a counter: the lane-0
        // add at the loop's head and the lane-0 store at its end let the compiler take
        // the two as a loop of lane 0 around one of the other lanes, which never ends.)
        for (int at = __builtin_amdgcn_readfirstlane(tid >> 6); at < n; at += 4) {
            const int l = s_l[at], x = s_x[at], y = s_y[at];
            const int tx = (x & 0x0FFFFFFF) + min(lane & 7, (int)((uint32_t)x >> 28));
            const int ty = (y & 0x0FFFFFFF) + min(lane >> 3, (int)((uint32_t)y >> 28));
            const float dm = ft[(int64_t)tile_level(l) * regions + (int64_t)ty * ((8 >> l) * rx) + tx];
            bool hit = __ballot(dm >= s_reach[at]) != 0;
            if (hit) {  // uniform across the wave
                int bx, by, bz;
                unpack_key(s_key[at], bx, by, bz);
                const int ix = 8 * bx + (lane & 7), iy = 8 * by + (lane >> 3);
                hit = __ballot(proj_any<0, 1>(f, vs, tau, maxr, ix, iy, 8 * bz)) != 0 ||
                      __ballot(proj_any<1, 8>(f, vs, tau, maxr, ix, iy, 8 * bz)) != 0;
            }
            if (lane == 0) s_hit[at] = hit;
        }
        __syncthreads();
        if (tid < n) {
            uint32_t out = 0;
            const int64_t j = s_j[tid];
            if (s_hit[tid]) {
                const uint64_t key = s_key[tid];
                const int64_t idx = hash_find(tkeys, tvals, tmask, key);
                if (idx >= 0) {
                    out = (uint32_t)idx + 1u;
                } else {
                    // the table holds twice as many slots as candidates; a stale
                    // read costs an atomic that changes nothing
                    uint64_t h = mix64(key) & fmask;
                    for (;; h = (h + 1) & fmask) {
                        unsigned long long k = *(const volatile uint64_t *)&fkeys[h];
                        if (k == kEmpty)
                            k = atomicCAS((unsigned long long *)&fkeys[h], (unsigned long long)kEmpty,
                                          (unsigned long long)key);
                        if (k == kEmpty || k == key) break;
                    }
                    if (*(const volatile uint32_t *)&finfo[h].x > (uint32_t)fi) atomicMin(&finfo[h].x, (uint32_t)fi);
                    out = kCandNew | (uint32_t)h;
                }
            }
            cand[(int64_t)fi * stride + j] = out;
        }
        __syncthreads();  // the lists are free again
    }
}

// Counts of a batch, by the last workgroup of k_batch_rank to end (one wave,
// F <= 64 frames).
__device__ void batch_commit(int F, int64_t *fcount, SubmapMeta *meta, int64_t cap, int64_t table_limit,
                             uint64_t *host_nb, uint64_t seq)
{
    const int lane = threadIdx.x & 63;
    const int64_t n0 = meta->n_blocks;
    // every read before the first use
    const int fl = min(lane, F - 1);
    const int32_t *fbox = (const int32_t *)(fcount + kCountBox);
    int64_t c = __hip_atomic_load(&fcount[fl], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int32_t box[6], old[6];
#pragma unroll
    for (int a = 0; a < 6; ++a) {
        box[a] = __hip_atomic_load(&fbox[6 * fl + a], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        old[a] = a < 3 ? meta->bmin[a] : meta->bmax[a - 3];
    }
    if (lane >= F) c = 0;
    int64_t incl = c;
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    const bool over = lane < F && (n0 + incl > cap || n0 + incl > table_limit);
    const uint64_t m = __ballot(over);
    const int committed = m ? __ffsll((long long)m) - 1 : F;
    if (lane < F) fcount[kCountOff + lane] = n0 + incl - c;
    // (all lanes take part in the shuffles)
    const int src = committed < F ? committed : 0;
    const int64_t before_fail = __shfl(incl - c, src, 64);
    const int64_t at_fail = __shfl(incl, src, 64);
    const int64_t total_all = __shfl(incl, 63, 64);
    const int64_t n_new = committed < F ? before_fail : total_all;
    // the box of the new blocks
#pragma unroll
    for (int a = 0; a < 6; ++a) {
        if (!(lane < committed && c > 0)) box[a] = a < 3 ? INT32_MAX : INT32_MIN;
        if (n_new == 0) continue;  // uniform
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t y = __shfl_xor(box[a], o, 64);
            box[a] = a < 3 ? min(box[a], y) : max(box[a], y);
        }
    }
    if (lane == 0) {
        if (committed < F) meta->status = n0 + at_fail > cap ? COVOX_EPOOL_FULL : COVOX_ETABLE_FULL;
        if (n_new > 0)
            for (int a = 0; a < 3; ++a) {
                meta->bmin[a] = n0 == 0 ? box[a] : min(old[a], box[a]);
                meta->bmax[a] = n0 == 0 ? box[3 + a] : max(old[3 + a], box[3 + a]);
            }
        meta->n_blocks = n0 + n_new;
        meta->n_new = (int32_t)n_new;
        meta->n_touched = 0;
        meta->batch_n0 = n0;
        meta->batch_frames = committed;
        publish_count(host_nb, seq, n0 + n_new);
    }
}

// Bound by latency (one workgroup a frame): a candidate's way was its key from the
// box, its slot by probing and its first frame, eight in turn to a lane, 18 us for
// 64 outdoor frames.  The candidate now names the slot, the four of a lane are in
// flight together, and places come from ballots: 13 us, with the counts' kernel
// (5 us) done by the last workgroup.
__global__ __launch_bounds__(1024) void k_batch_rank(const FrameArgs *__restrict__ frames,
                                                     const uint32_t *__restrict__ cand, int64_t stride,
                                                     const uint64_t *__restrict__ fkeys, uint2 *__restrict__ finfo,
                                                     int64_t *fcount, SubmapMeta *meta, int64_t cap,
                                                     int64_t table_limit, uint64_t *host_nb, uint64_t seq)
{
    constexpr int U = 4;  // runs of 64 candidates to a wave at once
    __shared__ int s_run[16 * U], s_box[16][6], s_last;
    const int fi = blockIdx.x, F = gridDim.x;
    const FrameArgs &f = frames[fi];
    const int64_t n_box = (int64_t)f.bdim[0] * f.bdim[1] * f.bdim[2];
    const uint32_t *cf = cand + (int64_t)fi * stride;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    int box[6] = {INT32_MAX, INT32_MAX, INT32_MAX, INT32_MIN, INT32_MIN, INT32_MIN};
    int64_t base = 0;
    for (int64_t j0 = 0; j0 < n_box; j0 += 1024 * U) {  // uniform
        uint32_t v[U], h[U];
        bool mine[U];
        uint64_t m[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int64_t j = j0 + 1024 * k + tid;
            v[k] = cf[j < n_box ? j : 0];
            if (j >= n_box) v[k] = 0;
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            h[k] = v[k] & kCandNew ? v[k] & ~kCandNew : 0u;  // slot 0 stands in
            mine[k] = finfo[h[k]].x == (uint32_t)fi;
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            mine[k] = mine[k] && (v[k] & kCandNew);
            m[k] = __ballot(mine[k]);
            if (lane == 0) s_run[16 * k + wid] = __popcll(m[k]);
        }
        __syncthreads();
        // every wave sums the 64 runs for itself
        const int c = s_run[lane];
        int incl = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int before = __shfl(incl - c, 16 * k + wid, 64);
            if (mine[k]) {
                finfo[h[k]].y = (uint32_t)(base + before + __popcll(m[k] & ((1ull << lane) - 1ull)));
                int b[3];
                unpack_key(fkeys[h[k]], b[0], b[1], b[2]);
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    box[a] = min(box[a], b[a]);
                    box[3 + a] = max(box[3 + a], b[a]);
                }
            }
        }
        base += __shfl(incl, 63, 64);
        __syncthreads();
    }
    if (base) {  // uniform: the box of the frame's new blocks (not read where it has none)
#pragma unroll
        for (int a = 0; a < 6; ++a) {
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_xor(box[a], o, 64);
                box[a] = a < 3 ? min(box[a], y) : max(box[a], y);
            }
            if (lane == 0) s_box[wid][a] = box[a];
        }
        __syncthreads();
        if (tid < 6) {
            int b = s_box[0][tid];
            for (int w = 1; w < 16; ++w) b = tid < 3 ? min(b, s_box[w][tid]) : max(b, s_box[w][tid]);
            int32_t *fbox = (int32_t *)(fcount + kCountBox) + 6 * fi;
            __hip_atomic_store(&fbox[tid], b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();
    if (tid == 0) {
        __hip_atomic_store(&fcount[fi], base, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __threadfence();  // (the workgroup's stores before the barrier too)
        s_last = atomicAdd((unsigned long long *)&fcount[kCountTicket], 1ull) == (unsigned long long)(F - 1);
        __threadfence();
    }
    __syncthreads();
    if (s_last && wid == 0) batch_commit(F, fcount, meta, cap, table_limit, host_nb, seq);
}

// Bound by atomics.  On shared addresses, six for the block box and one for the list
// per new block, they made 54 us of an outdoor batch (2000 new blocks); the box now
// comes with the ranks, new blocks are a range of indices that needs no list, and a
// workgroup takes its places in the list of the others together: 8 us.
__global__ __launch_bounds__(256) void k_batch_activate(const FrameArgs *__restrict__ frames,
                                                        const uint32_t *__restrict__ cand, int64_t stride,
                                                        const int64_t *__restrict__ fcount, SubmapMeta *meta,
                                                        uint64_t *keys, uint64_t *tkeys, uint32_t *tvals,
                                                        uint64_t tmask, const uint64_t *__restrict__ fkeys,
                                                        const uint2 *__restrict__ finfo, unsigned long long *touch,
                                                        uint32_t *list)
{
    __shared__ int s_n, s_at;
    const int fi = blockIdx.y;
    if (fi >= meta->batch_frames) return;  // uniform: frame not committed
    const FrameArgs &f = frames[fi];
    const int64_t n_box = (int64_t)f.bdim[0] * f.bdim[1] * f.bdim[2];
    const int64_t *foff = fcount + kCountOff;
    for (int64_t j0 = (int64_t)blockIdx.x * blockDim.x; j0 < n_box; j0 += (int64_t)gridDim.x * blockDim.x) {  // uniform
        if (threadIdx.x == 0) s_n = 0;
        __syncthreads();
        const int64_t j = j0 + threadIdx.x;
        const uint32_t v = j < n_box ? cand[(int64_t)fi * stride + j] : 0u;
        uint32_t idx = 0;
        int at = -1;
        if (v & kCandNew) {
            const uint32_t h = v & ~kCandNew;
            const uint2 first = finfo[h];
            idx = (uint32_t)(foff[first.x] + first.y);
            if (first.x == (uint32_t)fi) {
                const uint64_t key = fkeys[h];
                keys[idx] = key;
                hash_insert(tkeys, tvals, tmask, key, idx);
            }
            atomicOr(&touch[idx], 1ull << fi);
        } else if (v) {
            idx = v - 1u;  // existed before the batch
            if (atomicOr(&touch[idx], 1ull << fi) == 0) at = atomicAdd(&s_n, 1);  // the first to touch it
        }
        __syncthreads();
        if (threadIdx.x == 0 && s_n) s_at = atomicAdd(&meta->n_touched, s_n);
        __syncthreads();
        if (at >= 0) list[s_at + at] = idx;
        __syncthreads();
    }
}

// Storage rounding of a value kept in registers across frames, so that the
// batch matches per-frame calls that store after every frame.
template <typename S> __device__ __forceinline__ float stored(float v);
template <> __device__ __forceinline__ float stored<float>(float v) { return v; }
template <> __device__ __forceinline__ float stored<__half>(float v) { return __half2float(__float2half_rn(v)); }

// One workgroup a block, its four waves two z rows each.  A voxel's frames have to
// be applied in order, so the block seen by most frames sets the time: each step
// was a projection, a gather of depths and an update, one after the other, for
// eight voxels a lane (2.4 us a frame; 64 outdoor frames into 2000 blocks took 188
// us over the frames whose frustum holds the block, 157 over those that have a
// valid voxel in it, which the probe has found).  Now a lane has two voxels, and
// the next frame's depths are on their way while this one's are applied: 71 us.
// The registers that a second frame takes cost the eight-voxel form its occupancy.
constexpr int kBatchZ = 2;  // voxels of a lane

template <typename S, typename E>
__global__ __launch_bounds__(256) void k_integrate_batch(const E edt, const FrameArgs *__restrict__ frames,
                                                         SubmapMeta *__restrict__ meta,
                                                         const uint32_t *__restrict__ list,
                                                         const uint64_t *__restrict__ keys, S *D, S *W, float vs,
                                                         float tau, float maxr, uint8_t *__restrict__ dirty,
                                                         uint64_t *__restrict__ touch, int xcd)
{
    int64_t wg = blockIdx.x, n_wg = gridDim.x;
    if constexpr (E::rides) {
        __shared__ EdtZLds<1> elds;
        extern __shared__ __align__(16) uint32_t colw[];
        if (wg < edt.grid_z) {
            edt.run_z(elds, colw);
            return;
        }
        wg -= edt.grid_z;
        n_wg -= edt.grid_z;
    }
    __shared__ int s_ok[4];
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t n_new = meta->n_new, n0 = meta->batch_n0;
    const int64_t n_t = n_new + meta->n_touched;
    // the new blocks, then the listed ones, in a grid stride; with XCD order, the
    // workgroups on XCD r (w mod 8 = r) stride over the r-th eighth of them
    int64_t t0, t1, step, first;
    if (xcd) {
        const int r = (int)(wg & 7);
        t0 = n_t * r / 8;
        t1 = n_t * (r + 1) / 8;
        step = n_wg >> 3;
        first = wg >> 3;
    } else {
        t0 = 0;
        t1 = n_t;
        step = n_wg;
        first = wg;
    }
    int n_ok = 0;
    for (int64_t t = t0 + first; t < t1; t += step) {
        const bool is_new = t < n_new;
        const int64_t idx = is_new ? n0 + t : list[t - n_new];
        int bx, by, bz;
        unpack_key(keys[idx], bx, by, bz);
        const float cx = ((float)(8 * bx + (lane & 7)) + 0.5f) * vs;
        const float cy = ((float)(8 * by + (lane >> 3)) + 0.5f) * vs;
        float cz[kBatchZ];
#pragma unroll
        for (int z = 0; z < kBatchZ; ++z) cz[z] = ((float)(8 * bz + kBatchZ * wid + z) + 0.5f) * vs;
        S *Db = D + idx * 512 + lane + 64 * kBatchZ * wid;
        S *Wb = W + idx * 512 + lane + 64 * kBatchZ * wid;
        float dv[kBatchZ], wv[kBatchZ];
#pragma unroll
        for (int z = 0; z < kBatchZ; ++z) {
            dv[z] = is_new ? 0.0f : ld(Db + 64 * z);
            wv[z] = is_new ? 0.0f : ld(Wb + 64 * z);
        }
        // the frames with a valid voxel in the block, in order (uniform)
        const uint64_t tm = touch[idx];
        const uint32_t tl = __builtin_amdgcn_readfirstlane((uint32_t)tm);
        const uint32_t th = __builtin_amdgcn_readfirstlane((uint32_t)(tm >> 32));
        uint64_t left = ((uint64_t)th << 32) | tl;
        struct Look {
            float pz[kBatchZ], d[kBatchZ];
            bool in[kBatchZ];
        };
        int wmode = 0;
        auto look = [&](Look &l) {  // pixel and depth of each voxel in the next frame
            const FrameArgs &f = frames[__ffsll((unsigned long long)left) - 1];
            left &= left - 1;
            wmode = f.weight_mode;
            int64_t pix[kBatchZ];
#pragma unroll
            for (int z = 0; z < kBatchZ; ++z) pix[z] = proj_pixel(f, cx, cy, cz[z], l.pz[z]);
#pragma unroll
            for (int z = 0; z < kBatchZ; ++z) {
                l.in[z] = pix[z] >= 0;
                l.d[z] = f.depth[l.in[z] ? pix[z] : 0];  // pixel 0 stands in, unused
            }
        };
        Look cur;
        bool more = left != 0;
        if (more) look(cur);
        while (more) {  // uniform
            Look next = cur;
            more = left != 0;
            if (more) look(next);
#pragma unroll
            for (int z = 0; z < kBatchZ; ++z) {  // as proj_column and update_column
                const float d = cur.d[z], sdf = d - cur.pz[z];
                const bool ok = cur.in[z] && d > 0.0f && d <= maxr && sdf >= -tau;
                n_ok += __popcll(__ballot(ok));
                if (ok) {
                    const float w = wmode == COVOX_WEIGHT_INV_DEPTH2 ? 1.0f / (d * d) : 1.0f;
                    const float Wn = wv[z] + w;
                    const float Dn = ((dv[z] * wv[z]) + (fminf(sdf, tau) * w)) / Wn;
                    dv[z] = stored<S>(Dn);
                    wv[z] = stored<S>(Wn);
                }
            }
            cur = next;
        }
#pragma unroll
        for (int z = 0; z < kBatchZ; ++z) {
            st(Db + 64 * z, dv[z]);
            st(Wb + 64 * z, wv[z]);
        }
        __syncthreads();  // every wave has read the mask
        if (threadIdx.x == 0) {
            dirty[idx] = 1;
            touch[idx] = 0;  // masks are zero between batches
        }
    }
    if (lane == 0) s_ok[wid] = n_ok;
    __syncthreads();
    if (threadIdx.x == 0) {
        const int all = s_ok[0] + s_ok[1] + s_ok[2] + s_ok[3];
        if (all) atomicAdd(&meta->n_updates, (unsigned long long)all);
    }
}

// ---------------------------------------------------------------- host

void rigid_inverse(const double *T, double *O)
{
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) O[4 * r + c] = T[4 * c + r];
    for (int r = 0; r < 3; ++r)
        O[4 * r + 3] = -((O[4 * r + 0] * T[3] + O[4 * r + 1] * T[7]) + O[4 * r + 2] * T[11]);
    O[12] = 0; O[13] = 0; O[14] = 0; O[15] = 1;
}

void rigid_mul(const double *A, const double *B, double *O)
{
    double t[16];
    for (int r = 0; r < 3; ++r) {
        for (int c = 0; c < 3; ++c)
            t[4 * r + c] = (A[4 * r + 0] * B[c] + A[4 * r + 1] * B[4 + c]) + A[4 * r + 2] * B[8 + c];
        t[4 * r + 3] = ((A[4 * r + 0] * B[3] + A[4 * r + 1] * B[7]) + A[4 * r + 2] * B[11]) + A[4 * r + 3];
    }
    t[12] = 0; t[13] = 0; t[14] = 0; t[15] = 1;
    for (int k = 0; k < 16; ++k) O[k] = t[k];
}

bool is_rigid(const double *T)
{
    for (int k = 0; k < 16; ++k)
        if (!std::isfinite(T[k])) return false;
    if (T[12] != 0 || T[13] != 0 || T[14] != 0 || T[15] != 1) return false;
    double e = 0;
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) {
            double s = 0;
            for (int k = 0; k < 3; ++k) s += T[4 * k + r] * T[4 * k + c];
            e = std::max(e, std::fabs(s - (r == c ? 1.0 : 0.0)));
        }
    const double det = T[0] * (T[5] * T[10] - T[6] * T[9]) - T[1] * (T[4] * T[10] - T[6] * T[8]) +
                       T[2] * (T[4] * T[9] - T[5] * T[8]);
    return e <= 1e-6 && det > 0;
}

// Workgroups of the new-block integration after a fused probe: a frame adds a
// few new blocks, except the first ones; the waves walk the flags with a
// stride.  One more takes the counts.
constexpr unsigned kNewGrid = 64;

// Launches a kernel with the EDT pass that waits for the next one on the stream, or
// alone: launch(pass, its workgroups, its LDS).
template <typename F>
void with_xy(covox_ctx *ctx, F launch)
{
    EdtPass *q = ctx->edt_pass;
    if (!q || !q->grid_y) return launch(NoEdt{}, 0u, 0u);
    launch(*q, q->grid_y, q->lds_y);
    q->grid_y = 0;
}

template <typename F>
void with_z(covox_ctx *ctx, F launch)
{
    EdtPass *q = ctx->edt_pass;
    if (!q || !q->grid_z) return launch(NoEdt{}, 0u, 0u);
    launch(*q, q->grid_z, q->lds_z);
    q->grid_z = 0;
}

template <typename S>
void launch_frame(covox_ctx *ctx, covox_submap *s, const FrameArgs &f, float vs, float tau, float maxr, uint64_t tmask,
                  int64_t table_limit, int64_t n_box, unsigned grid, bool fused)
{
    S *D = (S *)s->D, *W = (S *)s->W;
    const int xcd = ctx->tune.mapping_xcd_order != 0;
    const unsigned grid8 = (grid + 7) / 8 * 8;  // a multiple of 8 for the XCD order
    {
        TimedLaunch tl(ctx, COVOX_K_PROBE);
        with_xy(ctx, [&](const auto &e, unsigned more, unsigned lds) {
            using E = std::decay_t<decltype(e)>;
            if (fused)
                hipLaunchKernelGGL((k_probe<S, true, E>), dim3(grid8 + more), dim3(256), lds, ctx->stream, e, f, vs, tau,
                                   maxr, s->tkeys, s->tvals, tmask, ctx->cand, n_box, D, W, s->meta, s->dirty, xcd);
            else
                hipLaunchKernelGGL((k_probe<S, false, E>), dim3(grid8 + more), dim3(256), lds, ctx->stream, e, f, vs,
                                   tau, maxr, s->tkeys, s->tvals, tmask, ctx->cand, n_box, D, W, s->meta, s->dirty, xcd);
        });
    }
    if (!fused) launch_block_scan(ctx, s, f, n_box, table_limit);
    TimedLaunch tl(ctx, COVOX_K_INTEGRATE);
    with_z(ctx, [&](const auto &e, unsigned more, unsigned lds) {
        using E = std::decay_t<decltype(e)>;
        if (fused)
            hipLaunchKernelGGL((k_integrate_new<S, E>), dim3(std::min(grid, kNewGrid) + 1 + more), dim3(256), lds,
                               ctx->stream, e, f, vs, tau, maxr, s->meta, (const uint8_t *)ctx->cand, n_box, s->keys, D,
                               W, s->tkeys, s->tvals, tmask, s->dirty, s->cap, table_limit, s->pin_nb_dev, s->seq);
        else
            hipLaunchKernelGGL((k_integrate<S, E>), dim3(grid + more), dim3(256), lds, ctx->stream, e, f, vs, tau, maxr,
                               s->meta, ctx->t_key, ctx->t_idx, s->keys, D, W, s->tkeys, s->tvals, tmask, s->dirty);
    });
}

}  // namespace

// Tightens the host's upper bound on the block count without stalling: the
// count the scan kernel of call q last published, plus the box sizes of the
// calls enqueued after q.  Then registers the next call with its box size.
void refresh_block_bound(covox_submap *s, int64_t next_box)
{
    const uint64_t v = *s->pin_nb;
    const uint64_t q = v >> 40, cnt = v & ((1ull << 40) - 1);
    const uint64_t behind = (s->seq - q) & 0xFFFFFFull;  // calls enqueued after q
    if (behind < (uint64_t)covox_submap::kSeqRing && behind <= s->seq) {
        int64_t b = (int64_t)cnt;
        for (uint64_t k = s->seq - behind + 1; k <= s->seq; ++k) b += s->box_ring[k % covox_submap::kSeqRing];
        s->nb_upper = std::min(s->nb_upper, b);
    }
    s->seq++;
    s->box_ring[s->seq % covox_submap::kSeqRing] = next_box;
}

// A replay's kernels publish their counts under the capture's sequence numbers, so a
// count that an earlier replay (or an eager call since) left would pass for the running
// one's.  The replay is therefore a call of its own, of up to nb_upper blocks, that
// publishes its count when it ends.
int register_replay(covox_ctx *ctx, covox_submap *s)
{
    s->seq++;
    s->box_ring[s->seq % covox_submap::kSeqRing] = s->nb_upper;
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(1), 0, ctx->stream, s->meta, s->pin_nb_dev, s->seq);
    return hip_check(ctx, hipGetLastError(), "block count after a replay");
}

// The compaction launch shared by both integrators (one workgroup).
void launch_block_scan(covox_ctx *ctx, covox_submap *s, const FrameArgs &f, int64_t n_box, int64_t table_limit)
{
    TimedLaunch tl(ctx, COVOX_K_SCAN);
    hipLaunchKernelGGL(k_scan, dim3(1), dim3(1024), 0, ctx->stream, ctx->cand, n_box, f, s->meta, s->cap,
                       table_limit, ctx->t_key, ctx->t_idx, s->pin_nb_dev, s->seq);
}

// Frame parameters (pose rounded once from binary64) and the block box of
// the frustum.
int prepare_frame(covox_ctx *ctx, const covox_submap *s, const float *depth, int32_t H, int32_t W, const float K[4],
                  const double T_wc[16], FrameArgs &f, int64_t &n_box)
{
    const covox_params &p = ctx->p;
    if (!depth || H <= 0 || W <= 0 || !K || !T_wc) return fail(ctx, COVOX_EINVAL, "integrate: bad argument");
    if (!(K[0] > 0) || !(K[1] > 0) || !std::isfinite(K[2]) || !std::isfinite(K[3]))
        return fail(ctx, COVOX_EINVAL, "integrate: fx and fy must be positive");
    if (!is_rigid(T_wc)) return fail(ctx, COVOX_EINVAL, "integrate: T_world_cam is not a rigid transform");

    // camera <- submap, binary64, rounded once to binary32
    double inv_wc[16], T_cs[16];
    rigid_inverse(T_wc, inv_wc);
    rigid_mul(inv_wc, s->T_ws, T_cs);
    for (int r = 0; r < 3; ++r) {
        for (int c = 0; c < 3; ++c) f.R[3 * r + c] = (float)T_cs[4 * r + c];
        f.t[r] = (float)T_cs[4 * r + 3];
    }
    for (int k = 0; k < 4; ++k) f.K[k] = K[k];
    f.H = H;
    f.W = W;
    f.depth = depth;
    f.weight_mode = p.weight_mode;
    {
        // side planes through the camera centre for u in [-1.5, W + 0.5]
        // and v in [-1.5, H + 0.5] (one pixel beyond the pixel-centre test)
        const double fx = K[0], fy = K[1], cx = K[2], cy = K[3];
        const double n[4][3] = {{fx, 0, cx + 1.5}, {-fx, 0, W + 0.5 - cx}, {0, fy, cy + 1.5}, {0, -fy, H + 0.5 - cy}};
        for (int k = 0; k < 4; ++k) {
            const double len = std::sqrt(n[k][0] * n[k][0] + n[k][1] * n[k][1] + n[k][2] * n[k][2]);
            for (int a = 0; a < 3; ++a) f.plane[k][a] = (float)(n[k][a] / len);
        }
        f.zfar = (float)(p.max_range + p.trunc_vox * p.voxel_size);
        f.cull_r = (float)(1.01 * std::sqrt(3.0) * 3.5 * p.voxel_size + 1e-4);
        for (int a = 0; a < 3; ++a)
            f.cull_e[a] = (float)(1.01 * 3.5 * p.voxel_size *
                                  (std::fabs(T_cs[4 * a]) + std::fabs(T_cs[4 * a + 1]) + std::fabs(T_cs[4 * a + 2])) + 1e-4);
    }

    // Block box containing every voxel centre of the frustum cut at
    // max_range + tau (conservative; validity decides exactly).
    double inv_ws[16], T_sc[16];
    rigid_inverse(s->T_ws, inv_ws);
    rigid_mul(inv_ws, T_wc, T_sc);
    // submap <- camera, rounded once, for raycasting
    for (int r = 0; r < 3; ++r) {
        for (int c = 0; c < 3; ++c) f.Rs[3 * r + c] = (float)T_sc[4 * r + c];
        f.o[r] = (float)T_sc[4 * r + 3];
    }
    f.ray_carve = p.ray_carve;
    const double tau = p.trunc_vox * p.voxel_size;
    const double zf = p.max_range + tau;
    double mn[3], mx[3];
    for (int a = 0; a < 3; ++a) mn[a] = mx[a] = T_sc[4 * a + 3];
    const double us[2] = {-0.5, W - 0.5}, vv[2] = {-0.5, H - 0.5};
    for (double u : us)
        for (double v : vv) {
            const double pc[3] = {(u - K[2]) / K[0] * zf, (v - K[3]) / K[1] * zf, zf};
            for (int a = 0; a < 3; ++a) {
                const double w = T_sc[4 * a] * pc[0] + T_sc[4 * a + 1] * pc[1] + T_sc[4 * a + 2] * pc[2] + T_sc[4 * a + 3];
                mn[a] = std::min(mn[a], w);
                mx[a] = std::max(mx[a], w);
            }
        }
    n_box = 1;
    for (int a = 0; a < 3; ++a) {
        const int64_t ilo = (int64_t)std::floor(mn[a] / p.voxel_size - 0.5) - 1;
        const int64_t ihi = (int64_t)std::ceil(mx[a] / p.voxel_size - 0.5) + 1;
        const int64_t blo = ilo >= 0 ? ilo / 8 : -((-ilo + 7) / 8);
        const int64_t bhi = ihi >= 0 ? ihi / 8 : -((-ihi + 7) / 8);
        if (blo < -kKeyOff + 1 || bhi > kKeyOff - 2)
            return fail(ctx, COVOX_EINVAL, "integrate: frustum outside the addressable block range");
        f.blo[a] = (int32_t)blo;
        f.bdim[a] = (int32_t)(bhi - blo + 1);
        n_box *= f.bdim[a];
    }
    return COVOX_OK;
}

namespace {

// Uploads the frame parameters of a batch through pinned staging: slot k is
// reused only once its previous upload has completed.
int stage_frames(covox_ctx *ctx, const FrameArgs *fr, int32_t F)
{
    int rc;
    const int slot = ctx->frames_slot;
    ctx->frames_slot ^= 1;
    if (!ctx->frames_pin[slot]) {
        if ((rc = hip_check(ctx, hipHostMalloc((void **)&ctx->frames_pin[slot], sizeof(FrameArgs) * kMaxBatch,
                                               hipHostMallocDefault), "frame staging")))
            return rc;
        if ((rc = hip_check(ctx, hipEventCreateWithFlags(&ctx->frames_ev[slot], hipEventDisableTiming),
                            "frame staging event")))
            return rc;
    } else if ((rc = hip_check(ctx, hipEventSynchronize(ctx->frames_ev[slot]), "frame staging wait"))) {
        return rc;
    }
    ::memcpy(ctx->frames_pin[slot], fr, sizeof(FrameArgs) * F);
    if ((rc = hip_check(ctx, hipMemcpyAsync(ctx->frames_dev, ctx->frames_pin[slot], sizeof(FrameArgs) * F,
                                            hipMemcpyHostToDevice, ctx->stream), "frame batch upload")))
        return rc;
    return hip_check(ctx, hipEventRecord(ctx->frames_ev[slot], ctx->stream), "frame staging record");
}

}  // namespace

// Host bounds after frames with the given boxes were enqueued.
void grow_bounds(covox_submap *s, const FrameArgs &f)
{
    for (int a = 0; a < 3; ++a) {
        const int32_t lo = f.blo[a], hi = f.blo[a] + f.bdim[a] - 1;
        if (!s->bound_valid) { s->bound_lo[a] = lo; s->bound_hi[a] = hi; }
        else { s->bound_lo[a] = std::min(s->bound_lo[a], lo); s->bound_hi[a] = std::max(s->bound_hi[a], hi); }
    }
    s->bound_valid = true;
}

int integrate_frame(covox_ctx *ctx, covox_submap *s, const float *depth, int32_t H, int32_t W,
                    const float K[4], const double T_wc[16], bool *maybe_full)
{
    const covox_params &p = ctx->p;
    if (p.integrator == COVOX_RAYCAST) return raycast_frame(ctx, s, depth, H, W, K, T_wc, maybe_full);
    FrameArgs f;
    int64_t n_box = 0;
    int rc = prepare_frame(ctx, s, depth, H, W, K, T_wc, f, n_box);
    if (rc) return rc;
    const double tau = p.trunc_vox * p.voxel_size;
    // (flag bytes are read 16 at a time)
    if ((rc = ensure_buffer(ctx, (void **)&ctx->cand, &ctx->cand_cap, n_box + 4, sizeof(uint32_t), "candidates")))
        return rc;
    if ((rc = ensure_buffer(ctx, (void **)&ctx->t_key, &ctx->t_key_cap, n_box, sizeof(uint64_t), "touched keys")))
        return rc;
    if ((rc = ensure_buffer(ctx, (void **)&ctx->t_idx, &ctx->t_idx_cap, n_box, sizeof(uint32_t), "touched index")))
        return rc;

    const float vs = (float)p.voxel_size, tau_f = (float)tau, maxr = (float)p.max_range;
    const uint64_t tmask = (uint64_t)s->tcap - 1;
    const int64_t table_limit = (int64_t)(0.85 * (double)s->tcap);
    const unsigned grid = (unsigned)((n_box + 3) / 4);
    refresh_block_bound(s, n_box);  // s->seq is now this frame's sequence number
    // Existing blocks are updated by the probe when no capacity failure is
    // possible for this frame (every box block new would still fit).
    const bool fused = s->nb_upper + n_box <= std::min<int64_t>(s->cap, table_limit);
    if (p.precision == COVOX_FP16)
        launch_frame<__half>(ctx, s, f, vs, tau_f, maxr, tmask, table_limit, n_box, grid, fused);
    else
        launch_frame<float>(ctx, s, f, vs, tau_f, maxr, tmask, table_limit, n_box, grid, fused);
    if ((rc = hip_check(ctx, hipGetLastError(), "integrate launch"))) return rc;

    // host-side bounds
    s->nb_upper += n_box;
    grow_bounds(s, f);
    s->version++;
    *maybe_full = s->nb_upper > s->cap || s->nb_upper > table_limit;
    return COVOX_OK;
}

int integrate_batch(covox_ctx *ctx, covox_submap *s, const float *depths, int32_t F, int32_t H, int32_t W,
                    const float K[4], const double *T_wc, bool *maybe_full)
{
    if (F <= 0) return COVOX_OK;
    if (F > kMaxBatch) return fail(ctx, COVOX_EINVAL, "integrate_batch: too many frames in one batch");
    const covox_params &p = ctx->p;
    std::vector<FrameArgs> fr(F);
    int64_t box_max = 0, box_sum = 0;
    for (int32_t i = 0; i < F; ++i) {
        int64_t n_box = 0;
        int rc = prepare_frame(ctx, s, depths + (size_t)i * H * W, H, W, K, T_wc + 16 * i, fr[i], n_box);
        if (rc) return rc;
        box_max = std::max(box_max, n_box);
        box_sum += n_box;
    }
    int rc;
    if ((rc = ensure_buffer(ctx, (void **)&ctx->frames_dev, &ctx->frames_cap, kMaxBatch, sizeof(FrameArgs),
                            "frame batch")))
        return rc;
    if ((rc = ensure_buffer(ctx, (void **)&ctx->cand, &ctx->cand_cap, box_max * F, sizeof(uint32_t), "candidates")))
        return rc;
    if ((rc = ensure_buffer(ctx, (void **)&ctx->blist, &ctx->blist_cap, std::max<int64_t>(1, s->cap),
                            sizeof(uint32_t), "batch block list")))
        return rc;
    // first-frame table: a power of two holding every candidate twice over (of boxes
    // beyond 2^30 blocks, whose frustum fills a third at most, 2^31 slots still do)
    int64_t fslots = 1;
    while (fslots < 2 * box_sum && fslots < int64_t(1) << 31) fslots <<= 1;
    if ((rc = ensure_buffer(ctx, (void **)&ctx->fkeys, &ctx->fkeys_cap, fslots, sizeof(uint64_t), "first-frame keys")))
        return rc;
    // first frame of a key and its rank there
    if ((rc = ensure_buffer(ctx, (void **)&ctx->finfo, &ctx->finfo_cap, fslots, sizeof(uint2), "first-frame values")))
        return rc;
    if ((rc = ensure_buffer(ctx, (void **)&ctx->fcount, &ctx->fcount_cap, kCountWords, sizeof(int64_t),
                            "frame counts")))
        return rc;
    const int rx = (W + 63) / 64, ry = (H + 63) / 64;
    if ((rc = ensure_buffer(ctx, (void **)&ctx->ftiles, &ctx->ftiles_cap, (int64_t)F * rx * ry * kTilesPerRegion,
                            sizeof(float), "depth maxima")))
        return rc;
    if (ctx->capturing) {
        // the graph keeps its own copy of the frame parameters
        void *h = nullptr;
        if ((rc = hip_check(ctx, hipHostMalloc(&h, sizeof(FrameArgs) * F, hipHostMallocDefault), "frame staging")))
            return rc;
        ctx->cap_host.push_back(h);
        ::memcpy(h, fr.data(), sizeof(FrameArgs) * F);
        if ((rc = hip_check(ctx, hipMemcpyAsync(ctx->frames_dev, h, sizeof(FrameArgs) * F, hipMemcpyHostToDevice,
                                                ctx->stream), "frame batch upload")))
            return rc;
    } else if ((rc = stage_frames(ctx, fr.data(), F))) {
        return rc;
    }
    const float vs = (float)p.voxel_size, tau_f = (float)(p.trunc_vox * p.voxel_size), maxr = (float)p.max_range;
    const uint64_t tmask = (uint64_t)s->tcap - 1;
    const int64_t table_limit = (int64_t)(0.85 * (double)s->tcap);
    refresh_block_bound(s, box_sum);
    {
        TimedLaunch tl(ctx, COVOX_K_PROBE);
        hipLaunchKernelGGL(k_batch_tiles, dim3((unsigned)(rx * ry), (unsigned)F), dim3(256), 0, ctx->stream,
                           ctx->frames_dev, rx, maxr, ctx->ftiles, ctx->fkeys, ctx->finfo, fslots, ctx->fcount);
        // a workgroup's share of a frame's box: small enough for some 4096 of them
        // (sixteen to a CU), at most one block a lane
        const int per = (int)(std::min<int64_t>(256, std::max<int64_t>(8, box_max * F / 4096)) + 7) / 8 * 8;
        const int64_t n_share = (box_max + per - 1) / per, items = n_share * F;
        const unsigned pgrid = (unsigned)((std::min<int64_t>(items, 1 << 20) + 7) / 8 * 8);
        with_xy(ctx, [&](const auto &e, unsigned more, unsigned lds) {
            using E = std::decay_t<decltype(e)>;
            hipLaunchKernelGGL(k_probe_batch<E>, dim3(pgrid + more), dim3(256), lds, ctx->stream, e, ctx->frames_dev, vs,
                               tau_f, maxr, s->tkeys, s->tvals, tmask, ctx->ftiles, rx, rx * ry, ctx->fkeys, ctx->finfo,
                               (uint64_t)fslots - 1, ctx->cand, box_max, per, n_share, F,
                               (int)(ctx->tune.mapping_xcd_order != 0));
        });
    }
    {
        TimedLaunch tl(ctx, COVOX_K_SCAN);
        const unsigned gx = (unsigned)std::min<int64_t>((box_max + 255) / 256, 256);
        hipLaunchKernelGGL(k_batch_rank, dim3((unsigned)F), dim3(1024), 0, ctx->stream, ctx->frames_dev, ctx->cand,
                           box_max, ctx->fkeys, ctx->finfo, ctx->fcount, s->meta, s->cap, table_limit, s->pin_nb_dev,
                           s->seq);
        hipLaunchKernelGGL(k_batch_activate, dim3(gx, (unsigned)F), dim3(256), 0, ctx->stream, ctx->frames_dev,
                           ctx->cand, box_max, ctx->fcount, s->meta, s->keys, s->tkeys, s->tvals, tmask, ctx->fkeys,
                           ctx->finfo, (unsigned long long *)s->touch, ctx->blist);
    }
    {
        // one workgroup per touched block (at most min(capacity, sum of the boxes),
        // mostly far fewer), eight to a CU at once
        const int64_t blocks = std::max<int64_t>(1, std::min(s->cap, s->nb_upper + box_sum));
        const unsigned grid = (unsigned)(std::min<int64_t>(blocks, 2048) + 7) / 8 * 8;
        const int xcd = ctx->tune.mapping_xcd_order != 0;
        TimedLaunch tl(ctx, COVOX_K_INTEGRATE);
        with_z(ctx, [&](const auto &e, unsigned more, unsigned lds) {
            using E = std::decay_t<decltype(e)>;
            if (p.precision == COVOX_FP16)
                hipLaunchKernelGGL((k_integrate_batch<__half, E>), dim3(grid + more), dim3(256), lds, ctx->stream, e,
                                   ctx->frames_dev, s->meta, ctx->blist, s->keys, (__half *)s->D, (__half *)s->W, vs,
                                   tau_f, maxr, s->dirty, s->touch, xcd);
            else
                hipLaunchKernelGGL((k_integrate_batch<float, E>), dim3(grid + more), dim3(256), lds, ctx->stream, e,
                                   ctx->frames_dev, s->meta, ctx->blist, s->keys, (float *)s->D, (float *)s->W, vs,
                                   tau_f, maxr, s->dirty, s->touch, xcd);
        });
    }
    if ((rc = hip_check(ctx, hipGetLastError(), "integrate batch launch"))) return rc;
    s->nb_upper += box_sum;
    for (int32_t i = 0; i < F; ++i) grow_bounds(s, fr[i]);
    s->version++;
    *maybe_full = s->nb_upper > s->cap || s->nb_upper > table_limit;
    return COVOX_OK;
}

}  // namespace covox
