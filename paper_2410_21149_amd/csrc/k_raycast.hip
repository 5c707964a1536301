// Raycast TSDF integration (paper Sec. III-C: a ray from the optical centre
// through every observed point updates each voxel it crosses up to the
// truncation distance behind the point; Sec. III-D: count and allocate the
// new blocks, then merge the frame's contributions per voxel).
//
// One frame is five launches on the context stream:
//   fill_u32        clears the block flags of the frustum's block box;
//   k_ray_walk      one lane per pixel walks its ray and adds w and t w of each
//                   contribution to the voxel: the workgroup's 16 x 16 pixel
//                   tile sums its voxels in an LDS table, which is flushed with
//                   global FP64 atomics into binary64 accumulators, one per
//                   voxel of the box, and flags the voxel's block; with constant
//                   weights, contributions clamped to tau travel as integer
//                   counts;
//   k_ray_resolve   one lane per box block: a flagged block that exists gets
//                   its buffer index, the others stay NEW;
//   k_scan          (shared with projection mapping) compacts the flags in
//                   key order, checks capacity, numbers the new blocks;
//   k_ray_apply     one wave per touched block: key and hash insert of a new one,
//                   W' = W + sw, D' = (D W + stw) / W' where sw > 0, and the
//                   accumulators are cleared (also when nothing is committed).
// A box of more blocks than the pool (whose size the accumulators have), or too
// wide for a 31-bit voxel index, takes seven, with two walks a frame:
//   fill_u32        as above;
//   k_ray_mark      one lane per pixel walks its ray and flags each box block
//                   that receives a contribution (in an LDS bitmap per
//                   workgroup, written out once per flagged block);
//   k_ray_resolve, k_scan   as above;
//   k_ray_activate  one wave per new block: key, hash insert, zeroed voxels;
//   k_ray_accum     one lane per pixel walks its ray again and adds w and t w
//                   of each contribution to the accumulators of the block's
//                   buffer index: lanes of a wave that reach the same voxel in
//                   the same step are summed in registers, then as above;
//   k_ray_apply     as above.
// The paper orders the merge by sorting the contributions by voxel address;
// here the sums are formed by hardware FP64 atomics instead, in any order.
// The walk takes each crossing parameter as ((i + [u > 0]) vs - o) * (1 / u)
// with the reciprocal rounded once per ray: a multiply per step instead of a
// division, and faithful to 2^-22 relative of the exact crossing.  A walk
// with correctly rounded crossings can therefore take another step only where
// two crossing parameters (or the nearest one and the segment end) lie within
// that margin of each other; elsewhere block keys, buffer indices and the set
// of contributions are those of the exact traversal.  The binary64 sums of
// binary32 products depend on their order only at rare rounding ties.
#include "covox_impl.h"

#include <math.h>

#include <algorithm>
#include <type_traits>

namespace covox {

namespace {

constexpr uint32_t kNewFlag = 0xFFFFFFFFu;  // the compaction's NEW marker

// A ray and the state of its grid walk (Amanatides and Woo, Eurographics
// 1987).  Voxel i spans [i vs, (i + 1) vs) per axis; sn[a] is the ray
// parameter of the next boundary along axis a, computed from the index.
struct Ray {
    float o[3], u[3], iu[3], r, s1, w;
    int32_t i[3];
    int32_t step[3];
    float sn[3];
    int32_t left;  // voxels the walk may still visit
};

__device__ __forceinline__ float next_boundary(const Ray &R, int a, float vs)
{
    return (((float)(R.i[a] + (R.step[a] > 0 ? 1 : 0)) * vs) - R.o[a]) * R.iu[a];
}

// Sets up the ray of pixel (col, row); false when its depth is invalid.
__device__ __forceinline__ bool ray_setup(const FrameArgs &f, float vs, float tau, float maxr, int col, int row,
                                          Ray &R)
{
    const float z = f.depth[(int64_t)row * f.W + col];
    if (!(z > 0.0f && z <= maxr)) return false;
    const float xc = (((float)col - f.K[2]) * z) / f.K[0];
    const float yc = (((float)row - f.K[3]) * z) / f.K[1];
    float d[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) d[k] = (f.Rs[3 * k] * xc + f.Rs[3 * k + 1] * yc) + f.Rs[3 * k + 2] * z;
    R.r = sqrtf((d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]);
    R.s1 = R.r + tau;
    const float s0 = f.ray_carve ? 0.0f : fmaxf(R.r - tau, 0.0f);
    R.left = 3 * (int32_t)ceilf((R.s1 - s0) / vs) + 6;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        R.u[a] = d[a] / R.r;
        R.o[a] = f.o[a];
        const float e = R.o[a] + s0 * R.u[a];
        R.i[a] = (int32_t)floorf(e / vs);
        R.step[a] = R.u[a] > 0.0f ? 1 : (R.u[a] < 0.0f ? -1 : 0);
        R.iu[a] = R.step[a] ? 1.0f / R.u[a] : 0.0f;
        R.sn[a] = R.step[a] ? next_boundary(R, a, vs) : INFINITY;
    }
    R.w = f.weight_mode == COVOX_WEIGHT_INV_DEPTH2 ? 1.0f / (z * z) : 1.0f;
    return true;
}

// Moves to the next voxel; false when the walk has ended (the nearest
// boundary lies at or beyond s1, or the step bound is reached).
// The axis is chosen and applied with selects only (constant indices), so
// that the ray stays in registers.
__device__ __forceinline__ bool ray_next(Ray &R, float vs)
{
    const bool y_first = R.sn[1] < R.sn[0];
    const float m01 = y_first ? R.sn[1] : R.sn[0];
    const bool z_first = R.sn[2] < m01;
    const float smin = z_first ? R.sn[2] : m01;
    if (!(smin < R.s1)) return false;
    if (--R.left <= 0) return false;
    const bool pick[3] = {!z_first && !y_first, !z_first && y_first, z_first};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        R.i[a] += pick[a] ? R.step[a] : 0;
        const float nb = next_boundary(R, a, vs);
        R.sn[a] = pick[a] ? nb : R.sn[a];
    }
    return true;
}

// Contribution of the current voxel: t = min(sdf, tau) when sdf >= -tau.
__device__ __forceinline__ bool ray_contrib(const Ray &R, float vs, float tau, float &t)
{
    float c[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) c[a] = ((float)R.i[a] + 0.5f) * vs;
    const float proj = ((c[0] - R.o[0]) * R.u[0] + (c[1] - R.o[1]) * R.u[1]) + (c[2] - R.o[2]) * R.u[2];
    const float sdf = R.r - proj;
    if (!(sdf >= -tau)) return false;
    t = fminf(sdf, tau);
    return true;
}

// Pixel of a lane: workgroups of 256 lanes cover 16 x 16 pixel tiles, each
// wave an 8 x 8 quarter, so that the rays of a wave stay close together.
__device__ __forceinline__ void lane_pixel(int &col, int &row)
{
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    col = (int)blockIdx.x * 16 + (wv & 1) * 8 + (lane & 7);
    row = (int)blockIdx.y * 16 + (wv >> 1) * 8 + (lane >> 3);
}

// Block flags of a workgroup are first set in an LDS bitmap over the box
// (boxes of up to kMarkBits blocks) and then written out once each.
constexpr int kMarkWords = 2048;
constexpr int64_t kMarkBits = 32 * kMarkWords;

__global__ __launch_bounds__(256) void k_ray_mark(FrameArgs f, float vs, float tau, float maxr,
                                                  uint32_t *__restrict__ cand, int64_t n_box)
{
    __shared__ uint32_t s_bits[kMarkWords];
    const bool local = n_box <= kMarkBits;  // uniform
    const int nw = (int)((n_box + 31) / 32);
    if (local) {
        for (int k = threadIdx.x; k < nw; k += blockDim.x) s_bits[k] = 0u;
        __syncthreads();
    }
    int col, row;
    lane_pixel(col, row);
    Ray R;
    if (col < f.W && row < f.H && ray_setup(f, vs, tau, maxr, col, row, R)) {
        int64_t last = -1;
        do {
            float t;
            if (ray_contrib(R, vs, tau, t)) {
                // the box holds every voxel a ray can cross (host-side construction)
                const int jx = (R.i[0] >> 3) - f.blo[0], jy = (R.i[1] >> 3) - f.blo[1], jz = (R.i[2] >> 3) - f.blo[2];
                if (jx >= 0 && jx < f.bdim[0] && jy >= 0 && jy < f.bdim[1] && jz >= 0 && jz < f.bdim[2]) {
                    const int64_t j = ((int64_t)jx * f.bdim[1] + jy) * f.bdim[2] + jz;
                    if (j != last) {
                        const uint32_t bit = 1u << (j & 31);
                        if (!local) cand[j] = kNewFlag;
                        else if (!(s_bits[j >> 5] & bit)) atomicOr(&s_bits[j >> 5], bit);  // set once
                        last = j;
                    }
                }
            }
        } while (ray_next(R, vs));
    }
    if (local) {
        __syncthreads();
        for (int k = threadIdx.x; k < nw; k += blockDim.x) {
            uint32_t bits = s_bits[k];
            while (bits) {
                const int b = __ffs(bits) - 1;
                cand[32 * (int64_t)k + b] = kNewFlag;
                bits &= bits - 1u;
            }
        }
    }
}

__global__ __launch_bounds__(256) void k_ray_resolve(FrameArgs f, const uint64_t *__restrict__ tkeys,
                                                     const uint32_t *__restrict__ tvals, uint64_t tmask,
                                                     uint32_t *__restrict__ cand, int64_t n_box)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n_box || cand[j] != kNewFlag) return;
    const int64_t nz = f.bdim[2], ny = f.bdim[1];
    const int32_t bz = f.blo[2] + (int32_t)(j % nz);
    const int32_t by = f.blo[1] + (int32_t)((j / nz) % ny);
    const int32_t bx = f.blo[0] + (int32_t)(j / (nz * ny));
    const int64_t idx = hash_find(tkeys, tvals, tmask, pack_key(bx, by, bz));
    if (idx >= 0) cand[j] = (uint32_t)idx + 1u;
}

__global__ __launch_bounds__(256) void k_ray_activate(const SubmapMeta *__restrict__ meta,
                                                      const uint64_t *__restrict__ t_key,
                                                      const uint32_t *__restrict__ t_idx, uint64_t *keys, float *D,
                                                      float *W, uint64_t *tkeys, uint32_t *tvals, uint64_t tmask)
{
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int lane = threadIdx.x & 63;
    const int64_t n_t = meta->n_touched;
    for (int64_t t = wave; t < n_t; t += nwaves) {
        const uint32_t v = t_idx[t];
        if (!(v >> 31)) continue;  // uniform across the wave
        const int64_t idx = v & 0x7FFFFFFFu;
        if (lane == 0) {
            keys[idx] = t_key[t];
            hash_insert(tkeys, tvals, tmask, t_key[t], (uint32_t)idx);
        }
#pragma unroll
        for (int z = 0; z < 8; ++z) {
            D[idx * 512 + lane + 64 * z] = 0.0f;
            W[idx * 512 + lane + 64 * z] = 0.0f;
        }
    }
}

// Per-workgroup accumulation table in LDS: the 256 rays of a 16 x 16 pixel
// tile run inside a narrow cone and cross mostly the same voxels, so their
// contributions are summed here and each voxel costs the workgroup one pair
// of global atomics when the table is flushed.  Open addressing with linear
// probing; a contribution that finds no slot within kAccProbe probes goes
// to the global accumulators directly.
constexpr int kAccSlots = 1024;
constexpr int kAccProbe = 16;
constexpr unsigned long long kAccEmpty = ~0ull;

__device__ __forceinline__ void add_global(double *acc, int64_t addr, double vw, double vtw)
{
    unsafeAtomicAdd(acc + 2 * addr, vw);
    unsafeAtomicAdd(acc + 2 * addr + 1, vtw);
}

// With constant weights, a contribution clamped to tau (free space: most of
// them) is (w, t w) = (1, tau), so it is counted instead: an integer per LDS
// slot, ballot popcounts for a wave's group.  The count c enters the binary64
// sums as c and c tau, both exact.
__global__ __launch_bounds__(256) void k_ray_accum(FrameArgs f, float vs, float tau, float maxr,
                                                   const SubmapMeta *__restrict__ meta,
                                                   const uint64_t *__restrict__ tkeys,
                                                   const uint32_t *__restrict__ tvals, uint64_t tmask,
                                                   double *__restrict__ acc)
{
    __shared__ unsigned long long s_key[kAccSlots];
    __shared__ double s_w[kAccSlots], s_tw[kAccSlots];
    __shared__ uint32_t s_cnt[kAccSlots];
    if (meta->n_touched == 0) return;  // uniform: nothing committed (capacity failure, or no contribution)
    for (int k = threadIdx.x; k < kAccSlots; k += blockDim.x) {
        s_key[k] = kAccEmpty;
        s_w[k] = 0.0;
        s_tw[k] = 0.0;
        s_cnt[k] = 0u;
    }
    __syncthreads();
    const bool counted = f.weight_mode == COVOX_WEIGHT_CONSTANT;  // uniform
    const double tau_d = (double)tau;
    const int lane = threadIdx.x & 63;
    int col, row;
    lane_pixel(col, row);
    Ray R;
    bool active = col < f.W && row < f.H && ray_setup(f, vs, tau, maxr, col, row, R);
    int32_t cb[3] = {INT32_MIN, INT32_MIN, INT32_MIN};
    int64_t base = -1;
    // The loop runs while any lane of the wave walks, so that every lane
    // takes part in the ballots and shuffles below.
    while (__ballot(active)) {
        bool has = false;
        int64_t addr = -1;
        double vw = 0.0, vtw = 0.0;
        uint32_t cnt = 0;  // clamped contributions carried as a count
        if (active) {
            float t;
            if (ray_contrib(R, vs, tau, t)) {
                const int32_t bx = R.i[0] >> 3, by = R.i[1] >> 3, bz = R.i[2] >> 3;
                if (bx != cb[0] || by != cb[1] || bz != cb[2]) {
                    cb[0] = bx; cb[1] = by; cb[2] = bz;
                    base = hash_find(tkeys, tvals, tmask, pack_key(bx, by, bz));
                }
                if (base >= 0) {
                    has = true;
                    addr = base * 512 + (R.i[0] & 7) + 8 * (R.i[1] & 7) + 64 * (R.i[2] & 7);
                    if (counted && t == tau) {
                        cnt = 1u;
                    } else {
                        vw = (double)R.w;
                        vtw = (double)t * (double)R.w;  // exact in binary64
                    }
                }
            }
            active = ray_next(R, vs);
        }
        // lanes that reached the first contributing lane's voxel: summed in
        // registers, the leader carries the sum
        const uint64_t m = __ballot(has);
        if (m) {
            const int leader = __ffsll((unsigned long long)m) - 1;
            const int64_t la = __shfl(addr, leader, 64);
            const bool in = has && addr == la;
            const uint64_t g = __ballot(in);
            if (__popcll(g) > 1) {
                const uint32_t gc = (uint32_t)__popcll(__ballot(in && cnt != 0u));
                double a = 0.0, b = 0.0;
                if (__ballot(in && cnt == 0u)) {  // some member carries a value
                    a = in ? vw : 0.0;
                    b = in ? vtw : 0.0;
#pragma unroll
                    for (int off = 32; off > 0; off >>= 1) {
                        a += __shfl_xor(a, off, 64);
                        b += __shfl_xor(b, off, 64);
                    }
                }
                if (in) {
                    has = lane == leader;
                    vw = a;
                    vtw = b;
                    cnt = gc;
                }
            }
        }
        if (has) {
            const unsigned long long key = (unsigned long long)addr;
            uint32_t h = (uint32_t)((key * 0x9E3779B97F4A7C15ull) >> 54);  // 10 bits
            bool done = false;
            for (int p = 0; p < kAccProbe && !done; ++p, h = (h + 1) & (kAccSlots - 1)) {
                unsigned long long k = s_key[h];
                if (k == kAccEmpty) {
                    k = atomicCAS(&s_key[h], kAccEmpty, key);  // the old value: empty, or the winner's key
                    if (k == kAccEmpty) k = key;
                }
                if (k == key) {
                    if (cnt) atomicAdd(&s_cnt[h], cnt);
                    if (vw != 0.0) {
                        __hip_atomic_fetch_add(&s_w[h], vw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        __hip_atomic_fetch_add(&s_tw[h], vtw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                    done = true;
                }
            }
            if (!done) add_global(acc, addr, (double)cnt + vw, (double)cnt * tau_d + vtw);
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < kAccSlots; k += blockDim.x)
        if (s_key[k] != kAccEmpty) {
            const double c = (double)s_cnt[k];
            add_global(acc, (int64_t)s_key[k], c + s_w[k], c * tau_d + s_tw[k]);
        }
}

// ------------------------------------------------------------- one walk a frame

// Voxels of the box as 31-bit numbers: the coordinates from the box's corner, z in
// the low bits.
struct BoxKey {
    int sy, sx;  // shifts of y and x
};

// Accumulator of a voxel: box blocks in order, 512 voxels each.
__device__ __forceinline__ int64_t box_address(const FrameArgs &f, const BoxKey &q, uint32_t key, int64_t &j)
{
    const int z = (int)(key & ((1u << q.sy) - 1u)), y = (int)((key >> q.sy) & ((1u << (q.sx - q.sy)) - 1u));
    const int x = (int)(key >> q.sx);
    j = ((int64_t)(x >> 3) * f.bdim[1] + (y >> 3)) * f.bdim[2] + (z >> 3);
    return j * 512 + (x & 7) + 8 * (y & 7) + 64 * (z & 7);
}

constexpr uint32_t kNoKey = 0xFFFFFFFFu;

// The table of a workgroup: weight of the contributions clamped to tau and of the
// others, and the sum of t w over the others.  COUNTED (constant weights): w = 1, and
// the weights are counts.
template <bool COUNTED>
struct RayTable {
    using Weight = std::conditional_t<COUNTED, uint32_t, double>;
    uint32_t key[kAccSlots];
    Weight w[2][kAccSlots];
    double tw[kAccSlots];

    // Slot of a key; -1 when the probes find none free.
    __device__ __forceinline__ int slot(uint32_t k)
    {
        uint32_t h = (k * 0x9E3779B1u) >> 22;  // 10 bits
        uint32_t at = key[h];
        if (at == k) return (int)h;
#pragma unroll 1
        for (int p = 0; p < kAccProbe; ++p) {
            if (at == kNoKey) {
                at = atomicCAS(&key[h], kNoKey, k);  // the old value: empty, or the winner's key
                if (at == kNoKey) at = k;
            }
            if (at == k) return (int)h;
            h = (h + 1) & (kAccSlots - 1);
            at = key[h];
        }
        return -1;
    }
};

template <typename T>
__device__ __forceinline__ void add_lds(T *p, T v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// An axis of a walk: the next boundary's index and its change with a step, as floats
// (exact: below 2^24), its ray parameter, and the change of the voxel's number.  What
// the index is measured from makes the boundary of an axis that the ray does not move
// along infinite.
struct WalkAxis {
    float at, dir, from, inv, s;
    uint32_t key;

    __device__ __forceinline__ void init(const Ray &R, int a, float vs, int shift)
    {
        at = (float)(R.i[a] + (R.step[a] > 0 ? 1 : 0));
        dir = (float)R.step[a];
        from = R.step[a] ? R.o[a] : -INFINITY;
        inv = R.step[a] ? R.iu[a] : 1.0f;
        s = R.sn[a];
        key = (uint32_t)R.step[a] << shift;
    }
    // The first boundary at or beyond parameter S (its parameter grows with every
    // boundary; the guess is off by rounding).
    __device__ __forceinline__ void seek(float S, float o, float u, float vs)
    {
        if (dir == 0.0f) return;
        const float e = (o + S * u) / vs;
        at = dir > 0.0f ? ceilf(e) : floorf(e);
        for (int k = 0; k < 8 && ((at * vs) - from) * inv < S; ++k) at += dir;
        for (int k = 0; k < 8 && (((at - dir) * vs) - from) * inv >= S; ++k) at -= dir;
        s = ((at * vs) - from) * inv;
    }
    __device__ __forceinline__ uint32_t step(bool taken, float vs)
    {
        at += taken ? dir : 0.0f;
        s = ((at * vs) - from) * inv;  // (of an axis not taken: the same again)
        return taken ? key : 0u;
    }
    __device__ __forceinline__ float index() const { return at - (dir > 0.0f ? 1.0f : 0.0f); }
};

struct Walk {
    WalkAxis x, y, z;
    uint32_t key;  // the voxel
    float s, s1;   // where the ray enters it, and its end

    // As ray_next, for the lanes that move (without a branch: the others keep their
    // state); false when such a lane's walk has ended.  The bound on its steps, three
    // times the length, is the wave's: a walk crosses at most sqrt(3) times it.
    __device__ __forceinline__ bool next(bool move, float vs)
    {
        const float sx = x.s, sy = y.s, sz = z.s;
        const bool y_first = sy < sx;
        const float m01 = y_first ? sy : sx;
        const bool z_first = sz < m01;
        const float smin = z_first ? sz : m01;
        const bool go = smin < s1;
        move = move && go;
        s = move ? smin : s;
        key += x.step(move && !z_first && !y_first, vs);
        key += y.step(move && !z_first && y_first, vs);
        key += z.step(move && z_first, vs);
        return go;
    }
    __device__ __forceinline__ bool outside(const FrameArgs &f) const
    {
        const float i[3] = {x.index(), y.index(), z.index()};
        bool out = false;
#pragma unroll
        for (int a = 0; a < 3; ++a)
            out = out || i[a] < (float)(8 * f.blo[a]) || i[a] >= (float)(8 * (f.blo[a] + f.bdim[a]));
        return out;
    }
};

// The lanes of m, a voxel number each, as groups of equal numbers: at most G groups,
// each with its lowest lane for a leader.  group(leader, its lanes).  What is left
// comes back.
template <int G, typename F>
__device__ __forceinline__ uint64_t by_voxel(uint64_t m, uint32_t key, F group)
{
#pragma unroll
    for (int q = 0; q < G; ++q) {
        if (!m) break;  // uniform
        const int leader = __builtin_ctzll(m);
        const uint32_t k = (uint32_t)__builtin_amdgcn_readlane((int)key, leader);
        const uint64_t g = __builtin_amdgcn_ballot_w64(key == k) & m;
        group(leader, g);
        m &= ~g;
    }
    return m;
}

// Bound by the instructions of a step, some ninety steps a ray.  Most of them are in
// free space, where t = tau: as long as the ray enters the voxel a voxel and more
// before the band begins, the centre is before it too (no centre is further than
// 0.87 vs from a point of its voxel) and nothing but the voxel's number is needed, a
// 32-bit word that a step changes by one addition.  The 8 x 8 neighbouring rays of a
// wave are in two voxels at a step (room, 5 cm): a lane each adds for its group, as
// 64 lanes on one address take the LDS 64 cycles.  With the walk for the block flags
// (66 us) and a sum a buffer index, merged by 64-bit shuffles (203 us), a room frame of
// 640 x 480 took 269 us; with an addition a lane, 194; with one a group, 145; with
// the groups' loop unrolled and a walk of its own for rays that might leave the box, 133.
// Images too small to fill the chip deal their rays out in parts along their length
// (blockIdx.z): 120 x 160, a frame 272 us before, 178 with whole rays, 52 in parts
// (640 x 480 in three parts: 157 for 145).
template <bool COUNTED>
__global__ __launch_bounds__(256) void k_ray_walk(FrameArgs f, float vs, float tau, float maxr, BoxKey q,
                                                  double *__restrict__ acc, uint32_t *__restrict__ cand)
{
    using Weight = typename RayTable<COUNTED>::Weight;
    __shared__ RayTable<COUNTED> tab;
    for (int k = threadIdx.x; k < kAccSlots; k += 256) {
        tab.key[k] = kNoKey;
        tab.w[0][k] = tab.w[1][k] = 0;
        tab.tw[k] = 0.0;
    }
    __syncthreads();
    const double tau_d = (double)tau;
    const int lane = threadIdx.x & 63;
    int col, row;
    lane_pixel(col, row);
    Ray R{};
    Walk w{};
    bool alive = col < f.W && row < f.H && ray_setup(f, vs, tau, maxr, col, row, R);
    bool guard = false;
    float lim = 0.0f;
    if (alive) {
        w.x.init(R, 0, vs, q.sx);
        w.y.init(R, 1, vs, q.sy);
        w.z.init(R, 2, vs, 0);
        w.s = f.ray_carve ? 0.0f : fmaxf(R.r - tau, 0.0f);
        w.s1 = R.s1;
        // This workgroup's part of the ray: the voxels entered at parameters from
        // `begin` (the first part: with the ray's first voxel) to w.s1.
        const float part = (R.s1 - w.s) / (float)gridDim.z, begin = w.s + (float)blockIdx.z * part;
        if (blockIdx.z + 1 < gridDim.z) w.s1 = w.s + (float)(blockIdx.z + 1) * part;
        if (blockIdx.z > 0) {
            w.x.seek(begin, R.o[0], R.u[0], vs);
            w.y.seek(begin, R.o[1], R.u[1], vs);
            w.z.seek(begin, R.o[2], R.u[2], vs);
        }
        w.key = ((uint32_t)((int)w.x.index() - 8 * f.blo[0]) << q.sx) +
                ((uint32_t)((int)w.y.index() - 8 * f.blo[1]) << q.sy) + (uint32_t)((int)w.z.index() - 8 * f.blo[2]);
        if (blockIdx.z > 0) alive = w.next(true, vs);
        // A walk moves one way along each axis, from its first voxel to the last:
        // both inside the box, or each voxel is looked at.
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int lo = 8 * f.blo[a], hi = lo + 8 * f.bdim[a];
            const float e = (R.o[a] + R.s1 * R.u[a]) / vs;
            guard = guard || !(R.i[a] >= lo && R.i[a] < hi && e >= (float)(lo + 1) && e < (float)(hi - 1));
        }
        lim = ((R.r - tau) - vs) - 4e-6f * (((fabsf(R.o[0]) + fabsf(R.o[1])) + fabsf(R.o[2])) + R.r);
    }
    int left = alive ? R.left : 0;
    for (int o = 1; o < 64; o <<= 1) left = max(left, __shfl_xor(left, o, 64));
    left = __builtin_amdgcn_readfirstlane(left);  // steps of the wave
    const double vw = (double)R.w;
    // One lane's sums into the table, or past it.
    auto add = [&](Weight clamped, Weight banded, double tw) {
        const int h = tab.slot(w.key);
        if (h < 0) {
            int64_t j;
            add_global(acc, box_address(f, q, w.key, j), (double)clamped + (double)banded, (double)clamped * tau_d + tw);
            cand[j] = kNewFlag;
            return;
        }
        if (clamped != 0) add_lds(&tab.w[0][h], clamped);
        if (banded != 0) {
            add_lds(&tab.w[1][h], banded);
            add_lds(&tab.tw[h], tw);
        }
    };
    auto walk = [&](auto guarded) __attribute__((always_inline)) {
        constexpr bool GUARD = decltype(guarded)::value;
        bool in = alive && w.s < lim;
        if (__builtin_amdgcn_ballot_w64(in)) do {  // (tested at the end: no copies of the walk's state)
            const bool ok = in && !(GUARD && guard && w.outside(f));
            Weight mine = 0;
            const uint64_t left = by_voxel<6>(__builtin_amdgcn_ballot_w64(ok), w.key, [&](int leader, uint64_t g) {
                if constexpr (COUNTED) {
                    mine = lane == leader ? (uint32_t)__popcll(g) : mine;
                } else {
                    const double sum = wave_sum(g >> lane & 1 ? vw : 0.0);
                    mine = lane == leader ? sum : mine;
                }
            });
            if (left) mine = left >> lane & 1 ? (COUNTED ? (Weight)1 : (Weight)vw) : mine;  // uniform
            if (mine != 0) add(mine, 0, 0.0);
            const bool go = w.next(in, vs);
            alive = alive && (go || !in);
            in = alive && w.s < lim;
        } while (--left > 0 && __builtin_amdgcn_ballot_w64(in));
        if (__builtin_amdgcn_ballot_w64(alive)) do {
            const float c0 = (w.x.index() + 0.5f) * vs, c1 = (w.y.index() + 0.5f) * vs, c2 = (w.z.index() + 0.5f) * vs;
            const float proj = ((c0 - R.o[0]) * R.u[0] + (c1 - R.o[1]) * R.u[1]) + (c2 - R.o[2]) * R.u[2];
            const float sdf = R.r - proj;
            const bool ok = alive && sdf >= -tau && !(GUARD && guard && w.outside(f));
            const bool clamped = sdf >= tau;
            const double vtw = (double)sdf * vw;  // exact in binary64
            const uint64_t mc = __builtin_amdgcn_ballot_w64(ok && clamped);
            Weight a = 0, b = 0;
            double t = 0.0;
            const uint64_t left = by_voxel<2>(__builtin_amdgcn_ballot_w64(ok), w.key, [&](int leader, uint64_t g) {
                const bool lead = lane == leader;
                const double tw = (g & ~mc) ? wave_sum((g & ~mc) >> lane & 1 ? vtw : 0.0) : 0.0;  // uniform
                t = lead ? tw : t;
                if constexpr (COUNTED) {
                    a = lead ? (uint32_t)__popcll(g & mc) : a;
                    b = lead ? (uint32_t)__popcll(g & ~mc) : b;
                } else {
                    const double sa = wave_sum((g & mc) >> lane & 1 ? vw : 0.0);
                    const double sb = wave_sum((g & ~mc) >> lane & 1 ? vw : 0.0);
                    a = lead ? sa : a;
                    b = lead ? sb : b;
                }
            });
            if (left >> lane & 1) {
                const Weight one = COUNTED ? (Weight)1 : (Weight)vw;
                a = clamped ? one : 0;
                b = clamped ? 0 : one;
                t = clamped ? 0.0 : vtw;
            }
            if (a != 0 || b != 0) add(a, b, t);
            const bool go = w.next(alive, vs);
            alive = alive && go;
        } while (--left > 0 && __builtin_amdgcn_ballot_w64(alive));
    };
    if (__builtin_amdgcn_ballot_w64(guard)) walk(std::true_type{});  // uniform
    else walk(std::false_type{});
    __syncthreads();
    for (int k = threadIdx.x; k < kAccSlots; k += 256) {
        if (tab.key[k] == kNoKey) continue;
        int64_t j;
        const int64_t addr = box_address(f, q, tab.key[k], j);
        const double c = (double)tab.w[0][k];
        add_global(acc, addr, c + (double)tab.w[1][k], c * tau_d + tab.tw[k]);
        if (cand[j] != kNewFlag) cand[j] = kNewFlag;
    }
}

// BOX: accumulators by box block (k_ray_walk), and the new blocks are entered here;
// else by buffer index.
template <bool BOX>
__global__ __launch_bounds__(256) void k_ray_apply(FrameArgs f, SubmapMeta *__restrict__ meta,
                                                   const uint64_t *__restrict__ t_key,
                                                   const uint32_t *__restrict__ t_idx,
                                                   const uint32_t *__restrict__ cand, int64_t n_box, uint64_t *keys,
                                                   uint64_t *tkeys, uint32_t *tvals, uint64_t tmask, float *D,
                                                   float *W, double *__restrict__ acc, uint8_t *__restrict__ dirty)
{
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int lane = threadIdx.x & 63;
    const int64_t n_t = meta->n_touched;
    if (BOX && n_t == 0) {  // nothing committed: the accumulators are zero again
        for (int64_t j = wave; j < n_box; j += nwaves) {
            if (cand[j] == 0) continue;
#pragma unroll
            for (int z = 0; z < 8; ++z) ((double2 *)acc)[j * 512 + lane + 64 * z] = make_double2(0.0, 0.0);
        }
        return;
    }
    for (int64_t t = wave; t < n_t; t += nwaves) {
        const uint32_t v = t_idx[t];
        const int64_t idx = v & 0x7FFFFFFFu;
        const bool is_new = BOX && (v >> 31) != 0;
        int64_t from = idx;
        if (BOX) {
            const uint64_t key = t_key[t];
            int bx, by, bz;
            unpack_key(key, bx, by, bz);
            from = ((int64_t)(bx - f.blo[0]) * f.bdim[1] + (by - f.blo[1])) * f.bdim[2] + (bz - f.blo[2]);
            if (is_new && lane == 0) {
                keys[idx] = key;
                hash_insert(tkeys, tvals, tmask, key, (uint32_t)idx);
            }
        }
        double2 sum[8];
        float Wv[8], Dv[8];
#pragma unroll
        for (int z = 0; z < 8; ++z) {
            const int64_t o = lane + 64 * z;
            sum[z] = ((const double2 *)acc)[from * 512 + o];
            Wv[z] = is_new ? 0.0f : W[idx * 512 + o];
            Dv[z] = is_new ? 0.0f : D[idx * 512 + o];
        }
        int n_ok = 0;
#pragma unroll
        for (int z = 0; z < 8; ++z) {
            const int64_t o = lane + 64 * z;
            const bool ok = sum[z].x > 0.0;
            n_ok += __popcll(__ballot(ok));
            if (ok) {
                const float Wn = Wv[z] + (float)sum[z].x;
                Dv[z] = ((Dv[z] * Wv[z]) + (float)sum[z].y) / Wn;
                Wv[z] = Wn;
                ((double2 *)acc)[from * 512 + o] = make_double2(0.0, 0.0);
            }
            if (ok || is_new) {
                D[idx * 512 + o] = Dv[z];
                W[idx * 512 + o] = Wv[z];
            }
        }
        if (lane == 0) {
            atomicAdd(&meta->n_updates, (unsigned long long)n_ok);
            dirty[idx] = 1;
        }
    }
}

constexpr int64_t kWalkGroups = 1280;  // resident at once: five to a CU

// Bits that hold 0 .. n - 1.
int bits_of(int64_t n)
{
    int b = 0;
    while ((int64_t(1) << b) < n) ++b;
    return b;
}

}  // namespace

int ensure_ray_acc(covox_ctx *ctx)
{
    const int64_t need = ctx->p.block_capacity;
    if (ctx->ray_acc && ctx->ray_acc_blocks >= need) return COVOX_OK;
    if (ctx->capturing) return fail(ctx, COVOX_EINVAL, "raycast accumulators cannot be allocated under capture");
    int rc;
    if (ctx->ray_acc) {
        if ((rc = hip_check(ctx, hipStreamSynchronize(ctx->stream), "raycast accumulator sync"))) return rc;
        (void)hipFree(ctx->ray_acc);
        ctx->ray_acc = nullptr;
        ctx->ray_acc_blocks = 0;
    }
    const size_t bytes = (size_t)need * 512 * 2 * sizeof(double);
    if ((rc = hip_check(ctx, hipMalloc((void **)&ctx->ray_acc, bytes), "raycast accumulators"))) return rc;
    if ((rc = hip_check(ctx, hipMemset(ctx->ray_acc, 0, bytes), "raycast accumulator clear"))) return rc;
    ctx->ray_acc_blocks = need;
    return COVOX_OK;
}

int raycast_frame(covox_ctx *ctx, covox_submap *s, const float *depth, int32_t H, int32_t W, const float K[4],
                  const double T_wc[16], bool *maybe_full)
{
    const covox_params &p = ctx->p;
    FrameArgs f;
    int64_t n_box = 0;
    int rc = prepare_frame(ctx, s, depth, H, W, K, T_wc, f, n_box);
    if (rc) return rc;
    if (p.precision != COVOX_FP32) return fail(ctx, COVOX_EINVAL, "integrate: raycasting needs FP32 storage");
    {
        // Longest ray: to depth max_range + tau through the outermost pixel
        // edge.  Walks are bounded by 3 x its length in voxels + 6 steps.
        const double zf = p.max_range + p.trunc_vox * p.voxel_size;
        const double ax = std::max(std::fabs(-0.5 - K[2]), std::fabs(W - 0.5 - K[2])) / K[0];
        const double ay = std::max(std::fabs(-0.5 - K[3]), std::fabs(H - 0.5 - K[3])) / K[1];
        if (zf * std::sqrt(1.0 + ax * ax + ay * ay) / p.voxel_size > 65536.0)
            return fail(ctx, COVOX_EINVAL, "integrate: rays longer than 65536 voxels (check K and max_range)");
    }
    if ((rc = ensure_ray_acc(ctx))) return rc;
    if ((rc = ensure_buffer(ctx, (void **)&ctx->cand, &ctx->cand_cap, n_box, sizeof(uint32_t), "candidates")))
        return rc;
    if ((rc = ensure_buffer(ctx, (void **)&ctx->t_key, &ctx->t_key_cap, n_box, sizeof(uint64_t), "touched keys")))
        return rc;
    if ((rc = ensure_buffer(ctx, (void **)&ctx->t_idx, &ctx->t_idx_cap, n_box, sizeof(uint32_t), "touched index")))
        return rc;

    const float vs = (float)p.voxel_size, tau = (float)(p.trunc_vox * p.voxel_size), maxr = (float)p.max_range;
    const uint64_t tmask = (uint64_t)s->tcap - 1;
    const int64_t table_limit = (int64_t)(0.85 * (double)s->tcap);
    const dim3 pix_grid((unsigned)((W + 15) / 16), (unsigned)((H + 15) / 16));
    const unsigned box_grid = (unsigned)((n_box + 255) / 256);
    const unsigned wave_grid = (unsigned)std::min<int64_t>((n_box + 3) / 4, 65536);
    float *Dp = (float *)s->D, *Wp = (float *)s->W;
    refresh_block_bound(s, n_box);
    const int bits[3] = {bits_of(8 * (int64_t)f.bdim[0]), bits_of(8 * (int64_t)f.bdim[1]), bits_of(8 * (int64_t)f.bdim[2])};
    const bool one_walk = n_box <= ctx->ray_acc_blocks && bits[0] + bits[1] + bits[2] <= 31;
    const BoxKey q{bits[2], bits[1] + bits[2]};
    auto resolve = [&] {
        hipLaunchKernelGGL(k_ray_resolve, dim3(box_grid), dim3(256), 0, ctx->stream, f, s->tkeys, s->tvals, tmask,
                           ctx->cand, n_box);
    };
    auto apply = [&](auto kernel) {
        TimedLaunch tl(ctx, COVOX_K_RAY_APPLY);
        hipLaunchKernelGGL(kernel, dim3(wave_grid), dim3(256), 0, ctx->stream, f, s->meta, ctx->t_key, ctx->t_idx,
                           ctx->cand, n_box, s->keys, s->tkeys, s->tvals, tmask, Dp, Wp, ctx->ray_acc, s->dirty);
    };
    if (one_walk) {
        {
            TimedLaunch tl(ctx, COVOX_K_RAY_ACCUM);
            fill_u32(ctx->stream, ctx->cand, 0u, n_box);
            // parts of a ray: for kWalkGroups workgroups, some twenty voxels of the
            // longest ray each at least (the set-up costs six)
            const int64_t tiles = (int64_t)pix_grid.x * pix_grid.y;
            const double len = p.ray_carve ? p.max_range / p.voxel_size + p.trunc_vox : 2.0 * p.trunc_vox;
            const int64_t parts = std::min<int64_t>(kWalkGroups / tiles, (int64_t)(len / 12.0));
            const dim3 walk_grid(pix_grid.x, pix_grid.y, (unsigned)std::max<int64_t>(1, std::min<int64_t>(parts, 16)));
            if (p.weight_mode == COVOX_WEIGHT_CONSTANT)
                hipLaunchKernelGGL(k_ray_walk<true>, walk_grid, dim3(256), 0, ctx->stream, f, vs, tau, maxr, q,
                                   ctx->ray_acc, ctx->cand);
            else
                hipLaunchKernelGGL(k_ray_walk<false>, walk_grid, dim3(256), 0, ctx->stream, f, vs, tau, maxr, q,
                                   ctx->ray_acc, ctx->cand);
        }
        {
            TimedLaunch tl(ctx, COVOX_K_RAY_MARK);
            resolve();
        }
        launch_block_scan(ctx, s, f, n_box, table_limit);
        apply(k_ray_apply<true>);
    } else {
        {
            TimedLaunch tl(ctx, COVOX_K_RAY_MARK);
            fill_u32(ctx->stream, ctx->cand, 0u, n_box);
            hipLaunchKernelGGL(k_ray_mark, pix_grid, dim3(256), 0, ctx->stream, f, vs, tau, maxr, ctx->cand, n_box);
            resolve();
        }
        launch_block_scan(ctx, s, f, n_box, table_limit);
        {
            TimedLaunch tl(ctx, COVOX_K_RAY_ACCUM);
            hipLaunchKernelGGL(k_ray_activate, dim3(wave_grid), dim3(256), 0, ctx->stream, s->meta, ctx->t_key,
                               ctx->t_idx, s->keys, Dp, Wp, s->tkeys, s->tvals, tmask);
            hipLaunchKernelGGL(k_ray_accum, pix_grid, dim3(256), 0, ctx->stream, f, vs, tau, maxr, s->meta, s->tkeys,
                               s->tvals, tmask, ctx->ray_acc);
        }
        apply(k_ray_apply<false>);
    }
    if ((rc = hip_check(ctx, hipGetLastError(), "raycast launch"))) return rc;
    s->nb_upper += n_box;
    grow_bounds(s, f);
    s->version++;
    *maybe_full = s->nb_upper > s->cap || s->nb_upper > table_limit;
    return COVOX_OK;
}

}  // namespace covox
