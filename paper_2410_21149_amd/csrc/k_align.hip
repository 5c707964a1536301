// Correspondence-free ESDF alignment of two submaps (paper Sec. I and
// Sec. III-F: the registration term of Eq. (1); registration points chosen
// by weight; residuals, Jacobians and the least-squares solve on the GPU).
//
// Registration points of B: zero crossings of D_B along voxel edges whose
// endpoints are both in the band with W >= w_reg (k_iso to count, k_iso_scan,
// k_iso to write, k_pbar for their centroid; order = block buffer index, in-block
// index, axis).
//
// Alignment (one problem per pair and start).  A problem's points are cut into
// segments of kSegPoints lanes' worth; every evaluation of the normal equations
// is one launch over the segments of all problems (k_align_step), and the sums
// of a segment go to memory.  The next launch reduces them in a fixed order and
// makes the solve and the pose update (6x6 binary64 Cholesky, T <- Exp(delta)
// T) before it evaluates.  So one pair fills as many CUs as it has segments,
// uneven problems leave no tail, nothing waits on another workgroup, and the
// sums of a problem do not depend on the batch it runs in.
//   k_align_tiles    phi of A as 9^3 tiles (a block and the next voxel of its
//                    neighbours): a point's cell is one page lookup and four
//                    8-byte reads of one tile;
//   k_align_step     per point (binary32): q = T p, trilinear ESDF of A and its
//                    gradient g, J = [g ; q x g]; exact binary64 products summed
//                    per lane in binary64, then a fixed tree over the workgroup
//                    into the 21 + 6 + 1 + 1 sums of the normal equations;
//   k_align_advance  the solves alone, where the segments outnumber the chip's
//                    workgroups;
//   k_align_finish   last solve test and results;
//   k_align_solo     all of it in one workgroup per problem (the same sums), for
//                    problems of few points and for iteration caps too long to
//                    enqueue ahead launch by launch.
#include "covox_impl.h"

#include <string.h>

#include <algorithm>
#include <type_traits>
#include <unordered_map>
#include <vector>

namespace covox {

namespace {

template <typename S> __device__ __forceinline__ float ldw(const S *p);
template <> __device__ __forceinline__ float ldw<float>(const float *p) { return *p; }
template <> __device__ __forceinline__ float ldw<__half>(const __half *p) { return __half2float(*p); }

struct DomArgs {
    int32_t lo[3], dim[3];
};

__device__ __forceinline__ DomArgs dom_of(const SubmapMeta *m)
{
    DomArgs d;
    for (int a = 0; a < 3; ++a) { d.lo[a] = m->dom_min[a]; d.dim[a] = m->dom_dim[a]; }
    return d;
}

// Buffer index of block (bx, by, bz) through a dense page, -1 when absent.
__device__ __forceinline__ int64_t page_lookup(const int32_t *page, const DomArgs &d, int bx, int by, int bz)
{
    const int x = bx - d.lo[0], y = by - d.lo[1], z = bz - d.lo[2];
    if (x < 0 || y < 0 || z < 0 || x >= d.dim[0] || y >= d.dim[1] || z >= d.dim[2]) return -1;
    return page[((int64_t)z * d.dim[1] + y) * d.dim[0] + x];
}

// Whether an edge's ends are both in the band and observed, of different sign.
__device__ __forceinline__ bool edge_crosses(bool base, float Di, float Dn, float Wn, float tau, float wreg)
{
    return base && Wn >= wreg && fabsf(Dn) < tau && ((Di < 0.0f) != (Dn < 0.0f));
}

// The +x, +y, +z edges of a block's voxels, one wave a block, lane = (x, y): counts
// (write = 0), or the points from place cnt[j] on, as far as pts has room, and their
// sums.  Bound by latency: all reads of a block, its own voxels and the planes of the
// three neighbours, are in flight together and the ends inside the block come from
// other lanes (z by z, with an inner prefix sum of shuffles, 13 us each for 1.4 k to
// 2 k blocks; now 8).
template <typename S>
__global__ __launch_bounds__(256) void k_iso(const SubmapMeta *__restrict__ meta, const uint64_t *__restrict__ keys,
                                             const int32_t *__restrict__ page, const S *__restrict__ D,
                                             const S *__restrict__ W, float vs, float tau, float wreg, int write,
                                             uint32_t *__restrict__ cnt, float *__restrict__ pts, int64_t room,
                                             double *__restrict__ psum)
{
    const int64_t nbk = meta->n_blocks;
    const DomArgs dm = dom_of(meta);
    const int lane = threadIdx.x & 63, x = lane & 7, y = lane >> 3;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const uint64_t below = (1ull << lane) - 1ull;
    for (int64_t j = wave; j < nbk; j += nwaves) {
        int bx, by, bz;
        unpack_key(keys[j], bx, by, bz);
        int64_t nb[3];
        nb[0] = page_lookup(page, dm, bx + 1, by, bz);
        nb[1] = page_lookup(page, dm, bx, by + 1, bz);
        nb[2] = page_lookup(page, dm, bx, by, bz + 1);
        float Dv[9], Wv[9], Dx[8], Wx[8], Dy[8], Wy[8];
#pragma unroll
        for (int z = 0; z < 8; ++z) {
            Dv[z] = ldw(D + j * 512 + lane + 64 * z);
            Wv[z] = ldw(W + j * 512 + lane + 64 * z);
        }
        // the neighbours' first planes; without a neighbour, distances outside any band
        // (no weight would do: the limit can be minus infinity)
        const int64_t oz = (nb[2] >= 0 ? nb[2] : j) * 512 + lane;
        Dv[8] = ldw(D + oz);
        Wv[8] = ldw(W + oz);
        if (nb[2] < 0) Dv[8] = INFINITY;
#pragma unroll
        for (int z = 0; z < 8; ++z) {
            Dx[z] = Dy[z] = INFINITY;
            Wx[z] = Wy[z] = 0.0f;
            if (x == 7 && nb[0] >= 0) {
                Dx[z] = ldw(D + nb[0] * 512 + lane + 64 * z - 7);
                Wx[z] = ldw(W + nb[0] * 512 + lane + 64 * z - 7);
            }
            if (y == 7 && nb[1] >= 0) {
                Dy[z] = ldw(D + nb[1] * 512 + lane + 64 * z - 56);
                Wy[z] = ldw(W + nb[1] * 512 + lane + 64 * z - 56);
            }
        }
        int64_t base = write ? (int64_t)cnt[j] : 0;
        uint32_t total = 0;
        double s0 = 0, s1 = 0, s2 = 0;
#pragma unroll
        for (int z = 0; z < 8; ++z) {
            const float Di = Dv[z];
            const bool in = Wv[z] >= wreg && fabsf(Di) < tau;
            const float Dr = __shfl_down(Di, 1, 64), Wr = __shfl_down(Wv[z], 1, 64);
            const float Du = __shfl_down(Di, 8, 64), Wu = __shfl_down(Wv[z], 8, 64);
            const float Dn[3] = {x < 7 ? Dr : Dx[z], y < 7 ? Du : Dy[z], Dv[z + 1]};
            const float Wn[3] = {x < 7 ? Wr : Wx[z], y < 7 ? Wu : Wy[z], Wv[z + 1]};
            bool ok[3];
            uint64_t m[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                ok[a] = edge_crosses(in, Di, Dn[a], Wn[a], tau, wreg);
                m[a] = __ballot(ok[a]);
            }
            const int wtot = __popcll(m[0]) + __popcll(m[1]) + __popcll(m[2]);
            if (write && (ok[0] || ok[1] || ok[2])) {
                // ascending lane = ascending in-block index, then axis
                int64_t at = base + (__popcll(m[0] & below) + __popcll(m[1] & below) + __popcll(m[2] & below));
                const int ix = 8 * bx + x, iy = 8 * by + y, iz = 8 * bz + z;
                const float cx = ((float)ix + 0.5f) * vs, cy = ((float)iy + 0.5f) * vs, cz = ((float)iz + 0.5f) * vs;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    if (!ok[a]) continue;
                    const float sfr = Di / (Di - Dn[a]);
                    float p[3] = {cx, cy, cz};
                    p[a] = p[a] + sfr * vs;
                    if (at < room) {
                        pts[3 * at + 0] = p[0];
                        pts[3 * at + 1] = p[1];
                        pts[3 * at + 2] = p[2];
                    }
                    s0 += (double)p[0];
                    s1 += (double)p[1];
                    s2 += (double)p[2];
                    ++at;
                }
            }
            base += wtot;
            total += (uint32_t)wtot;
        }
        if (!write) {
            if (lane == 0) cnt[j] = total;
        } else {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                s0 += __shfl_xor(s0, o, 64);
                s1 += __shfl_xor(s1, o, 64);
                s2 += __shfl_xor(s2, o, 64);
            }
            if (lane == 0) {
                psum[3 * j + 0] = s0;
                psum[3 * j + 1] = s1;
                psum[3 * j + 2] = s2;
            }
        }
    }
}

// Exclusive scan of cnt[0, n) in place (one 1024-lane workgroup, each lane a
// contiguous chunk), total into meta->n_points.
__global__ __launch_bounds__(1024) void k_iso_scan(SubmapMeta *meta, uint32_t *cnt)
{
    __shared__ int64_t lds[16];
    const int64_t n = meta->n_blocks;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, nw = blockDim.x >> 6;
    const int64_t C = (n + blockDim.x - 1) / blockDim.x;
    const int64_t beg = std::min<int64_t>((int64_t)tid * C, n), end = std::min<int64_t>(beg + C, n);
    int64_t s = 0;
    for (int64_t j = beg; j < end; ++j) s += cnt[j];
    int64_t x = s;
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) lds[wid] = x;
    __syncthreads();
    if (wid == 0) {
        int64_t w = lane < nw ? lds[lane] : 0;
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t y = __shfl_up(w, o, 64);
            if (lane >= o) w += y;
        }
        if (lane < nw) lds[lane] = w;
    }
    __syncthreads();
    int64_t run = (wid > 0 ? lds[wid - 1] : 0) + x - s;
    for (int64_t j = beg; j < end; ++j) {
        const uint32_t c = cnt[j];
        cnt[j] = (uint32_t)run;
        run += c;
    }
    if (tid == 0) meta->n_points = lds[nw - 1];
}

// Centroid of the points from per-block sums: lane i of one workgroup sums
// blocks i, i + 1024, ... in order, then the lanes in a fixed tree, so that the
// centroid does not depend on scheduling.  Bound by the latency of its reads:
// one lane that walked all blocks waited for each in turn (2043 outdoor
// blocks: 222 us); 1024 lanes have every block's read in flight at once.
constexpr int kPbarThreads = 1024;
__global__ __launch_bounds__(kPbarThreads) void k_pbar(SubmapMeta *meta, const double *__restrict__ psum)
{
    __shared__ double red[kPbarThreads / 64][3];
    const int64_t n = meta->n_blocks;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    double s[3] = {0, 0, 0};
    for (int64_t j = tid; j < n; j += kPbarThreads)
#pragma unroll
        for (int a = 0; a < 3; ++a) s[a] += psum[3 * j + a];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s[a] += __shfl_xor(s[a], o, 64);
        if (lane == 0) red[wid][a] = s[a];
    }
    __syncthreads();
    if (tid < 3) {
        double t = 0;
        for (int w = 0; w < kPbarThreads / 64; ++w) t += red[w][tid];
        meta->pbar[tid] = t / (double)(meta->n_points > 0 ? meta->n_points : 1);
    }
}

// ------------------------------------------------------------ alignment

__device__ __forceinline__ float phi_at(const float *phi, const int32_t *page, const DomArgs &d, int jx, int jy,
                                        int jz)
{
    const int64_t idx = page_lookup(page, d, jx >> 3, jy >> 3, jz >> 3);
    if (idx < 0) return __builtin_nanf("");
    return phi[idx * 512 + (jx & 7) + 8 * (jy & 7) + 64 * (jz & 7)];
}

// One submap's field as tiles: tile j holds the voxels (0..8)^3 of block j, the
// planes at 8 from its + neighbours (NaN where there is no block), so that the
// cell of every point of the block lies in one tile.  One wave per block; bound
// by its traffic, 2 KB read and 2.9 KB written a block (8 outdoor submaps of
// 1300 blocks: 50 MB; 25 us a value at a time, 20 with a block's reads in flight
// together).  Built for each call into the call's own memory: phi is
// whatever A holds then, and other contexts may align to A meanwhile.  Where that
// costs more than it saves (worth_tiles), or the memory is not there, the corners are
// read through the page, one look-up each.
constexpr int kTileEdge = 9, kTile = kTileEdge * kTileEdge * kTileEdge;

struct TileJob {
    const float *phi;
    const int32_t *page;
    const SubmapMeta *meta;
    const uint64_t *keys;
    float *tiles;
    int64_t nb;  // tiles that fit
};

__global__ __launch_bounds__(256) void k_align_tiles(const TileJob *__restrict__ jobs)
{
    const TileJob J = jobs[blockIdx.y];
    const DomArgs d = dom_of(J.meta);
    const int64_t nb = min((int64_t)J.meta->dom_nblocks, J.nb);
    const int lane = threadIdx.x & 63;
    for (int64_t j = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); j < nb; j += (int64_t)gridDim.x * 4) {
        int bx, by, bz;
        unpack_key(J.keys[j], bx, by, bz);
        int32_t idx = -1;  // lanes 0..7: the block at (lane & 1, lane >> 1 & 1, lane >> 2)
        if (lane < 8) idx = (int32_t)page_lookup(J.page, d, bx + (lane & 1), by + ((lane >> 1) & 1), bz + (lane >> 2));
        constexpr int kReads = (kTile + 63) / 64;  // all in flight before the first write
        float v[kReads];
#pragma unroll
        for (int k = 0; k < kReads; ++k) {
            const int e = min(lane + 64 * k, kTile - 1);
            const int x = e % kTileEdge, y = e / kTileEdge % kTileEdge, z = e / (kTileEdge * kTileEdge);
            const int32_t b = __shfl(idx, (x >> 3) | ((y >> 3) << 1) | ((z >> 3) << 2), 64);
            const float p = J.phi[(b >= 0 ? (int64_t)b * 512 : 0) + (x & 7) + 8 * (y & 7) + 64 * (z & 7)];
            v[k] = b >= 0 ? p : __builtin_nanf("");
        }
#pragma unroll
        for (int k = 0; k < kReads; ++k)
            if (lane + 64 * k < kTile) J.tiles[j * kTile + lane + 64 * k] = v[k];
    }
}

// x / b, correctly rounded, with rb = 1 / b rounded: a division by one number for all
// points.  The first correction leaves half an ulp and 2^-22 of one at most, so that the
// second adds less than the 2^-24 / m of an ulp (m: b's mantissa, 1 <= m < 2) by which a
// quotient misses every tie (Markstein, IBM J. Res. Dev. 34, 1990).  (Quotients below
// 2^-100 can be an ulp off.)  Five instructions for the sixteen slots of a general
// division, six a point: 94 -> 87 us an evaluation of 64 outdoor pairs' 512 problems,
// which is bound by vector instructions.
__device__ __forceinline__ float div_by(float x, float b, float rb)
{
    float q = x * rb;
    q = __builtin_fmaf(__builtin_fmaf(-q, b, x), rb, q);
    return __builtin_fmaf(__builtin_fmaf(-q, b, x), rb, q);
}

// Residual and Jacobian of U points (indices i0 + u stride, those at or beyond
// n are invalid) with all their loads issued before any is used; ok[u] false
// when a cell corner is unobserved or the point is far outside A.  Per
// point: q = T p; g = q / vs - 1/2, j0 = floor(g), f = g - j0; r is the
// trilinear value of the 8 corners and J = [grad; q x grad] with the
// gradient of the trilinear patch divided by vs.  TILED: a point's corners from the
// tile of its block; else each from its own block by the page (the same values).
template <int U, bool TILED>
__device__ __forceinline__ void residual_u(const float *Tf, const float *__restrict__ pts, int64_t i0, int64_t stride,
                                          int64_t n, float vs, const float *__restrict__ field, int64_t n_tiles,
                                          const int32_t *__restrict__ page, const DomArgs &d, float J[U][6], float r[U],
                                          bool ok[U])
{
    constexpr int kLooks = TILED ? 1 : 8;
    const float rvs = 1.0f / vs;
    float c[U][8], f[U][3], q[U][3];
    int32_t blk[U][kLooks], off[U][kLooks];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t i = i0 + u * stride;
        const bool in = i < n;
        const int64_t ii = in ? i : 0;
        const float p[3] = {pts[3 * ii], pts[3 * ii + 1], pts[3 * ii + 2]};
        int j0[3];
        bool fin = in;
#pragma unroll
        for (int a = 0; a < 3; ++a)
            q[u][a] = ((Tf[4 * a + 0] * p[0] + Tf[4 * a + 1] * p[1]) + Tf[4 * a + 2] * p[2]) + Tf[4 * a + 3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            float g = div_by(q[u][a], vs, rvs) - 0.5f;
            fin = fin && fabsf(g) < 1.0e8f;
            g = fabsf(g) < 1.0e8f ? g : 0.0f;  // keeps the clamped addresses sane
            const float fl = floorf(g);
            j0[a] = (int)fl;
            f[u][a] = g - fl;
        }
        ok[u] = fin;
#pragma unroll
        for (int k = 0; k < kLooks; ++k) {  // corner (k & 1, k >> 1 & 1, k >> 2)
            const int jx = j0[0] + (k & 1), jy = j0[1] + (k >> 1 & 1), jz = j0[2] + (k >> 2);
            const int x = (jx >> 3) - d.lo[0], y = (jy >> 3) - d.lo[1], z = (jz >> 3) - d.lo[2];
            const bool has = fin && x >= 0 && y >= 0 && z >= 0 && x < d.dim[0] && y < d.dim[1] && z < d.dim[2];
            const int32_t b = page[has ? ((int64_t)z * d.dim[1] + y) * d.dim[0] + x : 0];
            blk[u][k] = has ? b : -1;
            off[u][k] = TILED ? (jx & 7) + kTileEdge * ((jy & 7) + kTileEdge * (jz & 7))
                              : (jx & 7) + 8 * (jy & 7) + 64 * (jz & 7);
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if constexpr (TILED) {
            ok[u] = ok[u] && (uint32_t)blk[u][0] < (uint32_t)n_tiles;  // -1: no block
            const float *t = field + (ok[u] ? (int64_t)blk[u][0] * kTile + off[u][0] : 0);
#pragma unroll
            for (int k = 0; k < 4; ++k)  // the x pair of corner row (k & 1, k >> 1)
                __builtin_memcpy(&c[u][2 * k], t + kTileEdge * (k & 1) + kTileEdge * kTileEdge * (k >> 1), 8);
        } else {
#pragma unroll
            for (int k = 0; k < kLooks; ++k) {
                const float v = field[(blk[u][k] >= 0 ? (int64_t)blk[u][k] * 512 : 0) + off[u][k]];
                c[u][k] = blk[u][k] >= 0 ? v : __builtin_nanf("");
            }
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const float *cc = c[u];
        const float wx0 = 1.0f - f[u][0], wx1 = f[u][0], wy0 = 1.0f - f[u][1], wy1 = f[u][1], wz0 = 1.0f - f[u][2],
                    wz1 = f[u][2];
        const float c00 = cc[0] * wx0 + cc[1] * wx1, c10 = cc[2] * wx0 + cc[3] * wx1;
        const float c01 = cc[4] * wx0 + cc[5] * wx1, c11 = cc[6] * wx0 + cc[7] * wx1;
        const float c0 = c00 * wy0 + c10 * wy1, c1 = c01 * wy0 + c11 * wy1;
        r[u] = c0 * wz0 + c1 * wz1;
        ok[u] = ok[u] && r[u] == r[u];  // finite weights: NaN exactly when a corner is
        const float dx = ((cc[1] - cc[0]) * wy0 + (cc[3] - cc[2]) * wy1) * wz0 +
                         ((cc[5] - cc[4]) * wy0 + (cc[7] - cc[6]) * wy1) * wz1;
        const float dy = (c10 - c00) * wz0 + (c11 - c01) * wz1;
        const float dz = c1 - c0;
        const float g0 = div_by(dx, vs, rvs), g1 = div_by(dy, vs, rvs), g2 = div_by(dz, vs, rvs);
        J[u][0] = g0;
        J[u][1] = g1;
        J[u][2] = g2;
        J[u][3] = q[u][1] * g2 - q[u][2] * g1;
        J[u][4] = q[u][2] * g0 - q[u][0] * g2;
        J[u][5] = q[u][0] * g1 - q[u][1] * g0;
    }
}

// 4-DoF step (translation and yaw): rows and columns 0, 1, 2, 5 of the
// normal equations, diagonal damped by mu (0: Gauss-Newton), by Cholesky;
// x = (rho, 0, 0, theta_z).
__device__ bool solve_xyz_yaw(const double *ne, double mu, double x[6])
{
    const int sel[4] = {0, 1, 2, 5};
    double H[4][4], b[4], L[4][4];
    for (int a = 0; a < 4; ++a) {
        for (int c = 0; c < 4; ++c) {
            int r = sel[a], q = sel[c];
            if (r > q) { const int t = r; r = q; q = t; }
            H[a][c] = ne[r * 6 - r * (r - 1) / 2 + (q - r)];
            L[a][c] = 0.0;
        }
        b[a] = ne[21 + sel[a]];
    }
    if (mu != 0.0)
        for (int a = 0; a < 4; ++a) H[a][a] = H[a][a] + mu * H[a][a];
    for (int j = 0; j < 4; ++j) {
        double sj = H[j][j];
        for (int k = 0; k < j; ++k) sj -= L[j][k] * L[j][k];
        if (!(sj > 0.0)) return false;
        L[j][j] = sqrt(sj);
        for (int i = j + 1; i < 4; ++i) {
            double t = H[i][j];
            for (int k = 0; k < j; ++k) t -= L[i][k] * L[j][k];
            L[i][j] = t / L[j][j];
        }
    }
    double y[4], z[4];
    for (int i = 0; i < 4; ++i) {
        double t = -b[i];
        for (int k = 0; k < i; ++k) t -= L[i][k] * y[k];
        y[i] = t / L[i][i];
    }
    for (int i = 3; i >= 0; --i) {
        double t = y[i];
        for (int k = i + 1; k < 4; ++k) t -= L[k][i] * z[k];
        z[i] = t / L[i][i];
    }
    x[0] = z[0]; x[1] = z[1]; x[2] = z[2];
    x[3] = 0.0; x[4] = 0.0; x[5] = z[3];
    return true;
}

// 6x6 Cholesky solve of (H + mu diag(H)) x = -b (H from the packed upper
// triangle; mu = 0 is the Gauss-Newton step).  One lane's chain of dependent
// operations, of which a binary64 division is some twenty: one reciprocal a column,
// beside the square root's own, takes the place of 27 (an evaluation of one pair
// 9.1 us for 9.6).
__device__ bool solve6(const double *ne, double mu, double x[6])
{
    double L[6][6], inv[6];
    for (int j = 0; j < 6; ++j) {
        for (int i = 0; i < 6; ++i) L[j][i] = 0.0;
    }
    auto Hat = [&](int a, int b) {
        if (a > b) { const int t = a; a = b; b = t; }
        return ne[a * 6 - a * (a - 1) / 2 + (b - a)];
    };
    for (int j = 0; j < 6; ++j) {
        double s = Hat(j, j);
        if (mu != 0.0) s = s + mu * s;
        for (int k = 0; k < j; ++k) s -= L[j][k] * L[j][k];
        if (!(s > 0.0)) return false;
        inv[j] = 1.0 / sqrt(s);
        for (int i = j + 1; i < 6; ++i) {
            double t = Hat(i, j);
            for (int k = 0; k < j; ++k) t -= L[i][k] * L[j][k];
            L[i][j] = t * inv[j];
        }
    }
    double y[6];
    for (int i = 0; i < 6; ++i) {
        double t = -ne[21 + i];
        for (int k = 0; k < i; ++k) t -= L[i][k] * y[k];
        y[i] = t * inv[i];
    }
    for (int i = 5; i >= 0; --i) {
        double t = y[i];
        for (int k = i + 1; k < 6; ++k) t -= L[k][i] * x[k];
        x[i] = t * inv[i];
    }
    return true;
}

// Decrease of the sum of squares that the linear model predicts for the step
// d: -(2 d.b + d.H.d), from the packed normal equations.
__device__ double lm_predicted(const double *ne, const double d[6])
{
    double g = 0.0, q = 0.0;
    for (int a = 0; a < 6; ++a) {
        double s = 0.0;
        for (int b = 0; b < 6; ++b) {
            const int r = a < b ? a : b, c = a < b ? b : a;
            s += ne[r * 6 - r * (r - 1) / 2 + (c - r)] * d[b];
        }
        q += d[a] * s;
        g += d[a] * ne[21 + a];
    }
    return -(2.0 * g + q);
}

// T <- Exp(xi) T for xi = (rho, theta); T is the top 3x4 of a rigid
// transform, row-major.
__device__ void se3_left_update(const double xi[6], double T[12])
{
    const double *w = xi + 3;
    const double th2 = w[0] * w[0] + w[1] * w[1] + w[2] * w[2];
    const double th = sqrt(th2);
    double A, B, C;
    if (th < 1e-4) {
        A = 1.0 - th2 / 6.0 + th2 * th2 / 120.0;
        B = 0.5 - th2 / 24.0 + th2 * th2 / 720.0;
        C = 1.0 / 6.0 - th2 / 120.0 + th2 * th2 / 5040.0;
    } else {
        const double sh = sin(0.5 * th);
        A = sin(th) / th;
        B = 2.0 * sh * sh / th2;
        C = (th - sin(th)) / (th2 * th);
    }
    const double K[3][3] = {{0, -w[2], w[1]}, {w[2], 0, -w[0]}, {-w[1], w[0], 0}};
    double K2[3][3], Rm[3][3], V[3][3];
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) K2[r][c] = K[r][0] * K[0][c] + K[r][1] * K[1][c] + K[r][2] * K[2][c];
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) {
            const double I = r == c ? 1.0 : 0.0;
            Rm[r][c] = I + A * K[r][c] + B * K2[r][c];
            V[r][c] = I + B * K[r][c] + C * K2[r][c];
        }
    double tE[3];
    for (int r = 0; r < 3; ++r) tE[r] = V[r][0] * xi[0] + V[r][1] * xi[1] + V[r][2] * xi[2];
    double O[12];
    for (int r = 0; r < 3; ++r) {
        for (int c = 0; c < 3; ++c) O[4 * r + c] = (Rm[r][0] * T[c] + Rm[r][1] * T[4 + c]) + Rm[r][2] * T[8 + c];
        O[4 * r + 3] = ((Rm[r][0] * T[3] + Rm[r][1] * T[7]) + Rm[r][2] * T[11]) + tE[r];
    }
    for (int k = 0; k < 12; ++k) T[k] = O[k];
}

// LM ends as converged when the decrease L that the model predicts is
// within the cost's binary32 rounding noise, L <= 2^-19 Q sqrt(c): each
// residual carries an error of up to 16 u Q (u = 2^-24, Q the largest norm
// of a corner of A's ESDF domain, in metres), and over the residuals these
// errors add in root-sum-square to at most 2 * 16 u Q sqrt(c) in c = sum r^2;
// below that the gain ratio is rounding noise.
constexpr double kCostNoise32 = 1.0 / 524288.0;  // 2 * 16 * 2^-24
constexpr int kSums = 29;       // 21 of H, 6 of b, sum r^2, count
constexpr int kSumStride = 32;  // doubles per segment in memory
// Points per lane of a segment.  More lengthens the chain of one pair (a lane's
// points run one after another), fewer adds workgroup reductions to a batch: at
// 2, 4 and 8 one room pair (15 k points) took 253, 262 and 326 us, and 64
// outdoor pairs of 25 k points with 8 starts 4.15, 3.58 and 3.25 ms.
constexpr int kSegPoints = 4;

// A problem between evaluations.  Gauss-Newton takes every solve.
// Levenberg-Marquardt (the trust-region least squares Sec. III-F names) damps
// it by mu diag(H), evaluates the trial pose, and takes the step when the mean
// cost falls (gain ratio > 0); max_iter then caps the solves.
struct AlignState {
    double T[12];      // accepted pose
    double Te[12];     // pose of the next evaluation
    double ne[kSums];  // sums of the accepted pose (Gauss-Newton: set when done)
    double dl[6];      // LM: step to the trial pose
    double mu, nu;     // LM
    int32_t final_eval, solves, status;
    int32_t have, steps;  // LM: ne holds the accepted pose's sums; steps taken
    int32_t done;
};

struct AlignRun {
    float vs;
    double tol_rho, tol_theta;
    int n_min, dof, lm;
};

__device__ void align_init(AlignState &S, const AlignProblem &P)
{
    for (int k = 0; k < 12; ++k) S.T[k] = S.Te[k] = P.T[k];
    for (int k = 0; k < 6; ++k) S.dl[k] = 0.0;
    S.mu = 1e-4;
    S.nu = 2.0;
    S.final_eval = S.solves = S.have = S.steps = S.done = 0;
    S.status = COVOX_NOT_CONVERGED;
}

// Takes the sums of the evaluation at Te: ends the problem or sets the next Te.
__device__ void align_advance(AlignState &S, const double *tot, const AlignProblem &P, const AlignRun &A)
{
    double dl[6];
    if (!A.lm) {
        if (S.final_eval || S.solves >= P.max_iter) {
            S.done = 1;
        } else if (tot[28] < (double)A.n_min || !(A.dof == 4 ? solve_xyz_yaw(tot, 0.0, dl) : solve6(tot, 0.0, dl))) {
            S.status = COVOX_EDEGENERATE;
            S.done = 1;
        } else {
            se3_left_update(dl, S.T);
            for (int k = 0; k < 12; ++k) S.Te[k] = S.T[k];
            S.solves += 1;
            const double nr = sqrt(dl[0] * dl[0] + dl[1] * dl[1] + dl[2] * dl[2]);
            const double nt = sqrt(dl[3] * dl[3] + dl[4] * dl[4] + dl[5] * dl[5]);
            if (nr < A.tol_rho && nt < A.tol_theta) {
                S.status = COVOX_OK;
                S.final_eval = 1;  // one more evaluation at the final pose
            }
        }
        if (S.done)
            for (int k = 0; k < kSums; ++k) S.ne[k] = tot[k];
        return;
    }
    if (!S.have) {  // sums at the start pose
        for (int k = 0; k < kSums; ++k) S.ne[k] = tot[k];
        if (P.max_iter <= 0) {
            S.done = 1;
            return;
        }
        if (tot[28] < (double)A.n_min) {
            S.status = COVOX_EDEGENERATE;
            S.done = 1;
            return;
        }
        S.have = 1;
    } else {  // sums at the trial pose: take the step or raise the damping
        const double pred = lm_predicted(S.ne, S.dl);
        double rho = -1.0;
        if (tot[28] >= (double)A.n_min && pred > 0.0)
            rho = (S.ne[27] / S.ne[28] - tot[27] / tot[28]) / (pred / S.ne[28]);
        if (rho > 0.0) {
            for (int k = 0; k < 12; ++k) S.T[k] = S.Te[k];
            for (int k = 0; k < kSums; ++k) S.ne[k] = tot[k];
            S.steps += 1;
            const double s = 2.0 * rho - 1.0, f = 1.0 - s * s * s;
            S.mu *= f > 1.0 / 3.0 ? f : 1.0 / 3.0;
            S.nu = 2.0;
        } else {
            S.mu *= S.nu;
            S.nu *= 2.0;
        }
    }
    if (S.solves >= P.max_iter) {
        S.done = 1;
    } else if (!(A.dof == 4 ? solve_xyz_yaw(S.ne, S.mu, dl) : solve6(S.ne, S.mu, dl))) {
        S.status = COVOX_EDEGENERATE;
        S.done = 1;
    } else {
        S.solves += 1;
        double q2 = 0.0;  // the floor of the predicted decrease is noise sqrt(c)
        const DomArgs d = dom_of(P.metaA);
        for (int a = 0; a < 3; ++a) {
            const double e = 8.0 * (double)A.vs;
            const double m = fmax(fabs(e * (double)d.lo[a]), fabs(e * (double)(d.lo[a] + d.dim[a])));
            q2 += m * m;
        }
        const double noise = kCostNoise32 * sqrt(q2);
        const double nr = sqrt(dl[0] * dl[0] + dl[1] * dl[1] + dl[2] * dl[2]);
        const double nt = sqrt(dl[3] * dl[3] + dl[4] * dl[4] + dl[5] * dl[5]);
        if ((nr < A.tol_rho && nt < A.tol_theta) || lm_predicted(S.ne, dl) <= noise * sqrt(S.ne[27])) {
            S.status = COVOX_OK;  // converged; the step is not taken
            S.done = 1;
        } else {
            for (int k = 0; k < 12; ++k) S.Te[k] = S.T[k];
            se3_left_update(dl, S.Te);
            for (int k = 0; k < 6; ++k) S.dl[k] = dl[k];
        }
    }
}

// Sums of 32 values over the wave: lane l returns the sum of a[l / 2].  Each
// stage halves the values and the lanes that share one (32 + 16 register swaps,
// then DPP): 31 additions a lane, against 6 for each value by butterflies.
__device__ __forceinline__ double wave_sum32(double a[32])
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < 16; ++i) a[i] = swap_add<false>(a[i], a[i + 16]);
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = swap_add<true>(a[i], a[i + 8]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const bool up = lane & 8;
        a[i] = (up ? a[i + 4] : a[i]) + dpp_f64<0x128>(up ? a[i] : a[i + 4]);  // row_ror:8
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const bool up = lane & 4;
        a[i] = (up ? a[i + 2] : a[i]) + dpp_f64<0x141>(up ? a[i] : a[i + 2]);  // row_half_mirror
    }
    const bool up = lane & 2;
    a[0] = (up ? a[1] : a[0]) + dpp_f64<0x4E>(up ? a[0] : a[1]);  // quad_perm 2,3,0,1
    return a[0] + dpp_f64<0xB1>(a[0]);                            // quad_perm 1,0,3,2
}

template <int NT>
struct AlignShared {
    AlignState S;
    double red[NT / 32][kSumStride];
    double tot[kSumStride];
};

// Sums of one segment of a problem at the pose sh.S.Te, to out.
template <int NT, int U, bool TILED>
__device__ __forceinline__ void align_segment(AlignShared<NT> &sh, const AlignProblem &P, const DomArgs &d, int64_t seg,
                                              float vs, double *out)
{
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    float Tf[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) Tf[k] = (float)sh.S.Te[k];
    double acc[32];
#pragma unroll
    for (int k = 0; k < 32; ++k) acc[k] = 0.0;
    const int64_t i0 = seg * (kSegPoints * NT) + tid;
#pragma unroll 1
    for (int p = 0; p < kSegPoints; p += U) {
        float J[U][6], r[U];
        bool ok[U];
        residual_u<U, TILED>(Tf, P.pts, i0 + (int64_t)p * NT, NT, P.n_pts, vs, TILED ? P.tiles : P.phi, P.n_tiles, P.page,
                             d, J, r, ok);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!ok[u]) continue;
            double Jd[6];
#pragma unroll
            for (int a = 0; a < 6; ++a) Jd[a] = (double)J[u][a];
            const double rd = (double)r[u];
            int m = 0;
            // products of binary32 values are exact in binary64: a fused
            // multiply-add rounds as the product and the sum do
#pragma unroll
            for (int a = 0; a < 6; ++a)
#pragma unroll
                for (int b = a; b < 6; ++b, ++m) acc[m] = fma(Jd[a], Jd[b], acc[m]);
#pragma unroll
            for (int a = 0; a < 6; ++a) acc[21 + a] = fma(Jd[a], rd, acc[21 + a]);
            acc[27] = fma(rd, rd, acc[27]);
            acc[28] += 1.0;
        }
    }
    const double v = wave_sum32(acc);
    __syncthreads();  // red is free
    if (!(lane & 1)) sh.red[wid][lane >> 1] = v;
    __syncthreads();
    if (tid < kSums) {
        double s = 0.0;
        for (int w = 0; w < NT / 64; ++w) s += sh.red[w][tid];
        out[tid] = s;
    }
}

// Word that tells the host, while it enqueues evaluations, that no problem needs
// another one.
struct AlignEnd {
    int32_t *ended;  // problems that have ended (cleared by evaluation 0)
    uint64_t *host;  // pinned; null: nobody looks
    uint64_t token;  // this launch's
};

__device__ __forceinline__ void align_ended(const AlignEnd &E, int n)
{
    if (atomicAdd(E.ended, 1) == n - 1 && E.host) *(volatile uint64_t *)E.host = E.token;
}

// The state before evaluation `it` into sh.S: the start, or the last state with
// the sums of evaluation it - 1 (the segments' sums in a fixed order) taken.
// True where that ends the problem.
template <int NT>
__device__ __forceinline__ bool align_next_state(AlignShared<NT> &sh, const AlignProblem &P, int it,
                                                 const AlignState *old, const double *part,
                                                 const AlignRun &A)
{
    static_assert(sizeof(AlignState) % 8 == 0, "copied in 8-byte words");
    constexpr int kWords = sizeof(AlignState) / 8;
    const int tid = threadIdx.x;
    if (it == 0) {
        if (tid == 0) align_init(sh.S, P);
        __syncthreads();
        return false;
    }
    const int k = tid & 31, g = tid >> 5;
    for (int w = tid; w < kWords; w += NT) ((uint64_t *)&sh.S)[w] = ((const uint64_t *)old)[w];
    double s = 0.0;
    if (k < kSums)
        for (int q = g; q < P.n_segs; q += NT / 32) s += part[(int64_t)q * kSumStride + k];
    sh.red[g][k] = s;
    __syncthreads();
    if (sh.S.done) return false;  // uniform
    if (tid < kSums) {
        double t = 0.0;
        for (int w = 0; w < NT / 32; ++w) t += sh.red[w][tid];
        sh.tot[tid] = t;
    }
    __syncthreads();
    if (tid == 0) align_advance(sh.S, sh.tot, P, A);
    __syncthreads();
    return sh.S.done;
}

template <int NT>
__device__ __forceinline__ void store_state(const AlignShared<NT> &sh, AlignState *out)
{
    for (int w = threadIdx.x; w < (int)(sizeof(AlignState) / 8); w += NT)
        ((uint64_t *)out)[w] = ((const uint64_t *)&sh.S)[w];
}

// Evaluation `it` of every problem: workgroup w takes segment segs[w].  States
// and sums alternate between two buffers, so that no launch reads what it
// writes.  FUSED: each segment's workgroup makes the problem's solve itself (the
// first one stores the state); else k_align_advance has made it.  Bound by
// latency for few segments (a chain of point, page and tile reads, the
// reduction, the solve in one lane: 10 us a launch), by vector instructions for
// many.  One workgroup per problem took 120 us an evaluation of a room pair of
// 15 k points; 64 outdoor pairs with 8 starts went from 9.8 to 3.1 ms.
template <int NT, int U, bool TILED>
__global__ __launch_bounds__(NT) void k_align_step(const AlignProblem *__restrict__ probs,
                                                   const int2 *__restrict__ segs, int it, int fused, AlignState *states,
                                                   double *parts, int n, int64_t n_segs, AlignRun A, AlignEnd E)
{
    __shared__ AlignShared<NT> sh;
    const int2 w = segs[blockIdx.x];  // problem, segment
    const AlignProblem &P = probs[w.x];
    if (fused) {
        const int prev = (it + 1) & 1;
        const bool ends = align_next_state<NT>(sh, P, it, states + (int64_t)prev * n + w.x,
                                               parts + (prev * n_segs + P.seg0) * kSumStride, A);
        if (w.y == 0) store_state<NT>(sh, states + (int64_t)(it & 1) * n + w.x);
        if (threadIdx.x == 0 && w.y == 0 && ends) align_ended(E, n);
        if (threadIdx.x == 0 && blockIdx.x == 0 && it == 0) *E.ended = 0;
    } else {
        const AlignState *S = states + (int64_t)(it & 1) * n + w.x;
        for (int k = threadIdx.x; k < (int)(sizeof(AlignState) / 8); k += NT)
            ((uint64_t *)&sh.S)[k] = ((const uint64_t *)S)[k];
        __syncthreads();
    }
    if (sh.S.done) return;  // uniform
    align_segment<NT, U, TILED>(sh, P, dom_of(P.metaA), w.y, A.vs,
                                parts + ((it & 1) * n_segs + P.seg0 + w.y) * kSumStride);
}

template <int NT>
__global__ __launch_bounds__(NT) void k_align_advance(const AlignProblem *__restrict__ probs, int it,
                                                      AlignState *states, const double *__restrict__ parts, int n,
                                                      int64_t n_segs, AlignRun A, AlignEnd E)
{
    __shared__ AlignShared<NT> sh;
    const AlignProblem &P = probs[blockIdx.x];
    const int prev = (it + 1) & 1;
    const bool ends = align_next_state<NT>(sh, P, it, states + (int64_t)prev * n + blockIdx.x,
                                           parts + (prev * n_segs + P.seg0) * kSumStride, A);
    store_state<NT>(sh, states + (int64_t)(it & 1) * n + blockIdx.x);
    if (threadIdx.x == 0 && ends) align_ended(E, n);
    if (threadIdx.x == 0 && blockIdx.x == 0 && it == 0) *E.ended = 0;
}

__device__ void align_result(const AlignState &S, const AlignRun &A, AlignResult &R)
{
    for (int k = 0; k < 12; ++k) R.T[k] = S.T[k];
    R.T[12] = 0; R.T[13] = 0; R.T[14] = 0; R.T[15] = 1;
    for (int k = 0; k < kSums; ++k) R.ne[k] = S.ne[k];
    R.n_used = (int64_t)S.ne[28];
    R.cost = S.ne[28] > 0 ? S.ne[27] / S.ne[28] : __builtin_inf();
    R.iters = A.lm && S.have ? S.steps : S.solves;
    R.solves = S.solves;
    R.status = S.status;
}

// After evaluation it - 1, the last that any problem can need.
template <int NT>
__global__ __launch_bounds__(NT) void k_align_finish(const AlignProblem *__restrict__ probs, int it,
                                                     const AlignState *__restrict__ states,
                                                     const double *__restrict__ parts, int n, int64_t n_segs,
                                                     AlignRun A, AlignResult *res)
{
    __shared__ AlignShared<NT> sh;
    const AlignProblem &P = probs[blockIdx.x];
    const int prev = (it + 1) & 1;
    align_next_state<NT>(sh, P, it, states + (int64_t)prev * n + blockIdx.x,
                         parts + (prev * n_segs + P.seg0) * kSumStride, A);
    if (threadIdx.x == 0) align_result(sh.S, A, res[blockIdx.x]);
}

// One workgroup takes its problem to the end.  It reads back the sums that it
// wrote itself, in the same order as the launches above.
template <int NT, int U, bool TILED>
__global__ __launch_bounds__(NT) void k_align_solo(const AlignProblem *__restrict__ probs, AlignState *states,
                                                   double *parts, AlignRun A, AlignResult *res)
{
    __shared__ AlignShared<NT> sh;
    const AlignProblem &P = probs[blockIdx.x];
    const DomArgs d = dom_of(P.metaA);
    double *part = parts + (int64_t)P.seg0 * kSumStride;
    AlignState *S = states + blockIdx.x;
    for (int it = 0;; it = 1) {
        align_next_state<NT>(sh, P, it, S, part, A);
        if (sh.S.done) break;  // uniform
        for (int seg = 0; seg < P.n_segs; ++seg)
            align_segment<NT, U, TILED>(sh, P, d, seg, A.vs, part + (int64_t)seg * kSumStride);
        store_state<NT>(sh, S);
        __threadfence_block();
        __syncthreads();
    }
    if (threadIdx.x == 0) align_result(sh.S, A, res[blockIdx.x]);
}

// ---------------------------------------------------------------- summaries

// ESDF value at q by trilinear interpolation of the 8 cell corners (the
// residual's operation order); false when a corner is unobserved.
__device__ __forceinline__ bool phi_trilinear(const float q[3], float vs, const float *phi, const int32_t *page,
                                              const DomArgs &d, float &r)
{
    float f[3];
    int j0[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float g = (q[a] / vs) - 0.5f;
        if (!(fabsf(g) < 1.0e8f)) return false;
        const float fl = floorf(g);
        j0[a] = (int)fl;
        f[a] = g - fl;
    }
    float c[8];
#pragma unroll
    for (int k = 0; k < 8; ++k)
        c[k] = phi_at(phi, page, d, j0[0] + (k & 1), j0[1] + ((k >> 1) & 1), j0[2] + ((k >> 2) & 1));
#pragma unroll
    for (int k = 0; k < 8; ++k)
        if (isnan(c[k])) return false;
    const float wx0 = 1.0f - f[0], wx1 = f[0], wy0 = 1.0f - f[1], wy1 = f[1], wz0 = 1.0f - f[2], wz1 = f[2];
    const float c00 = c[0] * wx0 + c[1] * wx1, c10 = c[2] * wx0 + c[3] * wx1;
    const float c01 = c[4] * wx0 + c[5] * wx1, c11 = c[6] * wx0 + c[7] * wx1;
    const float c0 = c00 * wy0 + c10 * wy1, c1 = c01 * wy0 + c11 * wy1;
    r = c0 * wz0 + c1 * wz1;
    return true;
}

// One lane per cell of a 32^3 grid: cell centre ((i + 0.5) - 16) * cell in the
// grid frame, mapped to the submap by T (binary32, row-major 3x4); writes
// (clamp(phi / d_max, -1, 1), 1) or (0, 0) to channels chan, chan + 1 of a
// 4-channel NDHWC block.
__global__ __launch_bounds__(256) void k_summary(const SummaryReq *__restrict__ reqs, int n, float vs, float dmax)
{
    const int64_t total = (int64_t)n * 32768;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const SummaryReq &R = reqs[i >> 15];
        const int c = (int)(i & 32767);
        const int cx = c & 31, cy = (c >> 5) & 31, cz = c >> 10;
        const float g[3] = {(((float)cx + 0.5f) - 16.0f) * R.cell, (((float)cy + 0.5f) - 16.0f) * R.cell,
                            (((float)cz + 0.5f) - 16.0f) * R.cell};
        float q[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) q[a] = ((R.T[4 * a] * g[0] + R.T[4 * a + 1] * g[1]) + R.T[4 * a + 2] * g[2]) + R.T[4 * a + 3];
        const DomArgs d = dom_of(R.meta);
        float r, val = 0.0f, msk = 0.0f;
        if (phi_trilinear(q, vs, R.phi, R.page, d, r)) {
            val = fminf(1.0f, fmaxf(-1.0f, r / dmax));
            msk = 1.0f;
        }
        R.out[4 * c + R.chan] = val;
        R.out[4 * c + R.chan + 1] = msk;
    }
}

unsigned grid_waves(int64_t waves)
{
    const int64_t g = (waves + 3) / 4;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(g, 8192));
}

}  // namespace

int extract_points(covox_ctx *ctx, const covox_submap *Bc)
{
    // The registration points, the page and their versions are a cache the
    // library keeps inside the submap; the map itself (keys, D, W) is only
    // read here.
    covox_submap *B = const_cast<covox_submap *>(Bc);
    if (B->pts_version == B->version) return COVOX_OK;
    int rc;
    if ((rc = build_page(ctx, B))) return rc;
    const int64_t nbk = std::max<int64_t>(1, std::min(B->nb_upper, B->cap));
    if ((rc = ensure_buffer(ctx, (void **)&ctx->cnt, &ctx->cnt_cap, nbk, sizeof(uint32_t), "point counts"))) return rc;
    if ((rc = ensure_buffer(ctx, (void **)&ctx->psum, &ctx->psum_cap, nbk, 3 * sizeof(double), "point sums")))
        return rc;
    const covox_params &p = ctx->p;
    const float vs = (float)p.voxel_size, tau = (float)band_limit(p), wreg = (float)p.w_reg;
    const bool h = p.precision == COVOX_FP16;
    auto iso = [&](int write) {
        if (h)
            hipLaunchKernelGGL(k_iso<__half>, dim3(grid_waves(nbk)), dim3(256), 0, ctx->stream, B->meta, B->keys,
                               B->page, (const __half *)B->D, (const __half *)B->W, vs, tau, wreg, write, ctx->cnt,
                               B->pts, B->pts_cap, ctx->psum);
        else
            hipLaunchKernelGGL(k_iso<float>, dim3(grid_waves(nbk)), dim3(256), 0, ctx->stream, B->meta, B->keys,
                               B->page, (const float *)B->D, (const float *)B->W, vs, tau, wreg, write, ctx->cnt,
                               B->pts, B->pts_cap, ctx->psum);
    };
    auto points = [&]() -> int {
        TimedLaunch tl(ctx, COVOX_K_ISO);
        iso(1);
        hipLaunchKernelGGL(k_pbar, dim3(1), dim3(kPbarThreads), 0, ctx->stream, B->meta, ctx->psum);
        return hip_check(ctx, hipGetLastError(), "point write launch");
    };
    SubmapMeta m;
    auto read_meta = [&]() -> int {
        int rc2 = hip_check(ctx, hipMemcpyAsync(&m, B->meta, sizeof(m), hipMemcpyDeviceToHost, ctx->stream), "meta copy");
        return rc2 ? rc2 : hip_check(ctx, hipStreamSynchronize(ctx->stream), "point count sync");
    };
    {
        TimedLaunch tl(ctx, COVOX_K_ISO);
        iso(0);
        hipLaunchKernelGGL(k_iso_scan, dim3(1), dim3(1024), 0, ctx->stream, B->meta, ctx->cnt);
    }
    if ((rc = hip_check(ctx, hipGetLastError(), "point count launch"))) return rc;
    // Into the room of an earlier extraction without a look at the count, so with one
    // wait; again if that turns out to be short.
    const bool ahead = B->pts_cap > 0;
    if ((ahead && (rc = points())) || (rc = read_meta())) return rc;
    const int64_t n = m.n_points;
    if (!ahead || n > B->pts_cap) {
        if ((rc = ensure_buffer(ctx, (void **)&B->pts, &B->pts_cap, std::max<int64_t>(n, 1), 3 * sizeof(float), "points")))
            return rc;
        if ((rc = points()) || (rc = read_meta())) return rc;
    }
    B->n_pts = n;
    for (int a = 0; a < 3; ++a) B->pbar[a] = m.pbar[a];
    B->pts_version = B->version;
    return COVOX_OK;
}

int run_summaries(covox_ctx *ctx, const SummaryReq *reqs, int n)
{
    if (n <= 0) return COVOX_OK;
    int rc;
    const size_t bytes = sizeof(SummaryReq) * n;
    if ((rc = ensure_buffer(ctx, &ctx->sum_dev, &ctx->sum_cap, (int64_t)bytes, 1, "summary requests"))) return rc;
    if ((rc = hip_check(ctx, hipMemcpyAsync(ctx->sum_dev, reqs, bytes, hipMemcpyHostToDevice, ctx->stream),
                        "summary upload")))
        return rc;
    {
        TimedLaunch tl(ctx, COVOX_K_SUMMARY);
        const int64_t total = (int64_t)n * 32768;
        hipLaunchKernelGGL(k_summary, dim3((unsigned)std::min<int64_t>((total + 255) / 256, 1 << 20)), dim3(256), 0,
                           ctx->stream, (const SummaryReq *)ctx->sum_dev, n, (float)ctx->p.voxel_size,
                           (float)ctx->p.d_max);
    }
    return hip_check(ctx, hipGetLastError(), "summary launch");
}

AlignLaunch align_launch_of(const covox_ctx *ctx)
{
    AlignLaunch L;
    L.vs = (float)ctx->p.voxel_size;
    L.tol_rho = ctx->p.tol_rho;
    L.tol_theta = ctx->p.tol_theta;
    L.n_min = ctx->p.n_min;
    L.dof = ctx->p.align_dof;
    L.lm = ctx->p.align_solver == COVOX_LEVENBERG_MARQUARDT;
    L.threads = ctx->tune.align_threads == 512 ? 512 : 256;
    L.pps = ctx->tune.align_points_per_step == 2 ? 2 : 1;
    return L;
}

// Blocks of A's field: exact once the last integration's count has arrived in
// pinned memory, else the host's bound.
static int64_t field_blocks(covox_ctx *ctx, const covox_submap *A)
{
    // (waits only for work that the alignment would wait for too)
    if ((*A->pin_nb >> 40) != (A->seq & 0xFFFFFFull)) (void)hipStreamSynchronize(ctx->stream);
    int64_t nb = std::min(A->nb_upper, A->cap);
    const uint64_t v = *A->pin_nb;
    if ((v >> 40) == (A->seq & 0xFFFFFFull)) nb = std::min<int64_t>(nb, (int64_t)(v & ((1ull << 40) - 1)));
    return std::max<int64_t>(1, nb);
}

// Iteration caps up to this are enqueued as one launch an evaluation; under longer
// ones, launches that nobody waits for (sets and graphs, which would keep the host
// enqueueing, 4 us each, or hold a node each, 1.3 us a replay) take k_align_solo.  A
// call that waits for its results stops at the last evaluation needed whatever its
// cap (a room pair of 15 k points, 16 evaluations under a cap of 100: 923 us in one
// workgroup, 259 by launches).
constexpr int kMaxStepIters = 64;
// Problems of up to this many segments take k_align_solo too: one workgroup is as fast
// as a launch an evaluation (1 segment 6.2 us for 8.6, 2 segments 9.5 for 9.0, 3
// segments 12 for 9), and a problem that ends early has no launches left to drain (of
// 700 points outside the field: 41 us a call, 124 with 31 launches; Levenberg-
// Marquardt over 1900 points 92 us, 147).
constexpr int kSoloSegs = 2;
// Up to this many segments the chip holds all workgroups at once (four to a CU),
// and a solve in each of them is shorter than a launch of its own; beyond, the
// solves would take the CUs' time from other segments' points (64 outdoor pairs
// with 8 starts, 12 k segments: 4.6 ms with the solves in every workgroup, 3.1
// with a launch for them).
constexpr int64_t kFusedSegs = 1024;

// Whether the fields are worth their tiles.  Microseconds measured: tiles 3 and 1.6 for
// a thousand blocks; an evaluation by pages takes 2 more than by tiles (in one
// workgroup, 2 for each of a problem's segments) and 12.5 for a million points.  (8.7 k
// blocks: one evaluation of 15 k points 53 with tiles, 39 by pages; 30 of 10 k points
// over 2.5 k blocks 331 and 393.)  Ten evaluations are counted on: pairs that overlap
// take 7 to 30, the others one.
static bool worth_tiles(const std::vector<const covox_submap *> &fields, const AlignProblem *probs, int n, int n_min,
                        int iters, int max_segs)
{
    double blocks = 0.0, points = 0.0;
    for (const covox_submap *A : fields) blocks += (double)(*A->pin_nb & ((1ull << 40) - 1));  // (an estimate will do)
    for (int i = 0; i < n; ++i)
        if (probs[i].n_pts >= n_min) points += (double)probs[i].n_pts;  // (with fewer a problem ends at once)
    const int evals = points > 0.0 ? std::min(iters, 9) + 1 : 1;
    const double saved = 2.0 * (max_segs <= kSoloSegs ? max_segs : 1) + 12.5e-6 * points;
    return evals * saved > 3.0 + 1.6e-3 * blocks;
}

int plan_alignment(covox_ctx *ctx, AlignProblem *probs, int n, const AlignLaunch &L, int iters, AlignPlan &pl, bool tiles)
{
    pl.n = n;
    pl.launch = L;
    pl.max_iter = pl.max_segs = 0;
    const int64_t per = (int64_t)kSegPoints * L.threads;
    int64_t segs = 0;
    for (int i = 0; i < n; ++i) {
        AlignProblem &P = probs[i];
        P.seg0 = (int32_t)segs;
        P.n_segs = (int32_t)std::max<int64_t>(1, (P.n_pts + per - 1) / per);
        segs += P.n_segs;
        pl.max_segs = std::max(pl.max_segs, P.n_segs);
        if (segs > INT32_MAX) return fail(ctx, COVOX_EINVAL, "align: too many registration points in one call");
        pl.max_iter = std::max(pl.max_iter, P.max_iter);
    }
    pl.n_segs = segs;
    // the distinct fields
    std::vector<const covox_submap *> fields;
    std::vector<int32_t> of(n);
    std::unordered_map<const covox_submap *, int32_t> index;
    for (int i = 0; i < n; ++i) {
        if (i > 0 && probs[i].A == probs[i - 1].A) {
            of[i] = of[i - 1];
            continue;
        }
        const auto it = index.emplace(probs[i].A, (int32_t)fields.size());
        if (it.second) fields.push_back(probs[i].A);
        of[i] = it.first->second;
    }
    pl.tiled = tiles && ctx->align_field != 2 &&
               (ctx->align_field == 1 || worth_tiles(fields, probs, n, L.n_min, iters, pl.max_segs));
    if (!pl.tiled) fields.clear();
    std::vector<int64_t> nb(fields.size());
    for (size_t f = 0; f < fields.size(); ++f) nb[f] = field_blocks(ctx, fields[f]);
    pl.n_jobs = (int)fields.size();
    auto align16 = [](size_t b) { return (b + 15) / 16 * 16; };
    pl.off_segs = align16(sizeof(AlignProblem) * n);
    pl.off_jobs = align16(pl.off_segs + sizeof(int2) * segs);
    pl.up_bytes = align16(pl.off_jobs + sizeof(TileJob) * fields.size());
    pl.off_states = pl.up_bytes;
    pl.off_parts = align16(pl.off_states + sizeof(AlignState) * 2 * n);
    pl.off_end = align16(pl.off_parts + sizeof(double) * kSumStride * 2 * segs);
    pl.off_tiles = pl.off_end + 16;
    std::vector<size_t> at(fields.size());
    pl.total = pl.off_tiles;
    pl.tile_blocks = 0;
    for (size_t f = 0; f < fields.size(); ++f) {
        at[f] = pl.total;
        pl.total = align16(pl.total + sizeof(float) * kTile * nb[f]);
        pl.tile_blocks = std::max(pl.tile_blocks, nb[f]);
    }
    pl.stage.assign(pl.up_bytes, 0);
    // addresses relative to the plan's memory until bind_alignment
    TileJob *jobs = (TileJob *)(pl.stage.data() + pl.off_jobs);
    for (size_t f = 0; f < fields.size(); ++f) {
        const covox_submap *A = fields[f];
        jobs[f] = TileJob{A->phi, A->page, A->meta, A->keys, (float *)at[f], nb[f]};
    }
    for (int i = 0; i < n; ++i) {
        probs[i].phi = probs[i].A->phi;
        probs[i].tiles = pl.tiled ? (const float *)at[of[i]] : nullptr;
        probs[i].n_tiles = pl.tiled ? nb[of[i]] : 0;
    }
    ::memcpy(pl.stage.data(), probs, sizeof(AlignProblem) * n);
    int2 *sg = (int2 *)(pl.stage.data() + pl.off_segs);
    for (int i = 0; i < n; ++i)
        for (int q = 0; q < probs[i].n_segs; ++q) sg[probs[i].seg0 + q] = make_int2(i, q);
    return COVOX_OK;
}

int bind_alignment(covox_ctx *ctx, AlignPlan &pl, void *dev)
{
    pl.dev = (char *)dev;
    TileJob *jobs = (TileJob *)(pl.stage.data() + pl.off_jobs);
    for (int f = 0; f < pl.n_jobs; ++f) jobs[f].tiles = (float *)(pl.dev + (size_t)jobs[f].tiles);
    AlignProblem *probs = (AlignProblem *)pl.stage.data();
    for (int i = 0; i < pl.n && pl.tiled; ++i) probs[i].tiles = (const float *)(pl.dev + (size_t)probs[i].tiles);
    return hip_check(ctx, hipMemcpyAsync(pl.dev, pl.stage.data(), pl.up_bytes, hipMemcpyHostToDevice, ctx->stream),
                     "problem upload");
}

namespace {

template <int NT, int U, bool TILED>
void launch_shape(covox_ctx *ctx, const AlignPlan &pl, AlignResult *dres, bool waits)
{
    const AlignLaunch &L = pl.launch;
    const AlignRun A{L.vs, L.tol_rho, L.tol_theta, L.n_min, L.dof, L.lm};
    const AlignProblem *probs = (const AlignProblem *)pl.dev;
    const int2 *segs = (const int2 *)(pl.dev + pl.off_segs);
    AlignState *states = (AlignState *)(pl.dev + pl.off_states);
    double *parts = (double *)(pl.dev + pl.off_parts);
    if (pl.max_segs <= kSoloSegs || (pl.max_iter > kMaxStepIters && !(waits && ctx->align_pin))) {
        hipLaunchKernelGGL((k_align_solo<NT, U, TILED>), dim3(pl.n), dim3(NT), 0, ctx->stream, probs, states, parts, A, dres);
        return;
    }
    const int fused = pl.n_segs <= kFusedSegs;
    // The evaluations that no problem needs are not enqueued, as far as the GPU is
    // ahead of the host (15 k points outside the field: 66 us a call, 182 with all
    // 31).  A graph holds all of them, at 1.3 us each.
    volatile uint64_t *pin = ctx->capturing ? nullptr : ctx->align_pin;
    const AlignEnd E{(int32_t *)(pl.dev + pl.off_end), (uint64_t *)pin, ++ctx->align_token};
    int it = 0;
    for (; it <= pl.max_iter && !(pin && *pin == E.token); ++it) {
        if (!fused)
            hipLaunchKernelGGL((k_align_advance<NT>), dim3(pl.n), dim3(NT), 0, ctx->stream, probs, it, states, parts,
                               pl.n, pl.n_segs, A, E);
        hipLaunchKernelGGL((k_align_step<NT, U, TILED>), dim3((unsigned)pl.n_segs), dim3(NT), 0, ctx->stream, probs, segs, it,
                           fused, states, parts, pl.n, pl.n_segs, A, E);
    }
    hipLaunchKernelGGL((k_align_finish<NT>), dim3(pl.n), dim3(NT), 0, ctx->stream, probs, it, states, parts, pl.n,
                       pl.n_segs, A, dres);
}

}  // namespace

int launch_alignment(covox_ctx *ctx, const AlignPlan &pl, AlignResult *dres, bool tiles, bool waits)
{
    if (pl.n <= 0) return COVOX_OK;
    {
        TimedLaunch tl(ctx, COVOX_K_ALIGN);
        const bool wide = pl.launch.threads == 512, two = pl.launch.pps == 2;
        auto shape = [&](auto tiled) {
            constexpr bool T = decltype(tiled)::value;
            if (wide && two) launch_shape<512, 4, T>(ctx, pl, dres, waits);
            else if (wide) launch_shape<512, 2, T>(ctx, pl, dres, waits);
            else if (two) launch_shape<256, 4, T>(ctx, pl, dres, waits);
            else launch_shape<256, 2, T>(ctx, pl, dres, waits);
        };
        if (pl.tiled) {
            const unsigned gx = (unsigned)std::min<int64_t>((pl.tile_blocks + 3) / 4, 4096);
            if (tiles)
                hipLaunchKernelGGL(k_align_tiles, dim3(gx, (unsigned)pl.n_jobs), dim3(256), 0, ctx->stream,
                                   (const TileJob *)(pl.dev + pl.off_jobs));
            shape(std::true_type{});
        } else {
            shape(std::false_type{});
        }
    }
    return hip_check(ctx, hipGetLastError(), "align launch");
}

int place_alignment(covox_ctx *ctx, AlignProblem *probs, int n, int iters, AlignPlan &pl)
{
    const AlignLaunch L = align_launch_of(ctx);
    int rc;
    if ((rc = ensure_buffer(ctx, &ctx->res_dev, &ctx->res_cap, (int64_t)(sizeof(AlignResult) * n), 1, "results")) ||
        (rc = plan_alignment(ctx, probs, n, L, iters, pl)))
        return rc;
    rc = ensure_buffer(ctx, &ctx->prob_dev, &ctx->prob_cap, (int64_t)pl.total, 1, "problems");
    if (rc && pl.tiled) {  // no memory for the tiles: by pages
        (void)hipGetLastError();
        if ((rc = plan_alignment(ctx, probs, n, L, iters, pl, false))) return rc;
        rc = ensure_buffer(ctx, &ctx->prob_dev, &ctx->prob_cap, (int64_t)pl.total, 1, "problems");
    }
    return rc ? rc : bind_alignment(ctx, pl, ctx->prob_dev);
}

int run_alignment(covox_ctx *ctx, AlignProblem *probs, int n, AlignResult *res)
{
    if (n <= 0) return COVOX_OK;
    int rc;
    AlignPlan pl;
    if ((rc = place_alignment(ctx, probs, n, probs[0].max_iter, pl))) return rc;
    if ((rc = launch_alignment(ctx, pl, (AlignResult *)ctx->res_dev, true, true))) return rc;
    if ((rc = hip_check(ctx, hipMemcpyAsync(res, ctx->res_dev, sizeof(AlignResult) * n, hipMemcpyDeviceToHost,
                                            ctx->stream),
                        "result copy")))
        return rc;
    return hip_check(ctx, hipStreamSynchronize(ctx->stream), "align sync");
}

}  // namespace covox
