// Exact truncated ESDF from the TSDF (paper Sec. I: distance to the nearest
// obstacle built from the TSDF, reusing the in-band distances; Sec. III-E:
// an exact Euclidean distance transform in the PBA lineage, organised per
// block).
//
// The squared distance k(i) = min over sites s of |i - s|^2 is separable:
//   g1(x,y,z) = min_x' (x - x')^2 over sites on the x line
//   g2(x,y,z) = min_y' g1(x,y',z) + (y - y')^2          (with g1: k_edt_xy)
//   k(x,y,z)  = min_z' g2(x,y,z') + (z - z')^2          (k_edt_z_col)
// Only k <= R^2 (R = round(d_max / vs)) matters, so every pass looks at most
// R voxels (HB = ceil(R / 8) blocks) to each side and stores larger values as
// "infinite"; in each pass the search from the centre stops once d^2 reaches
// the best value, which makes the min exact.  The passes run over the dense
// block box of the allocated blocks: intermediate values are needed in
// unallocated blocks between allocated ones.
//
// Layout: every dense block keeps its 512 voxels contiguous (l = x + 8y +
// 64z), like the TSDF pool, so one wave64 owns one block with lane = (x, y)
// and z in registers.  Site masks are 8 64-bit words per block (word z, bit
// x+8y).  g2 is kept for the pass that reads it: 32-bit words of two voxels
// adjacent in x, z fastest (word z + 8 (x / 2 + 4 y)).
#include "covox_impl.h"
#include "edt_columns.h"
#include "edt_envelope.h"

#include <string.h>

#include <algorithm>
#include <vector>

namespace covox {

namespace {

constexpr int kBig = 1 << 24;

template <typename S> __device__ __forceinline__ float ldv(const S *p);
template <> __device__ __forceinline__ float ldv<float>(const float *p) { return *p; }
template <> __device__ __forceinline__ float ldv<__half>(const __half *p) { return __half2float(*p); }

// Page (dense block -> buffer index, -1 if unallocated), site masks and the
// snapshot of each submap's domain (block box and block count) that the later
// passes work on.  Two independent loops: one lane per dense block looks its
// key up in the hash table (64 lookups in flight per wave), writes the page
// and, for an unallocated block, empty site masks; one wave per allocated
// block reads its D and W and writes its site masks.  With SEEDS, that wave
// also writes the phi seed of each voxel: NaN when unobserved, D inside the
// band, and otherwise an infinity with the sign of D.  The EDT passes then
// never read the TSDF or the submap's bookkeeping, so that the next frames
// may be integrated while they run.
template <typename S, int NJ, bool SEEDS>
__global__ __launch_bounds__(256) void k_page_sites(const JobList<NJ> jl, int C, float vs, float tau,
                                                    uint64_t *__restrict__ sites, int32_t *__restrict__ blk,
                                                    uint8_t *__restrict__ ddirty)
{
    __shared__ Plan lds;
    PlanView<NJ, false> pv;
    pv.init(jl, C, lds);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (blockIdx.x == 0 && (int)threadIdx.x < jl.n) {
        const JobInfo d = pv.info(threadIdx.x);
        SubmapMeta *m = jl.j[threadIdx.x].meta;
        EsdfSnap *sn = jl.j[threadIdx.x].snap;
        for (int a = 0; a < 3; ++a) {
            m->dom_min[a] = sn->lo[a] = d.lo[a];
            m->dom_dim[a] = sn->dim[a] = d.dim[a];
        }
        m->dom_nblocks = sn->nb = (int32_t)d.nb;
        m->dom_valid = 1;
    }
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < pv.t[0];
         g += (int64_t)gridDim.x * blockDim.x) {
        const int j = pv.template job<&JobInfo::od>(g);
        const JobInfo d = pv.info(j);
        const EsdfJob &job = jl.j[j];
        const int64_t db = g - d.od;
        int x, y, z;
        dom_coords(d, db, x, y, z);
        const int64_t idx =
            hash_find(job.tkeys, job.tvals, job.tmask, pack_key(d.lo[0] + x, d.lo[1] + y, d.lo[2] + z));
        job.page[db] = (int32_t)idx;
        if (blk) blk[g] = (int32_t)idx;  // the launch's own copy, read by the column passes
        if (ddirty && idx < 0) ddirty[g] = 0;
        if (idx < 0) {
            uint4 *w = (uint4 *)(sites + g * 8);
#pragma unroll
            for (int k = 0; k < 4; ++k) w[k] = make_uint4(0u, 0u, 0u, 0u);
        }
    }
    for (int64_t w = (int64_t)blockIdx.x * 4 + wid; w < pv.t[1]; w += (int64_t)gridDim.x * 4) {
        const int jj = pv.template job<&JobInfo::ob>(w);
        const JobInfo d = pv.info(jj);
        const EsdfJob &job = jl.j[jj];
        const int64_t idx = w - d.ob;
        int bx, by, bz;
        unpack_key(job.keys[idx], bx, by, bz);
        const int64_t g = d.od + dom_index(d, bx - d.lo[0], by - d.lo[1], bz - d.lo[2]);
        if constexpr (SEEDS) {
            // an exact update consumes the block's change flag
            if (lane == 0) {
                if (ddirty) ddirty[g] = job.full ? 1 : job.dirty[idx];
                job.dirty[idx] = 0;
            }
        }
        const S *Db = (const S *)job.D + idx * 512 + lane;
        const S *Wb = (const S *)job.W + idx * 512 + lane;
        // all reads before the first write (the seeds), so that they overlap
        float Dk[8], Wk[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            Dk[k] = ldv(Db + 64 * k);
            Wk[k] = ldv(Wb + 64 * k);
        }
        uint64_t wm = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float Dv = Dk[k], Wv = Wk[k];
            const uint64_t m = __ballot(Wv > 0.0f && fabsf(Dv) <= vs);
            if (lane == k) wm = m;
            if constexpr (SEEDS)
                job.seeds[g * 512 + lane + 64 * k] =
                    !(Wv > 0.0f) ? __builtin_nanf("")
                                 : (fabsf(Dv) < tau ? Dv : (Dv > 0.0f ? __builtin_inff() : -__builtin_inff()));
        }
        if (lane < 8) sites[g * 8 + lane] = wm;
    }
}

// The x distances of the 8 voxels of one x-line of a block, as 8 bytes:
// byte x is the distance from bit 8 HB + x of the 128-bit site window
// (lo, hi) to its nearest set bit, or 255 when that exceeds R or the window
// has none.  The window holds the 2 HB + 1 blocks' bytes of the line (the
// own block's byte at bit 8 HB, in lo since HB <= 7; zero above).  The
// nearest sites below and above the own byte are found once per line, and
// each voxel then looks only inside its own byte.
__device__ __forceinline__ uint64_t line_dists(uint64_t lo, uint64_t hi, int HB, int R)
{
    constexpr int kNone = 1000;
    const int p0 = 8 * HB;
    const uint32_t b = (uint32_t)(lo >> p0) & 0xFFu;
    const uint64_t below = lo & ((1ull << p0) - 1ull);  // p0 <= 56
    const int dl0 = below ? p0 - (63 - __clzll((long long)below)) : kNone;  // from bit p0 down
    const uint64_t above = p0 + 8 < 64 ? lo >> (p0 + 8) : 0ull;
    const int dr7 = above ? __ffsll((long long)above)                        // from bit p0 + 7 up
                          : (hi ? 64 - (p0 + 7) + (__ffsll((long long)hi) - 1) : kNone);
    uint64_t out = 0;
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        const uint32_t ml = b & ((2u << x) - 1u);  // own sites at or below x
        const uint32_t mr = b >> x;                // own sites at or above x
        const int dl = ml ? x - (31 - __clz((int)ml)) : x + dl0;
        const int dr = mr ? __ffs((int)mr) - 1 : (7 - x) + dr7;
        const int d = min(dl, dr);
        out |= (uint64_t)(d <= R ? d : 255) << (8 * x);
    }
    return out;
}

// x pass of the per-line envelopes: one wave per dense block, lane = (y, z) line of
// the block.  The
// lane gathers byte y of site word z from the 2 HB + 1 blocks along x into a
// 128-bit mask and stores the 8 distances of its line (x = 0..7, contiguous
// in the block layout) as one 8-byte word; no LDS and no barriers, so
// consecutive blocks of a wave overlap their loads.
template <int NJ>
__global__ __launch_bounds__(256) void k_edt_x(const JobList<NJ> jl, const uint64_t *__restrict__ sites,
                                               uint8_t *__restrict__ g1, int R, int HB)
{
    __shared__ Plan lds;
    PlanView<NJ> pv;
    pv.init(jl, 8 * HB, lds);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int y = lane & 7, z = lane >> 3;
    for (int64_t g = (int64_t)blockIdx.x * 4 + wid; g < pv.t[0]; g += (int64_t)gridDim.x * 4) {
        const JobInfo d = pv.info(pv.template job<&JobInfo::od>(g));
        int bx, by, bz;
        dom_coords(d, g - d.od, bx, by, bz);
        // the site words of the 2 HB + 1 blocks along x, read together
        // (slots past the halo or outside the domain read this block's word
        // and drop it)
        uint64_t wv[2 * kMaxHalo + 1];
#pragma unroll
        for (int i = 0; i < 2 * kMaxHalo + 1; ++i) {
            const int nx = bx + i - HB;
            const bool ok = i < 2 * HB + 1 && nx >= 0 && nx < d.dim[0];
            const uint64_t v = sites[(ok ? g + (i - HB) : g) * 8 + z];
            wv[i] = ok ? v : 0ull;
        }
        uint64_t lo = 0, hi = 0;
#pragma unroll
        for (int i = 0; i < 2 * kMaxHalo + 1; ++i) {
            const uint64_t byte = (wv[i] >> (8 * y)) & 0xFFull;
            const int pos = 8 * i;
            if (pos < 64) lo |= byte << pos;
            else hi |= byte << (pos - 64);
        }
        *(uint64_t *)(g1 + g * 512 + 8 * lane) = line_dists(lo, hi, HB, R);
    }
}

// ------------------------------------------------------------------------
// The region of a partial update (jobs with full = 0): the blocks of the
// launch's page copy (blk) whose phi can change are those within HB blocks,
// along every axis, of a block whose TSDF changed since the last exact
// update -- a site HB + 1 blocks away along some axis is more than 8 HB >= R
// voxels away.  Two dilations of the change flags: k_esdf_dil_x along x into
// dx, then k_esdf_region clears blk for allocated blocks with no flagged dx
// within HB along y and z, which the column passes then neither write nor
// read.  Jobs with full = 1 have every allocated block flagged.
template <int NJ>
__global__ __launch_bounds__(256) void k_esdf_dil_x(const JobList<NJ> jl, int HB, const uint8_t *__restrict__ ddirty,
                                                    uint8_t *__restrict__ dx)
{
    __shared__ Plan lds;
    PlanView<NJ> pv;
    pv.init(jl, 8 * HB, lds);
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < pv.t[0];
         g += (int64_t)gridDim.x * blockDim.x) {
        const JobInfo d = pv.info(pv.template job<&JobInfo::od>(g));
        int x, y, z;
        dom_coords(d, g - d.od, x, y, z);
        uint8_t any = 0;
        for (int k = max(0, x - HB); k <= min(d.dim[0] - 1, x + HB); ++k) any |= ddirty[g + (k - x)];
        dx[g] = any;
    }
}

template <int NJ>
__global__ __launch_bounds__(256) void k_esdf_region(const JobList<NJ> jl, int HB, const uint8_t *__restrict__ dx,
                                                     int32_t *__restrict__ blk)
{
    __shared__ Plan lds;
    PlanView<NJ> pv;
    pv.init(jl, 8 * HB, lds);
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < pv.t[0];
         g += (int64_t)gridDim.x * blockDim.x) {
        if (blk[g] < 0) continue;
        const JobInfo d = pv.info(pv.template job<&JobInfo::od>(g));
        int x, y, z;
        dom_coords(d, g - d.od, x, y, z);
        bool any = false;
        for (int zz = max(0, z - HB); zz <= min(d.dim[2] - 1, z + HB) && !any; ++zz)
            for (int yy = max(0, y - HB); yy <= min(d.dim[1] - 1, y + HB) && !any; ++yy)
                any = dx[d.od + dom_index(d, x, yy, zz)] != 0;
        if (!any) blk[g] = -1;
    }
}

// ------------------------------------------------------------------------
// Column passes (edt_columns.h).
template <int NJ>
__global__ __launch_bounds__(256) void k_edt_xy(const JobList<NJ> jl, int Sseg, const uint64_t *__restrict__ sites,
                                                const int32_t *__restrict__ blk, uint16_t *__restrict__ g2, int R,
                                                int HB)
{
    __shared__ EdtXyLds<NJ> lds;
    extern __shared__ __align__(16) uint32_t colw[];
    edt_xy<NJ>(jl, Sseg, sites, blk, g2, R, HB, lds, colw, blockIdx.x, gridDim.x);
}

template <int NJ>
__global__ __launch_bounds__(256) void k_edt_z_col(const JobList<NJ> jl, int Sseg, const uint16_t *__restrict__ g2,
                                                   const int32_t *__restrict__ blk, int R, int HB, float vs,
                                                   float dmax)
{
    __shared__ EdtZLds<NJ> lds;
    extern __shared__ __align__(16) uint32_t colw[];
    edt_z<NJ>(jl, Sseg, g2, blk, R, HB, vs, dmax, lds, colw, blockIdx.x, gridDim.x);
}

// ------------------------------------------------------------------------
// Per-line passes: lower envelope of parabolas (Felzenszwalb and
// Huttenlocher, edt_envelope.h).  One wave per block column; lane = one
// line.  A line longer than kWin voxels is cut into output segments that each
// carry C = 8 HB >= R voxels of context on both sides, which is exact because
// only k <= R^2 is kept.  Work per voxel is a few LDS steps whatever the
// distances, which suits large domains with many lines.

__device__ __forceinline__ void segment(int L, int C, int seg, int S, int &y0, int &y1, int &w0, int &w1)
{
    y0 = seg * S;
    y1 = min(y0 + S, L);
    w0 = max(0, y0 - C);
    w1 = min(L, y1 + C);
}

// Lane = x + 8 z within the block column (bx, *, bz).
template <int NJ>
__global__ __launch_bounds__(64) void k_edt_y_env(const JobList<NJ> jl, const uint8_t *__restrict__ g1,
                                                  uint16_t *__restrict__ g2, int R, int HB)
{
    __shared__ Plan lds;
    __shared__ __align__(16) uint8_t col[kWin * 64];   // [position][lane]
    __shared__ __align__(16) uint8_t stk[kWin * 64];   // [entry][lane]
    __shared__ __align__(16) uint16_t ost[8 * 64];     // one block of outputs [y][lane]
    const int C = 8 * HB;
    PlanView<NJ> pv;
    pv.init(jl, C, lds);
    const int lane = threadIdx.x;
    const int Sg = kWin - 2 * C;
    const int R2 = R * R;
    auto getf = [&](int q) {
        const int a = col[q * 64 + lane];
        return a * a;
    };
    for (int64_t c = blockIdx.x; c < pv.t[2]; c += gridDim.x) {
        const JobInfo d = pv.info(pv.template job<&JobInfo::oy>(c));
        const int L = 8 * d.dim[1];
        const int nseg = (int)nsegments(L, Sg);
        const int64_t cl = c - d.oy;
        const int seg = (int)(cl % nseg);
        const int64_t cc = cl / nseg;
        const int bx = (int)(cc % d.dim[0]), bz = (int)(cc / d.dim[0]);
        int y0, y1, w0, w1;
        segment(L, C, seg, Sg, y0, y1, w0, w1);
        for (int j = w0 / 8; j < w1 / 8; ++j) {
            const int64_t g = d.od + dom_index(d, bx, j, bz);
            const uint64_t v = ((const uint64_t *)(g1 + g * 512))[lane];
            *(uint64_t *)&col[(8 * (j - w0 / 8) + (lane & 7)) * 64 + 8 * (lane >> 3)] = v;
        }
        wave_sync();
        Envelope e;
        env_clear(e);
        const int W = w1 - w0;
        for (int q = 0; q < W; ++q) {
            const int a = col[q * 64 + lane];
            if (a == 255) continue;
            env_push(e, stk, 64, lane, q, a * a, getf);
        }
        Walker wk;
        if (e.k >= 0) walk_init(wk, e, stk, 64, lane, getf);
        for (int yb = y0; yb < y1; yb += 8) {
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                int v = kInf16;
                if (e.k >= 0) {
                    const int val = walk_at(wk, e, stk, 64, lane, yb + t - w0, getf);
                    if (val <= R2) v = val;
                }
                ost[t * 64 + lane] = (uint16_t)v;
            }
            wave_sync();
            const int64_t g = d.od + dom_index(d, bx, yb / 8, bz);
            // words 4 lane .. 4 lane + 3 of the block: column (x pair, y), z from 4 (lane & 1)
            const int xp = (lane >> 1) & 3, ty = lane >> 3, z0 = 4 * (lane & 1);
            uint4 o;
            uint32_t *ow = (uint32_t *)&o;
#pragma unroll
            for (int k = 0; k < 4; ++k) ow[k] = *(const uint32_t *)&ost[ty * 64 + 2 * xp + 8 * (z0 + k)];
            *(uint4 *)(g2 + g * 512 + 8 * lane) = o;
            wave_sync();
        }
    }
}

// Lane = x + 8 y, the in-block layout, within the column (bx, by, *).
template <int NJ>
__global__ __launch_bounds__(64) void k_edt_z_env(const JobList<NJ> jl, const uint16_t *__restrict__ g2, int R,
                                                  int HB, float vs, float dmax)
{
    __shared__ Plan lds;
    __shared__ __align__(16) uint16_t col[kWin * 64];  // [position][lane]
    __shared__ __align__(16) uint8_t stk[kWin * 64];
    const int C = 8 * HB;
    PlanView<NJ> pv;
    pv.init(jl, C, lds);
    const int lane = threadIdx.x;
    const int Sg = kWin - 2 * C;
    const int R2 = R * R;
    auto getf = [&](int q) { return (int)col[q * 64 + lane]; };
    for (int64_t c = blockIdx.x; c < pv.t[3]; c += gridDim.x) {
        const int jj = pv.template job<&JobInfo::oz>(c);
        const JobInfo d = pv.info(jj);
        const EsdfJob &job = jl.j[jj];
        const int L = 8 * d.dim[2];
        const int nseg = (int)nsegments(L, Sg);
        const int64_t cl = c - d.oz;
        const int seg = (int)(cl % nseg);
        const int64_t cc = cl / nseg;
        const int bx = (int)(cc % d.dim[0]), by = (int)(cc / d.dim[0]);
        int z0, z1, w0, w1;
        segment(L, C, seg, Sg, z0, z1, w0, w1);
        // nothing to write when no block of the output range is allocated
        bool any = false;
        for (int j0 = z0 / 8; j0 < z1 / 8; j0 += 64) {
            const int j = j0 + lane;
            const bool a = j < z1 / 8 && job.page[dom_index(d, bx, by, j)] >= 0;
            any = any || __ballot(a) != 0;
        }
        if (!any) continue;
        for (int j = w0 / 8; j < w1 / 8; ++j) {
            // the lane's column: words z + 8 (x / 2 + 4 y), half x & 1
            const uint16_t *src = g2 + (d.od + dom_index(d, bx, by, j)) * 512 + 16 * ((lane & 7) / 2 + 4 * (lane >> 3)) + (lane & 1);
#pragma unroll
            for (int t = 0; t < 8; ++t) col[(8 * (j - w0 / 8) + t) * 64 + lane] = src[2 * t];
        }
        wave_sync();
        Envelope e;
        env_clear(e);
        const int Wn = w1 - w0;
        for (int q = 0; q < Wn; ++q) {
            const int a = col[q * 64 + lane];
            if (a > R2) continue;  // infinite
            env_push(e, stk, 64, lane, q, a, getf);
        }
        Walker wk;
        if (e.k >= 0) walk_init(wk, e, stk, 64, lane, getf);
        for (int zb = z0; zb < z1; zb += 8) {
            const int64_t idx = job.page[dom_index(d, bx, by, zb / 8)];
            if (idx < 0) continue;
            const float *Sb = job.seeds + (d.od + dom_index(d, bx, by, zb / 8)) * 512 + lane;
            float *Pb = job.phi + idx * 512 + lane;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const float seed = Sb[64 * t];  // from k_page_sites
                float out = seed;  // unobserved or in the band
                if (__builtin_isinf(seed)) {
                    const int best = e.k >= 0 ? walk_at(wk, e, stk, 64, lane, zb + t - w0, getf) : kBig;
                    out = phi_value(seed, best, R2, vs, dmax);
                }
                Pb[64 * t] = out;
            }
        }
        wave_sync();
    }
}

// Every ESDF kernel loops over its work items with a grid stride, so the
// grid only needs to fill the chip: the host's bounds on the dense domain
// and the block count are loose, and surplus workgroups would each pay
// their dispatch and set-up for nothing.  2048 workgroups of up to 512
// lanes keep 256 CUs busy.
unsigned clamp_grid(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>(n, 2048)); }
// The passes loop over their work with a grid stride, so a smaller grid is
// valid; while they run beside an integration (on their own stream or in its launches), the
// tuning's cap leaves CUs to it.
int64_t grid_limit(const covox_ctx *ctx)
{
    const int64_t cap = ctx->tune.edt_pipe_max_workgroups;
    return (ctx->esdf_edt_stream || ctx->edt_pass) && cap > 0 ? cap : INT64_MAX;
}
unsigned cap_grid(const covox_ctx *ctx, unsigned g) { return (unsigned)std::min<int64_t>(g, grid_limit(ctx)); }
// Single-wave workgroups (per-line envelopes): up to 64 waves per CU.
unsigned clamp_grid_w(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>(n, 16384)); }

int64_t bound_blocks(const covox_submap *s)
{
    if (!s->bound_valid) return 0;
    int64_t n = 1;
    for (int a = 0; a < 3; ++a) n *= (int64_t)(s->bound_hi[a] - s->bound_lo[a] + 1);
    return n;
}

// Columns (times segments) of a line pass over the host-side bound box:
// axes a and b span the columns, the third axis is the line.
int64_t bound_cols(const covox_submap *s, int a, int b, int HB)
{
    if (!s->bound_valid) return 0;
    const int c = 3 - a - b;
    const int64_t L = 8 * (int64_t)(s->bound_hi[c] - s->bound_lo[c] + 1);
    const int64_t S = kWin - 16 * HB;
    return (int64_t)(s->bound_hi[a] - s->bound_lo[a] + 1) * (s->bound_hi[b] - s->bound_lo[b] + 1) * ((L + S - 1) / S);
}

template <int NJ>
JobList<NJ> make_jobs(covox_submap *const *subs, int n, EsdfSnap *snap, float *seeds, bool partial)
{
    JobList<NJ> jl;
    memset(&jl, 0, sizeof(jl));
    jl.n = n;
    for (int i = 0; i < n; ++i) {
        covox_submap *s = subs[i];
        jl.j[i] = EsdfJob{s->meta, snap + i, s->keys, s->tkeys, s->tvals, (uint64_t)s->tcap - 1, s->D, s->W,
                          s->phi, s->page, seeds, s->dirty, (partial && s->esdf_exact) ? 0 : 1};
    }
    return jl;
}

// Page + site masks (and, with edt, the three EDT passes) for up to NJ
// submaps in one launch per kernel.
// Line segments of the y and z passes over the host bounds of the submaps.
void chunk_cols(covox_submap *const *subs, int n, int HB, int64_t &cy, int64_t &cz)
{
    cy = cz = 0;
    for (int i = 0; i < n; ++i) {
        cy += bound_cols(subs[i], 0, 2, HB);
        cz += bound_cols(subs[i], 0, 1, HB);
    }
}

// Column segments along axis `c` (columns spanned by the other two axes) of
// the column passes over the host-side bound box.
int64_t bound_segs(const covox_submap *s, int c, int S)
{
    if (!s->bound_valid) return 0;
    int64_t cols = 1;
    for (int a = 0; a < 3; ++a)
        if (a != c) cols *= (int64_t)(s->bound_hi[a] - s->bound_lo[a] + 1);
    const int64_t L = s->bound_hi[c] - s->bound_lo[c] + 1;
    return cols * ((L + S - 1) / S);
}

// Segment length of the column passes for halo HB along axis c: the tuning's, or (0) the
// longest that still gives the chip about kFillSegs workgroups (or as many as the
// tuning lets run), as a longer segment stages its halo for more blocks.  The dense box is taken as four times
// the blocks last counted (the host's own bound, the frames' frusta, is far
// looser); any length gives the same result.  (24 room frames with an update every
// second one, passes limited to 64 workgroups: 1446 us with segments for 768, 957 with
// segments for 64; the voxel-parallel passes took 1346.)  Small maps do not go below
// four blocks where the halo is wide (256 and 413 blocks, R = 40: 21.3 and 22.4 us at
// two, 20.4 and 21.7 at four, 20.8 and 23.4 by the voxel-parallel passes; R = 8: 16.6
// and 17.2, 16.9 and 17.3, 16.1 and 20.3).
constexpr int64_t kFillSegs = 768;
int col_segment(const covox_ctx *ctx, covox_submap *const *subs, int n, int HB, int c, int64_t want)
{
    // no longer than the box along c: a workgroup's LDS follows the segment
    int64_t most = 1;
    for (int i = 0; i < n; ++i)
        if (subs[i]->bound_valid) most = std::max<int64_t>(most, subs[i]->bound_hi[c] - subs[i]->bound_lo[c] + 1);
    most = std::min<int64_t>(most, kColMaxStage - 2 * HB);
    if (want > 0) return (int)std::min<int64_t>(want, most);
    int64_t dense = 0;
    for (int i = 0; i < n; ++i) dense += 4 * (int64_t)(*subs[i]->pin_nb & ((1ull << 40) - 1));
    const int64_t fill = std::min(kFillSegs, grid_limit(ctx));
    const int least = HB >= 3 ? 4 : 2;
    int S = 32;
    while (S > least && dense < fill * S) S /= 2;
    return (int)std::min<int64_t>(S, most);
}

// force < 0: pass shapes by the tuning (or COVOX_EDT_MODE); else the library's
// segments with bit 0 = y envelopes, bit 1 = z envelopes.
template <int NJ>
int esdf_chunk(covox_ctx *ctx, covox_submap *const *subs, int n, bool edt, int force = -1)
{
    const covox_params &p = ctx->p;
    const int R = (int)std::llround(p.d_max / p.voxel_size);
    const int HB = (R + 7) / 8;
    const int C = 8 * HB;
    int rc;
    // The page kernel runs on the context stream; the passes after it run
    // on ctx->esdf_edt_stream when a pipelined caller sets one (after
    // ev_paged, so that the caller may integrate meanwhile), else on the
    // context stream too.
    hipStream_t edt_stream = ctx->esdf_edt_stream ? ctx->esdf_edt_stream : ctx->stream;
    const int slot = ctx->esdf_slot;
    int64_t nd = 0, nb = 0, cy = 0, cz = 0;
    for (int i = 0; i < n; ++i) {
        covox_submap *s = subs[i];
        nd += std::max<int64_t>(bound_blocks(s), 1);
        nb += std::min(s->nb_upper, s->cap);
    }
    chunk_cols(subs, n, HB, cy, cz);
    // Pass shapes: the column passes, or per-line envelopes from the tuning's
    // numbers of lines up (or as forced by COVOX_EDT_MODE = window | envelope).
    // No default number: 16 outdoor submaps (25 k blocks, 6 k lines of y) take 387
    // us in the y envelopes, whose LDS leaves one wave per SIMD, and 89 in the
    // column pass with its x distances.
    const int64_t seg = force >= 0 ? 0 : ctx->tune.edt_col_seg;
    bool env_y = cy >= ctx->tune.edt_y_env_min_cols, env_z = cz >= ctx->tune.edt_z_env_min_cols;
    if (ctx->edt_mode == 2) env_y = env_z = true;
    if (force >= 0) {
        env_y = (force & 1) != 0;
        env_z = (force & 2) != 0;
    } else if (seg > 0 || ctx->edt_mode == 1) {
        env_y = env_z = false;
    }
    const int seg_y = col_segment(ctx, subs, n, HB, 1, seg), seg_z = col_segment(ctx, subs, n, HB, 2, seg);
    // a partial update (segments set by the tuning, never under capture): the
    // submaps whose phi is exact and whose changes since are all flagged
    bool partial = edt && seg > 0 && !ctx->capturing && !ctx->tune.esdf_full_recompute;
    if (partial) {
        bool any = false;
        for (int i = 0; i < n; ++i) any = any || subs[i]->esdf_exact;
        partial = any;
    }
    // a buffer that grows is freed: the passes of an earlier update on the
    // other stream may still read it
    bool grows = ctx->sites_cap[slot] < nd ||
                 (edt && (ctx->seeds_cap[slot] < nd || (env_y && ctx->g1_cap < nd) || ctx->g2_cap < nd ||
                          ctx->blk_cap[slot] < nd)) || (partial && ctx->ddirty_cap[slot] < 2 * nd);
    for (int i = 0; i < n; ++i) grows = grows || subs[i]->page_cap < std::max<int64_t>(bound_blocks(subs[i]), 1);
    if (grows && edt_stream != ctx->stream && !ctx->capturing &&
        (rc = hip_check(ctx, hipStreamSynchronize(edt_stream), "esdf stream sync")))
        return rc;
    for (int i = 0; i < n; ++i) {
        covox_submap *s = subs[i];
        const int64_t b = std::max<int64_t>(bound_blocks(s), 1);
        if ((rc = ensure_buffer(ctx, (void **)&s->page, &s->page_cap, b, sizeof(int32_t), "page"))) return rc;
    }
    if ((rc = ensure_buffer(ctx, (void **)&ctx->sites[slot], &ctx->sites_cap[slot], nd, 8 * sizeof(uint64_t),
                            "site masks")))
        return rc;
    if (!ctx->snap[slot] && (rc = hip_check(ctx, hipMalloc((void **)&ctx->snap[slot], sizeof(EsdfSnap) * kMaxJobs),
                                            "esdf snapshot")))
        return rc;
    if (edt) {
        if ((rc = ensure_buffer(ctx, (void **)&ctx->seeds[slot], &ctx->seeds_cap[slot], nd, 512 * sizeof(float),
                                "phi seeds")))
            return rc;
        if (env_y && (rc = ensure_buffer(ctx, (void **)&ctx->g1, &ctx->g1_cap, nd, 512, "edt g1"))) return rc;
        if ((rc = ensure_buffer(ctx, (void **)&ctx->g2, &ctx->g2_cap, nd, 1024, "edt g2"))) return rc;
    }
    if (edt && (rc = ensure_buffer(ctx, (void **)&ctx->blk[slot], &ctx->blk_cap[slot], nd, sizeof(int32_t),
                                    "esdf block index")))
        return rc;
    int32_t *const blk = edt ? ctx->blk[slot] : nullptr;
    if (partial && (rc = ensure_buffer(ctx, (void **)&ctx->ddirty[slot], &ctx->ddirty_cap[slot], 2 * nd, 1,
                                       "esdf change flags")))
        return rc;
    uint8_t *const ddirty = partial ? ctx->ddirty[slot] : nullptr;
    uint64_t *const sites = ctx->sites[slot];
    const JobList<NJ> jl = make_jobs<NJ>(subs, n, ctx->snap[slot], ctx->seeds[slot], partial);
    const float vs = (float)p.voxel_size, tau = (float)band_limit(p), dmax = (float)p.d_max;
    const bool h = p.precision == COVOX_FP16;
    {
        TimedLaunch tl(ctx, COVOX_K_ESDF_PAGE);
        const dim3 grid(clamp_grid(std::max((nd + 255) / 256, (nb + 3) / 4)));
        if (h && edt)
            hipLaunchKernelGGL((k_page_sites<__half, NJ, true>), grid, dim3(256), 0, ctx->stream, jl, C, vs, tau,
                               sites, blk, ddirty);
        else if (h)
            hipLaunchKernelGGL((k_page_sites<__half, NJ, false>), grid, dim3(256), 0, ctx->stream, jl, C, vs, tau,
                               sites, blk, ddirty);
        else if (edt)
            hipLaunchKernelGGL((k_page_sites<float, NJ, true>), grid, dim3(256), 0, ctx->stream, jl, C, vs, tau,
                               sites, blk, ddirty);
        else
            hipLaunchKernelGGL((k_page_sites<float, NJ, false>), grid, dim3(256), 0, ctx->stream, jl, C, vs, tau,
                               sites, blk, ddirty);
    }
    if ((rc = hip_check(ctx, hipGetLastError(), "page launch"))) return rc;
    for (int i = 0; i < n; ++i) subs[i]->page_version = subs[i]->version;
    if (!edt) return COVOX_OK;
    ctx->esdf_used_page = env_z;  // the z envelopes read the page
    // the passes read nothing the next integration writes: on their own
    // stream they wait for the page kernel only
    hipStream_t base = ctx->stream;
    if (edt_stream != base) {
        if ((rc = hip_check(ctx, hipEventRecord(ctx->ev_paged, base), "paged")) ||
            (rc = hip_check(ctx, hipStreamWaitEvent(edt_stream, ctx->ev_paged, 0), "paged wait")))
            return rc;
        ctx->stream = edt_stream;  // for the launches and their timing events below
    }
    if (partial) {
        const unsigned gd = cap_grid(ctx, clamp_grid((nd + 255) / 256));
        hipLaunchKernelGGL((k_esdf_dil_x<NJ>), dim3(gd), dim3(256), 0, ctx->stream, jl, HB, ddirty, ddirty + nd);
        hipLaunchKernelGGL((k_esdf_region<NJ>), dim3(gd), dim3(256), 0, ctx->stream, jl, HB, ddirty + nd, blk);
    }
    int64_t sy = 0, sz = 0;
    for (int i = 0; i < n; ++i) {
        sy += std::max<int64_t>(bound_segs(subs[i], 1, seg_y), 1);
        sz += std::max<int64_t>(bound_segs(subs[i], 2, seg_z), 1);
    }
    if constexpr (NJ == 1) {
        if (ctx->edt_pass && !env_y && !env_z) {  // taken along by the next integration, or flushed
            EdtPass &q = *ctx->edt_pass;
            q = EdtPass{jl, sites, blk, ctx->g2, seg_y, seg_z, R, HB, vs, dmax, cap_grid(ctx, clamp_grid(sy)),
                        cap_grid(ctx, clamp_grid(sz)), (unsigned)col_bytes(seg_y + 2 * HB),
                        (unsigned)col_bytes(seg_z + 2 * HB)};
            if ((rc = hip_check(ctx, hipGetLastError(), "esdf launch"))) {
                q.grid_y = q.grid_z = 0;
                return rc;
            }
            subs[0]->esdf_version = subs[0]->version;
            if (!ctx->capturing) subs[0]->esdf_exact = true;
            return COVOX_OK;
        }
    }
    if (env_y) {
        TimedLaunch tl(ctx, COVOX_K_EDT_X);
        hipLaunchKernelGGL((k_edt_x<NJ>), dim3(cap_grid(ctx, clamp_grid((nd + 3) / 4))), dim3(256), 0, ctx->stream, jl,
                           sites, ctx->g1, R, HB);
    }
    {
        TimedLaunch tl(ctx, COVOX_K_EDT_Y);
        if (env_y)
            hipLaunchKernelGGL((k_edt_y_env<NJ>), dim3(clamp_grid_w(cy)), dim3(64), 0, ctx->stream, jl, ctx->g1, ctx->g2,
                               R, HB);
        else
            hipLaunchKernelGGL((k_edt_xy<NJ>), dim3(cap_grid(ctx, clamp_grid(sy))), dim3(256), col_bytes(seg_y + 2 * HB),
                               ctx->stream, jl, seg_y, sites, blk, ctx->g2, R, HB);
    }
    {
        TimedLaunch tl(ctx, COVOX_K_EDT_Z);
        if (env_z)
            hipLaunchKernelGGL((k_edt_z_env<NJ>), dim3(clamp_grid_w(cz)), dim3(64), 0, ctx->stream, jl, ctx->g2, R, HB,
                               vs, dmax);
        else
            hipLaunchKernelGGL((k_edt_z_col<NJ>), dim3(cap_grid(ctx, clamp_grid(sz))), dim3(256), col_bytes(seg_z + 2 * HB),
                               ctx->stream, jl, seg_z, ctx->g2, blk, R, HB, vs, dmax);
    }
    ctx->stream = base;
    if ((rc = hip_check(ctx, hipGetLastError(), "esdf launch"))) return rc;
    for (int i = 0; i < n; ++i) {
        subs[i]->esdf_version = subs[i]->version;
        if (!ctx->capturing) subs[i]->esdf_exact = true;
    }
    return COVOX_OK;
}

}  // namespace

int build_page(covox_ctx *ctx, covox_submap *s)
{
    if (s->page_version == s->version) return COVOX_OK;
    return esdf_chunk<1>(ctx, &s, 1, false);
}

int build_page_and_sites(covox_ctx *ctx, covox_submap *s) { return esdf_chunk<1>(ctx, &s, 1, false); }

int update_esdf_batch(covox_ctx *ctx, covox_submap *const *subs, int n)
{
    std::vector<covox_submap *> todo;
    for (int i = 0; i < n; ++i)
        if (std::find(todo.begin(), todo.end(), subs[i]) == todo.end()) todo.push_back(subs[i]);
    if (todo.empty()) return COVOX_OK;
    if (ctx->p.esdf_mode == COVOX_ESDF_WAVEFRONT) {
        for (covox_submap *s : todo) {
            const int rc = update_esdf_wavefront(ctx, s);
            if (rc) return rc;
        }
        return COVOX_OK;
    }
    if (todo.size() == 1) return esdf_chunk<1>(ctx, todo.data(), 1, true);
    for (size_t i = 0; i < todo.size(); i += kMaxJobs) {
        const int m = (int)std::min<size_t>(kMaxJobs, todo.size() - i);
        const int rc = esdf_chunk<kMaxJobs>(ctx, todo.data() + i, m, true);
        if (rc) return rc;
    }
    return COVOX_OK;
}

int update_esdf(covox_ctx *ctx, covox_submap *s) { return update_esdf_batch(ctx, &s, 1); }

bool edt_can_ride(const covox_ctx *ctx)
{
    // (a timed launch is one kernel's)
    if (ctx->p.esdf_mode != COVOX_ESDF_EXACT || ctx->timing || ctx->edt_mode == 2) return false;
    return ctx->edt_mode == 1 || ctx->tune.edt_col_seg > 0 ||
           (ctx->tune.edt_y_env_min_cols == INT64_MAX && ctx->tune.edt_z_env_min_cols == INT64_MAX);
}

int flush_edt(covox_ctx *ctx)
{
    EdtPass *q = ctx->edt_pass;
    if (!q) return COVOX_OK;
    if (q->grid_y)
        hipLaunchKernelGGL(k_edt_xy<1>, dim3(q->grid_y), dim3(256), q->lds_y, ctx->stream, q->jl, q->seg_y, q->sites,
                           q->blk, q->g2, q->R, q->HB);
    if (q->grid_z)
        hipLaunchKernelGGL(k_edt_z_col<1>, dim3(q->grid_z), dim3(256), q->lds_z, ctx->stream, q->jl, q->seg_z, q->g2,
                           q->blk, q->R, q->HB, q->vs, q->dmax);
    q->grid_y = q->grid_z = 0;
    return hip_check(ctx, hipGetLastError(), "esdf launch");
}

int autotune_esdf(covox_ctx *ctx, covox_submap *const *subs, int n)
{
    std::vector<covox_submap *> todo;
    for (int i = 0; i < n && (int)todo.size() < kMaxJobs; ++i)
        if (std::find(todo.begin(), todo.end(), subs[i]) == todo.end()) todo.push_back(subs[i]);
    if (todo.empty()) return COVOX_OK;
    const int m = (int)todo.size();
    const int R = (int)std::llround(ctx->p.d_max / ctx->p.voxel_size);
    int64_t cy, cz;
    chunk_cols(todo.data(), m, (R + 7) / 8, cy, cz);
    auto run = [&](int force) {
        return m == 1 ? esdf_chunk<1>(ctx, todo.data(), 1, true, force)
                      : esdf_chunk<kMaxJobs>(ctx, todo.data(), m, true, force);
    };
    hipEvent_t e0, e1;
    int rc = hip_check(ctx, hipEventCreate(&e0), "autotune event");
    if (rc) return rc;
    if ((rc = hip_check(ctx, hipEventCreate(&e1), "autotune event"))) {
        (void)hipEventDestroy(e0);
        return rc;
    }
    const int32_t saved_timing = ctx->timing;
    ctx->timing = 0;  // no per-kernel events inside the measured region
    covox_tuning &t = ctx->tune;
    const int64_t saved_seg = t.edt_col_seg, saved_full = t.esdf_full_recompute;
    t.esdf_full_recompute = 1;  // every candidate times a whole update
    // candidates: columns or envelopes for each of y and z, then the column
    // passes at five segment lengths
    constexpr int kSegs[5] = {2, 4, 8, 16, 32};
    constexpr int kCand = 4 + 5;
    float best_ms[kCand];
    for (int cand = 0; cand < kCand && !rc; ++cand) {
        best_ms[cand] = 1e30f;
        const int force = cand < 4 ? cand : -1;
        if (cand >= 4) t.edt_col_seg = kSegs[cand - 4];
        rc = run(force);  // warm-up (buffers, caches)
        for (int rep = 0; rep < 3 && !rc; ++rep) {
            rc = hip_check(ctx, hipEventRecord(e0, ctx->stream), "autotune record");
            if (!rc) rc = run(force);
            if (!rc) rc = hip_check(ctx, hipEventRecord(e1, ctx->stream), "autotune record");
            if (!rc) rc = hip_check(ctx, hipEventSynchronize(e1), "autotune sync");
            float ms = 0;
            if (!rc) rc = hip_check(ctx, hipEventElapsedTime(&ms, e0, e1), "autotune elapsed");
            if (!rc) best_ms[cand] = std::min(best_ms[cand], ms);
        }
    }
    t.edt_col_seg = saved_seg;
    t.esdf_full_recompute = saved_full;
    ctx->timing = saved_timing;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc) return rc;
    int best = 0;
    for (int c = 1; c < kCand; ++c)
        if (best_ms[c] < best_ms[best]) best = c;
    if (best >= 4) {
        t.edt_col_seg = kSegs[best - 4];
        return COVOX_OK;
    }
    t.edt_col_seg = 0;
    if (best & 1) t.edt_y_env_min_cols = std::min(t.edt_y_env_min_cols, cy);
    else t.edt_y_env_min_cols = std::max(t.edt_y_env_min_cols, cy + 1);
    if (best & 2) t.edt_z_env_min_cols = std::min(t.edt_z_env_min_cols, cz);
    else t.edt_z_env_min_cols = std::max(t.edt_z_env_min_cols, cz + 1);
    return COVOX_OK;
}

}  // namespace covox
