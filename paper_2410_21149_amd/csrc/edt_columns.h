// The column passes of the exact ESDF and what a launch of them works on, for the
// kernels that run them alone (k_esdf.hip) or beside the next frames' integration
// in one launch (k_integrate.hip).
#pragma once

#include "covox_impl.h"

namespace covox {

constexpr int kWin = 256;     // envelope window positions (u8 stack entries)
constexpr int kMaxJobs = kEsdfMaxJobs;  // submaps per launch (the job list is a kernel argument)

// One submap of an ESDF launch.
struct EsdfJob {
    SubmapMeta *meta;
    EsdfSnap *snap;     // the update's domain (written by the page kernel)
    const uint64_t *keys;
    const uint64_t *tkeys;
    const uint32_t *tvals;
    uint64_t tmask;
    const void *D;
    const void *W;
    float *phi;
    int32_t *page;
    float *seeds;       // phi seed per voxel, by dense block index of the launch
    uint8_t *dirty;     // the submap's per-block change flags (cleared by the page kernel with SEEDS)
    int32_t full;       // every allocated block gets a new phi (else only those near a changed block)
};

template <int NJ>
struct JobList {
    EsdfJob j[NJ];
    int n;
};

// Per-workgroup view of a launch, derived from the submaps' device
// bookkeeping: each submap's domain (its allocated block box) and exclusive
// prefix sums of the work items of every pass over the submaps.  The dense
// prefix is also the offset of the submap's blocks in the shared scratch.
struct JobInfo {
    int32_t lo[3], dim[3];
    int64_t nd, nb;           // dense blocks of the box, allocated blocks
    int64_t od, ob, oy, oz;   // prefixes: dense, allocated, y columns, z columns
    int64_t oxy, ozc;         // prefixes: y and z column segments of the column passes
};

struct Plan {
    JobInfo info[kMaxJobs];
    int n;
    int64_t td, tb, ty, tz, txy, tzc;   // totals
};

// (L: a box's extent in voxels at most, so below 2^31)
__device__ __forceinline__ int64_t nsegments(int64_t L, int S)
{
    return L > 0 ? ((uint32_t)L + (uint32_t)S - 1u) / (uint32_t)S : 0;
}

// Work items of the column passes (segments of Sseg blocks along the pass
// axis; none when Sseg is 0).
struct ColCounts {
    int64_t cy, cz, cxy, czc;
};

// Fills the job info of one submap: from the live block count and block box
// (SNAP = false: the page kernel, which runs in order with the integration),
// or from the snapshot the page kernel stored (SNAP = true: the EDT passes,
// which may run while the next frames are integrated into the same submap).
template <bool SNAP>
__device__ __forceinline__ void job_info(const EsdfJob &job, int C, int Sseg, JobInfo &ji, ColCounts &cc)
{
    const SubmapMeta *m = job.meta;
    const EsdfSnap *sn = job.snap;
    for (int a = 0; a < 3; ++a) { ji.lo[a] = 0; ji.dim[a] = 0; }
    ji.nd = 0;
    ji.nb = 0;
    cc.cy = cc.cz = cc.cxy = cc.czc = 0;
    const int64_t nb = SNAP ? (int64_t)sn->nb : m->n_blocks;
    if (nb <= 0) return;
    ji.nb = nb;
    ji.nd = 1;
    for (int a = 0; a < 3; ++a) {
        ji.lo[a] = SNAP ? sn->lo[a] : m->bmin[a];
        ji.dim[a] = SNAP ? sn->dim[a] : m->bmax[a] - m->bmin[a] + 1;
        ji.nd *= ji.dim[a];
    }
    const int S = kWin - 2 * C;
    cc.cy = (int64_t)ji.dim[0] * ji.dim[2] * nsegments(8 * (int64_t)ji.dim[1], S);
    cc.cz = (int64_t)ji.dim[0] * ji.dim[1] * nsegments(8 * (int64_t)ji.dim[2], S);
    if (Sseg > 0) {
        cc.cxy = (int64_t)ji.dim[0] * ji.dim[2] * nsegments(ji.dim[1], Sseg);
        cc.czc = (int64_t)ji.dim[0] * ji.dim[1] * nsegments(ji.dim[2], Sseg);
    }
}

// The plan of a multi-submap launch: the first wave derives one submap per
// lane with wave prefix sums, then a workgroup barrier publishes it.  A
// single-submap launch keeps its one entry in registers instead (PlanView).
template <bool SNAP, int NJ>
__device__ void make_plan(const JobList<NJ> &jl, int C, int Sseg, Plan &pl)
{
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        JobInfo ji;
        ColCounts cc = {0, 0, 0, 0};
        for (int a = 0; a < 3; ++a) { ji.lo[a] = 0; ji.dim[a] = 0; }
        ji.nd = ji.nb = 0;
        if (lane < jl.n) job_info<SNAP>(jl.j[lane], C, Sseg, ji, cc);
        const int64_t v[6] = {ji.nd, ji.nb, cc.cy, cc.cz, cc.cxy, cc.czc};
        int64_t incl[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            int64_t x = v[k];
            for (int o = 1; o < 64; o <<= 1) {
                const int64_t y = __shfl_up(x, o, 64);
                if (lane >= o) x += y;
            }
            incl[k] = x;
        }
        if (lane < jl.n) {
            ji.od = incl[0] - v[0];
            ji.ob = incl[1] - v[1];
            ji.oy = incl[2] - v[2];
            ji.oz = incl[3] - v[3];
            ji.oxy = incl[4] - v[4];
            ji.ozc = incl[5] - v[5];
            pl.info[lane] = ji;
        }
        if (lane == 63) {
            pl.n = jl.n;
            pl.td = incl[0];
            pl.tb = incl[1];
            pl.ty = incl[2];
            pl.tz = incl[3];
            pl.txy = incl[4];
            pl.tzc = incl[5];
        }
    }
    __syncthreads();
}

// Submap owning global work item w of a pass (largest j with offset <= w).
template <int64_t JobInfo::*OFF>
__device__ __forceinline__ int find_job(const Plan &pl, int64_t w)
{
    int lo = 0, hi = pl.n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (pl.info[mid].*OFF <= w) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Uniform access to the plan: registers for one submap, LDS for several.
template <int NJ, bool SNAP = true>
struct PlanView {
    Plan *pl;
    JobInfo one;
    // totals: dense, allocated, y columns, z columns, y and z column segments
    int64_t t[6];

    template <typename L>
    __device__ void init(const JobList<NJ> &jl, int C, L &lds, int Sseg = 0)
    {
        if constexpr (NJ == 1) {
            ColCounts cc;
            job_info<SNAP>(jl.j[0], C, Sseg, one, cc);
            one.od = one.ob = one.oy = one.oz = one.oxy = one.ozc = 0;
            t[0] = one.nd;
            t[1] = one.nb;
            t[2] = cc.cy;
            t[3] = cc.cz;
            t[4] = cc.cxy;
            t[5] = cc.czc;
            pl = nullptr;
        } else {
            make_plan<SNAP>(jl, C, Sseg, lds);
            pl = &lds;
            t[0] = lds.td;
            t[1] = lds.tb;
            t[2] = lds.ty;
            t[3] = lds.tz;
            t[4] = lds.txy;
            t[5] = lds.tzc;
        }
    }
    template <int64_t JobInfo::*OFF>
    __device__ int job(int64_t w) const
    {
        if constexpr (NJ == 1) return 0;
        else return find_job<OFF>(*pl, w);
    }
    __device__ JobInfo info(int j) const
    {
        if constexpr (NJ == 1) return one;
        else return pl->info[j];
    }
};

// a / b with the remainder, a >= 0, b > 0: 32 bits where a has no more (a 64-bit
// division is some 130 instructions, a 32-bit one 20; these stand at the head of every
// workgroup's chain).
__device__ __forceinline__ int64_t divide(int64_t a, int b, int &rem)
{
    if ((uint64_t)a >> 32 == 0) {
        const uint32_t q = (uint32_t)a / (uint32_t)b;
        rem = (int)((uint32_t)a - q * (uint32_t)b);
        return q;
    }
    rem = (int)(a % b);
    return a / b;
}

__device__ __forceinline__ void dom_coords(const JobInfo &d, int64_t db, int &x, int &y, int &z)
{
    z = (int)divide(divide(db, d.dim[0], x), d.dim[1], y);
}

__device__ __forceinline__ int64_t dom_index(const JobInfo &d, int x, int y, int z)
{
    return ((int64_t)z * d.dim[1] + y) * d.dim[0] + x;
}

// phi of a voxel outside the band from its seed (an infinity with the sign
// of D) and the squared distance search result.
__device__ __forceinline__ float phi_value(float seed, int best, int R2, float vs, float dmax)
{
    const float sg = seed > 0.0f ? 1.0f : -1.0f;
    if (best > R2) return sg * dmax;
    return sg * fminf(dmax, vs * sqrtf((float)best));
}

// ------------------------------------------------------------------------
// Column passes.  Each workgroup owns a segment of Sseg blocks of one block
// column along the pass axis and stages the segment with HB halo blocks on
// each side once, so that no block is staged more than 1 + 2 HB / Sseg times.
//
// k_edt_xy fuses the x pass into the y pass: the squared x distances of the
// staged blocks of a y column (bx, *, bz) come from the site masks straight
// into LDS, and g2 is written only for the segment's blocks that the z pass
// reads (those with an allocated block within HB blocks along z).  k_edt_z_col
// stages g2 of a z column (bx, by, *) that holds an allocated block and writes
// phi of its allocated blocks.  Both read the launch's copy of the page (blk:
// buffer index per dense block, -1 when unallocated), never the submap's
// bookkeeping.
//
// Both searches are one routine, bound by vector instructions, so it works on
// pairs: a word holds two voxels adjacent in x as 16-bit squared distances, and
// a lane finds the minima of four consecutive positions of its column, that is
// of eight voxels; one wave covers a block.  Four offsets to each side cost two
// 16-byte LDS reads and 48 packed instructions (min of the two sides, plus e^2,
// min) for 64 candidates.  One voxel at a time, with byte reads, the same searches
// took about five instructions a pair of candidates and voxel: 16 outdoor submaps
// (25 k blocks) went from 56 + 387 us (x, y by envelopes) to 89 for k_edt_xy and
// from 98 to 67 for k_edt_z_col, a room frame (1.4 k blocks) from 6 + 14 to 14 and
// from 7 to 8 us with one launch less.
constexpr int kColMaxStage = 48;  // staged blocks of a segment: Sseg + 2 HB
// "No site within R": above every candidate that counts (at most 2 R^2 with R <=
// 56), and e^2 on top of it still fits 16 bits.
constexpr int kInf16 = 32400;
constexpr int kFarX = 180;  // the x distance that squares to it
static_assert(kFarX * kFarX == kInf16 && 2 * 56 * 56 < kInf16 && kInf16 + 64 * 64 <= 65535, "16-bit candidates");

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u16x2 as_pair(uint32_t v) { return __builtin_bit_cast(u16x2, v); }
__device__ __forceinline__ u16x2 pmin(u16x2 a, u16x2 b) { return __builtin_elementwise_min(a, b); }
__device__ __forceinline__ u16x2 pmax(u16x2 a, u16x2 b) { return __builtin_elementwise_max(a, b); }

// Words of a staged column: 8 rows a block and 4 words of padding (an odd number
// of 16-byte units, so that the columns of a wave spread over the banks).
__host__ __device__ constexpr int col_words(int nst) { return 8 * nst + 4; }
constexpr int kColumns = 32;  // x pairs by the eight positions along the third axis
inline size_t col_bytes(int nst) { return (size_t)kColumns * col_words(nst) * 4; }

// best[j] = min over |e| <= R of col[row + j + e] + e^2, j = 0..3, row a
// multiple of 4 with at least R rows staged to each side (rounded up to 8).
// Lanes with need = false do not keep the wave searching.
__device__ __forceinline__ void pair_search(const uint32_t *col, int row, int R, bool need, u16x2 best[4])
{
    const uint4 *c4 = (const uint4 *)col + (row >> 2);
    const uint4 cc = *c4;
    u16x2 dn[4] = {as_pair(cc.x), as_pair(cc.y), as_pair(cc.z), as_pair(cc.w)}, up[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) best[j] = up[j] = dn[j];
    for (int m = 0; 4 * m < R; m += 2) {
        // the next offset is e = 4 m + 1: past the best values nothing changes
        const u16x2 b = pmax(pmax(best[0], best[1]), pmax(best[2], best[3]));
        const int lim = (4 * m + 1) * (4 * m + 1);
        if (__ballot(need && max((int)b.x, (int)b.y) > lim) == 0) break;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int mm = m + h;  // rows row - 4 mm - 4 .. and row + 4 mm + 4 .., staged as 4 mm < 8 HB
            const uint4 lo = c4[-mm - 1], hi = c4[mm + 1];
            const u16x2 d[8] = {as_pair(lo.x), as_pair(lo.y), as_pair(lo.z), as_pair(lo.w), dn[0], dn[1], dn[2], dn[3]};
            const u16x2 u[8] = {up[0], up[1], up[2], up[3], as_pair(hi.x), as_pair(hi.y), as_pair(hi.z), as_pair(hi.w)};
#pragma unroll
            for (int q = 1; q <= 4; ++q) {
                const int e = 4 * mm + q;  // beyond R (the last step): above R^2, never kept
                const u16x2 ee = as_pair((uint32_t)(e * e) * 0x10001u);
#pragma unroll
                for (int j = 0; j < 4; ++j) best[j] = pmin(best[j], pmin(d[j - q + 4], u[j + q]) + ee);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                dn[j] = d[j];
                up[j] = u[4 + j];
            }
        }
    }
}

// The x distances inside one byte of a site mask (kFarX where it has no site),
// for the eight voxels of its line, as 16-bit values.
__device__ __forceinline__ void byte_dists(uint32_t b, uint32_t w[4])
{
    uint32_t d[8];
    uint32_t run = kFarX;
#pragma unroll
    for (int x = 0; x < 8; ++x) d[x] = run = (b >> x) & 1u ? 0u : min(run + 1u, (uint32_t)kFarX);
    run = kFarX;
#pragma unroll
    for (int x = 7; x >= 0; --x) {
        run = (b >> x) & 1u ? 0u : min(run + 1u, (uint32_t)kFarX);
        d[x] = min(d[x], run);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = d[2 * k] | (d[2 * k + 1] << 16);
}

// The plan of a launch in LDS: nothing for one submap, whose plan is in registers.
struct NoPlan {};
template <int NJ> struct LdsPlan { using type = Plan; };
template <> struct LdsPlan<1> { using type = NoPlan; };

template <int NJ>
struct EdtXyLds {
    uint4 lut[256];  // byte_dists
    uint64_t need;
    typename LdsPlan<NJ>::type plan;
};

// Workgroup wg of n_wg of the pass; colw: col_bytes() of LDS, columns x / 2 + 4 z,
// rows along y.
template <int NJ>
__device__ __forceinline__ void edt_xy(const JobList<NJ> &jl, int Sseg, const uint64_t *__restrict__ sites,
                                       const int32_t *__restrict__ blk, uint16_t *__restrict__ g2, int R, int HB,
                                       EdtXyLds<NJ> &lds, uint32_t *colw, int64_t wg, int64_t n_wg)
{
    PlanView<NJ> pv;
    pv.init(jl, 8 * HB, lds.plan, Sseg);
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    {
        uint32_t w[4];
        byte_dists(tid, w);
        lds.lut[tid] = make_uint4(w[0], w[1], w[2], w[3]);
    }
    const int R2 = R * R;
    for (int64_t c = wg; c < pv.t[4]; c += n_wg) {
        const JobInfo d = pv.info(pv.template job<&JobInfo::oxy>(c));
        const int nseg = (d.dim[1] + Sseg - 1) / Sseg;
        const int64_t cl = c - d.oxy;
        int seg, bx;
        const int64_t cc = divide(cl, nseg, seg);
        const int bz = (int)divide(cc, d.dim[0], bx);
        const int y0 = seg * Sseg, y1 = min(y0 + Sseg, d.dim[1]);
        const int nst = (y1 - y0) + 2 * HB;  // staged blocks y0 - HB .. y1 + HB - 1
        const int CW = col_words(nst);
        // output blocks that the z pass reads: an allocated block within HB along z
        if (tid < 64) {
            const int j = y0 + tid;
            int32_t most = -1;  // (every read issued together: a test of each would wait for it)
#pragma unroll
            for (int k = 0; k < 2 * kMaxHalo + 1; ++k) {
                const int zz = min(max(bz - HB + min(k, 2 * HB), 0), d.dim[2] - 1);
                most = max(most, blk[d.od + dom_index(d, bx, min(j, y1 - 1), zz)]);
            }
            const bool need = j < y1 && most >= 0;
            const uint64_t m = __ballot(need);
            if (tid == 0) lds.need = m;
        }
        __syncthreads();
        const uint64_t need = lds.need;
        if (need != 0) {
            // squared x distances of the staged blocks, one (y, z) row of 8
            // voxels per item: byte y of site word z of the 2 HB + 1 blocks
            // along x (outside the domain: no sites; staged blocks outside it:
            // none).  The nearest sites beside the own byte are found once a
            // row, those inside it come from the table.
#pragma unroll 2
            for (int e = tid; e < nst * 64; e += 256) {
                const int i = e >> 6, yr = e & 7, zr = (e >> 3) & 7;
                const int j = y0 - HB + i;
                uint32_t out[4] = {kInf16 * 0x10001u, kInf16 * 0x10001u, kInf16 * 0x10001u, kInf16 * 0x10001u};
                if (j >= 0 && j < d.dim[1]) {
                    const int64_t g = d.od + dom_index(d, bx, j, bz);
                    const uint32_t *sw = (const uint32_t *)sites + 2 * zr + (yr >> 2);
                    uint32_t wv[2 * kMaxHalo + 1];
#pragma unroll
                    for (int k = 0; k < 2 * kMaxHalo + 1; ++k) {
                        const int nx = bx + k - HB;
                        const bool ok = k < 2 * HB + 1 && nx >= 0 && nx < d.dim[0];
                        const uint32_t v = sw[(ok ? g + (k - HB) : g) * 16];
                        wv[k] = ok ? v : 0u;
                    }
                    uint32_t win[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                    for (int k = 0; k < 2 * kMaxHalo + 1; ++k) win[k >> 2] |= ((wv[k] >> (8 * (yr & 3))) & 0xFFu) << (8 * (k & 3));
                    const uint64_t lo = ((uint64_t)win[1] << 32) | win[0], hi = ((uint64_t)win[3] << 32) | win[2];
                    const int p0 = 8 * HB;  // the own byte's bit, at most 56
                    const uint64_t below = lo & ((1ull << p0) - 1ull);
                    const uint64_t above = p0 + 8 < 64 ? lo >> (p0 + 8) : 0ull;
                    // from voxel 0 down and from voxel 7 up
                    const int dl = below ? p0 - (63 - __clzll((long long)below)) : kFarX;
                    const int dr = above ? __ffsll((long long)above)
                                         : (hi ? min(64 - (p0 + 7) + __ffsll((long long)hi) - 1, kFarX) : kFarX);
                    const uint4 in = lds.lut[(uint32_t)(lo >> p0) & 0xFFu];
                    const uint32_t iw[4] = {in.x, in.y, in.z, in.w};
                    const u16x2 l2 = as_pair((uint32_t)dl * 0x10001u), r2 = as_pair((uint32_t)dr * 0x10001u);
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const u16x2 lx = l2 + as_pair((uint32_t)(2 * k) | ((uint32_t)(2 * k + 1) << 16));
                        const u16x2 rx = r2 + as_pair((uint32_t)(7 - 2 * k) | ((uint32_t)(6 - 2 * k) << 16));
                        const u16x2 v = pmin(as_pair(iw[k]), pmin(lx, rx));  // at most kFarX
                        out[k] = __builtin_bit_cast(uint32_t, v * v);
                    }
                }
                uint32_t *dst = colw + 4 * zr * CW + 8 * i + yr;
#pragma unroll
                for (int k = 0; k < 4; ++k) dst[k * CW] = out[k];
            }
            __syncthreads();
            // one wave a block: lane = (column, four rows)
            const uint32_t *col = colw + (lane >> 1) * CW;
            for (int io = wid; io < y1 - y0; io += 4) {
                if (!((need >> io) & 1ull)) continue;  // uniform
                u16x2 best[4];
                pair_search(col, 8 * (HB + io) + 4 * (lane & 1), R, true, best);
                // word z + 8 (x / 2 + 4 y)
                uint32_t *o = (uint32_t *)(g2 + (d.od + dom_index(d, bx, y0 + io, bz)) * 512) + (lane >> 3) +
                              8 * ((lane >> 1 & 3) + 16 * (lane & 1));
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const u16x2 v = {best[j].x <= R2 ? best[j].x : (unsigned short)kInf16,
                                     best[j].y <= R2 ? best[j].y : (unsigned short)kInf16};
                    o[32 * j] = __builtin_bit_cast(uint32_t, v);
                }
            }
        }
        __syncthreads();
    }
}

template <int NJ>
struct EdtZLds {
    int32_t blk[kColMaxStage + 2 * kMaxHalo];  // of z0 - 2 HB .. z1 + 2 HB - 1
    uint8_t need[kColMaxStage];                // staged block read by an allocated block
    typename LdsPlan<NJ>::type plan;
};

// As edt_xy; columns x / 2 + 4 y, rows along z.
template <int NJ>
__device__ __forceinline__ void edt_z(const JobList<NJ> &jl, int Sseg, const uint16_t *__restrict__ g2,
                                      const int32_t *__restrict__ blk, int R, int HB, float vs, float dmax,
                                      EdtZLds<NJ> &lds, uint32_t *colw, int64_t wg, int64_t n_wg)
{
    PlanView<NJ> pv;
    pv.init(jl, 8 * HB, lds.plan, Sseg);
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int R2 = R * R;
    for (int64_t c = wg; c < pv.t[5]; c += n_wg) {
        const int jj = pv.template job<&JobInfo::ozc>(c);
        const JobInfo d = pv.info(jj);
        const EsdfJob &job = jl.j[jj];
        const int nseg = (d.dim[2] + Sseg - 1) / Sseg;
        const int64_t cl = c - d.ozc;
        int seg, bx;
        const int64_t cc = divide(cl, nseg, seg);
        const int by = (int)divide(cc, d.dim[0], bx);
        const int z0 = seg * Sseg, z1 = min(z0 + Sseg, d.dim[2]);
        const int nst = (z1 - z0) + 2 * HB;  // staged blocks z0 - HB .. z1 + HB - 1
        const int CW = col_words(nst);
        for (int t = tid; t < nst + 2 * HB; t += 256) {
            const int zz = z0 - 2 * HB + t;
            lds.blk[t] = zz >= 0 && zz < d.dim[2] ? blk[d.od + dom_index(d, bx, by, zz)] : -1;
        }
        __syncthreads();
        bool any = false;
        for (int i = 0; i < z1 - z0; ++i) any = any || lds.blk[2 * HB + i] >= 0;
        if (any) {  // uniform
            // staged block i (z = z0 - HB + i) is written by k_edt_xy iff an
            // allocated block lies within HB of it: lds.blk[i .. i + 2 HB]
            for (int i = tid; i < nst; i += 256) {
                const int zz = z0 - HB + i;
                bool nd = false;
                for (int t = i; t <= i + 2 * HB; ++t) nd = nd || lds.blk[t] >= 0;
                lds.need[i] = nd && zz >= 0 && zz < d.dim[2];
            }
            __syncthreads();
            constexpr uint32_t inf2 = kInf16 * 0x10001u;
            constexpr int kAhead = 4;  // reads in flight
            for (int e0 = tid; e0 < nst * 64; e0 += kAhead * 256) {  // four rows of a column each
                uint4 v[kAhead];
#pragma unroll
                for (int k = 0; k < kAhead; ++k) {
                    const int e = min(e0 + 256 * k, nst * 64 - 1), i = e >> 6;
                    const bool in = lds.need[i] != 0;
                    v[k] = ((const uint4 *)(g2 + (d.od + dom_index(d, bx, by, in ? z0 - HB + i : z0)) * 512))[e & 63];
                    if (!in) v[k] = make_uint4(inf2, inf2, inf2, inf2);
                }
#pragma unroll
                for (int k = 0; k < kAhead; ++k) {
                    const int e = e0 + 256 * k, i = e >> 6, q = e & 63;
                    if (e < nst * 64) *(uint4 *)(colw + (q >> 1) * CW + 8 * i + 4 * (q & 1)) = v[k];
                }
            }
            __syncthreads();
            const uint32_t *col = colw + (lane >> 1) * CW;
            for (int io = wid; io < z1 - z0; io += 4) {
                const int32_t idx = lds.blk[2 * HB + io];
                if (idx < 0) continue;  // uniform
                // the lane's voxel pairs: x / 2 + 4 y = lane / 2, z = 4 (lane & 1) + j
                const int64_t v0 = 2 * (lane >> 1) + 256 * (lane & 1);
                const float *sd = job.seeds + (d.od + dom_index(d, bx, by, z0 + io)) * 512 + v0;  // from k_page_sites
                float2 seed[4];
                bool need = false;
#pragma unroll
                for (int j = 0; j < 4; ++j) seed[j] = *(const float2 *)(sd + 64 * j);
#pragma unroll
                for (int j = 0; j < 4; ++j) need = need || __builtin_isinf(seed[j].x) || __builtin_isinf(seed[j].y);
                u16x2 best[4];
                pair_search(col, 8 * (HB + io) + 4 * (lane & 1), R, need, best);
                float *out = job.phi + (int64_t)idx * 512 + v0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {  // unobserved (NaN) and in-band (D) seeds are the result
                    float2 o = seed[j];
                    if (__builtin_isinf(o.x)) o.x = phi_value(o.x, best[j].x, R2, vs, dmax);
                    if (__builtin_isinf(o.y)) o.y = phi_value(o.y, best[j].y, R2, vs, dmax);
                    *(float2 *)(out + 64 * j) = o;
                }
            }
        }
        __syncthreads();
    }
}

// The column passes of one submap's update, put off until the next frames'
// integration is launched on the same stream: its kernels take them along.  A second
// stream would overlap the two as well, but an event recorded on one stream and
// waited for on the other costs the host 14 us (a launch 4) and the frame 20.
struct EdtPass {
    static constexpr bool rides = true;
    JobList<1> jl;
    const uint64_t *sites;
    const int32_t *blk;
    uint16_t *g2;
    int seg_y, seg_z, R, HB;
    float vs, dmax;
    unsigned grid_y, grid_z;  // workgroups of the passes (0: not put off, or taken along already)
    unsigned lds_y, lds_z;    // bytes of LDS

    __device__ __forceinline__ void run_xy(EdtXyLds<1> &lds, uint32_t *colw) const
    {
        edt_xy<1>(jl, seg_y, sites, blk, g2, R, HB, lds, colw, blockIdx.x, grid_y);
    }
    __device__ __forceinline__ void run_z(EdtZLds<1> &lds, uint32_t *colw) const
    {
        edt_z<1>(jl, seg_z, g2, blk, R, HB, vs, dmax, lds, colw, blockIdx.x, grid_z);
    }
};

// A launch that takes none along.
struct NoEdt {
    static constexpr bool rides = false;
};

}  // namespace covox
