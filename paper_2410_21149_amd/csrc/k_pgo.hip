// Submap pose-graph optimisation (paper Eq. 1, Sec. III-F backend):
// registration, odometry and loop-closure terms over submap poses in
// R^3 x SO(2), solved by Levenberg-Marquardt with conjugate gradients on the
// reduced (block-sparse) system, all linear algebra on the GPU.
//
// One linearisation is three device steps:
//   k_pgo_move    the trial poses x + delta and T_i^-1 T_j of every pair;
//   registration normal equations of every pair: one batched alignment
//     evaluation with no pose update (k_align.hip);
//   k_pgo_terms   one wave per term: its four 4x4 blocks (ii, ij, ji, jj),
//                 two gradient pieces and its cost, in binary64;
//   k_pgo_reduce  one lane per output value (block entry, gradient entry,
//                 cost): sums its contributions in a fixed order, so the
//                 assembled system does not depend on scheduling.
// One step is one launch: (H + mu diag(H)) delta = -g by conjugate gradients
// with the inverses of the damped 4x4 diagonal blocks as preconditioner, then
// the model's predicted reduction -(2 delta.g + delta.H.delta):
//   k_pgo_cg_lds  one lane per unknown, the matrix in LDS (up to 64 free poses);
//   k_pgo_cg      one lane per block row, the matrix in memory (any size).
// The host runs the Levenberg-Marquardt loop (gain ratio, damping update of
// Madsen, Nielsen and Tingleff 2004, stopping on the step size) and reads seven
// numbers back once a step, after the linearisation at the trial poses.
#include "covox_impl.h"

#include <math.h>
#include <string.h>

#include <algorithm>
#include <map>
#include <vector>

namespace covox {

namespace {

struct PgoTerm {
    int32_t i, j;
    int32_t kind;  // 0 registration (normal equations `reg`), 1 relative-pose factor
    int32_t reg;
    double z[4];   // factor: measured (t, yaw) of T_i^-1 T_j
    double w[4];   // factor: 1 / sigma^2
};

constexpr int kTermOut = 4 * 16 + 2 * 4 + 1;  // blocks ii, ij, ji, jj; gradients i, j; cost

__device__ void rz3(double a, double R[9])
{
    double s, c;
    sincos(a, &s, &c);
    R[0] = c; R[1] = -s; R[2] = 0.0;
    R[3] = s; R[4] = c;  R[5] = 0.0;
    R[6] = 0.0; R[7] = 0.0; R[8] = 1.0;
}

__device__ double wrap_angle(double a)
{
    a = fmod(a + M_PI, 2.0 * M_PI);
    if (a <= 0.0) a += 2.0 * M_PI;
    return a - M_PI;
}

// One wave a term: with A_i, A_j (R x 4) the Jacobians of its R residuals at the two
// poses and B their weights, the blocks A_a^T B A_b, the gradients A_a^T v and the
// cost.  Bound by one lane's chain of some 600 dependent binary64 operations where a
// lane had a term (7.5 us, 16 submaps); a lane an entry, from LDS, 4.7.
__global__ __launch_bounds__(64) void k_pgo_terms(const PgoTerm *__restrict__ terms, const double *__restrict__ x,
                                                  const AlignResult *__restrict__ res, double w_reg,
                                                  double *__restrict__ out)
{
    __shared__ double Ad[36], M[2][24], A[2][24], B[36], v[6], BA[2][24];
    const int t = blockIdx.x, lane = threadIdx.x;
    const PgoTerm T = terms[t];
    const double *xi = x + 4 * T.i, *xj = x + 4 * T.j;
    double *o = out + (int64_t)t * kTermOut;
    const bool reg = T.kind == 0;  // uniform
    double scale = 1.0, cost = 0.0;
    if (reg) {
        // xi of T_ij = T_i^-1 T_j under T_k <- T(x_k + dx_k): Ad(T_i^-1) M(t_j) dx_j
        // - Ad(T_i^-1) M(t_i) dx_i, with M(t) dx = (dt - dyaw z x t, dyaw z)
        double Ri[9];
        rz3(xi[3], Ri);
        double Rt[9], ut[3];  // T_i^-1 = (Ri^T, -Ri^T t_i)
        for (int r = 0; r < 3; ++r)
            for (int c = 0; c < 3; ++c) Rt[3 * r + c] = Ri[3 * c + r];
        for (int r = 0; r < 3; ++r) ut[r] = -(Rt[3 * r] * xi[0] + Rt[3 * r + 1] * xi[1] + Rt[3 * r + 2] * xi[2]);
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                // [ut]x Rt
                const double hx[3] = {r == 0 ? 0.0 : (r == 1 ? ut[2] : -ut[1]),
                                      r == 0 ? -ut[2] : (r == 1 ? 0.0 : ut[0]),
                                      r == 0 ? ut[1] : (r == 1 ? -ut[0] : 0.0)};
                const double h = hx[0] * Rt[c] + hx[1] * Rt[3 + c] + hx[2] * Rt[6 + c];
                if (lane == 3 * r + c) {
                    Ad[6 * r + c] = Ad[6 * (r + 3) + c + 3] = Rt[3 * r + c];
                    Ad[6 * (r + 3) + c] = 0.0;
                    Ad[6 * r + c + 3] = h;
                }
            }
        if (lane < 48) {
            const double *tp = lane < 24 ? xi : xj;
            const int r = lane % 24 / 4, c = lane & 3;
            double m = r == c ? 1.0 : 0.0;
            if (c == 3) m = r == 0 ? tp[1] : (r == 1 ? -tp[0] : (r == 5 ? 1.0 : 0.0));
            M[lane / 24][lane % 24] = m;
        }
        const double *q = res[T.reg].ne;
        if (lane < 36) {
            const int r = min(lane / 6, lane % 6), c = max(lane / 6, lane % 6);
            B[lane] = q[r * 6 - r * (r - 1) / 2 + (c - r)];
        }
        if (lane < 6) v[lane] = q[21 + lane];
        scale = w_reg;
        cost = w_reg * q[27];
        __syncthreads();
        if (lane < 48) {
            const int r = lane % 24 / 4, c = lane & 3;
            double sum = 0.0;
#pragma unroll
            for (int k = 0; k < 6; ++k) sum += Ad[6 * r + k] * M[lane / 24][4 * k + c];
            A[lane / 24][lane % 24] = (lane < 24 ? -1.0 : 1.0) * sum;
        }
    } else {
        // e_t = Rz(-z_yaw) (Rz(-yaw_i) (t_j - t_i) - z_t), e_yaw = wrap(yaw_j - yaw_i - z_yaw)
        double Rzm[9], Rim[9], Q[9];
        rz3(-T.z[3], Rzm);
        rz3(-xi[3], Rim);
        for (int r = 0; r < 3; ++r)
            for (int c = 0; c < 3; ++c) Q[3 * r + c] = Rzm[3 * r] * Rim[c] + Rzm[3 * r + 1] * Rim[3 + c] + Rzm[3 * r + 2] * Rim[6 + c];
        const double d[3] = {xj[0] - xi[0], xj[1] - xi[1], xj[2] - xi[2]};
        double e[4];
        for (int r = 0; r < 3; ++r)
            e[r] = (Q[3 * r] * d[0] + Q[3 * r + 1] * d[1] + Q[3 * r + 2] * d[2]) -
                   (Rzm[3 * r] * T.z[0] + Rzm[3 * r + 1] * T.z[1] + Rzm[3 * r + 2] * T.z[2]);
        e[3] = wrap_angle(xj[3] - xi[3] - T.z[3]);
        const double zd[3] = {-d[1], d[0], 0.0};  // z x d
        const double we[4] = {T.w[0] * e[0], T.w[1] * e[1], T.w[2] * e[2], T.w[3] * e[3]};
        cost = e[0] * we[0] + e[1] * we[1] + e[2] * we[2] + e[3] * we[3];
        if (lane == 0) {
#pragma unroll
            for (int r = 0; r < 3; ++r) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    A[0][4 * r + c] = -Q[3 * r + c];
                    A[1][4 * r + c] = Q[3 * r + c];
                }
                A[0][4 * r + 3] = -(Q[3 * r] * zd[0] + Q[3 * r + 1] * zd[1] + Q[3 * r + 2] * zd[2]);
                A[1][4 * r + 3] = A[0][12 + r] = A[1][12 + r] = 0.0;
            }
            A[0][15] = -1.0;
            A[1][15] = 1.0;
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = we[k];
        }
    }
    __syncthreads();
    const int R = reg ? 6 : 4;
    // B A_b, and the gradients
    if (lane < 8 * R) {
        const int b = lane / (4 * R), e = lane % (4 * R), p = e >> 2, q = e & 3;
        double sum = 0.0;
        if (reg) {
#pragma unroll
            for (int k = 0; k < 6; ++k) sum += B[6 * p + k] * A[b][4 * k + q];
        } else {
            sum = terms[t].w[p] * A[b][e];  // B is diagonal
        }
        BA[b][e] = sum;
    }
    if (lane < 8) {
        double sum = 0.0;
        for (int k = 0; k < R; ++k) sum += A[lane >> 2][4 * k + (lane & 3)] * v[k];
        o[64 + lane] = scale * sum;
    }
    __syncthreads();
    {
        const int a = lane >> 5, b = lane >> 4 & 1, p = lane >> 2 & 3, q = lane & 3;
        double sum = 0.0;
        for (int k = 0; k < R; ++k) sum += A[a][4 * k + p] * BA[b][4 * k + q];
        o[lane] = scale * sum;
    }
    if (lane == 0) o[72] = cost;
}

// out[k] = sum of src[off[p]] for p in [ptr[k], ptr[k + 1]), in order; the last
// workgroup sums the terms' costs instead, in a fixed order.
__global__ __launch_bounds__(256) void k_pgo_reduce(int n_items, int n_terms, const int32_t *__restrict__ ptr,
                                                    const int32_t *__restrict__ off, const double *__restrict__ src,
                                                    double *__restrict__ out, double *__restrict__ cost)
{
    if (blockIdx.x == gridDim.x - 1) {
        __shared__ double red[4];
        double s = 0.0;
        for (int t = threadIdx.x; t < n_terms; t += 256) s += src[(int64_t)t * kTermOut + kTermOut - 1];
        s = wave_sum(s);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
        __syncthreads();
        if (threadIdx.x == 0) *cost = (red[0] + red[1]) + (red[2] + red[3]);
        return;
    }
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n_items) return;
    double s = 0.0;
    const int end = ptr[k + 1];
    constexpr int kAhead = 8;  // reads in flight
    for (int p = ptr[k]; p < end; p += kAhead) {
        double v[kAhead];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) v[q] = p + q < end ? src[off[p + q]] : 0.0;
#pragma unroll
        for (int q = 0; q < kAhead; ++q) s = p + q < end ? s + v[q] : s;
    }
    out[k] = s;
}

// T = [Rz(yaw) t; 0 1] of x = (t, yaw), row-major 4x4.
__device__ void pose_of(const double *x, double *T)
{
    double s, c;
    sincos(x[3], &s, &c);
    const double M[16] = {c, -s, 0, x[0], s, c, 0, x[1], 0, 0, 1, x[2], 0, 0, 0, 1};
    for (int k = 0; k < 16; ++k) T[k] = M[k];
}

// T_i^-1 T_j of two poses.
__device__ void relative_pose(const double *xi, const double *xj, double *T)
{
    double Ti[16], Tj[16];
    pose_of(xi, Ti);
    pose_of(xj, Tj);
    double Inv[16] = {0};
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) Inv[4 * r + c] = Ti[4 * c + r];
    for (int r = 0; r < 3; ++r) Inv[4 * r + 3] = -(Inv[4 * r] * Ti[3] + Inv[4 * r + 1] * Ti[7] + Inv[4 * r + 2] * Ti[11]);
    Inv[15] = 1.0;
    for (int r = 0; r < 4; ++r)
        for (int c = 0; c < 4; ++c)
            T[4 * r + c] = Inv[4 * r] * Tj[c] + Inv[4 * r + 1] * Tj[4 + c] + Inv[4 * r + 2] * Tj[8 + c] + Inv[4 * r + 3] * Tj[12 + c];
}

// xn = x + (0, delta) (delta null: the poses as they are), and the pose of every
// registration problem.
__global__ __launch_bounds__(64) void k_pgo_move(int n_poses, int n_terms, const PgoTerm *__restrict__ terms,
                                                 const double *x, const double *delta, double *xn,
                                                 AlignProblem *probs)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    auto at = [&](int k) { return x[k] + (delta && k >= 4 ? delta[k - 4] : 0.0); };
    if (t < 4 * n_poses) xn[t] = at(t);
    if (t >= n_terms || terms[t].kind != 0) return;
    double xi[4], xj[4], T[16];
    for (int a = 0; a < 4; ++a) {
        xi[a] = at(4 * terms[t].i + a);
        xj[a] = at(4 * terms[t].j + a);
    }
    relative_pose(xi, xj, T);
    for (int k = 0; k < 16; ++k) probs[terms[t].reg].T[k] = T[k];
}

constexpr int kCgThreads = 256;
constexpr int kCgWaves = kCgThreads / 64;

// Sums of (a, b) over the workgroup: butterfly within each wave, then the
// four wave totals in order (deterministic).  Two barriers.
__device__ void block_sum2(double &a, double &b, double *red)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_xor(a, off, 64);
        b += __shfl_xor(b, off, 64);
    }
    const int wid = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[2 * wid] = a;
        red[2 * wid + 1] = b;
    }
    __syncthreads();
    a = 0.0;
    b = 0.0;
    for (int w = 0; w < kCgWaves; ++w) {
        a += red[2 * w];
        b += red[2 * w + 1];
    }
    __syncthreads();
}

__device__ double block_max(double a, double *red)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) a = fmax(a, __shfl_xor(a, off, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
    __syncthreads();
    a = red[0];
    for (int w = 1; w < kCgWaves; ++w) a = fmax(a, red[w]);
    return a;
}

// Rows 4 r .. 4 r + 3 of (H + mu diag(H)) p.
__device__ __forceinline__ void bsr_row(int r, const int32_t *rp, const int32_t *ci, const double *vals,
                                        const int32_t *dslot, double mu, const double *p, double y[4])
{
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int s = rp[r]; s < rp[r + 1]; ++s) {
        const double *B = vals + 16 * (int64_t)s;
        const double *pc = p + 4 * ci[s];
        for (int a = 0; a < 4; ++a) acc[a] += B[4 * a] * pc[0] + B[4 * a + 1] * pc[1] + B[4 * a + 2] * pc[2] + B[4 * a + 3] * pc[3];
    }
    const double *Dg = vals + 16 * (int64_t)dslot[r];
    for (int a = 0; a < 4; ++a) y[a] = acc[a] + mu * Dg[5 * a] * p[4 * r + a];
}

// info[0] = iterations, info[1] = 1 on success (0: not positive definite),
// info[2] = predicted reduction, info[3] = final relative residual, info[4] =
// the largest |delta|.
// Each lane owns whole block rows (b = lane, lane + 256, ...), so that the
// preconditioner and the vector updates need no barrier; the five vectors
// (solution, r, z, p, Ap) live in LDS when they fit (dynamic shared memory
// of 40 n bytes), else in `work`.
__global__ __launch_bounds__(kCgThreads) void k_pgo_cg(int nb, const int32_t *__restrict__ rp,
                                                       const int32_t *__restrict__ ci, const double *__restrict__ vals,
                                                       const int32_t *__restrict__ dslot, const double *__restrict__ g,
                                                       double mu, double tol, int max_it, double *__restrict__ work,
                                                       double *__restrict__ delta_out, double *__restrict__ info,
                                                       int vec_in_lds)
{
    __shared__ double red[2 * kCgWaves];
    __shared__ int s_bad;
    extern __shared__ double dyn[];
    const int n = 4 * nb, tid = threadIdx.x;
    double *Pinv = work;
    double *vec = vec_in_lds ? dyn : work + 16 * (int64_t)nb;
    double *r = vec, *z = r + n, *p = z + n, *Ap = p + n, *x = Ap + n;
    if (tid == 0) s_bad = 0;
    __syncthreads();
    // inverses of the damped diagonal blocks (Cholesky)
    for (int b = tid; b < nb; b += kCgThreads) {
        const double *B = vals + 16 * (int64_t)dslot[b];
        double A[16], L[16] = {0}, Li[16] = {0};
        for (int k = 0; k < 16; ++k) A[k] = B[k];
        for (int a = 0; a < 4; ++a) A[5 * a] += mu * B[5 * a];
        bool ok = true;
        for (int j = 0; j < 4 && ok; ++j) {
            double sj = A[5 * j];
            for (int k = 0; k < j; ++k) sj -= L[4 * j + k] * L[4 * j + k];
            if (!(sj > 0.0)) { ok = false; break; }
            L[5 * j] = sqrt(sj);
            for (int i = j + 1; i < 4; ++i) {
                double t = A[4 * i + j];
                for (int k = 0; k < j; ++k) t -= L[4 * i + k] * L[4 * j + k];
                L[4 * i + j] = t / L[5 * j];
            }
        }
        if (!ok) {
            s_bad = 1;
            continue;
        }
        for (int c = 0; c < 4; ++c)  // L^-1 by forward substitution
            for (int i = 0; i < 4; ++i) {
                double t = i == c ? 1.0 : 0.0;
                for (int k = 0; k < i; ++k) t -= L[4 * i + k] * Li[4 * k + c];
                Li[4 * i + c] = t / L[5 * i];
            }
        double *P = Pinv + 16 * (int64_t)b;  // (L L^T)^-1 = L^-T L^-1
        for (int i = 0; i < 4; ++i)
            for (int j = 0; j < 4; ++j) {
                double t = 0.0;
                for (int k = 0; k < 4; ++k) t += Li[4 * k + i] * Li[4 * k + j];
                P[4 * i + j] = t;
            }
    }
    __syncthreads();
    if (s_bad) {
        if (tid == 0) { info[0] = 0; info[1] = 0; info[2] = 0; info[3] = 0; info[4] = 0; }
        return;
    }
    // z = P r for owned block row b (r already set)
    auto precond_row = [&](int b, double &rr, double &rzp) {
        const double *P = Pinv + 16 * (int64_t)b;
        const double *rb = r + 4 * b;
        for (int a = 0; a < 4; ++a) {
            const double za = P[4 * a] * rb[0] + P[4 * a + 1] * rb[1] + P[4 * a + 2] * rb[2] + P[4 * a + 3] * rb[3];
            z[4 * b + a] = za;
            rr += rb[a] * rb[a];
            rzp += rb[a] * za;
        }
    };
    double bb = 0.0, rz = 0.0;
    for (int b = tid; b < nb; b += kCgThreads) {
        for (int a = 0; a < 4; ++a) {
            x[4 * b + a] = 0.0;
            r[4 * b + a] = -g[4 * b + a];
        }
        precond_row(b, bb, rz);  // bb accumulates |r|^2 = |g|^2
        for (int a = 0; a < 4; ++a) p[4 * b + a] = z[4 * b + a];
    }
    block_sum2(bb, rz, red);  // also orders the p writes before the first product
    const double bnorm = sqrt(bb);
    int it = 0;
    int ok = 1;
    double rel = bnorm > 0.0 ? 1.0 : 0.0;
    while (bnorm > 0.0 && it < max_it) {
        double pap = 0.0, unused = 0.0;
        for (int b = tid; b < nb; b += kCgThreads) {
            double y[4];
            bsr_row(b, rp, ci, vals, dslot, mu, p, y);
            for (int a = 0; a < 4; ++a) {
                Ap[4 * b + a] = y[a];
                pap += p[4 * b + a] * y[a];
            }
        }
        block_sum2(pap, unused, red);
        if (!(pap > 0.0)) { ok = 0; break; }
        const double alpha = rz / pap;
        double rr = 0.0, rz2 = 0.0;
        for (int b = tid; b < nb; b += kCgThreads) {
            for (int a = 0; a < 4; ++a) {
                x[4 * b + a] += alpha * p[4 * b + a];
                r[4 * b + a] -= alpha * Ap[4 * b + a];
            }
            precond_row(b, rr, rz2);
        }
        block_sum2(rr, rz2, red);
        ++it;
        rel = sqrt(rr) / bnorm;
        if (rel <= tol) break;
        const double beta = rz2 / rz;
        rz = rz2;
        for (int b = tid; b < nb; b += kCgThreads)
            for (int a = 0; a < 4; ++a) p[4 * b + a] = z[4 * b + a] + beta * p[4 * b + a];
        __syncthreads();
    }
    // predicted reduction of the undamped model: -(2 x.g + x.H.x)
    __syncthreads();
    double pr = 0.0, unused = 0.0, big = 0.0;
    for (int b = tid; b < nb; b += kCgThreads) {
        double y[4];
        bsr_row(b, rp, ci, vals, dslot, 0.0, x, y);
        for (int a = 0; a < 4; ++a) {
            pr += 2.0 * x[4 * b + a] * g[4 * b + a] + x[4 * b + a] * y[a];
            delta_out[4 * b + a] = x[4 * b + a];
            big = fmax(big, fabs(x[4 * b + a]));
        }
    }
    block_sum2(pr, unused, red);
    big = block_max(big, red);
    if (tid == 0) {
        info[4] = big;
        info[0] = it;
        info[1] = ok;
        info[2] = -pr;
        info[3] = rel;
    }
}

// The same solve for up to 64 free poses: lane t owns unknown t (its x, r, z, p
// and Ap in registers), the matrix and p lie in LDS, and up to 16 poses need one
// wave and no barrier.  Bound by the chain of an iteration: one matrix row from
// LDS, two reductions, two divisions.  One lane per block row, with its blocks
// read from memory again in every iteration, took 152 us a solve for 15 free
// poses (60 unknowns, up to 240 iterations), with the rows read from LDS 71 us; with
// rows of up to kCgRow blocks in registers, so that an iteration reads only p, 41 us.
constexpr int kCgLdsPoses = 64;
constexpr size_t kCgLdsBytes = 60 * 1024;

constexpr int kCgRow = 8;  // blocks of a row held in registers

template <int NT>
__device__ __forceinline__ void cg_sync()
{
    if constexpr (NT == 64) wave_sync();
    else __syncthreads();
}

template <int NT>
__device__ __forceinline__ void cg_sum2(double &a, double &b, double *red)
{
    a = wave_sum(a);
    b = wave_sum(b);
    if constexpr (NT > 64) {
        const int wid = threadIdx.x >> 6;
        if ((threadIdx.x & 63) == 0) {
            red[2 * wid] = a;
            red[2 * wid + 1] = b;
        }
        __syncthreads();
        a = b = 0.0;
        for (int w = 0; w < NT / 64; ++w) {
            a += red[2 * w];
            b += red[2 * w + 1];
        }
        __syncthreads();
    }
}

template <int NT>
__global__ __launch_bounds__(NT) void k_pgo_cg_lds(int nb, int nnzb, const int32_t *__restrict__ rp,
                                                   const int32_t *__restrict__ ci, const double *__restrict__ vals,
                                                   const int32_t *__restrict__ dslot, const double *__restrict__ g,
                                                   double mu, double tol, int max_it, double *__restrict__ delta_out,
                                                   double *__restrict__ info)
{
    static_assert(NT == 64 || NT == kCgThreads, "one wave, or the width of block_sum2");
    __shared__ double red[2 * kCgWaves];
    __shared__ int s_bad;
    extern __shared__ double dyn[];  // matrix, p, columns
    double *B = dyn, *p = dyn + 16 * (size_t)nnzb;
    int32_t *col = (int32_t *)(p + 4 * nb);
    const int tid = threadIdx.x, n = 4 * nb;
    const bool own = tid < n;
    const int b = own ? tid >> 2 : 0, a = tid & 3;
    if (tid == 0) s_bad = 0;
    for (int k = tid; k < 16 * nnzb; k += NT) B[k] = vals[k];
    for (int k = tid; k < nnzb; k += NT) col[k] = ci[k];
    __syncthreads();
    const int s0 = rp[b], s1 = rp[b + 1];
    const double *Dg = B + 16 * dslot[b];
    const double diag = mu * Dg[5 * a];
    // row a of the inverse of the damped diagonal block (Cholesky)
    double Pa[4];
    {
        double A[16], L[16] = {0}, Li[16] = {0};
#pragma unroll
        for (int k = 0; k < 16; ++k) A[k] = Dg[k];
#pragma unroll
        for (int k = 0; k < 4; ++k) A[5 * k] += mu * Dg[5 * k];
        bool ok = true;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            double sj = A[5 * j];
#pragma unroll
            for (int k = 0; k < j; ++k) sj -= L[4 * j + k] * L[4 * j + k];
            ok = ok && sj > 0.0;
            L[5 * j] = sqrt(sj);
#pragma unroll
            for (int i = j + 1; i < 4; ++i) {
                double t = A[4 * i + j];
#pragma unroll
                for (int k = 0; k < j; ++k) t -= L[4 * i + k] * L[4 * j + k];
                L[4 * i + j] = t / L[5 * j];
            }
        }
        if (own && !ok) s_bad = 1;
#pragma unroll
        for (int c = 0; c < 4; ++c)  // L^-1 by forward substitution
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                double t = i == c ? 1.0 : 0.0;
#pragma unroll
                for (int k = 0; k < i; ++k) t -= L[4 * i + k] * Li[4 * k + c];
                Li[4 * i + c] = t / L[5 * i];
            }
#pragma unroll
        for (int j = 0; j < 4; ++j) {  // (L L^T)^-1 = L^-T L^-1
            double t = 0.0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const double lk = a == 0 ? Li[4 * k] : (a == 1 ? Li[4 * k + 1] : (a == 2 ? Li[4 * k + 2] : Li[4 * k + 3]));
                t += lk * Li[4 * k + j];
            }
            Pa[j] = t;
        }
    }
    __syncthreads();
    if (s_bad) {
        if (tid < 5) info[tid] = 0.0;
        return;
    }
    auto precond = [&](double r) {  // the pose's four residuals are in its quad of lanes
        const double z = Pa[0] * dpp_f64<0x00>(r) + Pa[1] * dpp_f64<0x55>(r) + Pa[2] * dpp_f64<0xAA>(r) +
                         Pa[3] * dpp_f64<0xFF>(r);
        return own ? z : 0.0;
    };
    // A row of up to kCgRow blocks stays in registers over the iterations.
    bool reg = s1 - s0 <= kCgRow;
    if constexpr (NT == 64) reg = __ballot(!reg) == 0;
    else reg = __syncthreads_and(reg) != 0;
    double Br[kCgRow][4];
    int pr4[kCgRow];
    if (reg) {  // uniform
#pragma unroll
        for (int q = 0; q < kCgRow; ++q) {
            const int sq = min(s0 + q, s1 - 1);
            pr4[q] = 4 * col[sq];
#pragma unroll
            for (int c = 0; c < 4; ++c) Br[q][c] = s0 + q < s1 ? B[16 * sq + 4 * a + c] : 0.0;
        }
    }
    auto row = [&](double damp, double pv) {  // (H + damp) p of this unknown
        double y = 0.0;
        if (reg) {
            double t[kCgRow];
#pragma unroll
            for (int q = 0; q < kCgRow; ++q) {
                const double *pc = p + pr4[q];
                t[q] = Br[q][0] * pc[0] + Br[q][1] * pc[1] + Br[q][2] * pc[2] + Br[q][3] * pc[3];
            }
#pragma unroll
            for (int q = 0; q < kCgRow; ++q) y += t[q];  // (0 beyond the row)
            return own ? y + damp * pv : 0.0;
        }
        // four blocks' reads at a time
        for (int s = s0; s < s1; s += 4) {
            double t[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int sq = min(s + q, s1 - 1);
                const double *Bs = B + 16 * sq + 4 * a, *pc = p + 4 * col[sq];
                t[q] = Bs[0] * pc[0] + Bs[1] * pc[1] + Bs[2] * pc[2] + Bs[3] * pc[3];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) y = s + q < s1 ? y + t[q] : y;
        }
        return own ? y + damp * pv : 0.0;
    };
    const double gv = own ? g[tid] : 0.0;
    double x = 0.0, r = -gv, z = precond(r), pv = z;
    double bb = r * r, rz = r * z;
    if (own) p[tid] = pv;
    cg_sum2<NT>(bb, rz, red);
    cg_sync<NT>();
    const double bnorm = sqrt(bb);
    // sqrt(rr) / bnorm <= tol is worked out only where it can hold
    const double near = 1.001 * (tol * bnorm) * (tol * bnorm);
    int it = 0, ok = 1;
    double rel = bnorm > 0.0 ? 1.0 : 0.0, rr = bb;
    while (bnorm > 0.0 && it < max_it) {
        const double Ap = row(diag, pv);
        double pap = pv * Ap, unused = 0.0;
        cg_sum2<NT>(pap, unused, red);
        if (!(pap > 0.0)) { ok = 0; break; }
        const double alpha = rz / pap;
        x += alpha * pv;
        r -= alpha * Ap;
        z = precond(r);
        double rz2 = r * z;
        rr = r * r;
        cg_sum2<NT>(rr, rz2, red);
        ++it;
        if (rr <= near && sqrt(rr) / bnorm <= tol) break;
        pv = z + rz2 / rz * pv;
        rz = rz2;
        cg_sync<NT>();  // every row has read the old p
        if (own) p[tid] = pv;
        cg_sync<NT>();
    }
    if (it > 0) rel = sqrt(rr) / bnorm;
    // predicted reduction of the undamped model: -(2 x.g + x.H.x)
    cg_sync<NT>();
    if (own) p[tid] = x;
    cg_sync<NT>();
    double pr = 2.0 * x * gv + x * row(0.0, x), unused = 0.0, big = fabs(x);
    cg_sum2<NT>(pr, unused, red);
    if constexpr (NT == 64) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) big = fmax(big, __shfl_xor(big, off, 64));
    } else {
        big = block_max(big, red);
    }
    if (own) delta_out[tid] = x;
    if (tid == 0) {
        info[0] = it;
        info[1] = ok;
        info[2] = -pr;
        info[3] = rel;
        info[4] = big;
    }
}

}  // namespace

void covox_default_pgo_cfg_impl(covox_pgo_cfg *c)
{
    c->max_iter = 20;
    c->cg_max_iter = 0;
    c->sigma_reg = 0.05;
    c->lambda0 = 1e-4;
    c->tol_step = 1e-8;
    c->cg_tol = 1e-12;
}

int pgo_solve(covox_ctx *ctx, covox_submap *const *subs, int32_t N, double *x, const int32_t *reg_pairs,
              int32_t n_reg, const covox_pose_factor *factors, int32_t n_fac, const covox_pgo_cfg *cfg_in,
              covox_pgo_stats *stats)
{
    covox_pgo_cfg cfg;
    if (cfg_in) cfg = *cfg_in;
    else covox_default_pgo_cfg_impl(&cfg);
    if (!subs || !x || N < 2 || n_reg < 0 || n_fac < 0 || (n_reg > 0 && !reg_pairs) || (n_fac > 0 && !factors))
        return fail(ctx, COVOX_EINVAL, "pgo: bad argument");
    if (cfg.max_iter < 0 || cfg.cg_max_iter < 0 || !(cfg.sigma_reg > 0) || !(cfg.lambda0 >= 0) ||
        !(cfg.tol_step >= 0) || !(cfg.cg_tol >= 0))
        return fail(ctx, COVOX_EINVAL, "pgo: bad configuration");
    for (int32_t k = 0; k < 4 * N; ++k)
        if (!std::isfinite(x[k])) return fail(ctx, COVOX_EINVAL, "pgo: poses must be finite");
    std::vector<PgoTerm> terms;
    for (int32_t k = 0; k < n_reg; ++k) {
        const int32_t i = reg_pairs[2 * k], j = reg_pairs[2 * k + 1];
        if (i < 0 || j < 0 || i >= N || j >= N || i == j || !subs[i] || !subs[j])
            return fail(ctx, COVOX_EINVAL, "pgo: bad registration pair");
        PgoTerm t{};
        t.i = i; t.j = j; t.kind = 0; t.reg = k;
        terms.push_back(t);
    }
    for (int32_t k = 0; k < n_fac; ++k) {
        const covox_pose_factor &f = factors[k];
        if (f.i < 0 || f.j < 0 || f.i >= N || f.j >= N || f.i == f.j)
            return fail(ctx, COVOX_EINVAL, "pgo: bad factor indices");
        PgoTerm t{};
        t.i = f.i; t.j = f.j; t.kind = 1; t.reg = -1;
        for (int a = 0; a < 4; ++a) {
            if (!(f.sigma[a] > 0) || !std::isfinite(f.z[a])) return fail(ctx, COVOX_EINVAL, "pgo: bad factor");
            t.z[a] = f.z[a];
            t.w[a] = 1.0 / (f.sigma[a] * f.sigma[a]);
        }
        terms.push_back(t);
    }
    const int n_terms = (int)terms.size();
    if (n_terms == 0) return fail(ctx, COVOX_EINVAL, "pgo: no terms");
    int rc;
    for (int32_t k = 0; k < n_reg; ++k) {
        covox_submap *A = subs[reg_pairs[2 * k]], *B = subs[reg_pairs[2 * k + 1]];
        if (A->esdf_version != A->version)
            return fail(ctx, COVOX_EINVAL, "pgo: an ESDF of a registration pair is out of date");
        if ((rc = extract_points(ctx, B))) return rc;
    }

    // block-sparse pattern over the free poses 1..N-1 (block row r = pose r + 1)
    const int nb = N - 1, n = 4 * nb;
    std::vector<std::vector<int>> cols(nb);
    for (int r = 0; r < nb; ++r) cols[r].push_back(r);
    for (const PgoTerm &t : terms)
        if (t.i > 0 && t.j > 0) {
            cols[t.i - 1].push_back(t.j - 1);
            cols[t.j - 1].push_back(t.i - 1);
        }
    std::vector<int32_t> rp(nb + 1, 0), ci, dslot(nb);
    std::map<std::pair<int, int>, int> slot;
    for (int r = 0; r < nb; ++r) {
        std::sort(cols[r].begin(), cols[r].end());
        cols[r].erase(std::unique(cols[r].begin(), cols[r].end()), cols[r].end());
        for (int c : cols[r]) {
            if (c == r) dslot[r] = (int32_t)ci.size();
            slot[{r, c}] = (int32_t)ci.size();
            ci.push_back(c);
        }
        rp[r + 1] = (int32_t)ci.size();
    }
    const int nnzb = (int)ci.size();
    // reduction plan: output = [blocks (16 nnzb) | gradient (n)]
    std::vector<std::vector<int32_t>> src(16 * nnzb + n);
    for (int t = 0; t < n_terms; ++t) {
        const int ends[2] = {terms[t].i, terms[t].j};
        for (int a = 0; a < 2; ++a) {
            if (ends[a] == 0) continue;
            for (int b = 0; b < 2; ++b) {
                if (ends[b] == 0) continue;
                const int s = slot[{ends[a] - 1, ends[b] - 1}];
                for (int e = 0; e < 16; ++e) src[16 * s + e].push_back(t * kTermOut + 16 * (2 * a + b) + e);
            }
            for (int e = 0; e < 4; ++e) src[16 * nnzb + 4 * (ends[a] - 1) + e].push_back(t * kTermOut + 64 + 4 * a + e);
        }
    }
    const int n_out = 16 * nnzb + n;
    std::vector<int32_t> pptr(1, 0), poff;
    for (int k = 0; k < n_out; ++k) {
        poff.insert(poff.end(), src[k].begin(), src[k].end());
        pptr.push_back((int32_t)poff.size());
    }

    // registration problems: laid out once, their poses written on the device
    std::vector<AlignProblem> probs(n_reg);
    for (int32_t k = 0; k < n_reg; ++k) {
        const covox_submap *A = subs[reg_pairs[2 * k]], *B = subs[reg_pairs[2 * k + 1]];
        AlignProblem &pr = probs[k];
        memset(&pr, 0, sizeof(pr));
        pr.A = A;
        pr.page = A->page;
        pr.metaA = A->meta;
        pr.pts = B->pts;
        pr.n_pts = B->n_pts;
        pr.max_iter = 0;
    }
    AlignPlan pl;
    if (n_reg > 0) {
        if ((rc = place_alignment(ctx, probs.data(), n_reg, cfg.max_iter, pl))) return rc;
    }
    AlignResult *dres = (AlignResult *)ctx->res_dev;

    // device arrays of the solve in the context's buffer, the constant ones and
    // the initial poses uploaded together
    size_t total = 0;
    auto take = [&](size_t bytes) {
        const size_t at = total;
        total += (bytes + 15) / 16 * 16;
        return at;
    };
    const size_t o_terms = take(sizeof(PgoTerm) * n_terms), o_rp = take(sizeof(int32_t) * rp.size()),
                 o_ci = take(sizeof(int32_t) * nnzb), o_dslot = take(sizeof(int32_t) * nb),
                 o_pptr = take(sizeof(int32_t) * pptr.size()), o_poff = take(sizeof(int32_t) * poff.size()),
                 o_x0 = take(sizeof(double) * 4 * N), up_bytes = total, o_x1 = take(sizeof(double) * 4 * N),
                 o_tout = take(sizeof(double) * kTermOut * n_terms), o_out0 = take(sizeof(double) * n_out),
                 o_out1 = take(sizeof(double) * n_out), o_work = take(sizeof(double) * (16 * (size_t)nb + 5 * (size_t)n)),
                 o_delta = take(sizeof(double) * n), o_info = take(sizeof(double) * 8);
    if ((rc = ensure_buffer(ctx, &ctx->pgo_dev, &ctx->pgo_cap, (int64_t)total, 1, "pgo buffers"))) return rc;
    if (!ctx->pgo_pin &&
        (rc = hip_check(ctx, hipHostMalloc((void **)&ctx->pgo_pin, sizeof(double) * 8, hipHostMallocDefault), "pgo step")))
        return rc;
    char *dev = (char *)ctx->pgo_dev;
    std::vector<char> stage(up_bytes);
    memcpy(stage.data() + o_terms, terms.data(), sizeof(PgoTerm) * n_terms);
    memcpy(stage.data() + o_rp, rp.data(), sizeof(int32_t) * rp.size());
    memcpy(stage.data() + o_ci, ci.data(), sizeof(int32_t) * nnzb);
    memcpy(stage.data() + o_dslot, dslot.data(), sizeof(int32_t) * nb);
    memcpy(stage.data() + o_pptr, pptr.data(), sizeof(int32_t) * pptr.size());
    if (!poff.empty()) memcpy(stage.data() + o_poff, poff.data(), sizeof(int32_t) * poff.size());
    memcpy(stage.data() + o_x0, x, sizeof(double) * 4 * N);
    hipStream_t st = ctx->stream;
    if ((rc = hip_check(ctx, hipMemcpyAsync(dev, stage.data(), up_bytes, hipMemcpyHostToDevice, st), "pgo upload")))
        return rc;
    const PgoTerm *dterms = (const PgoTerm *)(dev + o_terms);
    const int32_t *drp = (const int32_t *)(dev + o_rp), *dci = (const int32_t *)(dev + o_ci),
                  *ddslot = (const int32_t *)(dev + o_dslot);
    double *dx[2] = {(double *)(dev + o_x0), (double *)(dev + o_x1)};
    double *dout[2] = {(double *)(dev + o_out0), (double *)(dev + o_out1)};
    double *dtout = (double *)(dev + o_tout), *ddelta = (double *)(dev + o_delta), *dinfo = (double *)(dev + o_info);

    const double w_reg = 1.0 / (cfg.sigma_reg * cfg.sigma_reg);
    // F (to dinfo[5 + which]), g and H at the poses dx[which] = dx[from] + delta
    auto linearize = [&](int from, int which, const double *delta, bool first) -> int {
        hipLaunchKernelGGL(k_pgo_move, dim3((std::max(4 * N, n_terms) + 63) / 64), dim3(64), 0, st, N, n_terms, dterms,
                           dx[from], delta, dx[which], (AlignProblem *)ctx->prob_dev);
        int rc2;
        if (n_reg > 0 && (rc2 = launch_alignment(ctx, pl, dres, first))) return rc2;
        TimedLaunch tl(ctx, COVOX_K_PGO);
        hipLaunchKernelGGL(k_pgo_terms, dim3(n_terms), dim3(64), 0, st, dterms, dx[which], dres, w_reg, dtout);
        hipLaunchKernelGGL(k_pgo_reduce, dim3((n_out + 255) / 256 + 1), dim3(256), 0, st, n_out, n_terms,
                           (const int32_t *)(dev + o_pptr), (const int32_t *)(dev + o_poff), dtout, dout[which],
                           dinfo + 5 + which);
        return hip_check(ctx, hipGetLastError(), "pgo launch");
    };
    double *info = ctx->pgo_pin;
    auto read_info = [&]() -> int {
        int rc2;
        if ((rc2 = hip_check(ctx, hipMemcpyAsync(info, dinfo, sizeof(double) * 8, hipMemcpyDeviceToHost, st), "pgo info")))
            return rc2;
        return hip_check(ctx, hipStreamSynchronize(st), "pgo sync");
    };
    const int cg_max = cfg.cg_max_iter > 0 ? cfg.cg_max_iter : 4 * n;
    // the matrix in LDS where it and the unknowns fit, else the vectors up to
    // 48 KB (n <= 1228), beside the 2 KB reduction buffer
    const size_t mat_bytes = sizeof(double) * (16 * (size_t)nnzb + n) + sizeof(int32_t) * (size_t)nnzb;
    const bool small = nb <= kCgLdsPoses && mat_bytes <= kCgLdsBytes;
    const size_t lds_bytes = 5 * sizeof(double) * (size_t)n <= 48 * 1024 ? 5 * sizeof(double) * (size_t)n : 0;
    auto step = [&](int which, double mu) -> int {
        TimedLaunch tl(ctx, COVOX_K_PGO);
        const double *out = dout[which];
        if (small && n <= 64)
            hipLaunchKernelGGL(k_pgo_cg_lds<64>, dim3(1), dim3(64), mat_bytes, st, nb, nnzb, drp, dci, out, ddslot,
                               out + 16 * nnzb, mu, cfg.cg_tol, cg_max, ddelta, dinfo);
        else if (small)
            hipLaunchKernelGGL(k_pgo_cg_lds<kCgThreads>, dim3(1), dim3(kCgThreads), mat_bytes, st, nb, nnzb, drp, dci, out,
                               ddslot, out + 16 * nnzb, mu, cfg.cg_tol, cg_max, ddelta, dinfo);
        else
            hipLaunchKernelGGL(k_pgo_cg, dim3(1), dim3(kCgThreads), lds_bytes, st, nb, drp, dci, out, ddslot,
                               out + 16 * nnzb, mu, cfg.cg_tol, cg_max, (double *)(dev + o_work), ddelta, dinfo,
                               lds_bytes > 0 ? 1 : 0);
        return hip_check(ctx, hipGetLastError(), "pgo cg launch");
    };

    std::vector<double> xh(4 * (size_t)N);
    int cur = 0;
    if ((rc = linearize(0, 0, nullptr, true))) return rc;
    double F = 0.0, F0 = 0.0;
    if (cfg.max_iter == 0) {
        if ((rc = read_info())) return rc;
        F = F0 = info[5];
    }
    double mu = cfg.lambda0, nu = 2.0;
    int it = 0, acc = 0, conv = 0, cg_total = 0;
    while (it < cfg.max_iter) {
        ++it;
        // the step and, before its size is known here, the linearisation at the
        // trial poses: one wait a step
        if ((rc = step(cur, mu)) || (rc = linearize(cur, cur ^ 1, ddelta, false)) || (rc = read_info())) return rc;
        F = info[5 + cur];
        if (it == 1) F0 = F;
        if (info[1] == 0.0) return fail(ctx, COVOX_EINVAL, "pgo: the damped system is not positive definite");
        cg_total += (int)info[0];
        if (info[4] < cfg.tol_step) {
            conv = 1;
            break;
        }
        const double Fn = info[5 + (cur ^ 1)], pred = info[2];
        const double rho = pred > 0.0 ? (F - Fn) / pred : -1.0;
        if (rho > 0.0) {
            F = Fn;
            cur ^= 1;
            ++acc;
            mu *= std::max(1.0 / 3.0, 1.0 - (2.0 * rho - 1.0) * (2.0 * rho - 1.0) * (2.0 * rho - 1.0));
            nu = 2.0;
        } else {
            mu *= nu;
            nu *= 2.0;
        }
    }
    if ((rc = hip_check(ctx, hipMemcpyAsync(xh.data(), dx[cur], sizeof(double) * 4 * N, hipMemcpyDeviceToHost, st),
                        "pgo poses")) ||
        (rc = hip_check(ctx, hipStreamSynchronize(st), "pgo sync")))
        return rc;
    memcpy(x, xh.data(), sizeof(double) * 4 * N);
    if (stats) {
        stats->iterations = it;
        stats->accepted = acc;
        stats->converged = conv;
        stats->cg_iterations = cg_total;
        stats->cost_init = F0;
        stats->cost_final = F;
    }
    return COVOX_OK;
}

}  // namespace covox
