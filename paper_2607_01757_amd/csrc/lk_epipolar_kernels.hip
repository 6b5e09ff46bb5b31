// Epipolar check after LK (the geometric verification of temporal
// correspondences, Sec. III-C): eight-point models from caller-drawn
// samples, scored by the point-to-epipolar-line distance in pixels.
//
//   k_epi_hypotheses  64 hypotheses per workgroup.  The first wavefront
//                     solves them, one per lane: the 8 x 9 system on the
//                     normalized plane is reduced by Gaussian elimination
//                     with complete pivoting (binary64) in a lane-private
//                     LDS slab (entry (r, c) of lane l at [(9 r + c) 64 + l],
//                     so the lanes of a wavefront hit distinct banks) and the
//                     null vector is mapped to pixel space.  Four wavefronts
//                     then score the 64 models, a quarter of the
//                     correspondences each; these are staged in LDS, 512 at a
//                     time, and every lane reads each one from there (one
//                     broadcast read, no memory round trip per
//                     correspondence);
//   k_epi_best        one wavefront per set: the best hypothesis (most
//                     inliers, lowest index on ties), its model solved again
//                     by the whole wavefront, an entry of the system per lane
//                     (the same operations on every entry, so the same bits),
//                     and its inlier mask.
//
// Both are bound by chains of dependent binary64 operations: the slab leaves
// room for three workgroups in a CU and 64 sets of 512 hypotheses make two, so
// a chain has a SIMD to itself.  At that size (256 correspondences) scoring by
// the solving wavefront alone took 37 us in all, split in four 26 us; the best
// model solved by one lane took 20 us, by the wavefront 14 us.
//
// Neither function contracts multiply-adds, so the count of a hypothesis in
// the first kernel and its mask in the second come from identical arithmetic.
#include "lk_internal.h"

namespace lkmi {
namespace {

constexpr int kEpiLanes = 64;
constexpr int kEpiWaves = 4;               // wavefronts that score a workgroup's 64 models
constexpr int kEpiChunk = 512;             // correspondences staged in LDS at a time
constexpr double kEpiRankTol = 1e-10;

__device__ __forceinline__ double &slab(double *sa, int r, int c, int lane)
{
    return sa[(9 * r + c) * kEpiLanes + lane];
}

// The samples s[0..7] of a set of n correspondences, or false when one is out of
// range or two are equal.
__device__ __forceinline__ bool epi_samples(const int32_t *s, int n, int (&idx)[8])
{
    bool bad = false;
#pragma unroll
    for (int a = 0; a < 8; ++a) {
        idx[a] = s[a];
        bad |= idx[a] < 0 || idx[a] >= n;
    }
#pragma unroll
    for (int a = 0; a < 8; ++a)
#pragma unroll
        for (int b = a + 1; b < 8; ++b) bad |= idx[a] == idx[b];
    return !bad;
}

// Row x_q (x) x_p of correspondence i on the normalized plane.
__device__ __forceinline__ void epi_row(const EpiJob &J, int i, double ifx, double ify, double (&a)[9])
{
#pragma clang fp contract(off)
    const double xp = ((double)J.p[2 * i] - J.cx) * ifx, yp = ((double)J.p[2 * i + 1] - J.cy) * ify;
    const double xq = ((double)J.q[2 * i] - J.cx) * ifx, yq = ((double)J.q[2 * i + 1] - J.cy) * ify;
    a[0] = xq * xp;
    a[1] = xq * yp;
    a[2] = xq;
    a[3] = yq * xp;
    a[4] = yq * yp;
    a[5] = yq;
    a[6] = xp;
    a[7] = yp;
    a[8] = 1.0;
}

// F = K^-T E K^-1 with unit Frobenius norm, of the null vector e.
__device__ __forceinline__ void epi_pixel_model(const EpiJob &J, double ifx, double ify, const double (&e)[9], double (&F)[9])
{
#pragma clang fp contract(off)
    const double ax = -J.cx * ifx, ay = -J.cy * ify;
    double m[9];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        m[3 * i] = e[3 * i] * ifx;
        m[3 * i + 1] = e[3 * i + 1] * ify;
        m[3 * i + 2] = e[3 * i] * ax + e[3 * i + 1] * ay + e[3 * i + 2];
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        F[j] = ifx * m[j];
        F[3 + j] = ify * m[3 + j];
        F[6 + j] = ax * m[j] + ay * m[3 + j] + m[6 + j];
    }
    double nn = 0.0;
#pragma unroll
    for (int j = 0; j < 9; ++j) nn = nn + F[j] * F[j];
    const double inv = 1.0 / sqrt(nn);
#pragma unroll
    for (int j = 0; j < 9; ++j) F[j] = F[j] * inv;
}

// Pixel-space F (unit Frobenius norm) of the samples s[0..7] of job J, or
// false when the samples are invalid or the system has numerical rank < 8.
__device__ bool epi_model(const EpiJob &J, const int32_t *s, double *sa, int *scol, int lane, double (&F)[9])
{
#pragma clang fp contract(off)
    int idx[8];
    if (!epi_samples(s, J.n, idx)) return false;
    const double ifx = 1.0 / J.fx, ify = 1.0 / J.fy;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        double a[9];
        epi_row(J, idx[r], ifx, ify, a);
#pragma unroll
        for (int c = 0; c < 9; ++c) slab(sa, r, c, lane) = a[c];
    }
#pragma unroll
    for (int c = 0; c < 9; ++c) scol[c * kEpiLanes + lane] = c;
    double amax = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        // complete pivoting: the largest entry of the remaining block
        double best = -1.0;
        int br = k, bc = k;
#pragma unroll
        for (int r = k; r < 8; ++r)
#pragma unroll
            for (int c = k; c < 9; ++c) {
                const double v = fabs(slab(sa, r, c, lane));
                if (v > best) { best = v; br = r; bc = c; }
            }
        if (k == 0) amax = best;
        if (!(best > kEpiRankTol * amax)) return false;     // also catches NaN
        if (br != k)
#pragma unroll
            for (int c = 0; c < 9; ++c) {
                const double t = slab(sa, k, c, lane);
                slab(sa, k, c, lane) = slab(sa, br, c, lane);
                slab(sa, br, c, lane) = t;
            }
        if (bc != k) {
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const double t = slab(sa, r, k, lane);
                slab(sa, r, k, lane) = slab(sa, r, bc, lane);
                slab(sa, r, bc, lane) = t;
            }
            const int t = scol[k * kEpiLanes + lane];
            scol[k * kEpiLanes + lane] = scol[bc * kEpiLanes + lane];
            scol[bc * kEpiLanes + lane] = t;
        }
        const double piv = slab(sa, k, k, lane);
#pragma unroll
        for (int r = k + 1; r < 8; ++r) {
            const double f = slab(sa, r, k, lane) / piv;
#pragma unroll
            for (int c = k + 1; c < 9; ++c) slab(sa, r, c, lane) = slab(sa, r, c, lane) - f * slab(sa, k, c, lane);
        }
    }
    // null vector in the permuted columns (free column last), back substitution
    double y[9];
    y[8] = 1.0;
#pragma unroll
    for (int k = 7; k >= 0; --k) {
        double acc = 0.0;
#pragma unroll
        for (int c = k + 1; c < 9; ++c) acc = acc + slab(sa, k, c, lane) * y[c];
        y[k] = -acc / slab(sa, k, k, lane);
    }
    // undo the column permutation (through row 0 of the slab)
#pragma unroll
    for (int c = 0; c < 9; ++c) slab(sa, 0, scol[c * kEpiLanes + lane], lane) = y[c];
    double e[9];
#pragma unroll
    for (int c = 0; c < 9; ++c) e[c] = slab(sa, 0, c, lane);
    epi_pixel_model(J, ifx, ify, e, F);
    return true;
}

// The same by the 64 lanes of a workgroup of one wavefront, for one hypothesis:
// a lane per entry of the system (sa: its 72 entries, scol: its 9 columns).
// Every lane returns the model.
__device__ bool epi_model_wave(const EpiJob &J, const int32_t *s, double *sa, int *scol, int lane, double (&F)[9])
{
#pragma clang fp contract(off)
    int idx[8];
    if (!epi_samples(s, J.n, idx)) return false;               // (uniform, as every return here)
    const double ifx = 1.0 / J.fx, ify = 1.0 / J.fy;
    if (lane < 8) {
        double a[9];
        epi_row(J, s[lane], ifx, ify, a);
#pragma unroll
        for (int c = 0; c < 9; ++c) sa[9 * lane + c] = a[c];
    }
    if (lane < 9) scol[lane] = lane;
    __syncthreads();
    double amax = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        // the largest entry of the remaining block, the first in row order of
        // equal ones
        const int nc = 9 - k, ne = (8 - k) * nc;
        double best = -1.0;
        int at = 0;
#pragma unroll
        for (int e = lane; e < ne; e += 64) {
            const double v = fabs(sa[9 * (k + e / nc) + k + e % nc]);
            if (v > best) { best = v; at = e; }
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            const double v = __shfl_xor(best, o, 64);
            const int w = __shfl_xor(at, o, 64);
            if (v > best || (v == best && w < at)) { best = v; at = w; }
        }
        if (k == 0) amax = best;
        if (!(best > kEpiRankTol * amax)) return false;         // also catches NaN
        const int br = k + at / nc, bc = k + at % nc;
        if (br != k && lane < 9) {
            const double t = sa[9 * k + lane];
            sa[9 * k + lane] = sa[9 * br + lane];
            sa[9 * br + lane] = t;
        }
        __syncthreads();
        if (bc != k) {
            if (lane < 8) {
                const double t = sa[9 * lane + k];
                sa[9 * lane + k] = sa[9 * lane + bc];
                sa[9 * lane + bc] = t;
            }
            if (lane == 8) {
                const int t = scol[k];
                scol[k] = scol[bc];
                scol[bc] = t;
            }
        }
        __syncthreads();
        if (k < 7) {
            const int n = 8 - k;                               // columns right of the pivot
            const int r = k + 1 + lane / n, c = k + 1 + lane % n;
            if (r < 8) {
                const double f = sa[9 * r + k] / sa[9 * k + k];
                sa[9 * r + c] = sa[9 * r + c] - f * sa[9 * k + c];
            }
            __syncthreads();
        }
    }
    double y[9];
    y[8] = 1.0;
#pragma unroll
    for (int k = 7; k >= 0; --k) {
        double acc = 0.0;
#pragma unroll
        for (int c = k + 1; c < 9; ++c) acc = acc + sa[9 * k + c] * y[c];
        y[k] = -acc / sa[9 * k + k];
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 9; ++c)
        if (lane == c) sa[scol[c]] = y[c];
    __syncthreads();
    double e[9];
#pragma unroll
    for (int c = 0; c < 9; ++c) e[c] = sa[c];
    epi_pixel_model(J, ifx, ify, e, F);
    return true;
}

// Correspondence (p, q) is an inlier of F: the distance of q to the line
// F (p, 1) is at most the threshold (thr2 = threshold^2).
__device__ __forceinline__ bool epi_inlier(const double (&F)[9], float px, float py, float qx, float qy, double thr2)
{
#pragma clang fp contract(off)
    const double x = px, y = py;
    const double l0 = F[0] * x + F[1] * y + F[2];
    const double l1 = F[3] * x + F[4] * y + F[5];
    const double l2 = F[6] * x + F[7] * y + F[8];
    const double num = (double)qx * l0 + (double)qy * l1 + l2;
    const double den = l0 * l0 + l1 * l1;
    return (den > 0.0) & (num * num <= thr2 * den);
}

// Three wavefronts a SIMD: the slab leaves room for three workgroups in a CU,
// one wavefront of each to a SIMD, and at 169 registers only two fitted (768
// workgroups, 8 correspondences 75 us a call against 60; 16384 workgroups 1010
// against 882).
__global__ __launch_bounds__(kEpiLanes * kEpiWaves) __attribute__((amdgpu_waves_per_eu(3)))
void k_epi_hypotheses(const EpiJob *__restrict__ jobs, const int32_t *__restrict__ wg_job, double thr2)
{
    __shared__ double sa[72 * kEpiLanes];
    __shared__ int scol[9 * kEpiLanes];
    __shared__ float4 spq[kEpiChunk];
    __shared__ int s_cnt[kEpiWaves][kEpiLanes];
    const int lane = threadIdx.x & (kEpiLanes - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kEpiLanes);
    const EpiJob &J = jobs[__builtin_amdgcn_readfirstlane(wg_job[blockIdx.x])];
    const int n = __builtin_amdgcn_readfirstlane(J.n);
    const int k = (blockIdx.x - J.wg_begin) * kEpiLanes + lane;
    const bool live = k < J.h;
    double F[9];
    if (wv == 0) {
        // (a lane of its own for the solve: the scoring's addresses formed of `lane`
        // would be held through it)
        int ln = lane;
        asm("" : "+v"(ln));
        const bool solved = live && epi_model(J, J.samples + 8 * k, sa, scol, ln, F);
        if (solved)
#pragma unroll
            for (int j = 0; j < 9; ++j) slab(sa, 0, j, lane) = F[j];
        s_cnt[0][lane] = solved;
    }
    __syncthreads();
    // every lane stays to the end: the whole workgroup stages the correspondences
    const bool ok = s_cnt[0][lane] != 0;
#pragma unroll
    for (int j = 0; j < 9; ++j) F[j] = ok ? slab(sa, 0, j, lane) : 0.0;
    int cnt = 0;
    for (int i0 = 0; i0 < n; i0 += kEpiChunk) {
        const int m = min(kEpiChunk, n - i0);
        __syncthreads();                       // every lane has read the previous chunk (and its model)
        for (int i = threadIdx.x; i < m; i += kEpiLanes * kEpiWaves) {
            const int g = i0 + i;
            spq[i] = make_float4(J.p[2 * g], J.p[2 * g + 1], J.q[2 * g], J.q[2 * g + 1]);
        }
        __syncthreads();
        if (ok) {
#pragma unroll 4
            for (int i = wv; i < m; i += kEpiWaves) {
                const float4 v = spq[i];
                cnt += epi_inlier(F, v.x, v.y, v.z, v.w, thr2);
            }
        }
    }
    __syncthreads();                           // s_cnt[0] is read
    s_cnt[wv][lane] = cnt;
    __syncthreads();
    if (wv == 0 && live) {
#pragma unroll
        for (int w = 1; w < kEpiWaves; ++w) cnt += s_cnt[w][lane];
        J.counts[k] = ok ? cnt : -1;
    }
}

__global__ __launch_bounds__(kEpiLanes) void k_epi_best(const EpiJob *__restrict__ jobs, double thr2)
{
    __shared__ double sa[72];
    __shared__ int scol[9];
    const int lane = threadIdx.x;
    const EpiJob &J = jobs[blockIdx.x];
    // most inliers, then the lowest index: key = (count + 1) << 32 | ~index
    unsigned long long key = 0;
    for (int k = lane; k < J.h; k += kEpiLanes) {
        const int c = J.counts[k];
        if (c >= 0) {
            const unsigned long long v = ((unsigned long long)(c + 1) << 32) | (0xFFFFFFFFu - (uint32_t)k);
            key = v > key ? v : key;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long v = __shfl_xor(key, o, kEpiLanes);
        key = v > key ? v : key;
    }
    const int bk = key ? (int)(0xFFFFFFFFu - (uint32_t)key) : -1;
    const int bc = key ? (int)(key >> 32) - 1 : 0;
    double F[9];
    const bool ok = bk >= 0 && epi_model_wave(J, J.samples + 8 * bk, sa, scol, lane, F);
#pragma unroll
    for (int j = 0; j < 9; ++j) F[j] = ok ? F[j] : 0.0;
    for (int i = lane; i < J.n; i += kEpiLanes)
        J.inliers[i] = ok && epi_inlier(F, J.p[2 * i], J.p[2 * i + 1], J.q[2 * i], J.q[2 * i + 1], thr2) ? 1 : 0;
    if (lane == 0) {
        J.best[0] = bk;
        J.best[1] = bc;
    }
    if (J.model)
#pragma unroll
        for (int j = 0; j < 9; ++j)
            if (lane == j) J.model[j] = F[j];
}

}  // namespace

hipError_t launch_epipolar(const EpiJob *d_jobs, const int32_t *d_wg_job, int n_jobs, int total_wgs, double threshold,
                           hipStream_t s)
{
    const double thr2 = threshold * threshold;
    if (total_wgs > 0) {
        hipLaunchKernelGGL(k_epi_hypotheses, dim3(total_wgs), dim3(kEpiLanes * kEpiWaves), 0, s, d_jobs, d_wg_job, thr2);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (n_jobs > 0) hipLaunchKernelGGL(k_epi_best, dim3(n_jobs), dim3(kEpiLanes), 0, s, d_jobs, thr2);
    return hipGetLastError();
}

}  // namespace lkmi
