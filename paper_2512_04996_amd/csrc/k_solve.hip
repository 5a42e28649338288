// k_solve.hip -- the closed-form rigid transform of Eq. 1 per pair, in
// float64, and the ICP iteration bookkeeping (Sec. II.A; stop rule of
// Sec. IV.A).  One block per pair reduces the moment partials that the
// search blocks wrote, adds the queries resolved by the exhaustive search in
// index order (both in a fixed order), then one lane forms the cross-covariance
// H = sum (p - pbar)(q - qbar)^T = sum p q^T - m pbar qbar^T, takes its SVD
// H = U S V^T by one-sided Jacobi, and sets R = V diag(1, 1, det(V U^T)) U^T,
// t = qbar - R pbar; when det H is clearly positive the same R is taken as
// the orthogonal polar factor of H^T by a few Newton steps instead.  When the second singular value is below 1e-12 times the
// first, the rotation is not determined and the previous pose is kept.
#include <math.h>

#include "search_dev.hpp"
#include "solve_dev.hpp"
#include "vicp_internal.hpp"

namespace vicp {

namespace {

constexpr int kReplayThreads = 256;              // threads that replay the global-search list
constexpr int kReplayWaves = kReplayThreads / kWave;
constexpr int kFbWindow = 32 * kReplayThreads;   // queries per pass over the global-search list
constexpr int kUnitBatch = 16;                   // fold-unit loads in flight per thread
constexpr int kSolveThreads = 704;               // kUnitSlices threads per fold-unit sum
static_assert((kMoments + 2) * kUnitSlices <= kSolveThreads && kSolveThreads % kWave == 0, "unit slices");

// Adds the moments of one correspondence (p, q about the centre c, squared
// distance d) to a[].
__device__ __forceinline__ void add_moments(double* a, float px, float py, float pz, float qx, float qy, float qz,
                                            float d, double c0, double c1, double c2)
{
    const double p[3] = {(double)px - c0, (double)py - c1, (double)pz - c2};
    const double q[3] = {(double)qx - c0, (double)qy - c1, (double)qz - c2};
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        a[r] += p[r];
        a[3 + r] += q[r];
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) a[6 + 3 * r + cc] += p[r] * q[cc];
    }
    a[15] += p[0] * p[0] + p[1] * p[1] + p[2] * p[2];
    a[16] += q[0] * q[0] + q[1] * q[1] + q[2] * q[2];
    a[17] += (double)d;
    a[18] += 1.0;
}

// One block per pair.  (1) The pair's groups (moment-major, stride
// nunits) are summed per moment and counter by kUnitSlices threads each, in
// a fixed order.  (2) Queries resolved by the exhaustive search, when any were
// listed: their list is in arbitrary order, so it
// is replayed in windows of kFbWindow source indices through an LDS bitmap;
// each thread adds the correspondences of its own 32 indices per window in
// index order, and a fixed-order block reduction adds them to (1).  (3) The
// solve of Eq. 1 and the iteration bookkeeping on one lane.
__global__ __launch_bounds__(kSolveThreads) void k_solve(
    const PairDev* __restrict__ pd, const int32_t* __restrict__ fold_begin, int32_t nunits,
    const double* __restrict__ fpart, const unsigned long long* __restrict__ fctr, PairState* __restrict__ st,
    int32_t* __restrict__ fb_count, const uint32_t* __restrict__ fb_list, const unsigned long long* __restrict__ fb_key,
    const float* __restrict__ px, const float* __restrict__ py, const float* __restrict__ pz,
    const float* __restrict__ qx, const float* __restrict__ qy, const float* __restrict__ qz,
    int32_t* __restrict__ flags, double* __restrict__ rmse_hist, int32_t* __restrict__ fb_hist,
    int32_t* __restrict__ deg_hist, unsigned long long* __restrict__ ctr_hist, int k, int K, int early_stop,
    double eps, int32_t* __restrict__ nn_idx, float* __restrict__ nn_d2)
{
    __shared__ double tot[kMoments];
    __shared__ unsigned long long ctot[2];
    __shared__ double red[kMoments][kReplayWaves];
    __shared__ uint32_t wbits[kFbWindow / 32];
    __shared__ uint32_t wslot[kFbWindow];
    const int pair = blockIdx.x;
    PairState& S = st[pair];
    const PairDev& P = pd[pair];
    const int done = S.done;
    // uniform; only where pairs can stop early, as it delays the loads below (a
    // run that stops after 20 of 50 steps 2.37 -> 2.24 ms)
    if (early_stop && done) return;
    // a single pair owns every group: its range needs no table load
    const bool one = gridDim.x == 1;
    const int32_t u0 = one ? 0 : fold_begin[pair], u1 = one ? nunits : fold_begin[pair + 1];
    const int32_t nfb = fb_count[pair];
    const int32_t nmiss = fb_count[gridDim.x + pair];   // every global search, resolved in place or listed
    const double prev = S.prev_rmse;
    // the current rotation, the start of the polar refinement: read by every
    // thread (uniform loads, all in flight together; a per-thread condition
    // made the compiler wait for each in turn), used by thread 0
    double Rp[9];
#pragma unroll
    for (int j = 0; j < 9; ++j) Rp[j] = S.Rt[j];
    // the pair's groups: kUnitSlices threads (half a wave) per sum each add one
    // slice's groups in order (kUnitBatch loads in flight), then the half wave
    // adds the slices
    {
        const int j = threadIdx.x / kUnitSlices, sl = threadIdx.x % kUnitSlices;
        const bool last = sl == kUnitSlices - 1;
        double sm = 0.0;
        if (j < kMoments) {
            const double* row = fpart + (int64_t)j * nunits;
            for (int32_t u = u0 + sl; u < u1; u += kUnitSlices * kUnitBatch) {
                double v[kUnitBatch];
#pragma unroll
                for (int i = 0; i < kUnitBatch; ++i) {
                    const int32_t ui = u + i * kUnitSlices;
                    v[i] = ui < u1 ? row[ui] : 0.0;
                }
#pragma unroll
                for (int i = 0; i < kUnitBatch; ++i) sm += v[i];
            }
        } else if (j < kMoments + 2) {
            const unsigned long long* row = fctr + (int64_t)(j - kMoments) * nunits;
            // counts below 2^53 are exact in float64, in any order
            for (int32_t u = u0 + sl; u < u1; u += kUnitSlices) sm += (double)row[u];
        }
        sm = half_sum_f64(sm);
        if (last && j < kMoments) tot[j] = sm;
        if (last && j >= kMoments && j < kMoments + 2) ctot[j - kMoments] = (unsigned long long)sm;
    }
    __syncthreads();
    // a pair without source points, done from the start: tested after the
    // fold, whose loads do not depend on it, so that the flag's latency
    // overlaps theirs (its groups' sums are never used)
    if (done) return;   // uniform over the block
    const double cen[3] = {P.cx, P.cy, P.cz};
    if (nfb > 0) {   // uniform over the block
        const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
        double acc[kMoments];
#pragma unroll
        for (int j = 0; j < kMoments; ++j) acc[j] = 0.0;
        for (int64_t w0 = 0; w0 < P.m; w0 += kFbWindow) {
            if (threadIdx.x < kReplayThreads) wbits[threadIdx.x] = 0u;
            __syncthreads();
            for (int32_t e = threadIdx.x; e < nfb; e += kSolveThreads) {
                const int64_t r = (int64_t)fb_list[P.p_base + e] - w0;
                if (r >= 0 && r < kFbWindow) {
                    atomicOr(&wbits[r >> 5], 1u << (r & 31));
                    wslot[r] = (uint32_t)e;
                }
            }
            __syncthreads();
            uint32_t bits = threadIdx.x < kReplayThreads ? wbits[threadIdx.x] : 0u;
            while (bits) {
                const int u = __ffs(bits) - 1;
                bits &= bits - 1u;
                const int r = 32 * (int)threadIdx.x + u;
                const unsigned long long key = fb_key[P.p_base + wslot[r]];
                const uint32_t j = (uint32_t)(key & 0xFFFFFFFFull);
                if (j >= (uint64_t)P.n) {   // unresolved global search (never expected)
                    atomicOr(&flags[pair], 2);
                    continue;
                }
                const int64_t gp = P.p_base + w0 + r, gq = P.q_base + j;
                const float d = __uint_as_float((uint32_t)(key >> 32));
                add_moments(acc, px[gp], py[gp], pz[gp], qx[gq], qy[gq], qz[gq], d, cen[0], cen[1], cen[2]);
                if (nn_idx) {   // the correspondences, when asked for
                    nn_idx[gp] = (int32_t)j;
                    nn_d2[gp] = d;
                }
            }
            __syncthreads();
        }
#pragma unroll
        for (int j = 0; j < kMoments; ++j) {
            const double sm = wave_sum_f64(acc[j]);
            if (lane == 0 && w < kReplayWaves) red[j][w] = sm;
        }
        __syncthreads();
        if (threadIdx.x < kMoments) {
            double sm = tot[threadIdx.x];
#pragma unroll
            for (int q = 0; q < kReplayWaves; ++q) sm += red[threadIdx.x][q];
            tot[threadIdx.x] = sm;
        }
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    double Rt[12];   // written by kabsch only when it succeeds
    const double m = tot[18];
    const double rmse = m > 0.0 ? sqrt(tot[17] / m) : 0.0;
    const bool ok = kabsch(tot, cen, Rt, Rp, S.rot_ok != 0);
    if (ok) {
        for (int j = 0; j < 12; ++j) {
            S.Rt[j] = Rt[j];
            S.Rtf[j] = (float)Rt[j];
        }
        S.rot_ok = 1;
    } else {
        S.degenerate += 1;
    }
    const int64_t h = (int64_t)pair * K + k;
    rmse_hist[h] = rmse;
    fb_hist[h] = nmiss;
    deg_hist[h] = ok ? 0 : 1;
    ctr_hist[2 * h] = ctot[0];
    ctr_hist[2 * h + 1] = ctot[1];
    fb_count[pair] = 0;
    fb_count[gridDim.x + pair] = 0;
    S.iters = k + 1;
    if (early_stop && k >= 1 && fabs(rmse - prev) < eps) S.done = 1;
    S.prev_rmse = rmse;
    S.misses = nmiss;
}

// Initial state: pose rounded to float32 for the search; pairs with no
// source points are done from the start; the global-search counts and the
// fault flags start at zero.
struct PoseBlob {
    double rt[12 * kInlinePairs];
};

__device__ __forceinline__ void set_state_one(const PairDev* __restrict__ pd, PairState* __restrict__ st, int p,
                                              const double* rt, int npairs, int32_t* __restrict__ fb_count,
                                              int32_t* __restrict__ flags)
{
    init_pair_state(st, p, rt, pd[p].m, npairs, fb_count, flags);
}

// The poses travel in the launch's arguments (up to kInlinePairs pairs).
__global__ void k_set_state_inline(const PairDev* __restrict__ pd, PairState* __restrict__ st, PoseBlob b,
                                   int npairs, int32_t* __restrict__ fb_count, int32_t* __restrict__ flags)
{
    const int p = threadIdx.x;
    if (p < npairs) set_state_one(pd, st, p, b.rt + 12 * p, npairs, fb_count, flags);
}

__global__ void k_set_state(const PairDev* __restrict__ pd, PairState* __restrict__ st, const double* __restrict__ rt64,
                            int npairs, int32_t* __restrict__ fb_count, int32_t* __restrict__ flags)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= npairs) return;
    set_state_one(pd, st, p, rt64 + 12 * p, npairs, fb_count, flags);
}

}  // namespace

void launch_solve(const PairDev* pd, int npairs, const int32_t* fold_begin, int32_t nunits, const double* fpart,
                  const unsigned long long* fctr, PairState* st, int32_t* fb_count, const uint32_t* fb_list,
                  const unsigned long long* fb_key, const float* px, const float* py, const float* pz,
                  const float* qx, const float* qy, const float* qz, int32_t* flags, double* rmse_hist,
                  int32_t* fb_hist, int32_t* deg_hist, unsigned long long* ctr_hist, int k, int K, int early_stop,
                  double eps, int32_t* nn_idx, float* nn_d2, hipStream_t s)
{
    if (npairs <= 0) return;
    launch_timed(k_solve, dim3(npairs), dim3(kSolveThreads), s, pd, fold_begin, nunits, fpart, fctr, st, fb_count,
                 fb_list, fb_key, px, py, pz, qx, qy, qz, flags, rmse_hist, fb_hist, deg_hist, ctr_hist, k, K,
                 early_stop, eps, nn_idx, nn_d2);
}

void launch_set_state_inline(const PairDev* pd, PairState* st, const double* host_rt, int npairs,
                             int32_t* fb_count, int32_t* flags, hipStream_t s)
{
    if (npairs <= 0 || npairs > kInlinePairs) return;
    PoseBlob b{};
    for (int i = 0; i < 12 * npairs; ++i) b.rt[i] = host_rt[i];
    hipLaunchKernelGGL(k_set_state_inline, dim3(1), dim3(64), 0, s, pd, st, b, npairs, fb_count, flags);
}

void launch_set_state(const PairDev* pd, PairState* st, const double* rt64, int npairs, int32_t* fb_count,
                      int32_t* flags, hipStream_t s)
{
    if (npairs <= 0) return;
    hipLaunchKernelGGL(k_set_state, dim3((npairs + 63) / 64), dim3(64), 0, s, pd, st, rt64, npairs, fb_count, flags);
}

// Flags pairs whose source holds NaN or Inf (bit 0 of PairState::status).
__global__ void k_check_finite(const PairDev* __restrict__ pd, const BlockJob* __restrict__ jobs,
                               const float* __restrict__ px, const float* __restrict__ py,
                               const float* __restrict__ pz, int32_t* __restrict__ flags)
{
    const BlockJob job = jobs[blockIdx.x];
    const PairDev& P = pd[job.pair];
    const int64_t i = (int64_t)job.start + threadIdx.x;
    if (i >= P.m) return;
    const int64_t g = P.p_base + i;
    if (!(isfinite(px[g]) && isfinite(py[g]) && isfinite(pz[g]))) atomicOr(&flags[job.pair], 1);
}

void launch_check_finite(const PairDev* pd, const BlockJob* jobs, int njobs, const float* px, const float* py,
                         const float* pz, int32_t* flags, hipStream_t s)
{
    if (njobs <= 0) return;
    hipLaunchKernelGGL(k_check_finite, dim3(njobs), dim3(256), 0, s, pd, jobs, px, py, pz, flags);
}

}  // namespace vicp
