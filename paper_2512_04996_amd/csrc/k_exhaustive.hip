// k_exhaustive.hip -- a registration's search with every query compared with
// every target (the exact comparator; Table 2's "Brute").
//
// Bound by the vector units: 6.5 instructions a pair (three subtractions, a
// product, two fused steps, half a three-way minimum).  So k_exhaustive keeps
// only the smallest distance in its inner loop, and notes once per kExChunk
// targets which chunk it came from; k_exhaustive_record looks the index up in
// that chunk (the same arithmetic, so the same bits).  A thread keeps Q
// queries in registers, so that a target read from LDS (a broadcast) serves
// 64 Q pairs.  Blocks split the targets too, until they fill the device
// (exhaustive_split); their partial minima, one 8-byte word per query and
// split, are merged by the record kernel: atomics into one word per query
// (as the listed queries' search does) would be a million of them at once.
//
// The sums: a record per wave of 64 queries in source order, folded and solved
// like any search's records.
//
// 35,000 queries over 40,000 targets: 171 us (8.2e12 pairs/s, two thirds of
// the vector units' 78 T lane instructions/s) and 14 for the records, against
// 52 + 1256 + 237 us for the listing, 128 blocks that merged by atomics and a
// replay of the list in one block; 20 steps 29.9 -> 3.9 ms.  Eight queries a
// thread measured 1.5 % slower, chunks of 64 1 %.
#include <math.h>

#include <algorithm>

#include "search_dev.hpp"
#include "vicp_internal.hpp"

namespace vicp {

namespace {

constexpr int kExThreads = 256;
constexpr int kExChunk = 32;     // targets between two looks at the running minimum
constexpr int kExTile = 512;     // targets staged in LDS at a time
constexpr int kExFrom = 16384;   // source points from which a thread keeps kExMany queries
constexpr int kExMany = 4;
static_assert(kExTile % kExChunk == 0, "whole chunks a tile");

template <int Q>
__global__ __launch_bounds__(kExThreads) void k_exhaustive(const PairDev* __restrict__ pd,
                                                           const PairState* __restrict__ st,
                                                           const float* __restrict__ px, const float* __restrict__ py,
                                                           const float* __restrict__ pz, const float* __restrict__ qx,
                                                           const float* __restrict__ qy, const float* __restrict__ qz,
                                                           uint2* __restrict__ part, int64_t stride, int splits)
{
    __shared__ float4 t4[3][kExTile / 4];
    const int pair = blockIdx.y;
    const PairDev& P = pd[pair];
    const PairState& S = st[pair];
    const int64_t chunk0 = (int64_t)(blockIdx.x / splits) * (kExThreads * Q);
    if (chunk0 >= P.m || S.done) return;   // uniform
    const int split = blockIdx.x % splits;
    const int64_t nch = (P.n + kExChunk - 1) / kExChunk;
    const int64_t per = (nch + splits - 1) / splits;
    const int64_t c0 = min(nch, per * split), c1 = min(nch, c0 + per);
    float sx[Q], sy[Q], sz[Q], bd[Q];
    uint32_t bc[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int64_t i = P.p_base + min(chunk0 + q * kExThreads + (int64_t)threadIdx.x, P.m - 1);
        transform(S.Rtf, px[i], py[i], pz[i], sx[q], sy[q], sz[q]);
        bd[q] = INFINITY;
        bc[q] = 0u;
    }
    const float* src[3] = {qx + P.q_base, qy + P.q_base, qz + P.q_base};
    for (int64_t c = c0; c < c1; c += kExTile / kExChunk) {
        const int64_t t0 = c * kExChunk;
        const int tn = (int)min((int64_t)kExTile, min(c1 * kExChunk, P.n) - t0);
        __syncthreads();
        // targets past the end: infinitely far
        for (int j = threadIdx.x; j < kExTile; j += kExThreads)
#pragma unroll
            for (int a = 0; a < 3; ++a) reinterpret_cast<float*>(t4[a])[j] = j < tn ? src[a][t0 + j] : INFINITY;
        __syncthreads();
        const int nc = (tn + kExChunk - 1) / kExChunk;
        for (int h = 0; h < nc; ++h) {
            float lo[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) lo[q] = INFINITY;
#pragma unroll
            for (int j = h * (kExChunk / 4); j < (h + 1) * (kExChunk / 4); ++j) {
                const float4 x = t4[0][j], y = t4[1][j], z = t4[2][j];
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const float d0 = dist2(sx[q], sy[q], sz[q], x.x, y.x, z.x);
                    const float d1 = dist2(sx[q], sy[q], sz[q], x.y, y.y, z.y);
                    const float d2 = dist2(sx[q], sy[q], sz[q], x.z, y.z, z.z);
                    const float d3 = dist2(sx[q], sy[q], sz[q], x.w, y.w, z.w);
                    lo[q] = fminf(fminf(lo[q], d0), d1);
                    lo[q] = fminf(fminf(lo[q], d2), d3);
                }
            }
            const uint32_t hc = (uint32_t)(c + h);
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                bc[q] = lo[q] < bd[q] ? hc : bc[q];
                bd[q] = fminf(bd[q], lo[q]);
            }
        }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int64_t i = chunk0 + q * kExThreads + threadIdx.x;
        if (i < P.m) part[(int64_t)split * stride + P.p_base + i] = make_uint2(__float_as_uint(bd[q]), bc[q]);
    }
}

// The nearest target of every query from its splits' minima (the lowest chunk
// among equal distances, then the lowest index), and the moment records.
__global__ __launch_bounds__(kExThreads) void k_exhaustive_record(
    const PairDev* __restrict__ pd, const BlockJob* __restrict__ jobs, const PairState* __restrict__ st,
    const float* __restrict__ px, const float* __restrict__ py, const float* __restrict__ pz,
    const float* __restrict__ qx, const float* __restrict__ qy, const float* __restrict__ qz,
    const uint2* __restrict__ part, int64_t stride, int splits, int32_t* __restrict__ nn_idx,
    float* __restrict__ nn_d2, int32_t* __restrict__ fb_miss, double* __restrict__ rec,
    unsigned long long* __restrict__ ctr)
{
    const BlockJob job = jobs[blockIdx.x];
    const PairDev& P = pd[job.pair];
    const PairState& S = st[job.pair];
    const int64_t i = (int64_t)job.start + threadIdx.x;
    const bool active = i < P.m && S.done == 0;
    const int64_t gp = P.p_base + min(i, P.m - 1);
    if (active && i == 0) fb_miss[job.pair] = (int32_t)P.m;
    float x = 0.0f, y = 0.0f, z = 0.0f, bx = 0.0f, by = 0.0f, bz = 0.0f, bd = INFINITY;
    if (active) {
        x = px[gp];
        y = py[gp];
        z = pz[gp];
        uint32_t bc = 0u;
        constexpr int kBatch = 8;
        for (int s = 0; s < splits; s += kBatch) {
            uint2 v[kBatch];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) v[b] = part[(int64_t)min(s + b, splits - 1) * stride + gp];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const float d = __uint_as_float(v[b].x);
                bc = d < bd ? v[b].y : bc;
                bd = fminf(bd, d);
            }
        }
        float sx, sy, sz;
        transform(S.Rtf, x, y, z, sx, sy, sz);
        // no finite distance: the first target, as the listed search has it
        const int64_t t0 = bd < INFINITY ? (int64_t)bc * kExChunk : 0;
        const int last = (int)min((int64_t)kExChunk, P.n - t0) - 1;
        const float *tx = qx + P.q_base + t0, *ty = qy + P.q_base + t0, *tz = qz + P.q_base + t0;
        int at = last + 1;
        for (int j = 0; j <= last && bd < INFINITY && at > last; j += kBatch) {
            float cx[kBatch], cy[kBatch], cz[kBatch];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const int jj = min(j + b, last);
                cx[b] = tx[jj];
                cy[b] = ty[jj];
                cz[b] = tz[jj];
            }
#pragma unroll
            for (int b = kBatch - 1; b >= 0; --b)
                if (dist2(sx, sy, sz, cx[b], cy[b], cz[b]) == bd) at = min(j + b, last);
        }
        const int j = at > last ? 0 : at;
        bx = tx[j];
        by = ty[j];
        bz = tz[j];
        if (nn_idx) {
            nn_idx[gp] = (int32_t)(t0 + j);
            nn_d2[gp] = bd;
        }
    }
    const int64_t r = (int64_t)blockIdx.x * (kExThreads / kWave) + threadIdx.x / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t n = (uint32_t)__popcll(__ballot(active));
    wave_record<1>(active, x, y, z, bx, by, bz, bd, P.cx, P.cy, P.cz,
                   [&](int j, double v) { rec[r * kMoments + j] = v; });
    if (lane == 0) rec[r * kMoments + kMoments - 1] = (double)n;
    if (lane < 3) ctr[r * 3 + lane] = lane == 2 ? n : 0ull;
}

int queries_per_thread(int64_t total) { return total >= kExFrom ? kExMany : 1; }

}  // namespace

int exhaustive_max_splits(int64_t total)
{
    return (int)std::max<int64_t>(1, std::min<int64_t>(kExMaxSplits, kExWords / std::max<int64_t>(total, 1)));
}

int exhaustive_split(const int64_t* m, const int64_t* n, int npairs, int64_t total, int max_splits)
{
    const int64_t qpb = (int64_t)kExThreads * queries_per_thread(total);
    int64_t blocks = 0, most = 0;
    for (int p = 0; p < npairs; ++p) {
        blocks += (m[p] + qpb - 1) / qpb;
        if (m[p] > 0) most = std::max(most, (n[p] + kExChunk - 1) / kExChunk);
    }
    int best = 1;
    int64_t cost = -1;
    for (int t = 1; t <= max_splits && t <= most; ++t) {
        const int64_t deep = std::max<int64_t>(kExDeep, (blocks * t + kExCus - 1) / kExCus);
        const int64_t c = deep * ((most + t - 1) / t + kExCost);
        if (cost < 0 || c < cost) {
            cost = c;
            best = t;
        }
    }
    return best;
}

void launch_exhaustive(const PairDev* pd, int npairs, int64_t most_m, int64_t total, const PairState* st,
                       const float* px, const float* py, const float* pz, const float* qx, const float* qy,
                       const float* qz, uint2* part, int splits, hipStream_t s)
{
    const int Q = queries_per_thread(total);
    const int64_t qpb = (int64_t)kExThreads * Q;
    const int64_t nb = (most_m + qpb - 1) / qpb * splits;
    if (nb <= 0 || npairs <= 0) return;
    const dim3 grid((uint32_t)nb, (uint32_t)npairs);
    if (Q == 1)
        launch_timed(k_exhaustive<1>, grid, dim3(kExThreads), s, pd, st, px, py, pz, qx, qy, qz, part, total, splits);
    else
        launch_timed(k_exhaustive<kExMany>, grid, dim3(kExThreads), s, pd, st, px, py, pz, qx, qy, qz, part, total,
                     splits);
}

void launch_exhaustive_record(const PairDev* pd, const BlockJob* jobs, int njobs, int64_t total, const PairState* st,
                              const float* px, const float* py, const float* pz, const float* qx, const float* qy,
                              const float* qz, const uint2* part, int splits, int32_t* nn_idx, float* nn_d2,
                              int32_t* fb_miss, double* rec, unsigned long long* ctr, hipStream_t s)
{
    if (njobs <= 0) return;
    hipLaunchKernelGGL(k_exhaustive_record, dim3(njobs), dim3(kExThreads), 0, s, pd, jobs, st, px, py, pz, qx, qy, qz,
                       part, total, splits, nn_idx, nn_d2, fb_miss, rec, ctr);
}

}  // namespace vicp
