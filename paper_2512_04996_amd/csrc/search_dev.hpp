// search_dev.hpp -- device code shared by the search kernels (k_nns.hip) and
// the resident registration loop (k_loop.hip): candidate comparison, the exact
// global search, and the moment record of a search wave.
#pragma once

#include <math.h>

#include "vicp_internal.hpp"

namespace vicp {

namespace {

constexpr int kWave = 64;

__device__ __forceinline__ float dist2(float sx, float sy, float sz, float qx, float qy, float qz)
{
    const float dx = sx - qx, dy = sy - qy, dz = sz - qz;
    return __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
}

// The value of lane (this lane xor d): a DPP quad permutation for d = 1, 2
// (a VALU move), an LDS permute otherwise.
__device__ __forceinline__ uint32_t xor_lanes(uint32_t x, int d)
{
    if (d == 1) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, true);   // quad_perm 1,0,3,2
    if (d == 2) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, true);   // quad_perm 2,3,0,1
    return (uint32_t)__shfl_xor((int)x, d, kWave);
}

__device__ __forceinline__ float xor_lanes(float x, int d) { return __uint_as_float(xor_lanes(__float_as_uint(x), d)); }

// Selects, not branches: a branch lets the compiler sink the index load into
// the taken path and then wait for every load in flight.  kTies: candidates
// come in no particular order, so equal distances compare indices.
template <bool kTies>
__device__ __forceinline__ void consider(const float4& q, float sx, float sy, float sz, float& bd, uint32_t& bj)
{
    const float d = dist2(sx, sy, sz, q.x, q.y, q.z);
    const bool better = d < bd || (kTies && d == bd && __float_as_uint(q.w) < bj);
    bd = better ? d : bd;
    bj = better ? __float_as_uint(q.w) : bj;
}

// The same, keeping the candidate's position in the segment instead of its
// index (positions ascend with indices in a segment), so that a lane carries
// two values per candidate instead of five; the winner's coordinates are
// read once at the end.
__device__ __forceinline__ void consider_pos(const float4& q, uint32_t pos, float sx, float sy, float sz, float& bd,
                                             uint32_t& bk)
{
    const float d = dist2(sx, sy, sz, q.x, q.y, q.z);
    const bool better = d < bd;
    bd = better ? d : bd;
    bk = better ? pos : bk;
}

// Crowded voxels (8 lanes a query): the wave takes its queries' voxels one
// after the other, and every lane scans a 64th of a voxel's candidates for all
// the queries that look there.  So a loaded candidate serves up to eight
// distances, a load of the wave is one contiguous kilobyte, and the wave's time
// is the sum of its queries' candidates, not eight times the most of them.  The
// queries are in scalar registers.  The vector units bound it, so of each four
// candidates (64 apart) only the least distance is kept and compared; the eight
// lanes of a query look its last four up at the end.  Gives every lane of a
// query the least (distance, position); false, with nothing given, when two
// lanes held equal distances, whose order this does not know.  200,000 queries
// of 1470 candidates on average: 93 us query by query, 69 with every candidate
// compared, 52 so.  From 64 candidates every lane has one.
constexpr uint32_t kCrowd = 64;
__device__ __forceinline__ bool crowd_scan(const float4* __restrict__ qs4, int64_t start, uint32_t c, float sx, float sy,
                                           float sz, int lane, float& bd, uint32_t& bk)
{
    constexpr int Q = 8, N = 4;
    float x[Q], y[Q], z[Q], d[Q];
    uint32_t k[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        x[q] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sx), 8 * q));
        y[q] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sy), 8 * q));
        z[q] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sz), 8 * q));
        d[q] = INFINITY;
        k[q] = 0u;
    }
    unsigned long long todo = __ballot(c > 0u);
    while (todo) {   // uniform
        const int l = __ffsll((long long)todo) - 1;
        const uint32_t lc = (uint32_t)__builtin_amdgcn_readlane((int)c, l);
        const int64_t ls = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(start >> 32), l) << 32) |
                                     (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)start, l));
        const unsigned long long here = __ballot(c == lc && start == ls);
        todo &= ~here;
        const float4* seg = qs4 + ls;
        for (uint32_t k0 = 0; k0 < lc; k0 += N * kWave) {
            const uint32_t pos = k0 + (uint32_t)lane;
            float4 a[N];
#pragma unroll
            for (int n = 0; n < N; ++n) a[n] = seg[min(pos + (uint32_t)(n * kWave), lc - 1u)];
            // past the end: a coordinate that is infinitely far
            if (k0 + N * kWave > lc)
#pragma unroll
                for (int n = 0; n < N; ++n) a[n].x = pos + (uint32_t)(n * kWave) < lc ? a[n].x : INFINITY;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                if (!((here >> (8 * q)) & 1ull)) continue;
                float e[N];
#pragma unroll
                for (int n = 0; n < N; ++n) e[n] = dist2(x[q], y[q], z[q], a[n].x, a[n].y, a[n].z);
                const float lo = fminf(fminf(e[0], e[1]), fminf(e[2], e[3]));
                k[q] = lo < d[q] ? pos : k[q];
                d[q] = fminf(d[q], lo);
            }
        }
    }
    bool tie = false;
    const auto least = [&](float& ad, uint32_t& ak, float od, uint32_t ok) {
        tie |= od == ad && ok != ak && ad < INFINITY;
        ak = od < ad ? ok : ak;
        ad = fminf(ad, od);
    };
    // lanes 32 apart, then 16, then 8, share out the queries (lane l keeps query
    // l / 8), and a query's eight lanes combine
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const auto sd = __builtin_amdgcn_permlane32_swap(__float_as_uint(d[q]), __float_as_uint(d[q + 4]), false, false);
        const auto sk = __builtin_amdgcn_permlane32_swap(k[q], k[q + 4], false, false);
        d[q] = __uint_as_float(sd[0]);
        k[q] = sk[0];
        least(d[q], k[q], __uint_as_float(sd[1]), sk[1]);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const auto sd = __builtin_amdgcn_permlane16_swap(__float_as_uint(d[q]), __float_as_uint(d[q + 2]), false, false);
        const auto sk = __builtin_amdgcn_permlane16_swap(k[q], k[q + 2], false, false);
        d[q] = __uint_as_float(sd[0]);
        k[q] = sk[0];
        least(d[q], k[q], __uint_as_float(sd[1]), sk[1]);
    }
    const bool odd = (lane & 8) != 0;
    float wd = odd ? d[1] : d[0];
    uint32_t wk = odd ? k[1] : k[0];
    const float od = odd ? d[0] : d[1];
    const uint32_t ok = odd ? k[0] : k[1];
    // row_ror:8 (within 16 lanes): the value of lane xor 8
    least(wd, wk, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(od), 0x128, 0xF, 0xF, true)),
          (uint32_t)__builtin_amdgcn_update_dpp(0, (int)ok, 0x128, 0xF, 0xF, true));
#pragma unroll
    for (int i = 1; i < 8; i <<= 1) least(wd, wk, xor_lanes(wd, i), xor_lanes(wk, i));
    if (__ballot(tie)) return false;
    // the four candidates of the least distance: the first that has it
    const uint32_t at = wk + (uint32_t)((lane & (N - 1)) * kWave);
    bool has = false;
    if (at < c) {
        const float4 w = qs4[start + at];
        has = dist2(sx, sy, sz, w.x, w.y, w.z) == wd;
    }
    const uint32_t which = (uint32_t)(__ballot(has) >> (lane & ~7)) & ((1u << N) - 1u);
    bd = wd;
    bk = wk + (uint32_t)((which ? __ffs(which) - 1 : 0) * kWave);
    return true;
}

// Whether a wave's candidates are many enough for crowd_scan.
__device__ __forceinline__ bool crowded(uint32_t c) { return __ballot(c >= kCrowd) != 0ull; }

// consider(), also keeping the best candidate's coordinates.
template <bool kTies>
__device__ __forceinline__ void consider(const float4& q, float sx, float sy, float sz, float& bd, uint32_t& bj,
                                         float& bx, float& by, float& bz)
{
    const float d = dist2(sx, sy, sz, q.x, q.y, q.z);
    const bool better = d < bd || (kTies && d == bd && __float_as_uint(q.w) < bj);
    bd = better ? d : bd;
    bj = better ? __float_as_uint(q.w) : bj;
    bx = better ? q.x : bx;
    by = better ? q.y : by;
    bz = better ? q.z : bz;
}

// Exact global search on the occupancy pyramid.  A query whose voxel is empty
// and undilated, or outside the grid, takes the exact minimum of (d, j) over
// all n targets (Alg. 4's global search).  One wave resolves one query: the
// pyramid is a 64-ary tree (4 x 4 x 4 cells per cell above), so a lane holds
// one child of the current node, its occupied flag and a lower bound on the
// squared distance of any target in it; the wave takes the children nearest
// first and drops every child whose bound is above the best distance found.
// A query within reach of the surface first reads one cube of voxels around
// its own (clamped into the grid), which settles most misses in two rounds of
// loads.  The tree starts in the 16^3-voxel node around that voxel and climbs
// only while a target outside the node could still win; a far query descends
// from the top.  Level-1 cells (bricks of 64 voxels) are taken kN at a time.
// Voxels are read as rows along x, whose points are consecutive: two offsets
// give a whole row's.  Where a lane would scan more than kSerialPoints of them
// (crowded voxels), the first cube is dropped for the bricks, and a brick's
// voxels are taken nearest first, each scanned by the whole wave, until none
// left can hold a nearer target.
//
// Cells, and the grid box, are widened by a margin for the float32 rounding
// of the voxel assignment (floor((q - o) * inv)), so a target assigned to a
// voxel may lie slightly outside it; a bound must exceed the best distance
// by a factor 1 / (1 - 1e-4), far above the rounding of the float32
// distance, so a dropped target can neither win nor tie.  All 64 lanes call
// it with the same point; every lane gets the result.  False when the query
// is not finite or no finite distance was found, and with kCrowdBudget also once
// the budget of crowded voxels' points is used up (budget 0): it then goes to
// the exhaustive search.
//
// What bounds it: the latency of its dependent loads (flags, offsets,
// points).  Voxel cubes growing around the query, its former form, read
// 9^3 to 17^3 directory entries per miss and sent what lay farther than
// eight voxels to the exhaustive search.  A registration of two scans that
// overlap in part (140k / 120k points, 10 to 30% misses, 30 iterations):
// 88.3 ms before, 28.7 ms; the loss on 16 x 40k pairs (3.5% misses): 473 and
// 393 us; a 2k sphere with 2% misses, 20 iterations: 568 and 479 us.  Reading
// directory entries voxel by voxel instead of offsets row by row: 52.9 ms on
// the first, 466 and 578 us on the others.  Crowded voxels (a room of 200,000
// points on a 16^3 grid) scanned row by row, a 9^3 cube first: 10 steps with 860
// misses inside the grid took 8.8 ms, nearest voxel first 2.2 (cubes with a limit
// and the exhaustive search: 3.9); with 9,000 queries in overflowed blocks of
// the direct layout 20 to 30 ms, now 4.3 (9.3).
constexpr float kBoundSlack = 1.0f - 1e-4f;
constexpr uint32_t kSerialPoints = 96;   // points a lane scans alone; above that the wave scans voxel by voxel
constexpr uint32_t kSerialCost = 2048;   // what a round of over a quarter of them costs a small budget: 8 rounds of loads
constexpr int kN = 2;                    // rows per lane and round: of a cube, or of as many bricks
constexpr int kLoads = 4;                // point loads in flight per lane
constexpr int kCubeMin = 2;              // the first cube's smallest radius (registration): 5^3 voxels
constexpr int kCubeMinNN = 4;            // in the correspondence search, whose misses lie farther: 9^3 voxels
constexpr int kCubeMax = 4;

struct TreeBox {
    float s[3], o[3], mg[3], vox;
    int D[3];
};

// Lower bound on the squared distance from the query to any target in the
// cell (x, y, z) of level l.
__device__ __forceinline__ float cell_bound(const TreeBox& b, int l, int x, int y, int z)
{
    const uint32_t c[3] = {(uint32_t)x, (uint32_t)y, (uint32_t)z};   // (c + 1) 4^l < 2^32: D + 4^l < 2^31 + 2^30
    float lb = 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float lo = b.o[a] + (float)(c[a] << (2 * l)) * b.vox - b.mg[a];
        const float hi = b.o[a] + (float)min((c[a] + 1u) << (2 * l), (uint32_t)b.D[a]) * b.vox + b.mg[a];
        const float g = b.s[a] < lo ? lo - b.s[a] : (b.s[a] > hi ? b.s[a] - hi : 0.0f);
        lb += g * g;
    }
    return lb;
}

// A lower bound on the squared distance to the voxels [x0, x1) of row (y, z).
__device__ __forceinline__ float row_bound(const TreeBox& b, int x0, int x1, int y, int z)
{
    const float l[3] = {(float)x0, (float)y, (float)z}, h[3] = {(float)x1, (float)y + 1.0f, (float)z + 1.0f};
    float lb = 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float lo = b.o[a] + l[a] * b.vox - b.mg[a], hi = b.o[a] + h[a] * b.vox + b.mg[a];
        const float g = b.s[a] < lo ? lo - b.s[a] : (b.s[a] > hi ? b.s[a] - hi : 0.0f);
        lb += g * g;
    }
    return lb;
}

__device__ __forceinline__ TreeBox tree_box(const PairDev& P, float sx, float sy, float sz)
{
    TreeBox b;
    b.s[0] = sx, b.s[1] = sy, b.s[2] = sz;
    b.o[0] = P.ox, b.o[1] = P.oy, b.o[2] = P.oz;
    b.D[0] = P.Dx, b.D[1] = P.Dy, b.D[2] = P.Dz;
    b.vox = 1.0f / P.inv;
    // 1e-5 of the coordinates' magnitude and 1e-3 of a voxel: far above the
    // float32 rounding of the assignment and of the bounds' arithmetic
#pragma unroll
    for (int a = 0; a < 3; ++a) b.mg[a] = 1e-5f * (fabsf(b.o[a]) + ((float)b.D[a] + 1.0f) * b.vox) + 1e-3f * b.vox;
    return b;
}

// The points of the voxels [x0, x1) of row (y, z) as (first slot in qs4,
// number): consecutive voxels' segments follow each other, and every voxel
// before g has two header words in off[g].
__device__ __forceinline__ uint2 row_run(const PairDev& P, const TreeBox& b, const uint32_t* __restrict__ off, int x0,
                                         int x1, int y, int z)
{
    const int64_t g0 = P.v_base + x0 + (int64_t)b.D[0] * (y + (int64_t)b.D[1] * z), g1 = g0 + (x1 - x0);
    const uint32_t a0 = off[g0], a1 = off[g1];
    return make_uint2(a0 - 2u * (uint32_t)g0, a1 - a0 - 2u * (uint32_t)(x1 - x0));
}

// A search's best so far: the lane's own, and the wave's least distance.
struct TreeBest {
    float d, x, y, z, wave;
    uint32_t j;
    __device__ __forceinline__ void take(const float4& q, float sx, float sy, float sz)
    {
        const float e = dist2(sx, sy, sz, q.x, q.y, q.z);
        const uint32_t i = __float_as_uint(q.w);
        const bool better = e < d || (e == d && i < j);
        d = better ? e : d;
        j = better ? i : j;
        x = better ? q.x : x;
        y = better ? q.y : y;
        z = better ? q.z : z;
    }
    // Takes `points` from the budget; once that is used up the best is nearer
    // than any bound, so that the search ends by its own tests.
    __device__ __forceinline__ void spend(uint32_t& budget, uint32_t points)
    {
        budget -= min(points, budget);
        d = budget ? d : -1.0f;
        wave = budget ? wave : -1.0f;
    }
    // distances are >= 0: their bits order as the values do (and that of -1, in
    // all lanes, is itself)
    __device__ __forceinline__ void combine() { wave = __uint_as_float(wave_min_dpp(__float_as_uint(d))); }
};

// The voxels of a brick (of which (x0, y0, z0) is the first) nearest first, each
// scanned by the whole wave, with its row where the row is one round of loads.
// kGiveUp: within the budget.
template <bool kGiveUp>
__device__ __forceinline__ void crowd_brick(const PairDev& P, const TreeBox& b, const uint32_t* __restrict__ off,
                                            const float4* __restrict__ qs4, int x0, int y0, int z0, TreeBest& t,
                                            uint32_t& budget)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int x = x0 + (lane & 3), y = y0 + ((lane >> 2) & 3), z = z0 + (lane >> 4);
    uint2 ev = make_uint2(0u, 0u);
    if (x < b.D[0] && y < b.D[1] && z < b.D[2]) ev = row_run(P, b, off, x, x + 1, y, z);
    const float lb = row_bound(b, x, x + 1, y, z);
    // the row's run, in each of its four lanes
    uint2 rw = make_uint2((uint32_t)__builtin_amdgcn_update_dpp(0, (int)ev.x, 0x00, 0xF, 0xF, true), ev.y);   // quad_perm 0,0,0,0
    rw.y += xor_lanes(rw.y, 1);
    rw.y += xor_lanes(rw.y, 2);
    if (rw.y <= kLoads * kWave) ev = rw;
    unsigned long long left = __ballot(ev.y > 0u);
    while (left) {   // uniform
        const bool mine = (left >> lane) & 1ull;
        const float m = __uint_as_float(wave_min_dpp(mine ? __float_as_uint(lb) : 0xFFFFFFFFu));
        if (m * kBoundSlack > t.wave) break;
        const int L = __ffsll((long long)__ballot(mine && lb == m)) - 1;
        const uint32_t st = (uint32_t)__builtin_amdgcn_readlane((int)ev.x, L);
        const uint32_t cn = (uint32_t)__builtin_amdgcn_readlane((int)ev.y, L);
        left &= ~((uint32_t)__builtin_amdgcn_readlane((int)rw.y, L) <= kLoads * kWave ? 0xFull << (L & ~3) : 1ull << L);
        if (kGiveUp) {
            t.spend(budget, cn);
            if (budget == 0u) break;
        }
        for (uint32_t k = lane; k < cn; k += kLoads * kWave) {
            float4 q[kLoads];
#pragma unroll
            for (int i = 0; i < kLoads; ++i) q[i] = qs4[st + min(k + (uint32_t)(i * kWave), cn - 1u)];
#pragma unroll
            for (int i = 0; i < kLoads; ++i) t.take(q[i], b.s[0], b.s[1], b.s[2]);
        }
        t.combine();
    }
}

// What a search does among crowded voxels: scan them, scan them within the
// budget, or leave (budget 0, the results the best found so far).
enum Crowd { kCrowdScan, kCrowdBudget, kCrowdLeave };

// kFirst: the first cube's smallest radius.  kSeed: the results hold a target
// already found (or no finite distance), from which the search starts.
template <int kFirst, Crowd kCrowd, bool kSeed = false>
__device__ __forceinline__ bool tree_nearest(const PairDev& P, const uint32_t* __restrict__ off,
                                             const uint8_t* __restrict__ pyr, const float4* __restrict__ qs4, float sx,
                                             float sy, float sz, float& rd, uint32_t& rj, float& rx, float& ry,
                                             float& rz, uint32_t& budget)
{
    if (!(isfinite(sx) && isfinite(sy) && isfinite(sz))) return false;   // left to the exhaustive search
    const int lane = threadIdx.x & (kWave - 1);
    const int lx = lane & 3, ly = (lane >> 2) & 3, lz = lane >> 4;
    const TreeBox b = tree_box(P, sx, sy, sz);
    int v0[3];
    float d2box[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float f = (b.s[a] - b.o[a]) * P.inv;
        const int c = f < 0.0f ? 0 : (f >= (float)(b.D[a] - 1) ? b.D[a] - 1 : (int)floorf(f));
        v0[a] = __builtin_amdgcn_readfirstlane(c);
        const float lo = b.o[a] - b.mg[a], hi = b.o[a] + (float)b.D[a] * b.vox + b.mg[a];
        const float g = b.s[a] < lo ? lo - b.s[a] : (b.s[a] > hi ? b.s[a] - hi : 0.0f);
        d2box[a] = g * g;
    }
    // a lower bound on the squared distance of any target outside the voxels
    // [lo, hi): each of their faces that is not on the grid's boundary bounds
    // those beyond it on its axis, the grid box on the other two
    auto outside = [&](const int lo[3], const int hi[3]) {
        float out = INFINITY;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float rest = d2box[(a + 1) % 3] + d2box[(a + 2) % 3];
            if (lo[a] > 0) {
                const float g = b.s[a] - (b.o[a] + (float)lo[a] * b.vox + b.mg[a]);
                out = fminf(out, (g > 0.0f ? g * g : 0.0f) + rest);
            }
            if (hi[a] < b.D[a]) {
                const float g = (b.o[a] + (float)hi[a] * b.vox - b.mg[a]) - b.s[a];
                out = fminf(out, (g > 0.0f ? g * g : 0.0f) + rest);
            }
        }
        return out;
    };
    TreeBest t = {INFINITY, 0.0f, 0.0f, 0.0f, INFINITY, 0xFFFFFFFFu};
    if (kSeed && lane == 0) t = TreeBest{rd, rx, ry, rz, rd, rj};
    if (kSeed) t.wave = rd;
    // the first cube reaches one voxel past the dilation: a global search's
    // voxel has no occupied voxel within L1 distance L
    const int top = P.t_top;
    const int R = min(max(P.pad + 1, kFirst), kCubeMax);
    const int w = 2 * R + 1;
    static_assert((2 * kCubeMax + 1) * (2 * kCubeMax + 1) <= kN * kWave, "a cube's rows fit one round");
    const float reach = (float)R * b.vox;
    bool cube = top > 0 && d2box[0] + d2box[1] + d2box[2] <= reach * reach;
    const int ry_ = (lane >> 2) & 3, rz_ = lane >> 4;   // the lane's row in a brick
    // children of level l of the node (nx, ny, nz); `rem` are those still to
    // be looked at, kept per level in lane l of stk while a child's own
    // children are visited; `up` is the level the climb has reached.  A grid
    // of at most 4^3 voxels is one brick.
    int l = 1, up = 1, came = -1;
    int nx = v0[0] >> 4, ny = v0[1] >> 4, nz = v0[2] >> 4;
    uint32_t stk_lo = 0u, stk_hi = 0u;
    unsigned long long rem = 1ull;
    bool fresh = top > 0;
    // every round either moves in the tree or loads kN rows per lane and scans
    // their points
    while (true) {
        uint2 e[kN];   // runs of the lane: first point in qs4, points
        uint32_t bricks = 0u;            // the round's bricks: 1 + its place in the node, a byte each
        if (cube) {
#pragma unroll
            for (int u = 0; u < kN; ++u) {
                e[u] = make_uint2(0u, 0u);
                const int it = lane + u * kWave;
                const int z = it / w, y = it - z * w;
                // a voxel past 2^31 wraps to a negative index
                const int vy = (int)((uint32_t)v0[1] + (uint32_t)(y - R)), vz = (int)((uint32_t)v0[2] + (uint32_t)(z - R));
                const int x0 = max(v0[0] - R, 0), x1 = (int)min((uint32_t)v0[0] + R + 1u, (uint32_t)b.D[0]);
                if (it < w * w && vy >= 0 && vz >= 0 && vy < b.D[1] && vz < b.D[2]) e[u] = row_run(P, b, off, x0, x1, vy, vz);
            }
        } else {
            const int cx = 4 * nx + lx, cy = 4 * ny + ly, cz = 4 * nz + lz;
            if (fresh) {
                int64_t base = P.t_base;
                for (int k = 1; k < l; ++k) base += level_cells(b.D[0], b.D[1], b.D[2], k);
                const int dx = (int)level_dim(b.D[0], l), dy = (int)level_dim(b.D[1], l), dz = (int)level_dim(b.D[2], l);
                const bool in = cx < dx && cy < dy && cz < dz;
                const uint8_t f = in ? pyr[base + cx + (int64_t)dx * (cy + (int64_t)dy * cz)] : 0;
                rem = __ballot(f != 0);
                if (came >= 0) rem &= ~(1ull << came);
                came = -1;
                fresh = false;
            }
            float lb = (rem >> lane) & 1ull ? cell_bound(b, l, cx, cy, cz) : INFINITY;
            float m = __uint_as_float(wave_min_dpp(__float_as_uint(lb)));
            if (!rem || m * kBoundSlack > t.wave) {   // nothing left here
                if (top == 0) break;
                if (l < up) {   // back to the node above
                    ++l;
                    nx >>= 2, ny >>= 2, nz >>= 2;
                    rem = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)stk_hi, l) << 32) |
                          (uint32_t)__builtin_amdgcn_readlane((int)stk_lo, l);
                    continue;
                }
                if (l == top) break;   // everything has been looked at
                const int sh = 2 * (l + 1);
                // a node below the top ends at most one voxel row past 2^31
                const int lo[3] = {nx << sh, ny << sh, nz << sh};
                const int hi[3] = {(int)min((uint32_t)(nx + 1) << sh, (uint32_t)b.D[0]),
                                   (int)min((uint32_t)(ny + 1) << sh, (uint32_t)b.D[1]),
                                   (int)min((uint32_t)(nz + 1) << sh, (uint32_t)b.D[2])};
                if (outside(lo, hi) * kBoundSlack > t.wave) break;
                came = (nx & 3) | ((ny & 3) << 2) | ((nz & 3) << 4);
                nx >>= 2, ny >>= 2, nz >>= 2;
                up = ++l;
                fresh = true;
                continue;
            }
            if (l > 1) {   // into the nearest child
                const int pick = __ffsll((long long)__ballot(((rem >> lane) & 1ull) && lb == m)) - 1;
                rem &= ~(1ull << pick);
                stk_lo = lane == l ? (uint32_t)rem : stk_lo;
                stk_hi = lane == l ? (uint32_t)(rem >> 32) : stk_hi;
                nx = 4 * nx + (pick & 3), ny = 4 * ny + ((pick >> 2) & 3), nz = 4 * nz + (pick >> 4);
                --l;
                fresh = true;
                continue;
            }
            // the nearest kN bricks (one while there is no bound yet): 16 rows
            // of 4 voxels each, 4 lanes to a row
#pragma unroll
            for (int u = 0; u < kN; ++u) {
                e[u] = make_uint2(0u, 0u);
                if (u > 0) m = __uint_as_float(wave_min_dpp(__float_as_uint(lb)));
                if (!rem || m * kBoundSlack > t.wave || (u > 0 && t.wave == INFINITY)) continue;   // uniform
                const int pick = __ffsll((long long)__ballot(((rem >> lane) & 1ull) && lb == m)) - 1;
                rem &= ~(1ull << pick);
                lb = lane == pick ? INFINITY : lb;
                bricks |= (uint32_t)(pick + 1) << (8 * u);
                const int x0 = 4 * (4 * nx + (pick & 3)), vy = 4 * (4 * ny + ((pick >> 2) & 3)) + ry_,
                          vz = 4 * (4 * nz + (pick >> 4)) + rz_;
                const int x1 = (int)min((uint32_t)x0 + 4u, (uint32_t)b.D[0]);
                if (vy < b.D[1] && vz < b.D[2] && !(row_bound(b, x0, x1, vy, vz) * kBoundSlack > t.wave))
                    e[u] = row_run(P, b, off, x0, x1, vy, vz);
            }
        }
        // the lane's share of its runs' points (every 4th of a brick's row) as
        // one flat run, kLoads in flight (a lane past its last point repeats
        // it); where a lane would scan many, voxel by voxel
        const uint32_t first = cube ? 0u : (uint32_t)(lane & 3), sh = cube ? 0u : 2u;
        uint32_t own[kN], total = 0u;
#pragma unroll
        for (int u = 0; u < kN; ++u) {
            own[u] = e[u].y > first ? ((e[u].y - first - 1u) >> sh) + 1u : 0u;
            total += own[u];
        }
        const bool some = __ballot(total > kSerialPoints / 4) != 0ull;
        const bool crowd = some && __ballot(total > kSerialPoints) != 0ull;
        if (kCrowd == kCrowdBudget && some && !crowd && budget <= kStepBudget) t.spend(budget, kSerialCost);
        if (!crowd) {
            for (uint32_t t0 = 0; t0 < total; t0 += kLoads) {
                float4 q[kLoads];
#pragma unroll
                for (int i = 0; i < kLoads; ++i) {
                    uint32_t f = min(t0 + (uint32_t)i, total - 1u), slot = 0u;
                    bool found = false;
#pragma unroll
                    for (int u = 0; u < kN; ++u) {
                        const bool here = !found && f < own[u];
                        slot = here ? e[u].x + first + (f << sh) : slot;
                        found |= here;
                        f -= own[u];
                    }
                    q[i] = qs4[slot];
                }
#pragma unroll
                for (int i = 0; i < kLoads; ++i) t.take(q[i], sx, sy, sz);
            }
        } else if (kCrowd == kCrowdLeave) {
            budget = 0u;
            break;
        } else if (cube) {
            cube = false;
            continue;
        } else {
            for (; bricks; bricks >>= 8) {   // uniform
                const int pick = (int)(bricks & 0xFFu) - 1;
                const int x0 = 4 * (4 * nx + (pick & 3)), y0 = 4 * (4 * ny + ((pick >> 2) & 3)), z0 = 4 * (4 * nz + (pick >> 4));
                crowd_brick<kCrowd == kCrowdBudget>(P, b, off, qs4, x0, y0, z0, t, budget);
            }
        }
        t.combine();
        if (cube) {
            cube = false;
            const int lo[3] = {max(v0[0] - R, 0), max(v0[1] - R, 0), max(v0[2] - R, 0)};
            const int hi[3] = {(int)min((uint32_t)v0[0] + R + 1u, (uint32_t)b.D[0]),
                               (int)min((uint32_t)v0[1] + R + 1u, (uint32_t)b.D[1]),
                               (int)min((uint32_t)v0[2] + R + 1u, (uint32_t)b.D[2])};
            if (outside(lo, hi) * kBoundSlack > t.wave) break;
        }
    }
    if (!(t.wave < INFINITY) || (kCrowd == kCrowdBudget && t.wave < 0.0f)) return false;
    // the lowest index among the lanes at the best distance
    const uint32_t j = wave_min_dpp(t.d == t.wave ? t.j : 0xFFFFFFFFu);
    const int owner = __ffsll((long long)__ballot(t.d == t.wave && t.j == j)) - 1;
    rd = t.wave;
    rj = j;
    rx = __uint_as_float(__builtin_amdgcn_readlane((int)__float_as_uint(t.x), owner));
    ry = __uint_as_float(__builtin_amdgcn_readlane((int)__float_as_uint(t.y), owner));
    rz = __uint_as_float(__builtin_amdgcn_readlane((int)__float_as_uint(t.z), owner));
    return true;
}

// --------------------------------------------------------------------------
// The moment record of one search wave: the float64 moments of Eq. 1 over its
// found queries about the grid centre (sum p, sum q, sum p q^T, sum |p|^2,
// sum |q|^2, sum d), summed in a fixed order in registers.  Each step halves
// the values a lane holds while it doubles the lanes they are spread over:
// the LPQ lanes of a query take alternate entries, then the two halves of the
// wave (permlane32_swap exchanges a value's upper half for another's lower, so
// one addition serves two entries), then the odd and even rows of 16; the rest
// of a row is added by DPP.  The caller's store(entry, value) is called by the
// lane that ends with each entry.
//
// Bound by vector issue: about 130 (one lane per query) to 85 instructions a
// wave.  Its former form put every query's 18 values through LDS, 18 KB of
// traffic per wave: with 16 waves of 64 queries on a compute unit that took
// 2.8 us of a registration's iteration.
// --------------------------------------------------------------------------
constexpr int kRecSums = kMoments - 1;

// The value of the query's first lane, for each of its LPQ lanes.
template <int LPQ>
__device__ __forceinline__ float from_first(float v)
{
    const int i = __float_as_int(v);
    if (LPQ == 1) return v;
    if (LPQ == 2) return __int_as_float(__builtin_amdgcn_update_dpp(0, i, 0xA0, 0xF, 0xF, true));   // quad_perm 0,0,2,2
    if (LPQ == 4) return __int_as_float(__builtin_amdgcn_update_dpp(0, i, 0x00, 0xF, 0xF, true));   // quad_perm 0,0,0,0
    return __shfl(v, (int)(threadIdx.x & (kWave - 1)) & ~(LPQ - 1), kWave);
}

// a' + b' where the swap leaves a' = [a low, b low], b' = [a high, b high] of
// the wave (rows32) or of each pair of rows of 16: the sum of a's two parts in
// the low lanes, of b's in the high ones.
template <bool rows32>
__device__ __forceinline__ double swap_add(double a, double b)
{
    const auto swap = [](uint32_t x, uint32_t y) {
        if (rows32) return __builtin_amdgcn_permlane32_swap(x, y, false, false);
        return __builtin_amdgcn_permlane16_swap(x, y, false, false);
    };
    const auto lo = swap((uint32_t)__double2loint(a), (uint32_t)__double2loint(b));
    const auto hi = swap((uint32_t)__double2hiint(a), (uint32_t)__double2hiint(b));
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}

template <int LPQ, typename Store>
__device__ __forceinline__ void wave_record(bool found, float x, float y, float z, float bx, float by, float bz,
                                            float bd, float cx, float cy, float cz, Store&& store)
{
    const int lane = threadIdx.x & (kWave - 1), sub = lane % LPQ;
    // found counts on the query's first lane only; its other lanes hold other
    // entries of the same query
    const bool f = LPQ == 1 ? found : from_first<LPQ>(found ? 1.0f : 0.0f) != 0.0f;
    bx = from_first<LPQ>(bx);
    by = from_first<LPQ>(by);
    bz = from_first<LPQ>(bz);
    bd = from_first<LPQ>(bd);
    const double c0 = cx, c1 = cy, c2 = cz;
    const double p[3] = {f ? (double)x - c0 : 0.0, f ? (double)y - c1 : 0.0, f ? (double)z - c2 : 0.0};
    const double q[3] = {f ? (double)bx - c0 : 0.0, f ? (double)by - c1 : 0.0, f ? (double)bz - c2 : 0.0};
    double e[kRecSums + 2];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        e[r] = p[r];
        e[3 + r] = q[r];
#pragma unroll
        for (int c = 0; c < 3; ++c) e[6 + 3 * r + c] = p[r] * q[c];
    }
    e[15] = p[0] * p[0] + p[1] * p[1] + p[2] * p[2];
    e[16] = q[0] * q[0] + q[1] * q[1] + q[2] * q[2];
    e[17] = f ? (double)bd : 0.0;
    e[18] = e[19] = 0.0;
    // entry of value i in a lane: i 2^steps + the lane's bit of each step, the
    // first step's bit lowest
    constexpr int kSub = LPQ == 1 ? 0 : LPQ == 2 ? 1 : LPQ == 4 ? 2 : 3;
    constexpr int n0 = kRecSums, n1 = (n0 + (1 << kSub) - 1) >> kSub, n2 = (n1 + 1) / 2, n3 = (n2 + 1) / 2;
    int n = n0;
#pragma unroll
    for (int s = 0; s < kSub; ++s) {
        const bool odd = (sub >> s) & 1;
#pragma unroll
        for (int i = 0; 2 * i < n; ++i) e[i] = odd ? (2 * i + 1 < n ? e[2 * i + 1] : 0.0) : e[2 * i];
        n = (n + 1) / 2;
    }
#pragma unroll
    for (int i = 0; i < n2; ++i) e[i] = swap_add<true>(e[2 * i], 2 * i + 1 < n1 ? e[2 * i + 1] : 0.0);
#pragma unroll
    for (int i = 0; i < n3; ++i) e[i] = swap_add<false>(e[2 * i], 2 * i + 1 < n2 ? e[2 * i + 1] : 0.0);
    // a row's lanes of the same sub, in order: the total ends in the last
#pragma unroll
    for (int i = 0; i < n3; ++i) {
        if (LPQ <= 1) e[i] = dpp_add<0x111, 0xF>(e[i]);
        if (LPQ <= 2) e[i] = dpp_add<0x112, 0xF>(e[i]);
        if (LPQ <= 4) e[i] = dpp_add<0x114, 0xF>(e[i]);
        e[i] = dpp_add<0x118, 0xF>(e[i]);
    }
    if ((lane & 15) >= 16 - LPQ) {
        const int bits = sub | ((lane >> 5) << kSub) | (((lane >> 4) & 1) << (kSub + 1));
#pragma unroll
        for (int i = 0; i < n3; ++i) {
            const int j = (i << (kSub + 2)) | bits;
            if (j < kRecSums) store(j, e[i]);
        }
    }
}

__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sum over the wave of values held in every LPQ-th lane (zero elsewhere).
template <int LPQ>
__device__ __forceinline__ uint32_t wave_candidates(uint32_t c)
{
    const uint32_t cw = row_sum_u32<LPQ>(c);   // each 16-lane row's total in its lane 16 - LPQ
    return (uint32_t)__builtin_amdgcn_readlane((int)cw, 16 - LPQ) +
           (uint32_t)__builtin_amdgcn_readlane((int)cw, 32 - LPQ) +
           (uint32_t)__builtin_amdgcn_readlane((int)cw, 48 - LPQ) +
           (uint32_t)__builtin_amdgcn_readlane((int)cw, 64 - LPQ);
}

static_assert(kUnitSlices == kWave / 2, "one slice per lane of a half wave");

__device__ __forceinline__ double unit_sum(double (&v)[kUnitRecords])
{
#pragma unroll
    for (int w = kUnitRecords / 2; w >= 1; w >>= 1)
#pragma unroll
        for (int i = 0; i < w; ++i) v[i] += v[i + w];
    return v[0];
}

}  // namespace

}  // namespace vicp
