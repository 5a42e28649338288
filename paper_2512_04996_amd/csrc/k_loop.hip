// k_loop.hip -- the whole ICP loop of a registration in one launch (Sec. II.A;
// Alg. 4's search, Eq. 1's solve, the stop rule of Sec. IV.A).
//
// The blocks stay resident for all iterations.  A pair has one or more blocks;
// each searches its units (kUnitRecords wave records, one per wave of the
// block), and the pair's first block also gathers the units' moment sums,
// solves, and hands the next pose to the others.  Every sum is taken in the
// order of the launch-per-step kernels, so the two forms give the same bits.
//
// What bounds a step of the launch-per-step form on clouds of up to a few
// hundred thousand points is not work but its three launches, each a chain of
// a launch, a cold pose load and a reduction through memory: 17 to 20 us a step
// with 2,048 points (8 units at four lanes) and with 35,000 (137 units).  Here a
// step takes 12 us in both, of which 1.8 are the local search, 2.2 the solve's
// serial float64 chain, 2.7 the messages and their gather, and most of the rest
// the slowest block's global searches.  Registrations: 2,048 points, 20 steps
// 479 -> 308 us; 35,000, 50 steps 1468 -> 598; a 200,000-point room frame with
// its refill, 30 steps 812 -> 612; a 120,000-point frame of which a tenth has
// no counterpart, 30 steps 28.7 -> 13.4 ms (the global searches are spread over
// all waves of their block, and units interleave).
//
// Units of 16 waves, one block of 1024 threads: units of 8 double the messages
// that the solving block gathers, and measured slower.  A wave's 22 record sums
// are reduced in registers (wave_record); through LDS they took 2.8 us a step,
// the 16 waves of a block contending for it.
//
// Messages.  The eight XCDs' L2s are not coherent with each other, so blocks
// talk through agent-scope relaxed 64-bit accesses, and every word carries
// its own tag in its upper half (the iteration's number, from a counter that
// goes on over calls): a word whose tag matches is complete, so no fence
// orders a flag after its data.  A unit's sums are overwritten only after the
// next pose, which the first block publishes after it has read them all.
//
// Every wait ends: a block that has waited for `patience` ticks, or for
// `arrive` ticks while a block of the launch has not begun, raises the abort
// word (its lower half to one more than this call's tag, the upper to the
// reason), which every wait reads, and all blocks return; the host then runs the
// launch-per-step form.  The host launches at most as many blocks as fit the
// device at once, and one such loop per device at a time; blocks may still not
// all begin where another process' or another stream's kernels hold compute
// units, which a block sees after 2 ms in which it waits.
#include "search_dev.hpp"
#include "solve_dev.hpp"
#include "vicp_internal.hpp"

namespace vicp {

namespace {

constexpr int kLoopThreads = kWave * kUnitRecords;
constexpr int kLoopWaves = kUnitRecords;
constexpr int kSumCols = kMoments + 3;           // moments, candidates, dilated lookups, global searches
constexpr int kGather = kLoopAloneUnits;         // units gathered per round
constexpr int kGatherLoads = (kGather * kLoopWords + kLoopThreads - 1) / kLoopThreads;
static_assert(kLoopWords == 2 * kSumCols && kSumCols * kUnitSlices <= kLoopThreads && kGather % kGroupSpan == 0,
              "message and gather layout");

__device__ __forceinline__ unsigned long long ld_agent(const unsigned long long* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void st_tagged(unsigned long long* p, uint32_t tag, uint32_t v)
{
    __hip_atomic_store(p, ((unsigned long long)tag << 32) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A query's place in the block's list of global searches, and its result.
struct MissSlot {
    float s[3];
    float d, x, y, z;
    uint32_t j;
};
struct LoopShared {
    double rec[kLoopWaves][kSumCols + 1];                    // a unit's records
    double stage[kSumCols][kGather + 1];                     // units' sums at the solving block
    double tot[kSumCols];
    double Rt[12];                                           // the pose (solving block)
    float4 pt[kLoopThreads];                                 // the lanes' queries (a block with one unit)
    MissSlot slots[kLoopThreads];                            // the unit's global searches
    float pose[12];
    GridGeom geo;
    int32_t done, misses, stop;
};

// Eq. 1's solve from the totals in LDS: the pose Rt (in: the previous one), or
// false when the rotation cannot be refined from the previous one (nearly
// planar or degenerate sums, a turn of over 90 degrees): loop_solve_svd then.
// The rotation goes through LDS, so that the sums are read again for the
// translation instead of being held in registers through the refinement.
template <SolveStep kStep>
__device__ __forceinline__ bool solve_totals(LoopShared& sh, bool rot_ok)
{
    {
        double t[kMoments], Rp[9], R[9];
#pragma unroll
        for (int j = 0; j < kMoments; ++j) t[j] = sh.tot[j];
#pragma unroll
        for (int j = 0; j < 9; ++j) Rp[j] = sh.Rt[j];
        if (!kabsch_rotation<kStep>(t, Rp, rot_ok, R)) return false;
#pragma unroll
        for (int j = 0; j < 9; ++j) sh.Rt[j] = R[j];
    }
    asm volatile("" ::: "memory");
    double t[kMoments], R[9], tr[3];
#pragma unroll
    for (int j = 0; j < 6; ++j) t[j] = sh.tot[j];
    t[kMoments - 1] = sh.tot[kMoments - 1];
#pragma unroll
    for (int j = 0; j < 9; ++j) R[j] = sh.Rt[j];
    const double cen[3] = {sh.geo.cx, sh.geo.cy, sh.geo.cz};
    kabsch_translation(t, cen, R, tr);
#pragma unroll
    for (int j = 0; j < 3; ++j) sh.Rt[9 + j] = tr[j];
    return true;
}

// The solve without the refinement, out of line, so that its registers are not
// the loop's: false (pose untouched) when the sums do not determine a rotation.
__device__ __attribute__((noinline, cold)) bool loop_solve_svd(LoopShared* sh)
{
    return solve_totals<kAfterRefine>(*sh, false);
}

template <typename T>
__device__ __forceinline__ T* uniform_ptr(T* p)
{
    const uint64_t v = (uint64_t)p;
    return (T*)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32) |
                (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v));
}

// The block's global searches, shared out over its waves.  Out of line: most
// iterations have none, and inlined its registers would be the search's too.
// kRest: those that the first pass left, among crowded voxels, in a function of
// their own, as their registers and a call from within cost the ordinary ones
// more (a 2,048-point sphere, 20 steps: 295 us, 314 with a call from within).
// Returns kAllFound when every search of the wave has a finite distance, and
// kSomeLeft when some were left.
constexpr int kAllFound = 1, kSomeLeft = 2;
template <bool kRest>
__device__ __forceinline__ int wave_misses(const PairDev* P, const uint32_t* off, const uint8_t* pyr, const float4* qs4,
                                           MissSlot* slots, int n)
{
    P = uniform_ptr(P);
    off = uniform_ptr(off);
    pyr = uniform_ptr(pyr);
    qs4 = uniform_ptr(qs4);
    n = __builtin_amdgcn_readfirstlane(n);
    const int lane = threadIdx.x & (kWave - 1);
    int got = kAllFound;
    for (int e = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave); e < n; e += kLoopWaves) {
        float rd = INFINITY, rx = 0.0f, ry = 0.0f, rz = 0.0f;
        uint32_t rj = 0xFFFFFFFFu, budget = 1u;
        if (kRest) {
            // left: the negative of the best found, from which this goes on
            const uint32_t d = (uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(slots[e].d));
            if (!(d >> 31)) continue;
            rd = __uint_as_float(d & 0x7FFFFFFFu);
            rx = slots[e].x, ry = slots[e].y, rz = slots[e].z;
            rj = slots[e].j;
        }
        const bool ok = tree_nearest<kCubeMin, kRest ? kCrowdScan : kCrowdLeave, kRest>(
            *P, off, pyr, qs4, slots[e].s[0], slots[e].s[1], slots[e].s[2], rd, rj, rx, ry, rz, budget);
        if (!kRest && budget == 0u) {   // uniform
            got |= kSomeLeft;
            rd = __uint_as_float(__float_as_uint(rd) | 0x80000000u);
        } else if (!ok) {
            got &= ~kAllFound;
        }
        if (lane == 0) {
            slots[e].d = rd;
            slots[e].x = rx;
            slots[e].y = ry;
            slots[e].z = rz;
            slots[e].j = rj;
        }
    }
    return got;
}
__device__ __attribute__((noinline)) int block_misses(const PairDev* P, const uint32_t* off, const uint8_t* pyr,
                                                      const float4* qs4, MissSlot* slots, int n)
{
    return wave_misses<false>(P, off, pyr, qs4, slots, n);
}
__device__ __attribute__((noinline)) int block_crowd_misses(const PairDev* P, const uint32_t* off, const uint8_t* pyr,
                                                            const float4* qs4, MissSlot* slots, int n)
{
    return wave_misses<true>(P, off, pyr, qs4, slots, n);
}

// crowd_scan, out of line: most searches have no crowded voxel, and inlined its
// registers would be theirs too.  No position (the largest value): not found.
__device__ __attribute__((noinline)) uint2 block_crowd(const float4* qs4, uint32_t start, uint32_t c, float sx, float sy,
                                                       float sz)
{
    float bd = INFINITY;
    uint32_t bk = 0xFFFFFFFFu;
    if (!crowd_scan(uniform_ptr(qs4), (int64_t)start, c, sx, sy, sz, threadIdx.x & (kWave - 1), bd, bk))
        bk = 0xFFFFFFFFu;
    return make_uint2(__float_as_uint(bd), bk);
}

__device__ __forceinline__ void raise_abort(unsigned long long* word, uint32_t tag, uint32_t reason)
{
    __hip_atomic_store(word, ((unsigned long long)reason << 32) | (tag + 1u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

typedef const __attribute__((address_space(4))) LoopArgs* LoopArgsPtr;

// One pass of lane-wise polling: true when every lane's word carries the tag
// (lanes that have none pass ok = true); false when the loop is to stop.
__device__ __forceinline__ bool wait_over(bool ok, unsigned long long t0, LoopArgsPtr B, uint32_t tag)
{
    if (__ballot(!ok) == 0ull) return true;
    const unsigned long long waited = __builtin_amdgcn_s_memrealtime() - t0;
    if (waited > B->arrive && (waited > B->patience || ld_agent(B->begun) < B->begun_all))
        raise_abort(B->abort_word, tag, kAbortWait);
    __builtin_amdgcn_s_sleep(1);
    return false;
}

template <int LPQ, bool kSorted>
__global__ __launch_bounds__(kLoopThreads) void k_icp_loop(LoopArgs A)
{
    __shared__ LoopShared sh;
    constexpr int kQw = kWave / LPQ;
    // a single pair's blocks each take one unit in turn, neighbouring units on
    // one XCD; a batch has its blocks in a table
    LoopJob job;
    if (A.jobs)
        job = A.jobs[blockIdx.x];
    else
        job = LoopJob{0, xcd_slab((int)blockIdx.x, (int)gridDim.x), (int32_t)gridDim.x, 0};
    const PairDev& P = A.pd[job.pair];
    PairState& S = A.st[job.pair];
    const int64_t m = P.m;
    const int R = (int)((m + kQw - 1) / kQw), U = (R + kUnitRecords - 1) / kUnitRecords;
    const bool solver = job.u0 == 0, alone = job.stride == 1;
    const int64_t p_base = P.p_base;
    const uint2* dir = A.dir + P.v_base;
    unsigned long long* msg = A.msg + (int64_t)job.unit_base * kLoopWords;
    unsigned long long* pmsg = A.pose_msg + (int64_t)job.pair * kPoseWords;
    if (threadIdx.x < 12) {
        sh.pose[threadIdx.x] = S.Rtf[threadIdx.x];
        sh.Rt[threadIdx.x] = S.Rt[threadIdx.x];
    }
    if (threadIdx.x == 0) {
        __hip_atomic_fetch_add(A.begun, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sh.geo = GridGeom{P.ox, P.oy, P.oz, P.inv, P.fDx, P.fDy, P.fDz, P.cx, P.cy, P.cz, (uint32_t)P.Dx, (uint32_t)P.Dy};
        sh.done = 0;
        sh.misses = 0;
        sh.stop = 0;
    }
    bool rot_ok = S.rot_ok != 0;   // thread 0 of the solving block keeps the run's state
    double prev = S.prev_rmse;
    const bool once = job.u0 + job.stride >= U;   // one unit: its queries stay in LDS
    MissSlot* slots = sh.slots;
    __syncthreads();
    for (int k = 0; k < A.K; ++k) {
        // opaque to the compiler, which would otherwise work out every lane's
        // addresses before the loop and spill them
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        // the arguments that only some blocks or iterations use are read where
        // they are used, through a pointer that is opaque too
        auto B = (LoopArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(B));
        const int lane = tid & (kWave - 1), w = __builtin_amdgcn_readfirstlane(tid / kWave), sub = lane % LPQ;
        if (k > 0 && !alone && !solver) {
            if (w == 0) {
                const uint32_t tag = A.tag + (uint32_t)k;
                const unsigned long long t0 = __builtin_amdgcn_s_memrealtime();
                unsigned long long v = 0ull;
                bool over = false, quit = false;
                while (!over && !quit) {
                    v = lane < kPoseWords ? ld_agent(pmsg + lane) : (lane == kWave - 1 ? ld_agent(B->abort_word) : 0ull);
                    quit = __ballot(lane == kWave - 1 && (uint32_t)v == A.tag + 1u) != 0ull;
                    over = wait_over(lane >= kPoseWords || (uint32_t)(v >> 32) == tag, t0, B, A.tag);
                }
                if (lane < 12) sh.pose[lane] = __uint_as_float((uint32_t)v);
                if (lane == 12) sh.done = (int32_t)(uint32_t)v;
                if (lane == 0 && !over) sh.stop = 1;
            }
            __syncthreads();
        }
        if (sh.stop || sh.done) break;   // uniform: written before the last barrier
        for (int u = job.u0; u < U; u += job.stride) {
            const int r = u + w * U;
            const int64_t t = (int64_t)r * kQw + lane / LPQ;
            const bool active = r < R && t < m;
            // a lane's query goes through its own LDS slot: no other lane's
            // barrier is needed, and it holds no register through the iteration
            if (k == 0 || !once) {
                const int64_t tl = p_base + (active ? t : 0);
                sh.pt[tid] = kSorted ? A.ps4[tl]
                                     : make_float4(A.px[tl], A.py[tl], A.pz[tl], __uint_as_float((uint32_t)(tl - p_base)));
            }
            wave_lds_fence();
            const float x = sh.pt[tid].x, y = sh.pt[tid].y, z = sh.pt[tid].z;
            // no branch on the way to the directory entry (a lane outside the
            // grid or past the end reads voxel 0's and drops it)
            float sx, sy, sz;
            transform(sh.pose, x, y, z, sx, sy, sz);
            uint32_t v = 0u;
            const bool in = voxel_of(sh.geo, sx, sy, sz, v) & active;
            const uint2 ent = dir[in ? v : 0u];
            const uint32_t c = in ? ent.y & ~kMask : 0u, cs = ent.x;
            const bool dil = in && (ent.y & kMask) != 0u;
            float bd = INFINITY, bx = 0.0f, by = 0.0f, bz = 0.0f;
            uint32_t bk = 0xFFFFFFFFu;
            bool crowd = false;   // uniform over the wave
            if (LPQ == 8 && crowded(c)) {
                const uint2 got = block_crowd(A.qs4, cs, c, sx, sy, sz);
                crowd = __ballot(got.y == 0xFFFFFFFFu) == 0ull;
                bd = crowd ? __uint_as_float(got.x) : bd;
                bk = crowd ? got.y : bk;
            }
            if (!crowd && c > 0u) {
                constexpr int N = LPQ <= 2 ? 8 : 4;
                const float4* seg = A.qs4 + cs;
                const uint32_t last = c - 1u;
                for (uint32_t q0 = sub; q0 < c; q0 += N * LPQ) {
                    float4 a[N];
#pragma unroll
                    for (int n = 0; n < N; ++n) a[n] = seg[min(q0 + (uint32_t)(n * LPQ), last)];
#pragma unroll
                    for (int n = 0; n < N; ++n)
                        consider_pos(a[n], min(q0 + (uint32_t)(n * LPQ), last), sx, sy, sz, bd, bk);
                }
            }
#pragma unroll
            for (int d = 1; d < LPQ; d <<= 1) {
                const float od = xor_lanes(bd, d);
                const uint32_t ok = xor_lanes(bk, d);
                const bool take = (od < bd) | ((od == bd) & (ok < bk));
                bd = take ? od : bd;
                bk = take ? ok : bk;
            }
            uint32_t bj = 0u;
            if (c > 0u && sub == 0) {
                const float4 win = A.qs4[cs + min(bk, c - 1u)];
                bx = win.x, by = win.y, bz = win.z;
                bj = __float_as_uint(win.w);
            }
            // the block's global searches: listed here, shared out over its
            // waves below, and handed back to their lanes
            const bool miss = active && c == 0u && sub == 0;
            const unsigned long long mm = __ballot(miss);
            int place = 0;
            if (mm) {
                if (lane == 0) place = atomicAdd(&sh.misses, (int32_t)__popcll(mm));
                place = __shfl(place, 0, kWave) + (int)__popcll(mm & ((1ull << lane) - 1ull));
                if (miss) {
                    slots[place].s[0] = sx;
                    slots[place].s[1] = sy;
                    slots[place].s[2] = sz;
                }
            }
            // a wave without global searches writes its record at once, one with
            // some after the block has resolved them
            const bool found = active && sub == 0;
            bool recorded = false;
#pragma unroll 1
            for (int pass = 0; pass < 2; ++pass) {
                if (!recorded && (mm == 0ull || pass == 1)) {
                    recorded = true;
                    const float4 pt = sh.pt[tid];
                    if (found && B->nn_idx && (B->early_stop || k == B->K - 1)) {
                        const uint32_t i = __float_as_uint(pt.w);
                        B->nn_idx[p_base + i] = (int32_t)bj;
                        B->nn_d2[p_base + i] = bd;
                    }
                    wave_record<LPQ>(found, pt.x, pt.y, pt.z, bx, by, bz, bd, sh.geo.cx, sh.geo.cy, sh.geo.cz,
                                     [&](int j, double v) { sh.rec[w][j] = v; });
                    const uint32_t nf = (uint32_t)__popcll(__ballot(found));
                    const uint32_t nd = (uint32_t)__popcll(__ballot(dil && sub == 0));
                    const uint32_t nc = wave_candidates<LPQ>(sub == 0 ? c : 0u);
                    // the counters as float64 (exact below 2^53)
                    const uint32_t cnt = lane == 0 ? nf : lane == 1 ? nc : lane == 2 ? nd : (uint32_t)__popcll(mm);
                    if (lane < kSumCols - kRecSums) sh.rec[w][kRecSums + lane] = (double)cnt;
                }
                __syncthreads();
                const int nmiss = sh.misses;
                if (pass == 1 || nmiss == 0) break;   // uniform over the block
                int got = __builtin_amdgcn_readfirstlane(block_misses(&P, B->off, B->pyr, B->qs4, slots, nmiss));
                if (got & kSomeLeft)
                    got &= __builtin_amdgcn_readfirstlane(block_crowd_misses(&P, B->off, B->pyr, B->qs4, slots, nmiss));
                // no finite distance: the other form resolves it
                if (!(got & kAllFound) && lane == 0) sh.stop = 1;
                __syncthreads();
                if (miss) {
                    bd = slots[place].d;
                    bx = slots[place].x;
                    by = slots[place].y;
                    bz = slots[place].z;
                    bj = slots[place].j;
                }
                if (tid == 0) {
                    sh.misses = 0;
                    if (sh.stop) raise_abort(B->abort_word, A.tag, kAbortQuery);
                }
            }
            if (w == 0 && lane < kSumCols) {
                double v[kUnitRecords];
#pragma unroll
                for (int e = 0; e < kUnitRecords; ++e) v[e] = sh.rec[e][lane];
                const double sum = unit_sum(v);
                if (alone) {
                    sh.stage[lane][u] = sum;   // U <= kGather (kLoopAloneUnits)
                } else {
                    const uint32_t tag = A.tag + (uint32_t)k + 1u;
                    unsigned long long* out = msg + (int64_t)u * kLoopWords + 2 * lane;
                    st_tagged(out, tag, (uint32_t)__double2loint(sum));
                    st_tagged(out + 1, tag, (uint32_t)__double2hiint(sum));
                }
            }
            // the next unit's waves list misses and write records only once
            // wave 0 has read this unit's, and every wave its count of misses;
            // after the last unit the gather's or the next pose's barrier
            // orders them
            if (u + job.stride < U) __syncthreads();
        }
        if (!solver) continue;
        // the pair's units, kGather at a time: their words as they arrive, then
        // kUnitSlices threads per sum each add one slice's groups in order
        const int col = tid / kUnitSlices, sl = tid % kUnitSlices;
        double acc = 0.0;
        for (int g0 = 0; g0 < U; g0 += kGather) {
            const int n = min(kGather, U - g0);
            if (!alone) {
                const uint32_t tag = A.tag + (uint32_t)k + 1u;
                const unsigned long long* in = msg + (int64_t)g0 * kLoopWords;
                const unsigned long long t0 = __builtin_amdgcn_s_memrealtime();
                unsigned long long v[kGatherLoads];
                bool over = false, quit = false;
                while (!over && !quit) {
                    bool ok = true;
#pragma unroll
                    for (int e = 0; e < kGatherLoads; ++e) {
                        const int at = tid + e * kLoopThreads;
                        v[e] = at < n * kLoopWords ? ld_agent(in + at) : 0ull;
                    }
                    const unsigned long long ab = lane == 0 ? ld_agent(B->abort_word) : 0ull;
#pragma unroll
                    for (int e = 0; e < kGatherLoads; ++e)
                        ok &= tid + e * kLoopThreads >= n * kLoopWords || (uint32_t)(v[e] >> 32) == tag;
                    quit = __ballot(lane == 0 && (uint32_t)ab == A.tag + 1u) != 0ull;
                    over = wait_over(ok, t0, B, A.tag);
                }
                if (!over && lane == 0) sh.stop = 1;
                uint32_t* stage = reinterpret_cast<uint32_t*>(&sh.stage[0][0]);
#pragma unroll
                for (int e = 0; e < kGatherLoads; ++e) {
                    const int at = tid + e * kLoopThreads;
                    if (at >= n * kLoopWords) continue;
                    const int u = at / kLoopWords, q = at - u * kLoopWords;
                    stage[2 * ((q >> 1) * (kGather + 1) + u) + (q & 1)] = (uint32_t)v[e];
                }
            }
            __syncthreads();
            if (col < kSumCols) {
                for (int b = 0; b < n; b += kGroupSpan) {
                    double v[kGroupUnits], sum = 0.0;
#pragma unroll
                    for (int i = 0; i < kGroupUnits; ++i) {
                        const int u = b + sl + i * kUnitSlices;
                        v[i] = u < n ? sh.stage[col][u] : 0.0;
                    }
#pragma unroll
                    for (int i = 0; i < kGroupUnits; ++i) sum += v[i];
                    acc += sum;
                }
            }
            if (g0 + kGather < U) __syncthreads();   // the next round reuses the stage
        }
        acc = half_sum_f64(acc);
        if (col < kSumCols && sl == kUnitSlices - 1) sh.tot[col] = acc;
        __syncthreads();
        if (w == 0) {
            if (lane == 0) {
                const double n = sh.tot[kMoments - 1], rmse = n > 0.0 ? sqrt(sh.tot[17] / n) : 0.0;
                const bool ok = solve_totals<kRefine>(sh, rot_ok) || loop_solve_svd(&sh);
                if (ok) {
                    for (int j = 0; j < 12; ++j) sh.pose[j] = (float)sh.Rt[j];
                    rot_ok = true;
                } else {
                    S.degenerate += 1;   // the pose is kept
                }
                const bool end = B->early_stop && k >= 1 && fabs(rmse - prev) < B->eps;
                prev = rmse;
                sh.done = end ? 1 : 0;
                const int64_t h = (int64_t)job.pair * B->K + k;
                B->rmse_hist[h] = rmse;
                B->fb_hist[h] = (int32_t)sh.tot[kMoments + 2];
                B->deg_hist[h] = ok ? 0 : 1;
                B->ctr_hist[2 * h] = (unsigned long long)sh.tot[kMoments];
                B->ctr_hist[2 * h + 1] = (unsigned long long)sh.tot[kMoments + 1];
                if (end || k == B->K - 1) {
                    for (int j = 0; j < 12; ++j) {
                        S.Rt[j] = sh.Rt[j];
                        S.Rtf[j] = (float)sh.Rt[j];
                    }
                    S.rot_ok = rot_ok ? 1 : 0;
                    S.prev_rmse = prev;
                    S.iters = k + 1;
                    S.done = end ? 1 : 0;
                }
            }
            wave_lds_fence();
            if (!alone && k < B->K - 1 && lane < kPoseWords)
                st_tagged(pmsg + lane, A.tag + (uint32_t)k + 1u,
                          lane < 12 ? __float_as_uint(sh.pose[lane]) : (uint32_t)sh.done);
        }
        __syncthreads();
    }
}

}  // namespace

const void* loop_kernel(int lpq, bool sorted)
{
#define VICP_LOOP_K(L) (sorted ? (const void*)k_icp_loop<L, true> : (const void*)k_icp_loop<L, false>)
    switch (lpq) {
    case 1: return VICP_LOOP_K(1);
    case 2: return VICP_LOOP_K(2);
    case 4: return VICP_LOOP_K(4);
    default: return VICP_LOOP_K(8);
    }
#undef VICP_LOOP_K
}

int loop_threads() { return kLoopThreads; }

void launch_loop(const LoopArgs& a, int nblocks, int lpq, bool sorted, hipStream_t s)
{
    if (nblocks <= 0) return;
#define VICP_LOOP(L)                                                                                 \
    if (sorted)                                                                                      \
        hipLaunchKernelGGL((k_icp_loop<L, true>), dim3(nblocks), dim3(kLoopThreads), 0, s, a);       \
    else                                                                                             \
        hipLaunchKernelGGL((k_icp_loop<L, false>), dim3(nblocks), dim3(kLoopThreads), 0, s, a)
    switch (lpq) {
    case 1: VICP_LOOP(1); break;
    case 2: VICP_LOOP(2); break;
    case 4: VICP_LOOP(4); break;
    default: VICP_LOOP(8); break;
    }
#undef VICP_LOOP
}

}  // namespace vicp
