// k_nns.hip -- correspondence search (Alg. 4).
//
// Local search: one lane per source point.  The transformed point's voxel is
// found by the same float32 quantisation as the targets.  Its entry in the
// search directory (derived from the offsets and count words, and for a
// Mask(root) voxel from the root's, so still no replicated points) gives the
// start and count of its candidates in one 8-byte load, where reading
// offset -> count word -> root offset -> root count word would chain four
// dependent loads.  Candidates are read as float4 (x, y, z, index) from the
// segment-ordered copy of the target, a fixed number of 16-byte loads in
// flight per lane (indices past the end are clamped to the last candidate:
// a repeated candidate never changes a strict minimum); segments are in
// ascending index order, so a strict "<" keeps the lowest index among equal
// distances.
//
// Query order: lanes of a wave that look up different voxels diverge (the
// wave runs the longest segment) and gather from unrelated cache lines.  The
// search can therefore run over a copy of the source bucketed by target
// voxel at the current pose (a counting sort: LDS-hashed bucket counts, a
// plain scan, a placement pass), so neighbouring lanes share segments.
// Within a bucket the points are then put in ascending index order (each
// counts the smaller indices of its bucket), so the bucketed copy, and every
// per-block sum taken over it, is the same from run to run.
//
// Global search (empty undilated voxel or outside the grid): the wave
// resolves the query itself by an exact search of the occupancy pyramid.
// Exhaustive search (queries without a finite distance, or behind the budget of
// a wave among crowded voxels): the query is appended to a per-pair list and a
// brute force over all targets resolves it; partial minima from target tiles
// merge through a 64-bit atomic minimum of (distance bits << 32 | index), which
// is order-free, so the result is deterministic.
#include <math.h>

#include <algorithm>

#include "search_dev.hpp"
#include "vicp_internal.hpp"

namespace vicp {

namespace {

// LPQ lanes cooperate on one query: each scans every LPQ-th candidate of the
// segment in ascending order (so it keeps the lowest index among its equal
// distances), then the lanes combine by the lexicographic minimum of
// (distance, index) -- the same result as one lane scanning everything, with
// LPQ times more waves in flight to hide the load latency.
//
// kMom (registration): instead of writing each correspondence, each wave
// adds the float64 moments of Eq. 1 over the queries it resolves (sum p,
// sum q, sum p q^T, sum |p|^2, sum |q|^2 about the grid centre, sum d, count)
// in a fixed lane order and writes one record, with its counters
// (candidates scanned, dilated lookups, queries that needed a global search).
// Records are wave-major: wave w of job b is record r = b * (BS / 64) + w,
// entry j at [r * kMoments + j], counter k at [r * 3 + k].  Listed queries (see
// below) add their moments in the solve.  Launch blocks are mapped to jobs XCD
// by XCD (xcd_job, xcd_slab).
//
// kDirect: VANICP's monolithic layout (the comparator).  Voxel g's
// candidates are the records of its own fixed block, at g * cap, and its
// count word dcnt[g] (the root's count with the mask bit for a dilated
// voxel); a count above cap means an overflowed block and sends the query to
// the global search.  Records are in the order the voxelisation's atomics
// gave them, so ties compare indices.
//
// kMode 1 (registration over segments, for many candidates per query): each
// lane keeps the best distance and segment position only, and the winner's
// record is read once after the lanes combine (one more dependent load per
// query, three fewer selects per candidate).
//
// kOne (a single pair of one_m source points): a block's first query is its
// job index times the queries per block, so the query's load waits on no
// table, and the pair record, the pose and the query load go out together
// (with a table the chain is table -> pair record -> query).
//
// In registration nn_idx / nn_d2 are optional (null when not asked for): the
// correspondence and squared distance of each query resolved here (locally,
// or by the tree search) are written there too; the
// solve writes those of the exhaustively searched ones.
template <int BS, int LPQ, bool kSorted, bool kMom, bool kDirect, int kMode, bool kOne>
__global__ __launch_bounds__(BS) void k_nns_local(const PairDev* __restrict__ pd, const BlockJob* __restrict__ jobs,
                                                  const float* __restrict__ px, const float* __restrict__ py,
                                                  const float* __restrict__ pz, const float4* __restrict__ ps4,
                                                  const PairState* __restrict__ st, const uint2* __restrict__ dir,
                                                  const uint32_t* __restrict__ off, const uint8_t* __restrict__ pyr,
                                                  const float4* __restrict__ qs4, const float4* __restrict__ qsg,
                                                  int32_t* __restrict__ nn_idx, float* __restrict__ nn_d2,
                                                  int32_t* __restrict__ fb_count, int32_t* __restrict__ fb_miss,
                                                  uint32_t* __restrict__ fb_list,
                                                  unsigned long long* __restrict__ fb_key,
                                                  unsigned long long* __restrict__ ctr, double* __restrict__ part,
                                                  const uint32_t* __restrict__ dcnt, uint32_t cap,
                                                  int64_t one_m, int early, uint32_t most)
{
    static_assert(LPQ == 1 || LPQ == 2 || LPQ == 4 || LPQ == 8, "lanes per query");
    constexpr bool kReload = kMode == 1;
    static_assert(kMode == 0 || kMode == 1, "search mode");
    static_assert(!kReload || (kMom && !kDirect), "position tracking needs index-ordered segments");
    constexpr int kWaves = BS / kWave;
    // A batch gives each XCD one contiguous eighth of the jobs, whole pairs, so
    // that an L2 holds its pairs' directories and segments (64 pairs: 3.66
    // against 4.2 ms; the loss over 16 pairs: 242 against 257 us).  A single
    // pair keeps the rotating chunks.
    const int jb = kOne ? xcd_job((int)blockIdx.x, (int)gridDim.x) : xcd_slab((int)blockIdx.x, (int)gridDim.x);
    const BlockJob job = kOne ? BlockJob{0, jb * (BS / LPQ)} : jobs[jb];
    const PairDev& P = pd[job.pair];
    const PairState& S = st[job.pair];
    // where pairs can stop early, a finished one's blocks end here: 30 launches
    // behind the stop of a 200,000-point run took 12.4 us each, now 3.3 (the run
    // 2.70 -> 2.37 ms).  Only there, as the test delays the loads below by the
    // flag's latency.
    if (kMom && early && S.done) return;
    const int sub = threadIdx.x % LPQ;
    const int64_t t = (int64_t)job.start + threadIdx.x / LPQ;
    const bool inrange = t < (kOne ? one_m : P.m);
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    uint32_t c = 0, i = 0;
    int64_t cs = 0;
    float x = 0.0f, y = 0.0f, z = 0.0f;
    float sx = 0.0f, sy = 0.0f, sz = 0.0f;
    bool dil = false;
    // The query's load goes out unconditionally (a lane past the end reads
    // the block's first query, which exists).  Where no pair can stop early it
    // does not wait for the pair's done flag, so the two latencies overlap; the
    // flag then only says that a pair has no source points, which has no blocks.
    {
        const int64_t tl = (kOne ? (int64_t)0 : P.p_base) + (inrange ? t : (int64_t)job.start);
        if (kSorted) {
            const float4 pp = ps4[tl];
            x = pp.x;
            y = pp.y;
            z = pp.z;
            i = __float_as_uint(pp.w);
        } else {
            x = px[tl];
            y = py[tl];
            z = pz[tl];
            i = (uint32_t)(tl - (kOne ? (int64_t)0 : P.p_base));
        }
    }
    const bool active = inrange && S.done == 0;
    if (active) {
        transform(S.Rtf, x, y, z, sx, sy, sz);
        uint32_t v;
        if (voxel_of(P, sx, sy, sz, v)) {
            if (kDirect) {
                const uint32_t e = dcnt[P.v_base + v];
                const uint32_t cn = e & ~kMask;
                c = cn <= cap ? cn : 0u;
                cs = (P.v_base + (int64_t)v) * (int64_t)cap;
                dil = (e & kMask) != 0u && c != 0u;
            } else {
                const uint2 e = dir[P.v_base + v];
                c = e.y & ~kMask;
                cs = e.x;
                dil = (e.y & kMask) != 0u;
            }
        }
    }
    const int64_t gp = (kOne ? (int64_t)0 : P.p_base) + i;
    // queries for the global search (counted on their first lane)
    const bool miss = active && c == 0 && sub == 0;
    const unsigned long long mmask = __ballot(miss);
    float bd = INFINITY;
    uint32_t bj = 0xFFFFFFFFu;
    float bx = 0.0f, by = 0.0f, bz = 0.0f;
    bool crowd = false;   // uniform over the wave
    if (kReload && LPQ == 8 && crowded(c)) crowd = crowd_scan(qs4, cs, c, sx, sy, sz, lane, bd, bj);
    if (!crowd && active && c > 0) {
        // U candidates per lane per round, all loads issued before the first
        // compare; no serial remainder
        constexpr int U = LPQ <= 2 ? 8 : 4;
        const float4* seg = qs4 + cs;
        const uint32_t last = c - 1u;
        for (uint32_t k = sub; k < c; k += U * LPQ) {
            float4 a[U];
#pragma unroll
            for (int u = 0; u < U; ++u) a[u] = seg[min(k + (uint32_t)(u * LPQ), last)];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (kReload) consider_pos(a[u], min(k + (uint32_t)(u * LPQ), last), sx, sy, sz, bd, bj);
                else if (kMom) consider<kDirect>(a[u], sx, sy, sz, bd, bj, bx, by, bz);
                else consider<kDirect>(a[u], sx, sy, sz, bd, bj);
            }
        }
    }
    if (LPQ > 1) {
#pragma unroll
        for (int d = 1; d < LPQ; d <<= 1) {
            const float od = xor_lanes(bd, d);
            const uint32_t oj = xor_lanes(bj, d);
            float ox = 0.0f, oy = 0.0f, oz = 0.0f;
            if (kMom && !kReload) {
                ox = xor_lanes(bx, d);
                oy = xor_lanes(by, d);
                oz = xor_lanes(bz, d);
            }
            const bool take = od < bd || (od == bd && oj < bj);
            bd = take ? od : bd;
            bj = take ? oj : bj;
            if (kMom && !kReload) {
                bx = take ? ox : bx;
                by = take ? oy : by;
                bz = take ? oz : bz;
            }
        }
    }
    uint32_t bidx = bj;   // the winner's target index
    if (kReload && active && c > 0 && sub == 0) {
        const float4 wv = qs4[cs + min(bj, c - 1u)];   // bj < c: every distance is finite inside a grid
        bx = wv.x;
        by = wv.y;
        bz = wv.z;
        bidx = __float_as_uint(wv.w);
    }
    // Correspondence form: the wave's queries without a candidate go into its
    // mask (wave w of job b: word b * kWaves + w), for k_nns_global.
    if constexpr (!kMom) {
        if (lane == 0) {
            ctr[(int64_t)jb * kWaves + w] = mmask;
            if (mmask && fb_miss) atomicAdd(&fb_miss[job.pair], (int32_t)__popcll(mmask));
        }
        if (active && c > 0 && sub == 0) {
            nn_idx[gp] = (int32_t)bidx;
            nn_d2[gp] = bd;
        }
        return;
    }
    // Registration: the wave resolves its global searches itself, one query at
    // a time, by the exact tree search over the segments (qsg, whichever layout
    // the local search reads); those without a finite distance, and those behind
    // the wave's budget of crowded voxels' points, are appended to the pair's
    // list for the exhaustive search, one append per wave, each query at its rank
    // among the wave's unresolved ones.  Every global search is
    // counted in fb_miss.
    bool treed = false;
    unsigned long long left = mmask;
    if (mmask) {
        unsigned long long pend = mmask;
        left = 0ull;
        uint32_t budget = S.misses > kManyMisses ? kRareBudget : most;
        while (pend) {   // uniform over the wave
            const int L = __ffsll((long long)pend) - 1;
            pend &= pend - 1ull;
            float rd, rx, ry, rz;
            uint32_t rj;
            const float lx = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sx), L));
            const float ly = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sy), L));
            const float lz = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sz), L));
            if (tree_nearest<kCubeMin, kCrowdBudget>(P, off, pyr, qsg, lx, ly, lz, rd, rj, rx, ry, rz, budget)) {
                if (lane == L) {
                    treed = true;
                    bd = rd;
                    bidx = rj;
                    bx = rx;
                    by = ry;
                    bz = rz;
                }
            } else {
                left |= 1ull << L;
                if (budget == 0u) {   // the others lie in the same crowd
                    left |= pend;
                    pend = 0ull;
                }
            }
        }
        const int leader = __ffsll((long long)mmask) - 1;
        int32_t base = 0;
        if (lane == leader) {
            atomicAdd(&fb_miss[job.pair], (int32_t)__popcll(mmask));
            if (left) base = atomicAdd(&fb_count[job.pair], (int32_t)__popcll(left));
        }
        base = __shfl(base, leader, kWave);
        if ((left >> lane) & 1ull) {
            const int32_t pos = base + (int32_t)__popcll(left & ((1ull << lane) - 1ull));
            fb_list[P.p_base + pos] = i;
            fb_key[P.p_base + pos] = ~0ull;
        }
    }
    const bool found = (active && c > 0 && sub == 0) || treed;
    if (found && nn_idx) {
        nn_idx[gp] = (int32_t)bidx;
        nn_d2[gp] = bd;
    }
    // one record per wave, the float64 moments of Eq. 1 over
    // the wave's resolved queries about the grid centre and three exact
    // counters (candidates scanned, dilated lookups, queries sent to the
    // global search).  No block barrier: the waves of a block finish
    // independently.
    const int64_t rec = (int64_t)jb * kWaves + w;
    const uint32_t ndil = (uint32_t)__popcll(__ballot(dil && sub == 0));
    const uint32_t nfound = (uint32_t)__popcll(__ballot(found));
    const uint32_t ncand = wave_candidates<LPQ>(sub == 0 ? c : 0u);
    wave_record<LPQ>(found, x, y, z, bx, by, bz, bd, P.cx, P.cy, P.cz,
                     [&](int j, double v) { part[rec * kMoments + j] = v; });
    if (lane == 0) {
        part[rec * kMoments + kMoments - 1] = (double)nfound;
    } else if (lane >= 32 && lane < 35) {
        const int k = lane - 32;
        ctr[rec * 3 + k] = k == 0 ? (unsigned long long)ncand
                                  : (unsigned long long)(k == 1 ? ndil : (uint32_t)__popcll(mmask));
    }
}

// Global search.  Work item = (pair, chunk of kFbQ listed queries, tile of
// kFbT targets); items are enumerated from the device-side list lengths, so
// the launch shape is fixed (graph-capturable) whatever the number of misses.
constexpr int kFbThreads = kFbQueries;
constexpr int kFbQ = kFbQueries;
constexpr int kFbT = kFbTargets;
constexpr int kMaxPairs = kFbMaxPairs;

__global__ __launch_bounds__(kFbThreads) void k_fallback(const PairDev* __restrict__ pd, int npairs,
                                                         const float* __restrict__ qx, const float* __restrict__ qy,
                                                         const float* __restrict__ qz, const float* __restrict__ px,
                                                         const float* __restrict__ py, const float* __restrict__ pz,
                                                         const PairState* __restrict__ st,
                                                         const int32_t* __restrict__ fb_count,
                                                         const uint32_t* __restrict__ fb_list,
                                                         unsigned long long* __restrict__ fb_key,
                                                         const FoldJob* __restrict__ fjobs, int nfjobs,
                                                         const double* __restrict__ part,
                                                         const unsigned long long* __restrict__ ctr,
                                                         double* __restrict__ fpart,
                                                         unsigned long long* __restrict__ fctr)
{
    // the per-pair running sum of work items: npairs + 1 entries of dynamic
    // LDS (a single pair needs 16 bytes, not a table for the largest batch)
    extern __shared__ int64_t s_pref[];
    __shared__ float tx[kFbT], ty[kFbT], tz[kFbT];
    // the first kFbThreads pairs' list lengths and target counts do not
    // depend on the fold: loaded before it, used after it
    const bool own0 = (int)threadIdx.x < npairs;
    const int64_t F0 = own0 ? fb_count[threadIdx.x] : 0;
    const int64_t n0 = own0 ? pd[threadIdx.x].n : 0;
    // registration: first fold the search waves' moment records, one group of
    // kGroupUnits units per round (the launch runs anyway, and the fold does
    // not depend on the global search)
    if (fjobs && nfjobs > 0) {
        // rows padded by one element: the moment rows then start in different
        // banks, so neither the transposing stores nor the row sums conflict
        constexpr int kRecs = kGroupUnits * kUnitRecords;
        __shared__ double fv[kMoments][kRecs + 1];
        __shared__ double us[kMoments][kGroupUnits];
        __shared__ unsigned long long fc[2][kRecs + 1];
        for (int f = blockIdx.x; f < nfjobs; f += gridDim.x) {
            // a finished pair's groups are folded too (their sums go unused):
            // testing its flag first would delay every load behind it
            const FoldJob fj = fjobs[f];
            // record b of the round: the w-th of unit u + kUnitSlices i,
            // b = kGroupUnits w + i
            auto record = [&](int b) -> int64_t {
                const int u = fj.u + (b % kGroupUnits) * kUnitSlices, r = u + (b / kGroupUnits) * fj.U;
                return u < fj.U && r < fj.R ? (int64_t)fj.rec0 + r : -1;
            };
            // every load in flight before the first LDS store (a load-store
            // loop waits for each load in turn)
            constexpr int kVals = (kMoments * kRecs + kFbThreads - 1) / kFbThreads;
            static_assert(2 * kRecs <= kFbThreads, "one counter load per thread");
            double v[kVals];
#pragma unroll
            for (int r = 0; r < kVals; ++r) {
                const int e = threadIdx.x + r * kFbThreads, bb = e / kMoments;
                const int64_t rec = bb < kRecs ? record(bb) : -1;
                v[r] = rec >= 0 ? part[rec * kMoments + (e - bb * kMoments)] : 0.0;
            }
            const int ec = threadIdx.x;
            const int64_t crec = ec < 2 * kRecs ? record(ec / 2) : -1;
            const unsigned long long cv = crec >= 0 ? ctr[crec * 3 + (ec & 1)] : 0ull;
#pragma unroll
            for (int r = 0; r < kVals; ++r) {
                const int e = threadIdx.x + r * kFbThreads, bb = e / kMoments;
                if (bb < kRecs) fv[e - bb * kMoments][bb] = v[r];
            }
            if (ec < 2 * kRecs) fc[ec & 1][ec / 2] = cv;
            __syncthreads();
            if (threadIdx.x < kMoments * kGroupUnits) {
                const int j = threadIdx.x / kGroupUnits, i = threadIdx.x % kGroupUnits;
                double a[kUnitRecords];
#pragma unroll
                for (int w = 0; w < kUnitRecords; ++w) a[w] = fv[j][w * kGroupUnits + i];
                us[j][i] = unit_sum(a);
            } else if (threadIdx.x >= kFbThreads - 2) {
                const int j = threadIdx.x - (kFbThreads - 2);
                unsigned long long sm = 0;
                for (int w = 0; w < kRecs; ++w) sm += fc[j][w];
                fctr[(int64_t)j * nfjobs + fj.out] = sm;
            }
            __syncthreads();
            if (threadIdx.x < kMoments) {
                double sm = 0.0;
#pragma unroll
                for (int i = 0; i < kGroupUnits; ++i) sm += us[threadIdx.x][i];
                fpart[(int64_t)threadIdx.x * nfjobs + fj.out] = sm;
            }
        }
    }
    // items per pair (64-bit), loaded in parallel, then an in-LDS running sum
    for (int p = threadIdx.x; p < npairs; p += kFbThreads) {
        const bool first = p == (int)threadIdx.x;
        const int64_t F = first ? F0 : fb_count[p];
        const int64_t n = first ? n0 : pd[p].n;
        s_pref[p + 1] = fallback_items(F, n);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t acc = 0;
        s_pref[0] = 0;
        for (int p = 1; p <= npairs; ++p) {
            acc += s_pref[p];
            s_pref[p] = acc;
        }
    }
    __syncthreads();
    const int64_t total = s_pref[npairs];
    for (int64_t item = blockIdx.x; item < total; item += gridDim.x) {
        int lo = 0, hi = npairs;   // last p with s_pref[p] <= item
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (s_pref[mid] <= item) lo = mid;
            else hi = mid;
        }
        const int p = lo;
        const PairDev& P = pd[p];
        const int64_t local = item - s_pref[p];
        const int64_t ntile = (P.n + kFbT - 1) / kFbT;
        const int64_t qc = local / ntile, tile = local % ntile;
        const int64_t t0 = (int64_t)tile * kFbT;
        const int tn = (int)min((int64_t)kFbT, P.n - t0);
        __syncthreads();
        for (int j = threadIdx.x; j < tn; j += kFbThreads) {
            const int64_t g = P.q_base + t0 + j;
            tx[j] = qx[g];
            ty[j] = qy[g];
            tz[j] = qz[g];
        }
        __syncthreads();
        const int64_t slot = qc * kFbQ + threadIdx.x;
        if (slot < fb_count[p]) {
            const uint32_t i = fb_list[P.p_base + slot];
            const int64_t gp = P.p_base + i;
            float sx, sy, sz;
            transform(st[p].Rtf, px[gp], py[gp], pz[gp], sx, sy, sz);
            float bd = INFINITY;
            int bj = 0;
            for (int j = 0; j < tn; ++j) {
                const float d = dist2(sx, sy, sz, tx[j], ty[j], tz[j]);
                if (d < bd) {
                    bd = d;
                    bj = j;
                }
            }
            const unsigned long long key =
                ((unsigned long long)__float_as_uint(bd) << 32) | (unsigned long long)(uint32_t)(t0 + bj);
            atomicMin(&fb_key[P.p_base + slot], key);
        }
    }
}

// The correspondence form's global searches.  Block b takes the masks b,
// b + gridDim.x, ... of the search's waves, so that every block has its share
// of a region that misses together, lists their queries in LDS, and its waves
// resolve them one each at a time.  Resolved by the wave that met it, a query
// waits for the up to 63 before it, and the longest such chain is the launch:
// the search of a loss over 16 x 40,000 points of which 3 % have no candidate
// took 155 us, now 27 and this launch (forward and backward 390 -> 257 us in
// all); 2,000 queries of which 75 miss took 97 us, now 25.  768 blocks of 8
// waves fill the device; 1536 of 4 waves share less within a block (298 us),
// 256 of 16 waves as much (259).  A query without a finite distance goes to
// target 0, infinitely far.
// Block 0 also hands out the counts.
constexpr int kGlThreads = 512, kGlBatch = 256;
constexpr int kGlMaxBlocks = 768;
template <bool kSorted>
__global__ __launch_bounds__(kGlThreads) void k_nns_global(
    const PairDev* __restrict__ pd, const BlockJob* __restrict__ jobs, int npairs, int nrec, int waves, int lpq,
    const float* __restrict__ px, const float* __restrict__ py, const float* __restrict__ pz,
    const float4* __restrict__ ps4, const PairState* __restrict__ st, const uint32_t* __restrict__ off,
    const uint8_t* __restrict__ pyr, const float4* __restrict__ qs4, const unsigned long long* __restrict__ mask,
    const int32_t* __restrict__ fb_miss, int32_t* __restrict__ nn_idx, float* __restrict__ nn_d2,
    int32_t* __restrict__ n_fallback)
{
    __shared__ uint16_t list[kGlBatch * kWave];   // batch slot * 64 + lane
    __shared__ int32_t count, taken;
    if (blockIdx.x == 0 && n_fallback)
        for (int p = threadIdx.x; p < npairs; p += kGlThreads) n_fallback[p] = fb_miss[p];
    const int lane = threadIdx.x & (kWave - 1);
    for (int64_t b0 = blockIdx.x; b0 < nrec; b0 += (int64_t)kGlBatch * gridDim.x) {
        if (threadIdx.x == 0) count = taken = 0;
        __syncthreads();
        const int64_t r = b0 + (int64_t)threadIdx.x * gridDim.x;
        if (threadIdx.x < kGlBatch && r < nrec) {
            unsigned long long mm = mask[r];
            if (mm) {
                int at = atomicAdd(&count, (int32_t)__popcll(mm));
                for (; mm; mm &= mm - 1ull) list[at++] = (uint16_t)(threadIdx.x * kWave + __ffsll((long long)mm) - 1);
            }
        }
        __syncthreads();
        const int n = count;
        while (true) {
            int e = lane == 0 ? atomicAdd(&taken, 1) : 0;
            e = __builtin_amdgcn_readfirstlane(e);
            if (e >= n) break;
            const int item = __builtin_amdgcn_readfirstlane((int)list[e]);
            const int64_t rec = b0 + (int64_t)(item / kWave) * gridDim.x;
            const int64_t job_at = rec / waves;
            const BlockJob job = jobs[job_at];
            const PairDev& P = pd[job.pair];
            const int64_t at = P.p_base + job.start + ((rec - job_at * waves) * kWave + item % kWave) / lpq;
            const float4 p = kSorted ? ps4[at] : make_float4(px[at], py[at], pz[at], 0.0f);
            const int64_t t = kSorted ? P.p_base + __float_as_uint(p.w) : at;
            float s[3];
            transform(st[job.pair].Rtf, p.x, p.y, p.z, s[0], s[1], s[2]);
            const auto uniform = [](float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); };
            float rd, rx, ry, rz;
            uint32_t rj, budget;
            if (!tree_nearest<kCubeMinNN, kCrowdScan>(P, off, pyr, qs4, uniform(s[0]), uniform(s[1]), uniform(s[2]), rd, rj, rx, ry,
                                                 rz, budget)) {
                rd = INFINITY;
                rj = 0u;
            }
            if (lane == 0) {
                nn_idx[t] = (int32_t)rj;
                nn_d2[t] = rd;
            }
        }
        __syncthreads();
    }
}

}  // namespace

void launch_nns_local(const PairDev* pd, const BlockJob* jobs, int njobs, int block, int lpq, bool sorted, bool mom,
                      const float* px, const float* py, const float* pz, const float4* ps4, const PairState* st,
                      const uint2* dir, const uint32_t* off, const uint8_t* pyr, const float4* qs4, const float4* qsg,
                      int32_t* nn_idx, float* nn_d2, int32_t* fb_count, int32_t* fb_miss, uint32_t* fb_list, unsigned long long* fb_key, unsigned long long* ctr,
                      double* part, const uint32_t* dcnt, uint32_t cap, int mode, int64_t one_m,
                      int early, uint32_t budget, hipStream_t s)
{
    if (njobs <= 0) return;
    const bool one = one_m >= 0;
    // the position-tracking form, for many candidates per query: 4 or 8
    // lanes per query, registration over segments
    if (mode == 1 && mom && !dcnt) {
#define VICP_NNS_R(BS, L, SORTED)                                                                                  \
    if (one)                                                                                                       \
        launch_timed(k_nns_local<BS, L, SORTED, true, false, 1, true>, dim3(njobs), dim3(BS), s, pd, jobs, px, py,  \
                     pz, ps4, st, dir, off, pyr, qs4, qsg, nn_idx, nn_d2, fb_count, fb_miss, fb_list, fb_key, ctr, part, dcnt,    \
                     cap, one_m, early, budget);                                                            \
    else                                                                                                           \
        launch_timed(k_nns_local<BS, L, SORTED, true, false, 1, false>, dim3(njobs), dim3(BS), s, pd, jobs, px, py, \
                     pz, ps4, st, dir, off, pyr, qs4, qsg, nn_idx, nn_d2, fb_count, fb_miss, fb_list, fb_key, ctr, part, dcnt,    \
                     cap, one_m, early, budget)
#define VICP_NNS_RL(BS, SORTED)                                     \
    switch (lpq) {                                                  \
    case 1: VICP_NNS_R(BS, 1, SORTED); break;                       \
    case 2: VICP_NNS_R(BS, 2, SORTED); break;                       \
    case 4: VICP_NNS_R(BS, 4, SORTED); break;                       \
    default: VICP_NNS_R(BS, 8, SORTED); break;                      \
    }
#define VICP_NNS_RB(SORTED)                                         \
    switch (block) {                                                \
    case 128: { VICP_NNS_RL(128, SORTED) } break;                   \
    case 512: { VICP_NNS_RL(512, SORTED) } break;                   \
    default: { VICP_NNS_RL(256, SORTED) } break;                    \
    }
        if (sorted) {
            VICP_NNS_RB(true)
        } else {
            VICP_NNS_RB(false)
        }
#undef VICP_NNS_RB
#undef VICP_NNS_RL
#undef VICP_NNS_R
        return;
    }
#define VICP_NNS(BS, L, SORTED, MOM, DIRECT)                                                                       \
    if (one && !DIRECT)                                                                                            \
        launch_timed(k_nns_local<BS, L, SORTED, MOM, DIRECT, 0, true>, dim3(njobs), dim3(BS), s, pd, jobs, px, py,  \
                     pz, ps4, st, dir, off, pyr, qs4, qsg, nn_idx, nn_d2, fb_count, fb_miss, fb_list, fb_key, ctr, part, dcnt,    \
                     cap, one_m, early, budget);                                                            \
    else                                                                                                           \
        launch_timed(k_nns_local<BS, L, SORTED, MOM, DIRECT, 0, false>, dim3(njobs), dim3(BS), s, pd, jobs, px, py, \
                     pz, ps4, st, dir, off, pyr, qs4, qsg, nn_idx, nn_d2, fb_count, fb_miss, fb_list, fb_key, ctr, part, dcnt,    \
                     cap, one_m, early, budget)
#define VICP_NNS_L(BS, SORTED, MOM, DIRECT)                  \
    switch (lpq) {                                           \
    case 2: VICP_NNS(BS, 2, SORTED, MOM, DIRECT); break;     \
    case 4: VICP_NNS(BS, 4, SORTED, MOM, DIRECT); break;     \
    case 8: VICP_NNS(BS, 8, SORTED, MOM, DIRECT); break;     \
    default: VICP_NNS(BS, 1, SORTED, MOM, DIRECT); break;    \
    }
#define VICP_NNS_BS(SORTED, MOM, DIRECT)                     \
    switch (block) {                                         \
    case 128: VICP_NNS_L(128, SORTED, MOM, DIRECT); break;   \
    case 512: VICP_NNS_L(512, SORTED, MOM, DIRECT); break;   \
    default: VICP_NNS_L(256, SORTED, MOM, DIRECT); break;    \
    }
    // the direct layout serves registrations only
    if (dcnt && mom) {
        if (sorted) {
            VICP_NNS_BS(true, true, true)
        } else {
            VICP_NNS_BS(false, true, true)
        }
    } else if (mom) {
        if (sorted) {
            VICP_NNS_BS(true, true, false)
        } else {
            VICP_NNS_BS(false, true, false)
        }
    } else if (sorted) {
        VICP_NNS_BS(true, false, false)
    } else {
        VICP_NNS_BS(false, false, false)
    }
#undef VICP_NNS_BS
#undef VICP_NNS_L
#undef VICP_NNS
}

bool launch_fallback(const PairDev* pd, int npairs, int grid, const float* qx, const float* qy, const float* qz,
                     const float* px, const float* py, const float* pz, const PairState* st, const int32_t* fb_count,
                     const uint32_t* fb_list, unsigned long long* fb_key, const FoldJob* fjobs, int nfjobs,
                     const double* part, const unsigned long long* ctr, double* fpart,
                     unsigned long long* fctr, hipStream_t s)
{
    if (npairs <= 0 || npairs > kMaxPairs || grid <= 0) return false;
    launch_timed_lds(k_fallback, dim3(grid), dim3(kFbThreads), sizeof(int64_t) * (npairs + 1), s, pd, npairs, qx, qy,
                     qz, px, py, pz, st, fb_count, fb_list, fb_key, fjobs, nfjobs, part, ctr, fpart, fctr);
    return true;
}

void launch_nns_global(const PairDev* pd, const BlockJob* jobs, int npairs, int njobs, int block, int lpq, bool sorted,
                       const float* px, const float* py, const float* pz, const float4* ps4, const PairState* st,
                       const uint32_t* off, const uint8_t* pyr, const float4* qs4, const unsigned long long* mask, const int32_t* fb_miss,
                       int32_t* nn_idx, float* nn_d2, int32_t* n_fallback, hipStream_t s)
{
    if (njobs <= 0) return;
    const int waves = block / kWave;
    const int64_t nrec = (int64_t)njobs * waves;
    const int nb = (int)std::min<int64_t>((nrec + kGlThreads / kWave - 1) / (kGlThreads / kWave), kGlMaxBlocks);
    launch_timed(sorted ? k_nns_global<true> : k_nns_global<false>, dim3(nb), dim3(kGlThreads), s, pd, jobs, npairs,
                 (int)nrec, waves, lpq, px, py, pz, ps4, st, off, pyr, qs4, mask, fb_miss, nn_idx, nn_d2, n_fallback);
}

}  // namespace vicp
