// vicp_api.hip -- host runtime behind the C ABI of include/vicp.h.
//
// It sizes grids, owns device memory, builds the per-block work tables,
// queues the kernels of k_*.hip on the caller's stream, captures the ICP
// iterations in a hipGraph when asked, and reads results back.  No
// arithmetic of the method runs on the host except the grid specification
// (float32 scalar code, identical rounding to the device's).
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <chrono>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "vicp.h"
#include "vicp_internal.hpp"

using namespace vicp;

namespace {

thread_local std::string g_err;

int fail(int code, const std::string& msg)
{
    g_err = msg;
    return code;
}

#define VICP_HIP(expr)                                                                         \
    do {                                                                                       \
        hipError_t e_ = (expr);                                                                \
        if (e_ != hipSuccess) return fail(VICP_ERR_HIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

// ---------------------------------------------------------------- utilities

// Small host -> device uploads travel as kernel arguments, so they never
// depend on the lifetime of the caller's host buffer and can be captured.
constexpr int kBlobWords = 512;
struct Blob {
    uint32_t w[kBlobWords];
};

__global__ void k_upload(Blob b, uint32_t* dst, int nwords)
{
    for (int i = threadIdx.x; i < nwords; i += blockDim.x) dst[i] = b.w[i];
}

// Zeroes up to four arrays (u32, u64, u32, u32) and writes one blob, in one
// launch.
__global__ void k_clear4_blob(Blob blob, uint32_t* __restrict__ dst, int nwords, uint32_t* __restrict__ a, int64_t na,
                              unsigned long long* __restrict__ b, int64_t nb, uint32_t* __restrict__ c, int64_t nc,
                              uint32_t* __restrict__ d, int64_t nd, int64_t n)
{
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < nwords; i += blockDim.x) dst[i] = blob.w[i];
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        if (i < na) a[i] = 0u;
        if (i < nb) b[i] = 0ull;
        if (i < nc) c[i] = 0u;
        if (i < nd) d[i] = 0u;
    }
}

// The first launch of a paired refill and plan (vicp_rebuild_register): the
// pair records (block 0), the zeroing of the refill's histogram, scan states,
// tickets and error words and of the plan's bucket counts, scan states,
// tickets and cap flags, and each pair's state at its pose (poses and source
// sizes travel in the launch: at most kInlinePairs pairs).
struct FrameStart {
    double rt[12 * kInlinePairs];
    int64_t m[kInlinePairs];
    uint32_t* z32[6];
    int64_t n32[6];
    unsigned long long* z64[2];
    int64_t n64[2];
};

__global__ void k_start_frame(Blob blob, uint32_t* __restrict__ dst, int nwords, FrameStart f, int npairs,
                              PairState* __restrict__ st, int32_t* __restrict__ fb_count, int32_t* __restrict__ flags,
                              int64_t n)
{
    if (blockIdx.x == 0) {
        for (int i = threadIdx.x; i < nwords; i += blockDim.x) dst[i] = blob.w[i];
        if ((int)threadIdx.x < npairs)
            init_pair_state(st, threadIdx.x, f.rt + 12 * threadIdx.x, f.m[threadIdx.x], npairs, fb_count, flags);
    }
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
#pragma unroll
        for (int k = 0; k < 6; ++k)
            if (i < f.n32[k]) f.z32[k][i] = 0u;
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (i < f.n64[k]) f.z64[k][i] = 0ull;
    }
}

void launch_clear4_blob(const Blob& blob, uint32_t* dst, int nwords, uint32_t* a, int64_t na, unsigned long long* b,
                        int64_t nb, uint32_t* c, int64_t nc, uint32_t* d, int64_t nd, hipStream_t s)
{
    const int64_t n = std::max(std::max(na, nb), std::max(nc, nd));
    const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 2048));
    hipLaunchKernelGGL(k_clear4_blob, dim3(blocks), dim3(256), 0, s, blob, dst, nwords, a, na, b, nb, c, nc, d, nd, n);
}

// Waits until each of `count` words in pinned host memory, `stride` words
// apart, holds the tag (device kernels write it after the values it
// guards).  Spins on the host for up to a millisecond (no stream
// synchronisation, whose wake-up is slower); a longer wait synchronises
// the stream instead (no busy host thread) and then looks once more.
hipError_t wait_tags(const uint32_t* first, int count, size_t stride, uint32_t tag, hipStream_t s)
{
    const auto t0 = std::chrono::steady_clock::now();
    int next = 0;
    for (;;) {
        while (next < count && __atomic_load_n(&first[stride * (size_t)next], __ATOMIC_ACQUIRE) == tag) ++next;
        if (next == count) return hipSuccess;
        if (std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(1)) break;
    }
    const hipError_t e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    for (; next < count; ++next)
        if (__atomic_load_n(&first[stride * (size_t)next], __ATOMIC_ACQUIRE) != tag) return hipErrorUnknown;
    return hipSuccess;
}

// Copies the registration's result block (state, histories, counters,
// flags) into mapped pinned host memory, block b the words [b * chunk,
// (b + 1) * chunk), then writes the call's tag into the b-th word after the
// block: each thread's stores are fenced at system scope before the
// barrier, and the tag is the block's last store.
constexpr int kPublishMaxBlocks = 64;
constexpr int64_t kPublishChunk = 2048;   // words per block (a batch's histories span many)

__global__ __launch_bounds__(256) void k_publish(const uint32_t* __restrict__ src, uint32_t* dst, int64_t words,
                                                 uint32_t tag)
{
    const int64_t chunk = (words + gridDim.x - 1) / gridDim.x;
    const int64_t w0 = (int64_t)blockIdx.x * chunk, w1 = min(words, w0 + chunk);
    for (int64_t i = w0 + threadIdx.x; i < w1; i += blockDim.x) dst[i] = src[i];
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(dst + words + blockIdx.x, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

int publish_blocks(int64_t words)
{
    return (int)std::max<int64_t>(1, std::min<int64_t>(kPublishMaxBlocks, (words + kPublishChunk - 1) / kPublishChunk));
}

void launch_publish(const uint32_t* src, uint32_t* dst, int64_t words, uint32_t tag, hipStream_t s)
{
    hipLaunchKernelGGL(k_publish, dim3(publish_blocks(words)), dim3(256), 0, s, src, dst, words, tag);
}

void upload(const void* host, size_t bytes, void* dst, hipStream_t s)
{
    const uint32_t* src = (const uint32_t*)host;
    size_t words = bytes / 4;
    uint32_t* d = (uint32_t*)dst;
    while (words > 0) {
        Blob b;
        const int n = (int)std::min<size_t>(words, kBlobWords);
        memcpy(b.w, src, (size_t)n * 4);
        hipLaunchKernelGGL(k_upload, dim3(1), dim3(256), 0, s, b, d, n);
        src += n;
        d += n;
        words -= n;
    }
}

__global__ void k_export_off(const uint32_t* __restrict__ off, int64_t count, uint32_t base, uint32_t* __restrict__ out)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = off[i] - base;
}

__global__ void k_grid_stats(const uint32_t* __restrict__ hist, const uint32_t* __restrict__ off,
                             const uint32_t* __restrict__ vm, int64_t V, unsigned long long* out)
{
    unsigned long long occ = 0, dil = 0, mx = 0;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < V; v += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t h = hist[v];
        const uint32_t o = off[v];   // loaded with the count, not after it
        if (h) {
            occ += 1;
            mx = max(mx, (unsigned long long)h);
        } else if (vm[(int64_t)o + 1] & kMask) {
            dil += 1;
        }
    }
    // one set of atomics per wave
    for (int d = 32; d > 0; d >>= 1) {
        occ += __shfl_xor(occ, d, 64);
        dil += __shfl_xor(dil, d, 64);
        mx = max(mx, __shfl_xor(mx, d, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        if (occ) atomicAdd(&out[0], occ);
        if (dil) atomicAdd(&out[1], dil);
        if (mx) atomicMax(&out[2], mx);
    }
}

// ----------------------------------------------------------- per-kernel timing

struct ProfRec {
    const char* name;
    hipEvent_t a, b;
};

struct Prof {
    std::mutex mu;
    bool on = false;
    std::vector<ProfRec> recs;
    std::vector<hipEvent_t> pool;
    std::map<std::string, std::pair<int64_t, double>> acc;
    std::map<std::string, std::vector<double>> samples;   // each launch's milliseconds, in launch order
} g_prof;

// Host-side work timed on the host clock (e.g. the host offset scan).
void prof_add_host(const char* name, double ms)
{
    std::lock_guard<std::mutex> lk(g_prof.mu);
    if (!g_prof.on) return;
    auto& x = g_prof.acc[name];
    x.first += 1;
    x.second += ms;
}

hipEvent_t prof_event()
{
    if (!g_prof.pool.empty()) {
        hipEvent_t e = g_prof.pool.back();
        g_prof.pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    (void)hipEventCreate(&e);
    return e;
}

void prof_flush_locked()
{
    for (auto& r : g_prof.recs) {
        float ms = 0.0f;
        (void)hipEventSynchronize(r.b);
        if (hipEventElapsedTime(&ms, r.a, r.b) == hipSuccess) {
            auto& x = g_prof.acc[r.name];
            x.first += 1;
            x.second += ms;
            g_prof.samples[r.name].push_back(ms);
        }
        g_prof.pool.push_back(r.a);
        g_prof.pool.push_back(r.b);
    }
    g_prof.recs.clear();
}

// Events recorded while a registration is being captured: they become event
// nodes of the graph and time each kernel of every replay.
thread_local std::vector<ProfRec>* t_capture_events = nullptr;

// Brackets one launch with events when timing is on.  Outside capture the
// pair is read at the next vicp_prof_read; inside capture it is kept with the
// graph and read after each replay.
// Records an event on a stream.  Under capture, the event goes in as an
// explicit event-record node after the stream's current dependencies (an
// event recorded through capture cannot be timed on this runtime; an
// explicit node can).
void record_event(hipEvent_t e, hipStream_t s, bool capturing)
{
    if (!capturing) {
        (void)hipEventRecord(e, s);
        return;
    }
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    unsigned long long id = 0;
    hipGraph_t graph = nullptr;
    const hipGraphNode_t* deps = nullptr;
    size_t ndeps = 0;
    if (hipStreamGetCaptureInfo_v2(s, &cs, &id, &graph, &deps, &ndeps) != hipSuccess ||
        cs != hipStreamCaptureStatusActive) {
        (void)hipGetLastError();
        return;
    }
    hipGraphNode_t node = nullptr;
    if (hipGraphAddEventRecordNode(&node, graph, deps, ndeps, e) != hipSuccess ||
        hipStreamUpdateCaptureDependencies(s, &node, 1, hipStreamSetCaptureDependencies) != hipSuccess)
        (void)hipGetLastError();
}

// The events of the open timed scope, for a launch that records them at the
// kernel's own start and end (launch_timed).
struct ExtEvents {
    hipEvent_t a = nullptr, b = nullptr;
    bool used = false;
};
thread_local ExtEvents* t_ext = nullptr;

// A timed scope: events around the work queued inside it.  With ext set and
// no capture, a launch_timed launch inside the scope takes the events
// instead, which excludes the launch overhead from the measured time.
struct ProfScope {
    hipStream_t s;
    const char* name;
    bool cap;
    hipEvent_t a = nullptr, b = nullptr;
    ExtEvents ext;
    bool use_ext = false;
    ProfScope(const char* nm, hipStream_t st, bool capturing, bool ext_launch = false) : s(st), name(nm), cap(capturing)
    {
        if (!g_prof.on) return;
        if (capturing && !t_capture_events) return;
        std::lock_guard<std::mutex> lk(g_prof.mu);
        a = prof_event();
        b = prof_event();
        use_ext = ext_launch && !capturing;
        if (use_ext) {
            ext.a = a;
            ext.b = b;
            t_ext = &ext;
        } else {
            record_event(a, s, cap);
        }
        if (capturing)
            t_capture_events->push_back({name, a, b});
        else
            g_prof.recs.push_back({name, a, b});
    }
    ~ProfScope()
    {
        if (!b) return;
        if (use_ext) {
            t_ext = nullptr;
            if (!ext.used) {   // nothing was launched: an empty interval
                (void)hipEventRecord(a, s);
                (void)hipEventRecord(b, s);
            }
        } else {
            record_event(b, s, cap);
        }
    }
};

}  // namespace

bool vicp::prof_take_ext_events(hipEvent_t* start, hipEvent_t* stop)
{
    if (!t_ext || t_ext->used) return false;
    t_ext->used = true;
    *start = t_ext->a;
    *stop = t_ext->b;
    return true;
}

namespace {

// After a replay has finished: add the graph's kernel times.  Runtimes that
// cannot time events recorded by a graph report an error here; it is cleared
// and the graph's kernels simply go untimed.
void prof_add_graph(const std::vector<ProfRec>& evs)
{
    std::lock_guard<std::mutex> lk(g_prof.mu);
    for (auto& r : evs) {
        float ms = 0.0f;
        if (hipEventElapsedTime(&ms, r.a, r.b) == hipSuccess && ms >= 0.0f) {
            auto& x = g_prof.acc[r.name];
            x.first += 1;
            x.second += ms;
            g_prof.samples[r.name].push_back(ms);
        } else {
            (void)hipGetLastError();
            g_prof.acc["graph_untimed"].first += 1;
        }
    }
}

void prof_return(std::vector<ProfRec>& evs)
{
    std::lock_guard<std::mutex> lk(g_prof.mu);
    for (auto& r : evs) {
        g_prof.pool.push_back(r.a);
        g_prof.pool.push_back(r.b);
    }
    evs.clear();
}

// ---------------------------------------------------------------- memory

struct Mem {
    vicp_allocator a{};
    bool custom = false;
    void* get(size_t bytes, hipStream_t s)
    {
        bytes = std::max<size_t>(bytes, 256);
        if (custom) return a.alloc(bytes, s, a.user);
        void* p = nullptr;
        if (hipMallocAsync(&p, bytes, s) != hipSuccess) {
            (void)hipGetLastError();
            if (hipMalloc(&p, bytes) != hipSuccess) return nullptr;
        }
        return p;
    }
    void put(void* p, size_t bytes, hipStream_t s)
    {
        if (!p) return;
        bytes = std::max<size_t>(bytes, 256);
        if (custom) {
            a.free(p, bytes, s, a.user);
            return;
        }
        if (hipFreeAsync(p, s) != hipSuccess) {
            (void)hipGetLastError();
            (void)hipFree(p);
        }
    }
};

struct Buf {
    void* p = nullptr;
    size_t bytes = 0;
};

// One allocation that holds a set of buffers laid out together: measured by a
// first pass over the same calls, then taken from.  A set that is laid out
// again (another voxel or source count) keeps the allocation while it fits and
// is not four times too large.
struct Arena {
    Buf buf;
    size_t used = 0, need = 0;
    bool measuring = false;
};

struct PairHost {
    int64_t n = 0, q_base = 0, V = 0, v_base = 0, vm_base = 0, t_base = 0;
    float origin[3] = {0, 0, 0}, inv = 0, voxel = 0;
    int32_t dims[3] = {0, 0, 0};
};

// Block table: every block serves one pair; `items` items per block.
void make_jobs(const std::vector<int64_t>& counts, int items, std::vector<BlockJob>& jobs, std::vector<int32_t>* begin)
{
    jobs.clear();
    if (begin) begin->assign(1, 0);
    for (size_t p = 0; p < counts.size(); ++p) {
        for (int64_t s = 0; s < counts[p]; s += items) jobs.push_back({(int32_t)p, (int32_t)s});
        if (begin) begin->push_back((int32_t)jobs.size());
    }
}

// Work tables of source points: queries per block.
constexpr int kNumTables = 6;
constexpr int kQpb[kNumTables] = {16, 32, 64, 128, 256, 512};
constexpr int kT256 = 4;   // the 256-per-block table (one lane per point kernels)
// The resident loop: most units of all pairs (their messages: 1.4 MB) and most
// blocks.
constexpr int64_t kLoopMaxUnits = 4096;
constexpr int kLoopMaxBlocks = 512;
// The most units a block of the loop takes in turn.  With 196 units of 1024
// queries on 196 blocks (200,000 points) a step takes 11 us against 18 in three
// launches; with two units a block (120,000 points at four lanes, a
// tenth without counterpart) 30 steps take 13.4 ms against 28.8, by its balanced
// global searches; with seven (1.8M points) it took 3.5 ms
// for 30 steps against 2.6: the launch-per-step search then has twice the waves
// in flight on each compute unit, and its launches no longer count.  Between, on a
// 64^3 grid over a room of 226,000, four lanes: 25.9 against 29.4 us with two units,
// 35.8 and 36.5 with three, 41.7 and 43.1 with four, 60.1 and 56.0 with six.
constexpr int64_t kLoopRounds = 2;
static_assert(kLoopRounds <= kLoopAloneUnits, "a pair on one block keeps its units' sums there");
// One on a crowded grid, whose steps are the search's time and nothing else: a
// 16^3 grid over the same room, four lanes, 400 units in pairs take 200.8 us,
// 155.6 in launches, and 8^3 499 and 411; with 7 points a voxel (32^3) 59.7 and
// 49.8, with 3 34.6 and 33.8.
constexpr int64_t kLoopRoundsCrowded = 1;
// A crowded grid: its voxels hold this many points on average.
constexpr int64_t kCrowdedPoints = 4;
// Waves per search block (128, 256 or 512 threads): the search writes one
// moment record per wave.
constexpr int kNumWpb = 3;
constexpr int kWpb[kNumWpb] = {2, 4, 8};

int wpb_index(int nns_block)
{
    const int w = nns_block / 64;
    return w <= 2 ? 0 : (w <= 4 ? 1 : 2);
}

int table_of(int qpb)
{
    for (int i = 0; i < kNumTables; ++i)
        if (kQpb[i] == qpb) return i;
    return kT256;
}

}  // namespace

// ------------------------------------------------------------------ the grid

struct vicp_grid {
    int B = 0;
    const float *qx = nullptr, *qy = nullptr, *qz = nullptr;
    int64_t n_total = 0, V_total = 0, vm_words = 0;
    int32_t pad = 0, rings_applied = 0;
    bool dilated = false;
    std::vector<PairHost> pairs;
    std::vector<float> voxels;
    Mem mem;
    Arena owned;     // sized by the target point counts (fixed for the grid)
    Arena vbufs;     // sized by the voxel counts (change when a rebuild changes V)

    PairDev* d_pd = nullptr;
    uint32_t* err = nullptr;
    BlockJob* jobs_q = nullptr;      // 256 target points per block
    int njobs_q = 0;
    BlockJob* jobs_q512 = nullptr;   // 512 and 1024 target points per block (count schedules)
    int njobs_q512 = 0;
    BlockJob* jobs_q1024 = nullptr;
    int njobs_q1024 = 0;
    BlockJob* jobs_q8 = nullptr;     // 2048 target points per block (bounding box)
    int njobs_q8 = 0;
    uint32_t *vox = nullptr, *rank = nullptr, *slots = nullptr;
    uint32_t* big_list = nullptr;   // voxels whose segments are sorted whole (fixed grids)
    float4* qs4 = nullptr;
    uint32_t *hist = nullptr, *off = nullptr, *vm = nullptr;
    uint8_t* pyr = nullptr;   // occupancy pyramids of the pairs, in the words after hist (zeroed with it)
    int64_t pyr_words = 0;
    uint2* dir = nullptr;   // per voxel: (start in qs4, count | mask), root's entry for a dilated voxel
    BlockJob* jobs_v = nullptr;
    int njobs_v = 0;
    BlockJob* jobs_t[kDilateShapes] = {};   // voxel tiles of the one-launch dilation, per tile shape
    int njobs_t[kDilateShapes] = {};
    unsigned long long* scan_status = nullptr;
    uint32_t* scan_ticket = nullptr;
    uint32_t *dil_a = nullptr, *dil_b = nullptr;

    // schedule choices (never change a result)
    int count_block = 256;   // target points per count block
    bool dil_fused = true;   // 1-4 rings in one launch (else one launch per ring)
    int dil_shape = 0;       // tile shape of the one-launch dilation
    int ring_block = 256;    // threads per block of the ring-by-ring dilation
    int nns_block = 256;
    int nns_lpq = 4;
    int fb_grid = 128;
    bool sort_src = true;
    int search_mode = 0;   // 0 gather, 1 position tracking (4 or 8 lanes per query)

    // source workspace
    std::vector<int64_t> m;   // source layout currently in d_pd / tables
    int64_t m_total = -1;
    int64_t ws_V = -1;
    int K_cap = 0;
    PairState* st = nullptr;
    // every per-registration output (state, histories, counters, flags) lives
    // in one device block, read back with one copy into pinned host memory
    char* res = nullptr;
    size_t res_bytes = 0;
    size_t o_rmse = 0, o_ctr = 0, o_fb = 0, o_deg = 0, o_flags = 0, o_abort = 0;
    // pinned host memory mapped for the device: the result block, then the
    // tag of the registration that wrote it (res_gen)
    void* h_res = nullptr;
    void* d_hres = nullptr;
    size_t h_res_cap = 0;
    uint32_t res_gen = 0;
    // pinned host memory mapped for the device: the per-block bounding-box
    // partials, each tagged with its build's number (box_gen)
    uint32_t* h_box = nullptr;
    uint32_t* d_box = nullptr;
    uint32_t box_gen = 0;
    std::vector<PairDev> h_pd;   // the pair records of the last refill, written by its first launch
    // a given grid geometry (single pair) instead of the target's padded box
    bool fixed = false;
    bool usable = true;   // false from a refill's grid specification until its kernels are queued, or after it failed
    // the Alg. 1 ablation: host-side offset scan, fused 32-bit LDS hash entries
    bool host_offsets = false, packed_hash = false;
    std::vector<uint32_t> h_hist, h_off;
    float f_origin[3] = {0, 0, 0};
    int32_t f_dims[3] = {0, 0, 0};
    // VANICP's monolithic layout, built beside the segmented one as a
    // comparator (single pair): V fixed blocks of dcap 16-byte records and a
    // count word per voxel.  Allocated directly (tens of GB at 64 KiB per
    // voxel), freed by vicp_direct_free or with the grid.
    float4* dblk = nullptr;
    size_t dblk_bytes = 0;
    uint32_t* dcnt = nullptr;
    size_t dcnt_bytes = 0;
    uint32_t dcap = 0;
    bool direct_ready = false;   // false again after any rebuild
    std::vector<BlockJob> h_jobs_q8;
    void* staging = nullptr;
    int32_t* fb_count = nullptr;
    uint32_t* fb_list = nullptr;
    unsigned long long* fb_key = nullptr;
    int32_t* nn_idx = nullptr;
    float* nn_d2 = nullptr;
    double* part = nullptr;
    int32_t* job_begin = nullptr;       // per pair, blocks of the 256-point table (inside job_begin6)
    int32_t* job_begin6 = nullptr;      // per pair, blocks of each source table
    BlockJob* jobs_p[kNumTables] = {};
    int njobs_p[kNumTables] = {};
    // fold jobs of the search's per-wave records, per search table and waves
    // per block (kWpb)
    FoldJob* fjobs[kNumTables][kNumWpb] = {};
    int nfjobs[kNumTables][kNumWpb] = {};
    int32_t* fold_begin6 = nullptr;     // per table, waves per block and pair: first fold unit
    double* fpart = nullptr;            // per fold unit: folded moment partials
    unsigned long long* fctr = nullptr; // per fold unit: folded counters
    int32_t* flags = nullptr;
    double* jl6 = nullptr;
    double* rmse_hist = nullptr;
    int32_t* fb_hist = nullptr;
    int32_t* deg_hist = nullptr;
    unsigned long long* ctr = nullptr;        // per search block: candidates, dilated lookups, global searches
    unsigned long long* ctr_hist = nullptr;   // candidates and dilated lookups per pair and iteration
    double* npart = nullptr;                  // per search block: the moment partials (registration)
    uint32_t *sh = nullptr, *soff = nullptr, *skey = nullptr, *srank = nullptr, *sidx = nullptr;
    int32_t* sbig = nullptr;   // per pair: a bucket exceeded kRankCap (index order)
    float4* ps4 = nullptr;
    unsigned long long* s_status = nullptr;
    uint32_t* s_ticket = nullptr;
    Arena ws_bufs;   // sized by the source point counts
    Arena wv_bufs;   // the source buckets', by the voxel counts too
    Arena ex_bufs;   // the exhaustive search's, from its first use

    // the exhaustive search's partial minima (null until its first use)
    uint2* ex_part = nullptr;
    int ex_splits = 1;
    // the resident loop's messages, and the last tag used in them (no tag is 0)
    unsigned long long *loop_msg = nullptr, *loop_pose = nullptr;
    int64_t loop_units = 0;
    uint32_t loop_tag = 0;
    uint64_t loop_begun = 0;        // blocks of all loops launched since the layout
    uint64_t loop_arrive = kLoopArrive, loop_patience = kLoopPatience;
    int loop_rest = 0;              // registrations to run without the loop (kLoopRest)
    LoopJob* loop_jobs = nullptr;   // a batch's blocks, for loop_lpq lanes per query
    int loop_lpq = 0, loop_blocks = 0;
    uint32_t step_budget = kRareBudget;   // of the launch-per-step search's waves (kStepBudget)
    int32_t last_form = VICP_FORM_NONE;   // how the last registration ran

    // Captured work: the registration (plan + iterations).
    struct Captured {
        hipGraphExec_t exec = nullptr;
        std::vector<uintptr_t> key;
        std::vector<ProfRec> events;   // per-kernel event pairs inside the graph (timing on)
        void drop()
        {
            if (exec) (void)hipGraphExecDestroy(exec);
            exec = nullptr;
            key.clear();
            prof_return(events);
        }
    };
    Captured reg;
    hipStream_t cap_stream = nullptr;

    // A buffer of the arena (only its size is noted while it is measured).
    static void* take(size_t bytes, Arena& a, bool& ok)
    {
        bytes = (std::max<size_t>(bytes, 1) + 255) & ~(size_t)255;
        if (a.measuring) {
            a.need += bytes;
            return nullptr;
        }
        if (a.used + bytes > a.buf.bytes) {
            ok = false;
            return nullptr;
        }
        void* p = (char*)a.buf.p + a.used;
        a.used += bytes;
        return p;
    }
    // Lays the arena out: body(ok) takes its buffers.  An allocation that does
    // not fit is replaced (by one an eighth larger, so that a count that moves
    // a little from frame to frame does not replace it each time).
    template <typename F>
    bool lay_out(Arena& a, hipStream_t s, F&& body)
    {
        bool ok = true;
        a.measuring = true;
        a.need = 0;
        body(ok);
        a.measuring = false;
        if (a.buf.bytes < a.need || a.buf.bytes / 4 > a.need) {
            const size_t spare = a.buf.p ? a.need / 8 : 0;
            if (a.buf.p && hipStreamSynchronize(s) != hipSuccess) return false;
            release(a, s);
            a.buf.bytes = a.need + spare;
            a.buf.p = mem.get(a.buf.bytes, s);
            if (!a.buf.p && spare) {   // near the end of the memory: what it needs
                a.buf.bytes = a.need;
                a.buf.p = mem.get(a.buf.bytes, s);
            }
            if (!a.buf.p) {
                a.buf.bytes = 0;
                return false;
            }
        }
        a.used = 0;
        body(ok);
        return ok;
    }
    void release(Arena& a, hipStream_t s)
    {
        mem.put(a.buf.p, a.buf.bytes, s);
        a.buf = Buf{};
        a.used = 0;
    }
    void drop_graph() { reg.drop(); }
    int64_t extra_bytes() const
    {
        int64_t b = 0;
        for (const Arena* x : {&owned, &vbufs, &ws_bufs, &wv_bufs, &ex_bufs}) b += (int64_t)x->buf.bytes;
        // the paper's accounting: histogram + offsets (8 V) and the dilated voxel index (4 (n + 2V))
        return b - 8 * V_total - 4 * (n_total + 2 * V_total);
    }
};

namespace {

bool capturing(hipStream_t s)
{
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cs) != hipSuccess) return false;
    return cs == hipStreamCaptureStatusActive;
}

// The target and grid fields of one pair's device record.
void fill_grid_fields(const PairHost& h, int32_t pad, PairDev& d)
{
    d.q_base = h.q_base;
    d.n = h.n;
    d.v_base = h.v_base;
    d.V = h.V;
    d.ox = h.origin[0];
    d.oy = h.origin[1];
    d.oz = h.origin[2];
    d.inv = h.inv;
    d.Dx = h.dims[0];
    d.Dy = h.dims[1];
    d.Dz = h.dims[2];
    d.fDx = (float)h.dims[0];
    d.fDy = (float)h.dims[1];
    d.fDz = (float)h.dims[2];
    d.cx = h.origin[0] + 0.5f * (float)h.dims[0] * h.voxel;
    d.cy = h.origin[1] + 0.5f * (float)h.dims[1] * h.voxel;
    d.cz = h.origin[2] + 0.5f * (float)h.dims[2] * h.voxel;
    d.pad = pad;
    d.t_base = h.t_base;
    d.t_top = pyramid_top(h.dims);
}

void fill_pairdev(const vicp_grid* g, std::vector<PairDev>& pd)
{
    pd.assign(g->B, PairDev{});
    int64_t pb = 0, sb = 0;
    for (int p = 0; p < g->B; ++p) {
        const PairHost& h = g->pairs[p];
        PairDev& d = pd[p];
        fill_grid_fields(h, g->pad, d);
        if ((int)g->m.size() == g->B) {
            d.p_base = pb;
            d.m = g->m[p];
            const SrcChunks sc = src_chunks(h.V, g->m[p]);
            d.s_base = sb;
            d.s_chunks = sc.chunks;
            d.s_shift = sc.shift;
            pb += g->m[p];
            sb += h.V * sc.chunks + (g->m[p] + kOutChunk - 1) / kOutChunk;
        }
    }
}

// Source buckets of a layout: per pair, V voxel buckets (times the index
// chunks of a coarse grid) and the "outside" chunks.
int64_t source_buckets(const vicp_grid* g, const std::vector<int64_t>& m)
{
    int64_t nb = 0;
    for (int p = 0; p < g->B; ++p)
        nb += g->pairs[p].V * src_chunks(g->pairs[p].V, m[p]).chunks + (m[p] + kOutChunk - 1) / kOutChunk;
    return nb;
}

// The source buckets' workspaces, which depend on the voxel counts.
int ensure_buckets(vicp_grid* g, hipStream_t s)
{
    const int64_t nb = source_buckets(g, g->m);
    g->ws_V = -1;
    const bool ok = g->lay_out(g->wv_bufs, s, [&](bool& ok) {
        g->sh = (uint32_t*)g->take(sizeof(uint32_t) * nb, g->wv_bufs, ok);
        g->soff = (uint32_t*)g->take(sizeof(uint32_t) * (nb + 1), g->wv_bufs, ok);
        g->s_status = (unsigned long long*)g->take(sizeof(unsigned long long) * std::max(scan_tiles(nb), 1), g->wv_bufs, ok);
    });
    if (!ok) return fail(VICP_ERR_OOM, "workspace allocation failed");
    g->ws_V = g->V_total;
    return VICP_OK;
}

// A table's place in a block of host tables.
template <typename T>
size_t add_table(std::vector<char>& block, const std::vector<T>& t)
{
    const size_t at = (block.size() + 255) & ~(size_t)255;
    block.resize(at + std::max<size_t>(sizeof(T) * t.size(), 1));
    if (!t.empty()) memcpy(block.data() + at, t.data(), sizeof(T) * t.size());
    return at;
}

// (Re)build the source-side device state for a per-pair source layout.
// Synchronises when the layout changes (rare), so that host staging can be
// released safely.
int ensure_source(vicp_grid* g, const int64_t* m_per_pair, int K, hipStream_t s)
{
    std::vector<int64_t> m(m_per_pair, m_per_pair + g->B);
    for (auto v : m)
        if (v < 0 || v > (int64_t)INT32_MAX) return fail(VICP_ERR_INVALID_ARG, "source size out of range");
    if (m == g->m && K <= g->K_cap) {
        if (g->ws_V == g->V_total) return VICP_OK;
        g->drop_graph();
        return ensure_buckets(g, s);
    }
    g->drop_graph();
    g->release(g->ex_bufs, s);
    g->ex_part = nullptr;
    g->m.clear();
    g->K_cap = 0;
    g->ws_V = -1;
    const int B = g->B;
    int64_t mt = 0;
    for (auto v : m) mt += v;
    const int Kc = std::max(K, 1);
    std::vector<BlockJob> jobs[kNumTables];
    std::vector<int32_t> begin;
    std::vector<int32_t> begin6;
    std::vector<FoldJob> folds[kNumTables][kNumWpb];
    std::vector<int32_t> fbegin6;
    size_t max_rec = 1, max_units = 1;
    for (int k = 0; k < kNumTables; ++k) {
        make_jobs(m, kQpb[k], jobs[k], &begin);
        begin6.insert(begin6.end(), begin.begin(), begin.end());
        for (int wi = 0; wi < kNumWpb; ++wi) {
            // pair p's records are the first R from begin[p] * wpb (the waves
            // of its last block past its last query add nothing)
            const int32_t wpb = kWpb[wi], lpq = 64 * wpb / kQpb[k];
            int32_t units = 0;
            fbegin6.push_back(0);
            for (int p = 0; p < B; ++p) {
                const int32_t R = lpq >= 1 && lpq <= 8 ? (int32_t)wave_records(m[p], lpq) : 0;
                const int32_t U = (int32_t)record_units(R);
                // groups in the order of their sums: slice by slice
                for (int32_t g0 = 0; g0 < U; g0 += kGroupSpan)
                    for (int32_t u = g0; u < std::min(U, g0 + kUnitSlices); ++u)
                        folds[k][wi].push_back({p, begin[p] * wpb, R, U, u, units++});
                fbegin6.push_back(units);
            }
            if (units) max_rec = std::max(max_rec, (size_t)begin[B] * wpb);
            max_units = std::max(max_units, (size_t)units);
        }
    }
    const size_t mt1 = (size_t)std::max<int64_t>(mt, 1);
    {
        auto a8 = [](size_t x) { return (x + 7) & ~(size_t)7; };
        const size_t bk = (size_t)B * Kc;
        g->o_rmse = a8(sizeof(PairState) * B);
        g->o_ctr = g->o_rmse + sizeof(double) * bk;
        g->o_fb = g->o_ctr + sizeof(unsigned long long) * 2 * bk;
        g->o_deg = g->o_fb + sizeof(int32_t) * bk;
        g->o_flags = g->o_deg + sizeof(int32_t) * bk;
        g->o_abort = a8(g->o_flags + sizeof(int32_t) * B);
        g->res_bytes = g->o_abort + 16;   // the abort word and the count of blocks begun
        if (g->h_res_cap < g->res_bytes) {
            if (g->h_res) (void)hipHostFree(g->h_res);
            g->h_res = nullptr;
            g->d_hres = nullptr;
            g->h_res_cap = 0;
            const size_t bytes = g->res_bytes + 4 * kPublishMaxBlocks;   // the tags after the block
            if (hipHostMalloc(&g->h_res, bytes, hipHostMallocMapped | hipHostMallocCoherent) == hipSuccess &&
                hipHostGetDevicePointer(&g->d_hres, g->h_res, 0) == hipSuccess) {
                memset(g->h_res, 0, bytes);   // no tag is 0
                g->h_res_cap = g->res_bytes;
            } else {
                if (g->h_res) (void)hipHostFree(g->h_res);
                g->h_res = nullptr;
                g->d_hres = nullptr;
                return fail(VICP_ERR_OOM, "pinned host allocation failed");
            }
        }
    }
    // messages of the finest schedule (8 lanes per query) the loop takes
    g->loop_units = 0;
    for (int p = 0; p < B; ++p) g->loop_units += record_units(wave_records(m[p], 8));
    g->loop_units = std::min<int64_t>(g->loop_units, kLoopMaxUnits);
    const int64_t loop_words = g->loop_units * kLoopWords + (int64_t)B * kPoseWords;
    // all tables in one host block, for one copy
    std::vector<char> tables;
    size_t t_jobs[kNumTables], t_folds[kNumTables][kNumWpb];
    for (int k = 0; k < kNumTables; ++k) {
        t_jobs[k] = add_table(tables, jobs[k]);
        g->njobs_p[k] = (int)jobs[k].size();
        for (int wi = 0; wi < kNumWpb; ++wi) {
            t_folds[k][wi] = add_table(tables, folds[k][wi]);
            g->nfjobs[k][wi] = (int)folds[k][wi].size();
        }
    }
    const size_t t_fbegin = add_table(tables, fbegin6), t_begin = add_table(tables, begin6);
    char* d_tables = nullptr;
    const bool ok = g->lay_out(g->ws_bufs, s, [&](bool& ok) {
    Arena& L = g->ws_bufs;
    g->res = (char*)g->take(g->res_bytes, L, ok);
    d_tables = (char*)g->take(tables.size(), L, ok);
    g->staging = g->take(sizeof(double) * 12 * B, L, ok);
    // per pair: the global-search list's length, then (fb_count + B) every
    // query that needed a global search, resolved in place or listed
    g->fb_count = (int32_t*)g->take(sizeof(int32_t) * 2 * B, L, ok);
    g->fb_list = (uint32_t*)g->take(sizeof(uint32_t) * mt1, L, ok);
    g->fb_key = (unsigned long long*)g->take(sizeof(unsigned long long) * mt1, L, ok);
    g->nn_idx = (int32_t*)g->take(sizeof(int32_t) * mt1, L, ok);
    g->nn_d2 = (float*)g->take(sizeof(float) * mt1, L, ok);
    g->part = (double*)g->take(sizeof(double) * kMoments * std::max<size_t>(jobs[kT256].size(), 1), L, ok);
    g->jl6 = (double*)g->take(sizeof(double) * 36 * B, L, ok);
    g->ctr = (unsigned long long*)g->take(sizeof(unsigned long long) * 3 * max_rec, L, ok);
    g->npart = (double*)g->take(sizeof(double) * kMoments * max_rec, L, ok);
    g->fpart = (double*)g->take(sizeof(double) * kMoments * max_units, L, ok);
    g->fctr = (unsigned long long*)g->take(sizeof(unsigned long long) * 2 * max_units, L, ok);
    g->skey = (uint32_t*)g->take(sizeof(uint32_t) * mt1, L, ok);
    g->srank = (uint32_t*)g->take(sizeof(uint32_t) * mt1, L, ok);
    g->sidx = (uint32_t*)g->take(sizeof(uint32_t) * (mt1 + 4), L, ok);   // +4: rank_in reads 16-byte chunks
    g->sbig = (int32_t*)g->take(sizeof(int32_t) * B, L, ok);
    g->ps4 = (float4*)g->take(sizeof(float4) * mt1, L, ok);
    g->s_ticket = (uint32_t*)g->take(sizeof(uint32_t) * 4, L, ok);
    g->loop_msg = (unsigned long long*)g->take(sizeof(unsigned long long) * std::max<int64_t>(loop_words, 1), L, ok);
    g->loop_jobs = (LoopJob*)g->take(sizeof(LoopJob) * kLoopMaxBlocks, L, ok);
    });
    if (!ok) return fail(VICP_ERR_OOM, "workspace allocation failed");
    g->loop_pose = g->loop_msg + g->loop_units * kLoopWords;
    g->loop_lpq = 0;
    g->loop_tag = 0;
    g->loop_begun = 0;
    g->st = (PairState*)g->res;
    g->rmse_hist = (double*)(g->res + g->o_rmse);
    g->ctr_hist = (unsigned long long*)(g->res + g->o_ctr);
    g->fb_hist = (int32_t*)(g->res + g->o_fb);
    g->deg_hist = (int32_t*)(g->res + g->o_deg);
    g->flags = (int32_t*)(g->res + g->o_flags);
    for (int k = 0; k < kNumTables; ++k) {
        g->jobs_p[k] = (BlockJob*)(d_tables + t_jobs[k]);
        for (int wi = 0; wi < kNumWpb; ++wi) g->fjobs[k][wi] = (FoldJob*)(d_tables + t_folds[k][wi]);
    }
    g->fold_begin6 = (int32_t*)(d_tables + t_fbegin);
    g->job_begin6 = (int32_t*)(d_tables + t_begin);
    g->job_begin = g->job_begin6 + kT256 * (B + 1);
    g->m = m;
    std::vector<PairDev> pd;
    fill_pairdev(g, pd);
    VICP_HIP(hipMemcpyAsync(g->d_pd, pd.data(), sizeof(PairDev) * B, hipMemcpyHostToDevice, s));
    VICP_HIP(hipMemcpyAsync(d_tables, tables.data(), tables.size(), hipMemcpyHostToDevice, s));
    launch_clear4((uint32_t*)g->fb_count, 2 * B, g->loop_msg, loop_words, (uint32_t*)(g->res + g->o_abort), 4, nullptr, 0, s);
    VICP_HIP(hipStreamSynchronize(s));   // the host tables go out of scope
    g->m_total = mt;
    g->K_cap = Kc;
    return ensure_buckets(g, s);
}

int check_grid(const vicp_grid* g)
{
    if (!g) return fail(VICP_ERR_INVALID_ARG, "null grid");
    if (!g->hist) return fail(VICP_ERR_STATE, "grid not built");
    if (!g->usable) return fail(VICP_ERR_STATE, "the last build failed: rebuild the grid first");
    return VICP_OK;
}

// Bucket the source by target voxel at the pose now in g->st (a counting
// sort into g->ps4), so that the search's neighbouring lanes share segments.
void queue_plan(vicp_grid* g, const float* px, const float* py, const float* pz, hipStream_t s, bool cap)
{
    ProfScope ps("src_plan", s, cap);
    const int64_t nb = source_buckets(g, g->m);
    launch_clear4(g->sh, nb, g->s_status, scan_tiles(nb), g->s_ticket, 4, (uint32_t*)g->sbig, g->B, s);
    launch_src_bucket(g->d_pd, g->jobs_p[kT256], g->njobs_p[kT256], px, py, pz, g->st, g->sh, g->skey, g->srank,
                      g->sbig, g->flags, s);
    launch_scan(g->sh, nb, g->soff, nullptr, nullptr, g->s_status, g->s_ticket, s);
    launch_src_place(g->d_pd, g->jobs_p[kT256], g->njobs_p[kT256], g->skey, g->srank, g->soff, g->sidx, s);
    launch_src_rank(g->d_pd, g->jobs_p[kT256], g->njobs_p[kT256], px, py, pz, g->skey, g->soff, g->sidx, g->sbig,
                    g->ps4, s);
}

// Per-pair state at the given host poses (12 per pair), with the
// global-search counts and fault flags zeroed.  Up to kInlinePairs poses travel
// in the launch itself.
void queue_state(vicp_grid* g, const double* rt_host, hipStream_t s)
{
    if (g->B <= kInlinePairs) {
        launch_set_state_inline(g->d_pd, g->st, rt_host, g->B, g->fb_count, g->flags, s);
    } else {
        upload(rt_host, sizeof(double) * 12 * g->B, g->staging, s);
        launch_set_state(g->d_pd, g->st, (const double*)g->staging, g->B, g->fb_count, g->flags, s);
    }
}

// The same and the source's finiteness check, which rides on the bucketing pass
// when the search buckets the source (that pass then follows).
void queue_start(vicp_grid* g, const double* rt_host, const float* px, const float* py, const float* pz,
                 hipStream_t s)
{
    queue_state(g, rt_host, s);
    if (!g->sort_src) launch_check_finite(g->d_pd, g->jobs_p[kT256], g->njobs_p[kT256], px, py, pz, g->flags, s);
}

// Registration search for every pair at the poses in g->st (Alg. 4): the
// moment records, their fold, and the per-query results when nn_idx is not
// null.  direct: search VANICP's monolithic layout instead.  False when the
// batch is too large for the global search (nothing of it queued).
bool queue_search(vicp_grid* g, const float* px, const float* py, const float* pz, int32_t* nn_idx, float* nn_d2,
                  hipStream_t s, bool cap, bool direct = false, int early = 0)
{
    const int tab = table_of(g->nns_block / g->nns_lpq);
    {
        ProfScope ps(direct ? "nns_direct" : "nns_local", s, cap, true);
        launch_nns_local(g->d_pd, g->jobs_p[tab], g->njobs_p[tab], g->nns_block, g->nns_lpq, g->sort_src, true, px, py,
                         pz, g->ps4, g->st, g->dir, g->off, g->pyr, direct ? g->dblk : g->qs4, g->qs4, nn_idx, nn_d2,
                         g->fb_count, g->fb_count + g->B, g->fb_list, g->fb_key, g->ctr, g->npart,
                         direct ? g->dcnt : nullptr, g->dcap, g->search_mode, g->B == 1 ? g->m[0] : -1, early,
                         g->step_budget, s);
    }
    ProfScope ps("fallback", s, cap, true);
    return launch_fallback(g->d_pd, g->B, g->fb_grid, g->qx, g->qy, g->qz, px, py, pz, g->st, g->fb_count,
                           g->fb_list, g->fb_key, g->fjobs[tab][wpb_index(g->nns_block)],
                           g->nfjobs[tab][wpb_index(g->nns_block)], g->npart, g->ctr, g->fpart, g->fctr, s);
}

bool crowded_grid(const vicp_grid* g) { return g->n_total >= kCrowdedPoints * g->V_total; }

// Whether a single search buckets its source by target voxel first.  The five
// launches of that cost about 20 us with 100,000 queries and 150 with 900,000,
// more than they save where voxels hold few points (a room of 226,000: 35 us
// against 103 with as many queries on a 64^3 grid, 95 against 243 with 900,000; at
// 7 points a voxel 132 against 113), but not where a wave in index order waits for
// the most crowded of its voxels: 576 against 280 us on a 16^3 grid (55 points a
// voxel), 1460 against 748 on 8^3.  Below 50,000 queries, and below 1.5M points of
// average voxels to scan, the two are within 5 us or bucketing is the slower (35
// against 49 us with 40,000 queries at 10 points a voxel).
bool bucket_single_search(const vicp_grid* g)
{
    return g->sort_src && crowded_grid(g) && g->m_total >= 50000 &&
           (double)g->n_total * (double)g->m_total >= 1.5e6 * (double)g->V_total;
}

// The correspondences of every pair at the poses in g->st and (unless null)
// each pair's count of global searches, over the source in index order or
// bucketed (bucket_single_search).
void queue_correspondences(vicp_grid* g, const float* px, const float* py, const float* pz, int32_t* nn_idx, float* nn_d2,
                           int32_t* n_fallback, hipStream_t s, bool cap)
{
    const int tab = table_of(g->nns_block / g->nns_lpq);
    int32_t* miss = n_fallback ? g->fb_count + g->B : nullptr;
    const bool sorted = bucket_single_search(g);
    if (sorted) queue_plan(g, px, py, pz, s, cap);
    {
        ProfScope ps("nns_local", s, cap, true);
        launch_nns_local(g->d_pd, g->jobs_p[tab], g->njobs_p[tab], g->nns_block, g->nns_lpq, sorted, false, px, py, pz,
                         g->ps4, g->st, g->dir, g->off, g->pyr, g->qs4, g->qs4, nn_idx, nn_d2, nullptr, miss, nullptr,
                         nullptr, g->ctr, nullptr, nullptr, 0u, 0, g->B == 1 ? g->m[0] : -1, 0, 0u, s);
    }
    ProfScope ps("nns_global", s, cap, true);
    launch_nns_global(g->d_pd, g->jobs_p[tab], g->B, g->njobs_p[tab], g->nns_block, g->nns_lpq, sorted, px, py, pz,
                      g->ps4, g->st, g->off, g->pyr, g->qs4, g->ctr, miss, nn_idx, nn_d2, n_fallback, s);
}

// The registration form of the search with every query compared with every
// target, and the fold of its records (one lane per query in blocks of 256,
// the source in index order).
bool queue_exhaustive(vicp_grid* g, const float* px, const float* py, const float* pz, int32_t* nn_idx, float* nn_d2,
                      hipStream_t s, bool cap)
{
    if (g->B > kFbMaxPairs) return false;
    uint2* part = g->ex_part ? g->ex_part : (uint2*)g->fb_key;
    {
        ProfScope ps("exhaustive", s, cap, true);
        launch_exhaustive(g->d_pd, g->B, *std::max_element(g->m.begin(), g->m.end()), g->m_total, g->st, px, py, pz,
                          g->qx, g->qy, g->qz, part, g->ex_splits, s);
    }
    {
        ProfScope ps("exhaustive_record", s, cap);
        launch_exhaustive_record(g->d_pd, g->jobs_p[kT256], g->njobs_p[kT256], g->m_total, g->st, px, py, pz, g->qx,
                                 g->qy, g->qz, part, g->ex_splits, nn_idx, nn_d2, g->fb_count + g->B, g->npart,
                                 g->ctr, s);
    }
    const int wi = wpb_index(256);
    ProfScope ps("fallback", s, cap, true);
    return launch_fallback(g->d_pd, g->B, g->fb_grid, g->qx, g->qy, g->qz, px, py, pz, g->st, g->fb_count,
                           g->fb_list, g->fb_key, g->fjobs[kT256][wi], g->nfjobs[kT256][wi], g->npart, g->ctr,
                           g->fpart, g->fctr, s);
}

// The exhaustive search's splits, and the words of their minima: taken with
// the first such registration of a source (not while a stream is captured,
// and when there is no memory, one split, whose words are fb_key's).
void plan_exhaustive(vicp_grid* g, hipStream_t s)
{
    if (g->m_total == 0) return;
    const int most = exhaustive_max_splits(g->m_total);
    if (most > 1 && !g->ex_part && !capturing(s)) {
        const bool ok = g->lay_out(g->ex_bufs, s, [&](bool& ok) {
            g->ex_part = (uint2*)g->take(sizeof(uint2) * (size_t)most * (size_t)g->m_total, g->ex_bufs, ok);
        });
        if (!ok) (void)hipGetLastError();
    }
    std::vector<int64_t> n(g->B);
    for (int p = 0; p < g->B; ++p) n[p] = g->pairs[p].n;
    g->ex_splits = g->ex_part ? exhaustive_split(g->m.data(), n.data(), g->B, g->m_total, most) : 1;
}

// One ICP iteration (search, global search with the fold, solve); nn_idx /
// nn_d2 (optional) receive the iteration's correspondences.
bool queue_iteration(vicp_grid* g, const float* px, const float* py, const float* pz, int k, int K, int early,
                     double eps, hipStream_t s, bool cap, bool all_global, bool direct, int32_t* nn_idx, float* nn_d2)
{
    if (!(all_global ? queue_exhaustive(g, px, py, pz, nn_idx, nn_d2, s, cap)
                     : queue_search(g, px, py, pz, nn_idx, nn_d2, s, cap, direct, early)))
        return false;
    ProfScope ps("solve", s, cap, true);
    const int tab = all_global ? kT256 : table_of(g->nns_block / g->nns_lpq);
    const int wi = wpb_index(all_global ? 256 : g->nns_block);
    launch_solve(g->d_pd, g->B, g->fold_begin6 + (tab * kNumWpb + wi) * (g->B + 1), g->nfjobs[tab][wi], g->fpart,
                 g->fctr, g->st,
                 g->fb_count, g->fb_list, g->fb_key, px, py, pz, g->qx, g->qy, g->qz, g->flags, g->rmse_hist,
                 g->fb_hist, g->deg_hist, g->ctr_hist, k, K, early, eps, nn_idx, nn_d2, s);
    return true;
}

// The grid box [origin, origin + dims * voxel] within the coordinate limit.
bool box_fits(const float origin[3], const int32_t dims[3], float voxel)
{
    float lo[3], hi[3];
    for (int a = 0; a < 3; ++a) {
        lo[a] = origin[a];
        hi[a] = (float)((double)origin[a] + (double)dims[a] * (double)voxel);
    }
    return grid_box_fits(lo, hi);
}

// float32 grid specification of one pair from its bounding box (host code,
// compiled without contraction: the same roundings as the device).
int grid_spec(PairHost& h, const float lo[3], const float hi[3], float voxel, int32_t pad)
{
    const float inv = 1.0f / voxel;
    const float padw = (float)pad * voxel;
    int64_t V = 1;
    for (int a = 0; a < 3; ++a) {
        h.origin[a] = lo[a] - padw;
        const float f = (hi[a] - h.origin[a]) * inv;
        if (!(f < 1073741824.0f)) return fail(VICP_ERR_GRID_TOO_LARGE, "grid too large (voxels per axis)");
        const int64_t d = (int64_t)floorf(f) + 1 + pad;
        if (d > INT32_MAX) return fail(VICP_ERR_GRID_TOO_LARGE, "grid too large (voxels per axis)");
        h.dims[a] = (int32_t)d;
        V *= d;
        if (V >= (int64_t)1 << 31) return fail(VICP_ERR_GRID_TOO_LARGE, "grid has 2^31 voxels or more");
    }
    if (h.n + 2 * V >= (int64_t)1 << 32) return fail(VICP_ERR_GRID_TOO_LARGE, "n + 2V does not fit 32-bit offsets");
    if (!box_fits(h.origin, h.dims, voxel))
        return fail(VICP_ERR_INVALID_ARG, "the grid reaches beyond +-1e18: float32 squared distances could overflow");
    h.inv = inv;
    h.voxel = voxel;
    h.V = V;
    return VICP_OK;
}

// A given grid: origin and dims as given, 1/voxel rounded once.
int fixed_grid_spec(PairHost& h, const float origin[3], const int32_t dims[3], float voxel)
{
    int64_t V = 1;
    for (int a = 0; a < 3; ++a) {
        h.origin[a] = origin[a];
        h.dims[a] = dims[a];
        V *= dims[a];
    }
    if (V >= (int64_t)1 << 31) return fail(VICP_ERR_GRID_TOO_LARGE, "grid has 2^31 voxels or more");
    if (h.n + 2 * V >= (int64_t)1 << 32) return fail(VICP_ERR_GRID_TOO_LARGE, "n + 2V does not fit 32-bit offsets");
    if (!box_fits(origin, dims, voxel))
        return fail(VICP_ERR_INVALID_ARG, "the grid reaches beyond +-1e18: float32 squared distances could overflow");
    h.inv = 1.0f / voxel;
    h.voxel = voxel;
    h.V = V;
    return VICP_OK;
}

float unordered(uint32_t k)
{
    const uint32_t u = (k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k;
    float f;
    memcpy(&f, &u, 4);
    return f;
}

// The count (Alg. 1 GPU part) under the grid's count schedule (the
// packed-hash ablation always runs 256 points per block).
void queue_count(vicp_grid* g, const float* qx, const float* qy, const float* qz, bool packed, hipStream_t s,
                 bool cap = false, bool list_long = false)
{
    ProfScope ps("count", s, cap, true);
    const BlockJob* jobs = g->jobs_q;
    int nj = g->njobs_q, bs = 256;
    if (!packed && g->count_block == 512) {
        jobs = g->jobs_q512;
        nj = g->njobs_q512;
        bs = 512;
    } else if (!packed && g->count_block == 1024) {
        jobs = g->jobs_q1024;
        nj = g->njobs_q1024;
        bs = 1024;
    }
    launch_count(qx, qy, qz, g->d_pd, jobs, nj, bs, g->hist, g->vox, g->rank, g->err, packed, s,
                 list_long ? g->big_list : nullptr, list_long ? g->err + 1 : nullptr);
}

// `rings` dilation rings (Alg. 3) under the grid's dilation schedule: all in
// one launch on LDS tiles (1 to 4 rings), or one launch per ring.  Running it
// again on the same grid rewrites the same words.
void queue_dilate(vicp_grid* g, int rings, hipStream_t s, bool cap)
{
    if (rings < 1) return;
    if (rings <= kFusedRings && g->dil_fused) {
        ProfScope ps("dilate", s, cap, true);
        launch_dilate_fused(g->d_pd, g->jobs_t[g->dil_shape], g->njobs_t[g->dil_shape], rings, g->dil_shape, g->vm,
                            g->dir, s);
        return;
    }
    uint32_t* a = g->dil_a;
    uint32_t* b = g->dil_b;
    for (int r = 1; r <= rings; ++r) {
        ProfScope ps("dilate_ring", s, cap);
        launch_dilate_ring(g->d_pd, g->jobs_v, g->njobs_v, g->ring_block, g->hist, g->off, g->vm, g->dir,
                           r == 1 ? nullptr : a, r == rings ? nullptr : b, r == 1, r == rings, s);
        std::swap(a, b);
    }
}

// The host part of a refill: the bounding box (read back), the grid
// specification, new buffers when the shape changes, and the pair records
// on the device (passed in launch arguments, so no pageable copy holds the
// host).
int grid_fill_host(vicp_grid* g, const float* qx, const float* qy, const float* qz, hipStream_t s)
{
    const int B = g->B;
    g->direct_ready = false;
    std::vector<PairHost> pairs = g->pairs;
    int64_t Vt = 0, words = 0;
    if (g->fixed) {
        int rc = fixed_grid_spec(pairs[0], g->f_origin, g->f_dims, g->voxels[0]);
        if (rc) return rc;
        Vt = pairs[0].V;
        words = pairs[0].n + 2 * pairs[0].V;
    } else {
    const size_t nbox = 8 * (size_t)g->njobs_q8;
    if (!g->h_box && nbox) {
        if (hipHostMalloc((void**)&g->h_box, sizeof(uint32_t) * nbox, hipHostMallocMapped | hipHostMallocCoherent) !=
            hipSuccess) {
            g->h_box = nullptr;
            return fail(VICP_ERR_OOM, "pinned host allocation failed");
        }
        memset(g->h_box, 0, sizeof(uint32_t) * nbox);   // no tag is 0
        if (hipHostGetDevicePointer((void**)&g->d_box, g->h_box, 0) != hipSuccess) {
            (void)hipHostFree(g->h_box);
            g->h_box = nullptr;
            return fail(VICP_ERR_HIP, "pinned host memory not mapped for the device");
        }
    }
    if (++g->box_gen == 0) g->box_gen = 1;
    {
        ProfScope ps("aabb", s, false, true);
        launch_aabb(qx, qy, qz, g->d_pd, g->jobs_q8, g->njobs_q8, 2048, g->d_box, g->box_gen, s);
    }
    VICP_HIP(hipGetLastError());
    if (nbox) VICP_HIP(wait_tags(g->h_box + 7, g->njobs_q8, 8, g->box_gen, s));
    // per pair: min of the block minima, max of the block maxima, any
    // non-finite flag (a pair with no points keeps the empty box)
    std::vector<uint32_t> hbox(8 * (size_t)B);
    for (int p = 0; p < B; ++p)
        for (int f = 0; f < 8; ++f) hbox[8 * p + f] = f < 3 ? 0xFFFFFFFFu : 0u;
    for (int j = 0; j < g->njobs_q8; ++j) {
        uint32_t* d = &hbox[8 * (size_t)g->h_jobs_q8[j].pair];
        const uint32_t* b = &g->h_box[8 * (size_t)j];
        for (int f = 0; f < 3; ++f) d[f] = std::min(d[f], b[f]);
        for (int f = 3; f < 7; ++f) d[f] = std::max(d[f], b[f]);
    }
    for (int p = 0; p < B; ++p) {
        const uint32_t* b = &hbox[8 * p];
        if (b[6]) return fail(VICP_ERR_NONFINITE, "non-finite target coordinates");
        float lo[3], hi[3];
        for (int a = 0; a < 3; ++a) {
            lo[a] = unordered(b[a]);
            hi[a] = unordered(b[3 + a]);
        }
        int rc = grid_spec(pairs[p], lo, hi, g->voxels[p], g->pad);
        if (rc) return rc;
        pairs[p].v_base = Vt;
        pairs[p].vm_base = words;
        Vt += pairs[p].V;
        words += pairs[p].n + 2 * pairs[p].V;
    }
    }
    if (Vt >= ((int64_t)1 << 31) || words >= ((int64_t)1 << 32))
        return fail(VICP_ERR_GRID_TOO_LARGE, "batch exceeds 2^31 voxels or 2^32 index words");
    // the pyramids' bytes and the dilation's tiles depend on the dims, not on V alone
    int64_t pyr_bytes = 0;
    for (int p = 0; p < B; ++p) {
        pairs[p].t_base = pyr_bytes;
        pyr_bytes += pyramid_bytes(pairs[p].dims);
    }
    bool same_shape = g->hist != nullptr;
    for (int p = 0; p < B && same_shape; ++p) same_shape = memcmp(pairs[p].dims, g->pairs[p].dims, sizeof(pairs[p].dims)) == 0;
    g->qx = qx;
    g->qy = qy;
    g->qz = qz;
    g->pairs = pairs;
    g->dilated = false;
    g->rings_applied = 0;
    if (!same_shape) {
        // voxel-sized buffers follow the new grid; captured work referring to
        // the old ones is dropped, the source buckets are laid out on demand
        g->drop_graph();
        g->ws_V = -1;
        g->V_total = Vt;
        g->vm_words = words;
        std::vector<int64_t> vcount(B);
        for (int p = 0; p < B; ++p) vcount[p] = pairs[p].V;
        std::vector<BlockJob> jv, jt[kDilateShapes];
        make_jobs(vcount, 256, jv, nullptr);
        for (int sh = 0; sh < kDilateShapes; ++sh) {
            std::vector<int64_t> tcount(B);
            for (int p = 0; p < B; ++p)
                tcount[p] = dilate_tiles(sh, pairs[p].dims[0], pairs[p].dims[1], pairs[p].dims[2]);
            make_jobs(tcount, 1, jt[sh], nullptr);
        }
        std::vector<char> tables;
        const size_t t_v = add_table(tables, jv);
        size_t t_t[kDilateShapes];
        for (int sh = 0; sh < kDilateShapes; ++sh) {
            t_t[sh] = add_table(tables, jt[sh]);
            g->njobs_t[sh] = (int)jt[sh].size();
        }
        g->njobs_v = (int)jv.size();
        const int tiles = scan_tiles(Vt);
        char* d_tables = nullptr;
        g->pyr_words = pyr_bytes / 4;
        const bool ok = g->lay_out(g->vbufs, s, [&](bool& ok) {
            Arena& L = g->vbufs;
            g->hist = (uint32_t*)g->take(sizeof(uint32_t) * (Vt + g->pyr_words), L, ok);
            g->off = (uint32_t*)g->take(sizeof(uint32_t) * (Vt + 1), L, ok);
            g->vm = (uint32_t*)g->take(sizeof(uint32_t) * words, L, ok);
            g->dir = (uint2*)g->take(sizeof(uint2) * Vt, L, ok);
            d_tables = (char*)g->take(tables.size(), L, ok);
            g->scan_status = (unsigned long long*)g->take(sizeof(unsigned long long) * tiles, L, ok);
            g->scan_ticket = (uint32_t*)g->take(sizeof(uint32_t) * 4, L, ok);
            g->dil_a = (uint32_t*)g->take(sizeof(uint32_t) * Vt, L, ok);
            g->dil_b = (uint32_t*)g->take(sizeof(uint32_t) * Vt, L, ok);
        });
        if (!ok) {
            g->hist = nullptr;
            return fail(VICP_ERR_OOM, "grid allocation failed");
        }
        g->pyr = (uint8_t*)(g->hist + Vt);
        g->jobs_v = (BlockJob*)(d_tables + t_v);
        for (int sh = 0; sh < kDilateShapes; ++sh) g->jobs_t[sh] = (BlockJob*)(d_tables + t_t[sh]);
        VICP_HIP(hipMemcpyAsync(d_tables, tables.data(), tables.size(), hipMemcpyHostToDevice, s));
        VICP_HIP(hipStreamSynchronize(s));   // the host tables go out of scope
    }
    fill_pairdev(g, g->h_pd);
    return VICP_OK;
}

// The first launch of a refill's device part: zeroes the histogram, the
// scan's tile states, its tickets and the error words, and writes the pair
// records when they fit the launch (else a separate upload first).
void clear_for_build(vicp_grid* g, hipStream_t s)
{
    const int64_t Vt = g->V_total;
    const size_t bytes = sizeof(PairDev) * g->h_pd.size();
    if (bytes <= sizeof(Blob)) {
        Blob b;
        memcpy(b.w, g->h_pd.data(), bytes);
        launch_clear4_blob(b, (uint32_t*)g->d_pd, (int)(bytes / 4), g->hist, Vt + g->pyr_words, g->scan_status, scan_tiles(Vt),
                           g->scan_ticket, 4, g->err, 4, s);
    } else {
        upload(g->h_pd.data(), bytes, g->d_pd, s);
        launch_clear4(g->hist, Vt + g->pyr_words, g->scan_status, scan_tiles(Vt), g->scan_ticket, 4, g->err, 4, s);
    }
}

// The packed-hash ablation applies when every pair's voxel ids fit its key.
bool count_packed(const vicp_grid* g)
{
    bool packed = g->packed_hash;
    for (int p = 0; p < g->B && packed; ++p) packed = count_packed_fits(g->pairs[p].V);
    return packed;
}

// The device part of a refill whose pair records are on the device:
// histogram (Alg. 1 GPU part), offsets, and the segments in ascending
// order (Alg. 2).  The fixed-grid check and the host-side offset scan
// synchronise, so grid_fill runs those forms itself.
void queue_build_rest(vicp_grid* g, hipStream_t s, bool cap)
{
    const int64_t Vt = g->V_total;
    queue_count(g, g->qx, g->qy, g->qz, count_packed(g), s, cap);
    {
        ProfScope ps("scan", s, cap, true);
        launch_scan(g->hist, Vt, g->off, g->vm, g->dir, g->scan_status, g->scan_ticket, s);
    }
    {
        ProfScope ps("place", s, cap, true);
        launch_place(g->d_pd, g->jobs_q, g->njobs_q, g->vox, g->rank, g->off, g->slots, s);
    }
    {
        ProfScope ps("rank_sort", s, cap, true);
        launch_rank_sort(g->qx, g->qy, g->qz, g->d_pd, g->jobs_q, g->njobs_q, g->vox, g->hist, g->off, g->slots,
                         g->vm, g->qs4, g->pyr, s);
    }
}

void queue_build(vicp_grid* g, hipStream_t s, bool cap)
{
    clear_for_build(g, s);
    queue_build_rest(g, s, cap);
}

// Fills (or refills) a grid from target coordinates: bounding box (the one
// synchronisation), grid specification, then counts, offsets, segments.
int grid_fill(vicp_grid* g, const float* qx, const float* qy, const float* qz, hipStream_t s)
{
    int rc = grid_fill_host(g, qx, qy, qz, s);
    if (rc) return rc;
    g->usable = false;   // the grid's words are stale until the refill below is queued
    const int64_t Vt = g->V_total;
    if (!g->fixed && !g->host_offsets) {
        queue_build(g, s, false);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(VICP_ERR_HIP, std::string("grid build: ") + hipGetErrorString(e));
        g->usable = true;
        return VICP_OK;
    }
    // a fixed grid (the paper's coarse 2^N grids hold thousands of points in a
    // voxel) sorts its long segments whole; the count lists them (err[1]
    // counts the list)
    const bool seg_sort = g->fixed && !count_packed(g);
    clear_for_build(g, s);
    queue_count(g, qx, qy, qz, count_packed(g), s, false, seg_sort);
    if (g->fixed) {   // the one synchronisation of a fixed-grid build: every target inside the grid?
        uint32_t herr = 0;
        VICP_HIP(hipMemcpyAsync(&herr, g->err, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
        VICP_HIP(hipStreamSynchronize(s));
        if (herr) {
            g->usable = false;   // until a successful rebuild
            return fail(VICP_ERR_INVALID_ARG, "a target point lies outside the given grid");
        }
    }
    if (g->host_offsets) {
        // Alg. 1's CPU part as the paper runs it: the histogram comes to the
        // host, the offsets are a serial running sum of count + 2 there, and
        // go back; a kernel then writes the segment headers and directory
        g->h_hist.resize((size_t)Vt);
        g->h_off.resize((size_t)Vt + 1);
        VICP_HIP(hipMemcpyAsync(g->h_hist.data(), g->hist, sizeof(uint32_t) * Vt, hipMemcpyDeviceToHost, s));
        VICP_HIP(hipStreamSynchronize(s));
        const auto t0 = std::chrono::steady_clock::now();
        uint64_t head = 0;
        for (int64_t v = 0; v < Vt; ++v) {
            g->h_off[v] = (uint32_t)head;
            head += (uint64_t)g->h_hist[v] + 2;
        }
        g->h_off[Vt] = (uint32_t)head;
        const auto t1 = std::chrono::steady_clock::now();
        prof_add_host("moc_host", std::chrono::duration<double, std::milli>(t1 - t0).count());
        VICP_HIP(hipMemcpyAsync(g->off, g->h_off.data(), sizeof(uint32_t) * (Vt + 1), hipMemcpyHostToDevice, s));
        launch_seg_headers(g->hist, g->off, Vt, g->vm, g->dir, s);
        VICP_HIP(hipStreamSynchronize(s));   // the host arrays are reused by the next build
    } else {
        ProfScope ps("scan", s, false, true);
        launch_scan(g->hist, Vt, g->off, g->vm, g->dir, g->scan_status, g->scan_ticket, s);
    }
    {
        ProfScope ps("place", s, false, true);
        launch_place(g->d_pd, g->jobs_q, g->njobs_q, g->vox, g->rank, g->off, g->slots, s);
    }
    {
        ProfScope ps("rank_sort", s, false, true);
        launch_rank_sort(qx, qy, qz, g->d_pd, g->jobs_q, g->njobs_q, g->vox, g->hist, g->off, g->slots, g->vm,
                         g->qs4, g->pyr, s, seg_sort ? kSegSortMin : 0xFFFFFFFFu);
    }
    if (seg_sort) {
        ProfScope ps("seg_sort", s, false, true);
        launch_sort_segments(qx, qy, qz, g->d_pd, g->big_list, g->err + 1, g->hist, g->off, g->slots, g->vm, g->qs4,
                             g->pyr, s);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(VICP_ERR_HIP, std::string("grid build: ") + hipGetErrorString(e));
    g->usable = true;
    return VICP_OK;
}

}  // namespace

// ====================================================================== C ABI

extern "C" {

const char* vicp_version(void) { return "vicp 0.2 (gfx950)"; }

const char* vicp_last_error(void) { return g_err.c_str(); }

const char* vicp_status_str(int code)
{
    switch (code) {
    case VICP_OK: return "ok";
    case VICP_ERR_INVALID_ARG: return "invalid argument";
    case VICP_ERR_GRID_TOO_LARGE: return "grid too large";
    case VICP_ERR_OOM: return "out of device memory";
    case VICP_ERR_HIP: return "HIP runtime error";
    case VICP_ERR_STATE: return "call out of order";
    case VICP_ERR_NONFINITE: return "non-finite coordinates";
    case VICP_ERR_DEGENERATE: return "degenerate cross-covariance (pose kept)";
    default: return "unknown status";
    }
}

namespace {

struct FixedGrid {
    float origin[3];
    int32_t dims[3];
};

int build_grid_impl(const float* qx, const float* qy, const float* qz, const int64_t* n_per_pair, int32_t npairs,
                    const float* voxel_per_pair, int32_t pad_rings, const vicp_allocator* alloc, hipStream_t s,
                    vicp_grid** out, const FixedGrid* fixed)
{
    (void)hipGetLastError();   // an error left by other code is not ours to report
    if (!out) return fail(VICP_ERR_INVALID_ARG, "null output");
    *out = nullptr;
    if (!qx || !qy || !qz || !n_per_pair || !voxel_per_pair) return fail(VICP_ERR_INVALID_ARG, "null pointer");
    if (npairs < 1 || npairs > 4096) return fail(VICP_ERR_INVALID_ARG, "npairs must be in [1, 4096]");
    if (pad_rings < 0 || pad_rings > 1024) return fail(VICP_ERR_INVALID_ARG, "pad_rings must be in [0, 1024]");
    if (alloc && (!alloc->alloc || !alloc->free)) return fail(VICP_ERR_INVALID_ARG, "allocator without functions");
    std::vector<PairHost> pairs(npairs);
    int64_t nt = 0;
    for (int p = 0; p < npairs; ++p) {
        if (n_per_pair[p] <= 0 || n_per_pair[p] > (int64_t)INT32_MAX)
            return fail(VICP_ERR_INVALID_ARG, "every pair needs 1 .. 2^31-1 target points");
        const float vx = voxel_per_pair[p];
        if (!(vx > 0.0f) || !isfinite(vx)) return fail(VICP_ERR_INVALID_ARG, "voxel must be finite and > 0");
        pairs[p].n = n_per_pair[p];
        pairs[p].q_base = nt;
        nt += n_per_pair[p];
    }
    if (nt >= ((int64_t)1 << 32)) return fail(VICP_ERR_INVALID_ARG, "too many target points");
    vicp_grid* g = new vicp_grid();
    g->B = npairs;
    g->pad = pad_rings;
    if (fixed) {
        g->fixed = true;
        for (int a = 0; a < 3; ++a) {
            g->f_origin[a] = fixed->origin[a];
            g->f_dims[a] = fixed->dims[a];
        }
    }
    g->n_total = nt;
    g->pairs = pairs;
    g->voxels.assign(voxel_per_pair, voxel_per_pair + npairs);
    if (alloc) {
        g->mem.a = *alloc;
        g->mem.custom = true;
    }
    auto bail = [&](int rc) {
        std::string msg = g_err;
        vicp_grid_free(g);
        g_err = msg;
        return rc;
    };
    std::vector<int64_t> ncount(npairs);
    for (int p = 0; p < npairs; ++p) ncount[p] = pairs[p].n;
    std::vector<BlockJob> jq, jq8, jq512, jq1024;
    make_jobs(ncount, 256, jq, nullptr);
    make_jobs(ncount, 2048, jq8, nullptr);
    make_jobs(ncount, 512, jq512, nullptr);
    make_jobs(ncount, 1024, jq1024, nullptr);
    std::vector<PairDev> pd;
    fill_pairdev(g, pd);   // target fields only; the grid fields follow the bounding box
    std::vector<char> tables;
    const size_t t_pd = add_table(tables, pd), t_q = add_table(tables, jq), t_q8 = add_table(tables, jq8);
    const size_t t_512 = add_table(tables, jq512), t_1024 = add_table(tables, jq1024);
    char* d_tables = nullptr;
    const bool ok = g->lay_out(g->owned, s, [&](bool& ok) {
        Arena& L = g->owned;
        d_tables = (char*)g->take(tables.size(), L, ok);
        g->err = (uint32_t*)g->take(sizeof(uint32_t) * 4, L, ok);
        g->vox = (uint32_t*)g->take(sizeof(uint32_t) * nt, L, ok);
        g->rank = (uint32_t*)g->take(sizeof(uint32_t) * nt, L, ok);
        g->slots = (uint32_t*)g->take(sizeof(uint32_t) * (nt + 4), L, ok);   // +4: rank_in reads 16-byte chunks
        // the long segments a fixed grid's count lists (at most n / kSegSortMin)
        g->big_list = (uint32_t*)g->take(sizeof(uint32_t) * (nt / kSegSortMin + 1), L, ok);
        g->qs4 = (float4*)g->take(sizeof(float4) * nt, L, ok);
    });
    if (!ok) return bail(fail(VICP_ERR_OOM, "allocation failed"));
    g->d_pd = (PairDev*)(d_tables + t_pd);
    g->jobs_q = (BlockJob*)(d_tables + t_q);
    g->jobs_q8 = (BlockJob*)(d_tables + t_q8);
    g->jobs_q512 = (BlockJob*)(d_tables + t_512);
    g->jobs_q1024 = (BlockJob*)(d_tables + t_1024);
    g->njobs_q = (int)jq.size();
    g->njobs_q8 = (int)jq8.size();
    g->njobs_q512 = (int)jq512.size();
    g->njobs_q1024 = (int)jq1024.size();
    g->h_jobs_q8 = jq8;
    // (the tables go out of scope: grid_fill waits for work queued after them
    // or copies its own and synchronises)
    if (hipMemcpyAsync(d_tables, tables.data(), tables.size(), hipMemcpyHostToDevice, s) != hipSuccess)
        return bail(fail(VICP_ERR_HIP, "upload failed"));
    int rc = grid_fill(g, qx, qy, qz, s);
    if (rc) return bail(rc);
    *out = g;
    return VICP_OK;
}

}  // namespace

int vicp_build_grid_batched(const float* qx, const float* qy, const float* qz, const int64_t* n_per_pair, int32_t npairs,
                            const float* voxel_per_pair, int32_t pad_rings, const vicp_allocator* alloc,
                            hipStream_t s, vicp_grid** out)
{
    return build_grid_impl(qx, qy, qz, n_per_pair, npairs, voxel_per_pair, pad_rings, alloc, s, out, nullptr);
}

int vicp_build_grid(const float* qx, const float* qy, const float* qz, int64_t n, float voxel, int32_t pad_rings,
                    const vicp_allocator* alloc, hipStream_t s, vicp_grid** out)
{
    return build_grid_impl(qx, qy, qz, &n, 1, &voxel, pad_rings, alloc, s, out, nullptr);
}

int vicp_build_grid_fixed(const float* qx, const float* qy, const float* qz, int64_t n, const float origin[3],
                          float voxel, const int32_t dims[3], int32_t max_rings, const vicp_allocator* alloc,
                          hipStream_t s, vicp_grid** out)
{
    if (!origin || !dims) return fail(VICP_ERR_INVALID_ARG, "null pointer");
    FixedGrid fg;
    for (int a = 0; a < 3; ++a) {
        if (!isfinite(origin[a])) return fail(VICP_ERR_INVALID_ARG, "origin must be finite");
        if (dims[a] < 1) return fail(VICP_ERR_INVALID_ARG, "dims must be >= 1");
        fg.origin[a] = origin[a];
        fg.dims[a] = dims[a];
    }
    return build_grid_impl(qx, qy, qz, &n, 1, &voxel, max_rings, alloc, s, out, &fg);
}

int vicp_grid_rebuild(vicp_grid* g, const float* qx, const float* qy, const float* qz, hipStream_t s)
{
    (void)hipGetLastError();   // an error left by other code is not ours to report
    if (!g) return fail(VICP_ERR_INVALID_ARG, "null grid");
    if (!g->hist) return fail(VICP_ERR_STATE, "grid not built");
    if (!qx || !qy || !qz) return fail(VICP_ERR_INVALID_ARG, "null pointer");
    return grid_fill(g, qx, qy, qz, s);
}

int vicp_grid_npairs(const vicp_grid* g) { return g ? g->B : 0; }

int vicp_last_form(const vicp_grid* g, int32_t* form)
{
    if (!g || !form) return fail(VICP_ERR_INVALID_ARG, "null pointer");
    *form = g->last_form;
    return VICP_OK;
}

int vicp_set_build_options(vicp_grid* g, int32_t host_offsets, int32_t packed_hash)
{
    if (!g) return fail(VICP_ERR_INVALID_ARG, "null grid");
    g->host_offsets = host_offsets != 0;
    g->packed_hash = packed_hash != 0;
    return VICP_OK;
}

// VANICP's layout for the comparison (Sec. II.B; Sec. III and Fig. 1
// contrast it with the segmented layout): the target is voxelised straight
// into fixed per-voxel blocks, the same rings of dilation run on the block
// counts, and every dilated voxel's block receives a copy of its root's
// records.
int vicp_direct_build(vicp_grid* g, int64_t block_bytes, hipStream_t s)
{
    (void)hipGetLastError();   // an error left by other code is not ours to report
    int rc = check_grid(g);
    if (rc) return rc;
    if (g->B != 1) return fail(VICP_ERR_INVALID_ARG, "the direct layout needs a single-pair grid");
    if (!g->dilated) return fail(VICP_ERR_STATE, "dilate the grid first (the direct layout uses the same rings)");
    if (block_bytes < 16 || block_bytes % 16 != 0 || block_bytes / 16 > 0x7FFFFFFF)
        return fail(VICP_ERR_INVALID_ARG, "block_bytes must be a positive multiple of 16 below 2^35");
    const int64_t V = g->V_total;
    if (V > (int64_t)(SIZE_MAX / 2) / block_bytes) return fail(VICP_ERR_GRID_TOO_LARGE, "direct layout too large");
    const size_t need = (size_t)V * (size_t)block_bytes, need_c = sizeof(uint32_t) * (size_t)V;
    g->direct_ready = false;
    if (g->dblk_bytes != need || g->dcnt_bytes != need_c) {
        VICP_HIP(hipStreamSynchronize(s));
        vicp_direct_free(g);
        void* b = nullptr;
        void* c = nullptr;
        if (hipMalloc(&b, need) != hipSuccess || hipMalloc(&c, need_c) != hipSuccess) {
            (void)hipGetLastError();
            if (b) (void)hipFree(b);
            return fail(VICP_ERR_OOM, "direct layout: device allocation of " + std::to_string(need) + " bytes failed");
        }
        g->dblk = (float4*)b;
        g->dblk_bytes = need;
        g->dcnt = (uint32_t*)c;
        g->dcnt_bytes = need_c;
    }
    g->dcap = (uint32_t)(block_bytes / 16);
    const bool cap = capturing(s);
    {
        ProfScope ps("direct_count", s, cap);
        launch_fill_u32(g->dcnt, 0u, V, s);
        launch_count_direct(g->qx, g->qy, g->qz, g->d_pd, g->jobs_q, g->njobs_q, g->dcnt, g->err, g->dblk, g->dcap,
                            s);
    }
    // the segmented grid's ring-state arrays are free once it is dilated
    uint32_t* a = g->dil_a;
    uint32_t* b = g->dil_b;
    const int rings = g->rings_applied;
    for (int r = 1; r <= rings; ++r) {
        ProfScope ps("direct_dilate_ring", s, cap);
        launch_dilate_ring(g->d_pd, g->jobs_v, g->njobs_v, 256, g->dcnt, nullptr, nullptr, nullptr,
                           r == 1 ? nullptr : a, b, r == 1, 0, s);
        std::swap(a, b);
    }
    {
        ProfScope ps("direct_replicate", s, cap);
        launch_replicate(g->d_pd, V, rings > 0 ? a : nullptr, g->dcnt, g->dblk, g->dcap, s);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(VICP_ERR_HIP, std::string("direct build: ") + hipGetErrorString(e));
    g->direct_ready = true;
    return VICP_OK;
}

int vicp_direct_free(vicp_grid* g)
{
    if (!g) return fail(VICP_ERR_INVALID_ARG, "null grid");
    if (!g->dblk && !g->dcnt) return VICP_OK;
    (void)hipDeviceSynchronize();
    g->drop_graph();   // a captured registration may point at the blocks
    if (g->dblk) (void)hipFree(g->dblk);
    if (g->dcnt) (void)hipFree(g->dcnt);
    g->dblk = nullptr;
    g->dcnt = nullptr;
    g->dblk_bytes = g->dcnt_bytes = 0;
    g->direct_ready = false;
    return VICP_OK;
}

int vicp_dilate(vicp_grid* g, int32_t rings, hipStream_t s)
{
    (void)hipGetLastError();   // an error left by other code is not ours to report
    int rc = check_grid(g);
    if (rc) return rc;
    if (g->dilated) return fail(VICP_ERR_STATE, "grid already dilated");
    if (rings < 0 || rings > g->pad) return fail(VICP_ERR_INVALID_ARG, "rings must be in [0, pad_rings]");
    g->dilated = true;
    g->rings_applied = rings;
    queue_dilate(g, rings, s, capturing(s));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(VICP_ERR_HIP, std::string("dilate: ") + hipGetErrorString(e));
    return VICP_OK;
}

int vicp_nns_batched(const vicp_grid* gc, const float* px, const float* py, const float* pz, const int64_t* m_per_pair,
                     const float* Rt, int32_t* nn_idx, float* nn_d2, int32_t* n_fallback, hipStream_t s)
{
    (void)hipGetLastError();   // an error left by other code is not ours to report
    vicp_grid* g = const_cast<vicp_grid*>(gc);
    int rc = check_grid(g);
    if (rc) return rc;
    if (!m_per_pair || !Rt) return fail(VICP_ERR_INVALID_ARG, "null pointer");
    int64_t mt = 0;
    for (int p = 0; p < g->B; ++p) mt += std::max<int64_t>(m_per_pair[p], 0);
    rc = ensure_source(g, m_per_pair, 1, s);
    if (rc) return rc;
    if (mt == 0) {
        if (n_fallback) launch_fill_u32((uint32_t*)n_fallback, 0u, g->B, s);
        return VICP_OK;
    }
    if (!px || !py || !pz || !nn_idx || !nn_d2) return fail(VICP_ERR_INVALID_ARG, "null pointer");
    for (int i = 0; i < 12 * g->B; ++i)
        if (!isfinite(Rt[i])) return fail(VICP_ERR_INVALID_ARG, "non-finite pose");
    const bool cap = capturing(s);
    std::vector<double> rt64(12 * g->B);
    for (int i = 0; i < 12 * g->B; ++i) rt64[i] = (double)Rt[i];
    queue_state(g, rt64.data(), s);
    queue_correspondences(g, px, py, pz, nn_idx, nn_d2, n_fallback, s, cap);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(VICP_ERR_HIP, std::string("nns: ") + hipGetErrorString(e));
    return VICP_OK;
}

int vicp_nns(const vicp_grid* g, const float* px, const float* py, const float* pz, int64_t m, const float Rt[12],
             int32_t* nn_idx, float* nn_d2, int32_t* n_fallback, hipStream_t s)
{
    if (!g) return fail(VICP_ERR_INVALID_ARG, "null grid");
    if (g->B != 1) return fail(VICP_ERR_INVALID_ARG, "vicp_nns needs a single-pair grid");
    if (m < 0) return fail(VICP_ERR_INVALID_ARG, "m < 0");
    return vicp_nns_batched(g, px, py, pz, &m, Rt, nn_idx, nn_d2, n_fallback, s);
}

}  // extern "C"

// ------------------------------------------------- the allocation-free search
//
// vicp_nns_noalloc keeps every intermediate of one search in `scratch`, a
// fixed device array of this translation unit.  In host code the array's
// name only stands for the symbol: its device address on the current GPU is
// found once per device with hipGetSymbolAddress and kept, and only that
// address is ever handed to a kernel.
namespace {

constexpr int64_t kNaMaxQ = VICP_NOALLOC_MAX_QUERIES;
constexpr int64_t kNaMinQpb = 16;                        // fewest queries per block of any schedule
constexpr int64_t kNaMaxJobs = kNaMaxQ / kNaMinQpb;      // search blocks
constexpr int64_t kNaMaxMasks = kNaMaxQ / 8 + 8;          // search waves: a mask word each (8 lanes a query, the last block's)
constexpr size_t kNaOffPd = 0;                           // PairDev
constexpr size_t kNaOffSt = 256;                         // PairState
constexpr size_t kNaOffCnt = 512;                        // queries that needed a global search
constexpr size_t kNaOffJobs = 768;
constexpr size_t kNaOffMask = kNaOffJobs + sizeof(BlockJob) * kNaMaxJobs;
constexpr size_t kNaBytes = kNaOffMask + sizeof(unsigned long long) * kNaMaxMasks;
static_assert(sizeof(PairDev) <= 256 && sizeof(PairState) <= 256, "scratch header slots");
static_assert(kNaOffMask % 256 == 0, "scratch sections stay 256-byte aligned");
static_assert(kNaBytes == 1573696, "the size the header states");

}  // namespace

static __device__ __align__(256) unsigned char scratch[kNaBytes];

namespace {

std::mutex g_na_mu;
std::map<int, unsigned char*> g_na_ptr;   // device ordinal -> address of `scratch` on that device

// The address of `scratch` on the current device (located on first use).
int noalloc_scratch(unsigned char** out)
{
    int devi = 0;
    VICP_HIP(hipGetDevice(&devi));
    std::lock_guard<std::mutex> lk(g_na_mu);
    auto it = g_na_ptr.find(devi);
    if (it == g_na_ptr.end()) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(VICP_ERR_HIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        it = g_na_ptr.emplace(devi, (unsigned char*)p).first;
    }
    *out = it->second;
    return VICP_OK;
}

struct NaSetup {
    PairDev pd;
    float rt[12];
};

// One launch prepares the search: the pair record and pose, the global-search
// count and fault flags at zero, and the two block tables (search blocks of
// qpb queries, result blocks of 256 points).
__global__ void k_noalloc_setup(NaSetup a, int32_t njobs, int32_t qpb, unsigned char* base)
{
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (tid == 0) {
        *reinterpret_cast<PairDev*>(base + kNaOffPd) = a.pd;
        PairState& S = *reinterpret_cast<PairState*>(base + kNaOffSt);
        for (int j = 0; j < 12; ++j) {
            S.Rt[j] = (double)a.rt[j];
            S.Rtf[j] = a.rt[j];
        }
        S.prev_rmse = 0.0;
        S.done = 0;
        S.iters = 0;
        S.degenerate = 0;
        S.status = 0;
        S.rot_ok = 0;
        S.misses = 0;
        int32_t* cnt = reinterpret_cast<int32_t*>(base + kNaOffCnt);
        cnt[0] = 0;
    }
    BlockJob* jobs = reinterpret_cast<BlockJob*>(base + kNaOffJobs);
    for (int64_t j = tid; j < njobs; j += (int64_t)gridDim.x * blockDim.x) jobs[j] = BlockJob{0, (int32_t)(j * qpb)};
}

}  // namespace

extern "C" {

int vicp_nns_noalloc(const vicp_grid* g, const float* px, const float* py, const float* pz, int64_t m,
                     const float Rt[12], int32_t* nn_idx, float* nn_d2, int32_t* n_fallback, hipStream_t s)
{
    (void)hipGetLastError();   // an error left by other code is not ours to report
    int rc = check_grid(g);
    if (rc) return rc;
    if (g->B != 1) return fail(VICP_ERR_INVALID_ARG, "vicp_nns_noalloc needs a single-pair grid");
    if (m < 0) return fail(VICP_ERR_INVALID_ARG, "m < 0");
    if (m > kNaMaxQ)
        return fail(VICP_ERR_INVALID_ARG, "vicp_nns_noalloc takes at most " + std::to_string(kNaMaxQ) +
                                              " source points (its fixed scratch array); use vicp_nns");
    unsigned char* base = nullptr;
    rc = noalloc_scratch(&base);
    if (rc) return rc;
    int32_t* cnt = reinterpret_cast<int32_t*>(base + kNaOffCnt);
    if (m == 0) {
        if (n_fallback) launch_fill_u32((uint32_t*)n_fallback, 0u, 1, s);
        return VICP_OK;
    }
    if (!px || !py || !pz || !nn_idx || !nn_d2 || !Rt) return fail(VICP_ERR_INVALID_ARG, "null pointer");
    for (int i = 0; i < 12; ++i)
        if (!isfinite(Rt[i])) return fail(VICP_ERR_INVALID_ARG, "non-finite pose");
    // the grid's search schedule, over the source in index order (bucketing
    // the source would need the grid's workspace)
    const int qpb = g->nns_block / g->nns_lpq;
    const int64_t njobs = (m + qpb - 1) / qpb;
    NaSetup a{};
    fill_grid_fields(g->pairs[0], g->pad, a.pd);
    a.pd.p_base = 0;
    a.pd.m = m;
    a.pd.s_chunks = 1;
    a.pd.s_shift = 62;
    for (int i = 0; i < 12; ++i) a.rt[i] = Rt[i];
    const PairDev* pd = reinterpret_cast<const PairDev*>(base + kNaOffPd);
    PairState* st = reinterpret_cast<PairState*>(base + kNaOffSt);
    const BlockJob* jobs = reinterpret_cast<const BlockJob*>(base + kNaOffJobs);
    unsigned long long* mask = reinterpret_cast<unsigned long long*>(base + kNaOffMask);
    const int setup_blocks = (int)std::min<int64_t>((njobs + 255) / 256, 256);
    hipLaunchKernelGGL(k_noalloc_setup, dim3(setup_blocks), dim3(256), 0, s, a, (int32_t)njobs, (int32_t)qpb, base);
    launch_nns_local(pd, jobs, (int)njobs, g->nns_block, g->nns_lpq, false, false, px, py, pz, nullptr, st, g->dir,
                     g->off, g->pyr, g->qs4, g->qs4, nn_idx, nn_d2, nullptr, cnt, nullptr, nullptr, mask, nullptr,
                     nullptr, 0u, 0, m, 0, 0u, s);
    launch_nns_global(pd, jobs, 1, (int)njobs, g->nns_block, g->nns_lpq, false, px, py, pz, nullptr, st, g->off, g->pyr,
                      g->qs4, mask, cnt, nn_idx, nn_d2, n_fallback, s);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(VICP_ERR_HIP, std::string("nns_noalloc: ") + hipGetErrorString(e));
    return VICP_OK;
}

}  // extern "C"

namespace {

// Captures the work `body` queues on the capture stream into c, unless c
// already holds it under the same key.  With timing on, the first attempt
// records kernel events inside the graph; if the runtime refuses that, the
// work is captured without them.  body returns false when the batch is too
// large for the global search: nothing is kept and the result is
// INVALID_ARG.
template <class F>
int capture_into(vicp_grid* g, vicp_grid::Captured& c, const std::vector<uintptr_t>& key, F&& body)
{
    if (c.exec && key == c.key) return VICP_OK;
    c.drop();
    if (!g->cap_stream) VICP_HIP(hipStreamCreateWithFlags(&g->cap_stream, hipStreamNonBlocking));
    std::string why;
    for (int attempt = (g_prof.on ? 0 : 1); attempt < 2 && !c.exec; ++attempt) {
        hipGraph_t graph = nullptr;
        VICP_HIP(hipStreamBeginCapture(g->cap_stream, hipStreamCaptureModeThreadLocal));
        t_capture_events = attempt == 0 ? &c.events : nullptr;
        const bool queued = body(g->cap_stream);
        t_capture_events = nullptr;
        hipError_t ec = hipStreamEndCapture(g->cap_stream, &graph);
        hipError_t e = ec;
        if (ec == hipSuccess) {
            e = hipGraphInstantiate(&c.exec, graph, nullptr, nullptr, 0);
            (void)hipGraphDestroy(graph);
        }
        if (e != hipSuccess || !queued) {
            (void)hipGetLastError();
            if (c.exec) (void)hipGraphExecDestroy(c.exec);
            c.exec = nullptr;
            prof_return(c.events);
            if (!queued) return fail(VICP_ERR_INVALID_ARG, "too many pairs for the global search");
            why = hipGetErrorString(e);
        }
    }
    if (!c.exec) return fail(VICP_ERR_HIP, "graph capture: " + why);
    c.key = key;
    return VICP_OK;
}

// ---------------------------------------------------- the resident loop's host side

// One resident loop at a time per device: two that together exceed the device
// could each hold what the other waits for.  A call that finds it taken runs
// the launch-per-step form.
constexpr int kMaxDevices = 64;
// Registrations that a grid runs without the loop after one whose blocks did not
// meet: 2 ms lost in one of 33.
constexpr int kLoopRest = 32;
std::mutex g_loop_mu[kMaxDevices];

// Blocks of the loop kernel that fit the device together (0 when unknown).
int loop_capacity(int dev, int lpq, bool sorted)
{
    static std::mutex mu;
    static int cap[kMaxDevices][4][2];   // 0: not asked yet
    const int li = lpq == 1 ? 0 : lpq == 2 ? 1 : lpq == 4 ? 2 : 3;
    std::lock_guard<std::mutex> lk(mu);
    int& c = cap[dev][li][sorted ? 1 : 0];
    if (c == 0) {
        int per = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, loop_kernel(lpq, sorted), loop_threads(), 0) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || per < 1 || cus < 1) {
            (void)hipGetLastError();
            return 0;
        }
        c = std::min(per * cus, kLoopMaxBlocks);
    }
    return c;
}

// Whether the stream's kernels may use every compute unit (the loop's blocks
// might otherwise not all be resident).
bool whole_device(hipStream_t s, int dev)
{
    constexpr int kWords = 32;
    uint32_t mask[kWords] = {};
    int cus = 0, bits = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus > 32 * kWords ||
        hipExtStreamGetCUMask(s, (uint32_t)(cus + 31) / 32, mask) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    for (uint32_t w : mask) bits += __builtin_popcount(w);
    return bits == 0 || bits >= cus;
}

// Blocks of pair p's U units when every block takes at most r of them.
int32_t loop_pair_blocks(int64_t U, int64_t r) { return (int32_t)((U + r - 1) / r); }

// The loop's blocks for the grid's source and schedule, U the units of each
// pair and r the most of them a block takes; 0 when the loop does not take it.
int loop_fit(const vicp_grid* g, int capacity, std::vector<int64_t>& U, int64_t& r)
{
    const int lpq = g->nns_lpq, B = g->B;
    U.resize(B);
    int64_t total = 0, most = 0;
    for (int p = 0; p < B; ++p) {
        U[p] = record_units(wave_records(g->m[p], lpq));
        total += U[p];
        most = std::max(most, U[p]);
    }
    if (total < 1 || total > g->loop_units || capacity < 1) return 0;
    // the fewest units per block for which all blocks fit; with more than
    // kLoopRounds the launch-per-step form, which has more waves in flight, is
    // the faster
    r = std::max<int64_t>(1, (total + capacity - 1) / capacity);
    auto blocks = [&](int64_t rr) {
        int64_t n = 0;
        for (int p = 0; p < B; ++p) n += loop_pair_blocks(U[p], rr);
        return n;
    };
    while (r < most && blocks(r) > capacity) ++r;
    const int64_t nb = blocks(r);
    if (nb > capacity || r > (crowded_grid(g) ? kLoopRoundsCrowded : kLoopRounds)) return 0;
    return (int)nb;
}

// loop_fit, with a batch's table on the device.
int loop_plan(vicp_grid* g, int capacity, hipStream_t s)
{
    const int lpq = g->nns_lpq, B = g->B;
    std::vector<int64_t> U;
    int64_t r = 0;
    const int nb = loop_fit(g, capacity, U, r);
    if (nb == 0 || B == 1) return nb;
    if (g->loop_lpq == lpq && g->loop_blocks == nb) return nb;
    // blocks b, b + 8, ... share an XCD: a pair's blocks go there together,
    // the largest pairs first, each to the XCD with the most room
    std::vector<int> order(B);
    for (int p = 0; p < B; ++p) order[p] = p;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return U[a] > U[b]; });
    std::vector<LoopJob> jobs((size_t)nb);
    std::vector<int32_t> base(B);
    int32_t acc = 0;
    for (int p = 0; p < B; ++p) {
        base[p] = acc;
        acc += (int32_t)U[p];
    }
    int next[kXcds];
    for (int x = 0; x < kXcds; ++x) next[x] = x;
    for (int p : order) {
        if (U[p] == 0) continue;
        const int32_t n = loop_pair_blocks(U[p], r);
        for (int32_t b = 0, x = -1; b < n; ++b) {
            if (x < 0 || next[x] >= nb) {
                x = 0;
                for (int y = 1; y < kXcds; ++y)
                    if (next[y] < next[x]) x = y;
            }
            jobs[next[x]] = LoopJob{p, b, n, base[p]};
            next[x] += kXcds;
        }
    }
    upload(jobs.data(), sizeof(LoopJob) * jobs.size(), g->loop_jobs, s);
    g->loop_lpq = lpq;
    g->loop_blocks = nb;
    return nb;
}

// What the launch-per-step search may scan of crowded voxels, by the grid and by
// whether the loop could take the same registration.
void set_step_budget(vicp_grid* g)
{
    std::vector<int64_t> U;
    int64_t r = 0;
    int dev = -1;
    g->step_budget = kRareBudget;
    if (crowded_grid(g) && hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices &&
        loop_fit(g, loop_capacity(dev, g->nns_lpq, g->sort_src), U, r) == 0)
        g->step_budget = kStepBudget;
}

// The loop's launch: K iterations from the state now in g->st on nloop blocks
// (loop_plan).
void queue_loop(vicp_grid* g, const float* px, const float* py, const float* pz, int nloop, int K, int early, double eps,
                int32_t* out_idx, float* out_d2, hipStream_t s)
{
    const int B = g->B;
    if (g->loop_tag > 0xFFFFFFFFu - 200000u) {   // the tags are used up: start again
        launch_fill_u64(g->loop_msg, 0ull, g->loop_units * kLoopWords + (int64_t)B * kPoseWords, s);
        launch_fill_u64((unsigned long long*)(g->res + g->o_abort), 0ull, 1, s);
        g->loop_tag = 0;
    }
    LoopArgs a{};
    a.pd = g->d_pd;
    a.st = g->st;
    a.jobs = B == 1 ? nullptr : g->loop_jobs;
    a.px = px;
    a.py = py;
    a.pz = pz;
    a.ps4 = g->ps4;
    a.dir = g->dir;
    a.off = g->off;
    a.pyr = g->pyr;
    a.qs4 = g->qs4;
    a.nn_idx = out_idx;
    a.nn_d2 = out_d2;
    a.msg = g->loop_msg;
    a.pose_msg = g->loop_pose;
    a.abort_word = (unsigned long long*)(g->res + g->o_abort);
    a.rmse_hist = g->rmse_hist;
    a.fb_hist = g->fb_hist;
    a.deg_hist = g->deg_hist;
    a.ctr_hist = g->ctr_hist;
    a.begun = a.abort_word + 1;
    g->loop_begun += (uint64_t)nloop;
    a.begun_all = g->loop_begun;
    a.arrive = g->loop_arrive;
    a.patience = g->loop_patience;
    a.eps = eps;
    a.tag = g->loop_tag;
    a.K = K;
    a.early_stop = early;
    launch_loop(a, nloop, g->nns_lpq, g->sort_src, s);
    g->loop_tag += (uint32_t)K;
}

// The registration's argument checks (none touches the grid).
int check_register(const vicp_grid* g, const float* px, const float* py, const float* pz,
                   const int64_t* m_per_pair, const vicp_icp_opts* o, const double* Rt_io)
{
    if (!m_per_pair || !o || !Rt_io) return fail(VICP_ERR_INVALID_ARG, "null pointer");
    if (o->max_iter < 0 || o->max_iter > 100000) return fail(VICP_ERR_INVALID_ARG, "max_iter out of range");
    if (!(o->rmse_eps >= 0.0)) return fail(VICP_ERR_INVALID_ARG, "rmse_eps must be >= 0");
    for (int i = 0; i < 12 * g->B; ++i)
        if (!isfinite(Rt_io[i])) return fail(VICP_ERR_INVALID_ARG, "non-finite initial pose");
    int64_t mt = 0;
    for (int p = 0; p < g->B; ++p) {
        if (m_per_pair[p] < 0 || m_per_pair[p] > (int64_t)INT32_MAX)
            return fail(VICP_ERR_INVALID_ARG, "source size out of range");
        mt += m_per_pair[p];
    }
    if (mt > 0 && o->max_iter > 0 && (!px || !py || !pz)) return fail(VICP_ERR_INVALID_ARG, "null pointer");
    if (o->layout != 0 && o->global_only != 0)
        return fail(VICP_ERR_INVALID_ARG, "global_only and the direct layout exclude each other");
    if ((o->nn_idx == nullptr) != (o->nn_d2 == nullptr))
        return fail(VICP_ERR_INVALID_ARG, "nn_idx and nn_d2 are given together or not at all");
    return VICP_OK;
}

// The registration (vicp_register_batched).
// started: the per-pair state and the source plan are already queued (by
// vicp_rebuild_register, on its second stream, which s waits for).
int register_impl(vicp_grid* g, const float* px, const float* py, const float* pz, const int64_t* m_per_pair,
                  const vicp_icp_opts* o, double* Rt_io, vicp_icp_stats* stats, hipStream_t s,
                  bool started = false, bool allow_loop = true)
{
    int rc = check_grid(g);
    if (rc) return rc;
    rc = check_register(g, px, py, pz, m_per_pair, o, Rt_io);
    if (rc) return rc;
    const int B = g->B;
    int64_t mt = 0;
    for (int p = 0; p < B; ++p) mt += m_per_pair[p];
    if (stats)
        for (int p = 0; p < B; ++p) {
            stats[p].iters = 0;
            stats[p].degenerate = 0;
        }
    const int K = o->max_iter;
    g->last_form = VICP_FORM_NONE;
    if (mt == 0 || K == 0) return ensure_source(g, m_per_pair, 1, s);
    if (!px || !py || !pz) return fail(VICP_ERR_INVALID_ARG, "null pointer");
    rc = ensure_source(g, m_per_pair, K, s);
    if (rc) return rc;
    const int early = o->early_stop ? 1 : 0;
    const double eps = o->rmse_eps;
    const bool all_global = o->global_only != 0;
    const bool direct = o->layout != 0;
    if (direct && all_global) return fail(VICP_ERR_INVALID_ARG, "global_only and the direct layout exclude each other");
    if (direct && !g->direct_ready) return fail(VICP_ERR_STATE, "no direct layout: call vicp_direct_build first");
    if ((o->nn_idx == nullptr) != (o->nn_d2 == nullptr))
        return fail(VICP_ERR_INVALID_ARG, "nn_idx and nn_d2 are given together or not at all");
    int32_t* out_idx = o->nn_idx;
    float* out_d2 = o->nn_d2;
    constexpr const char* kTooMany = "too many pairs for the global search";
    if (!started) queue_start(g, Rt_io, px, py, pz, s);
    set_step_budget(g);
    bool plan = g->sort_src && !started;
    vicp_grid::Captured& cg = g->reg;
    int dev = -1;
    std::unique_lock<std::mutex> loop_lock;
    int nloop = 0;
    if (allow_loop && !all_global && !direct && !g_prof.on && !capturing(s) && hipGetDevice(&dev) == hipSuccess &&
        dev >= 0 && dev < kMaxDevices) {
        loop_lock = std::unique_lock<std::mutex>(g_loop_mu[dev], std::try_to_lock);
        if (g->loop_rest > 0) --g->loop_rest;
        else if (loop_lock.owns_lock() && whole_device(s, dev)) nloop = loop_plan(g, loop_capacity(dev, g->nns_lpq, g->sort_src), s);
    }
    if (all_global) plan_exhaustive(g, s);
    g->last_form = nloop > 0 ? VICP_FORM_LOOP : (allow_loop ? VICP_FORM_STEPS : VICP_FORM_HANDED_OVER);
    if (nloop > 0) {
        if (plan) queue_plan(g, px, py, pz, s, false);
        queue_loop(g, px, py, pz, nloop, K, early, eps, out_idx, out_d2, s);
    } else if (o->use_graph) {
        std::vector<uintptr_t> key = {(uintptr_t)px, (uintptr_t)py, (uintptr_t)pz, (uintptr_t)K, (uintptr_t)early,
                                      (uintptr_t)g->nns_block, (uintptr_t)g->nns_lpq, (uintptr_t)g->fb_grid,
                                      (uintptr_t)g->search_mode,
                                      (uintptr_t)g->sort_src, (uintptr_t)all_global, (uintptr_t)direct,
                                      (uintptr_t)g->dblk,
                                      (uintptr_t)g->qx, (uintptr_t)g->qy, (uintptr_t)g->qz,
                                      (uintptr_t)out_idx, (uintptr_t)out_d2};
        uint64_t eb;
        memcpy(&eb, &eps, 8);
        key.push_back((uintptr_t)eb);
        key.push_back((uintptr_t)(g_prof.on ? 1 : 0));
        key.push_back((uintptr_t)(plan ? 1 : 0));
        rc = capture_into(g, cg, key, [&](hipStream_t cs) {
            if (plan) queue_plan(g, px, py, pz, cs, true);
            bool queued = true;
            for (int k = 0; k < K && queued; ++k)
                queued = queue_iteration(g, px, py, pz, k, K, early, eps, cs, true, all_global, direct, out_idx,
                                         out_d2);
            return queued;
        });
        if (rc) return rc;
        ProfScope ps("icp_graph", s, false);
        VICP_HIP(hipGraphLaunch(cg.exec, s));
    } else {
        const bool cap = capturing(s);
        if (plan) queue_plan(g, px, py, pz, s, cap);
        for (int k = 0; k < K; ++k)
            if (!queue_iteration(g, px, py, pz, k, K, early, eps, s, cap, all_global, direct, out_idx, out_d2))
                return fail(VICP_ERR_INVALID_ARG, kTooMany);
    }
    // the results go into mapped pinned memory, followed by this call's tag,
    // which the host waits for (the stream itself is synchronised only when
    // timing events are to be read)
    if (++g->res_gen == 0) g->res_gen = 1;
    const int64_t rwords = (int64_t)(g->res_bytes / 4);
    // the tags' words may hold another layout's data from an earlier call
    const int npub = publish_blocks(rwords);
    for (int b = 0; b < npub; ++b) __atomic_store_n((uint32_t*)g->h_res + rwords + b, 0u, __ATOMIC_RELEASE);
    launch_publish((const uint32_t*)g->res, (uint32_t*)g->d_hres, rwords, g->res_gen, s);
    VICP_HIP(hipGetLastError());
    VICP_HIP(wait_tags((const uint32_t*)g->h_res + rwords, npub, 1, g->res_gen, s));
    if (g_prof.on) VICP_HIP(hipStreamSynchronize(s));
    const char* hb = (const char*)g->h_res;
    const unsigned long long gave_up = *(const unsigned long long*)(hb + g->o_abort);
    if (nloop > 0 && (uint32_t)gave_up == g->loop_tag - (uint32_t)K + 1u) {
        // the loop gave up (blocks that never met, or a query without a finite
        // distance): again by the launch-per-step form
        loop_lock.unlock();
        if ((uint32_t)(gave_up >> 32) == kAbortWait) g->loop_rest = kLoopRest;
        return register_impl(g, px, py, pz, m_per_pair, o, Rt_io, stats, s, false, false);
    }
    const PairState* hst = (const PairState*)hb;
    const double* hr = (const double*)(hb + g->o_rmse);
    const unsigned long long* hc = (const unsigned long long*)(hb + g->o_ctr);
    const int32_t* hf = (const int32_t*)(hb + g->o_fb);
    const int32_t* hflags = (const int32_t*)(hb + g->o_flags);
    if (o->use_graph && g_prof.on) prof_add_graph(cg.events);
    bool nonfinite = false, degenerate = false, internal = false;
    for (int p = 0; p < B; ++p) {
        memcpy(Rt_io + 12 * p, hst[p].Rt, sizeof(double) * 12);
        nonfinite |= (hflags[p] & 1) != 0;
        internal |= (hflags[p] & 2) != 0;
        degenerate |= hst[p].degenerate != 0;
        if (stats) {
            vicp_icp_stats& S = stats[p];
            S.iters = hst[p].iters;
            S.degenerate = hst[p].degenerate;
            for (int k = 0; k < hst[p].iters && k < K; ++k) {
                const size_t h = (size_t)p * K + k;
                if (S.rmse) S.rmse[k] = hr[h];
                if (S.fallbacks) S.fallbacks[k] = hf[h];
                if (S.candidates) S.candidates[k] = (int64_t)hc[2 * h];
                if (S.dilated_lookups) S.dilated_lookups[k] = (int64_t)hc[2 * h + 1];
            }
        }
    }
    if (internal) return fail(VICP_ERR_HIP, "internal: unresolved global search");
    if (nonfinite) return fail(VICP_ERR_NONFINITE, "non-finite source coordinates");
    if (degenerate) return fail(VICP_ERR_DEGENERATE, "a solve kept the previous pose (rank < 2)");
    return VICP_OK;
}

// Refill, dilation and registration in one call (vicp_rebuild_register).
// The refill's host part (bounding box, grid specification) comes first;
// then the pair records and the per-pair state are written, and each of the
// refill's count, scan, scatter and order passes runs in one launch with the
// source plan's matching pass (the two are independent: the plan reads the
// pair records, the pose state and the source, and writes only its own
// buffers, the state, the global-search counts and the fault flags, none of
// which the refill touches).  The dilation and the loop follow.  Forms that
// synchronise inside the refill (given geometry, host-side offsets), searches
// over the source in index order (no plan), the direct layout and the
// exhaustive comparator run the three steps in turn.
int rebuild_register_impl(vicp_grid* g, const float* qx, const float* qy, const float* qz, int32_t rings,
                          const float* px, const float* py, const float* pz, const int64_t* m_per_pair,
                          const vicp_icp_opts* o, double* Rt_io, vicp_icp_stats* stats, hipStream_t s)
{
    if (!g) return fail(VICP_ERR_INVALID_ARG, "null grid");
    if (!g->hist) return fail(VICP_ERR_STATE, "grid not built");
    if (!qx || !qy || !qz) return fail(VICP_ERR_INVALID_ARG, "null pointer");
    if (rings < 0 || rings > g->pad) return fail(VICP_ERR_INVALID_ARG, "rings must be in [0, pad_rings]");
    int rc = check_register(g, px, py, pz, m_per_pair, o, Rt_io);
    if (rc) return rc;
    int64_t mt = 0;
    for (int p = 0; p < g->B; ++p) mt += m_per_pair[p];
    const bool paired = !g->fixed && !g->host_offsets && !g->packed_hash && g->sort_src && mt > 0 &&
                        o->max_iter > 0 && o->layout == 0 && o->global_only == 0;
    if (!paired) {
        rc = grid_fill(g, qx, qy, qz, s);
        if (rc) return rc;
        rc = vicp_dilate(g, rings, s);
        if (rc) return rc;
        return register_impl(g, px, py, pz, m_per_pair, o, Rt_io, stats, s);
    }
    rc = grid_fill_host(g, qx, qy, qz, s);
    if (rc) return rc;
    g->usable = false;   // the grid's words are stale until the refill below is queued
    rc = ensure_source(g, m_per_pair, o->max_iter, s);
    if (rc) return rc;
    fill_pairdev(g, g->h_pd);   // the pair records with the source's fields
    const bool cap = capturing(s);
    const int64_t Vt = g->V_total;
    const int64_t nb = source_buckets(g, g->m);
    const BlockJob* pj = g->jobs_p[kT256];
    const int np = g->njobs_p[kT256];
    const size_t pd_bytes = sizeof(PairDev) * g->h_pd.size();
    if (g->B <= kInlinePairs && pd_bytes <= sizeof(Blob)) {
        // one launch for the records, both passes' clears and the states
        Blob bl;
        memcpy(bl.w, g->h_pd.data(), pd_bytes);
        FrameStart f{};
        for (int p = 0; p < g->B; ++p) {
            for (int j = 0; j < 12; ++j) f.rt[12 * p + j] = Rt_io[12 * p + j];
            f.m[p] = g->m[p];
        }
        uint32_t* z32[6] = {g->hist, g->scan_ticket, g->err, g->sh, g->s_ticket, (uint32_t*)g->sbig};
        const int64_t n32[6] = {Vt + g->pyr_words, 4, 4, nb, 4, g->B};
        for (int k = 0; k < 6; ++k) {
            f.z32[k] = z32[k];
            f.n32[k] = n32[k];
        }
        f.z64[0] = g->scan_status;
        f.n64[0] = scan_tiles(Vt);
        f.z64[1] = g->s_status;
        f.n64[1] = scan_tiles(nb);
        const int64_t n = std::max(Vt + g->pyr_words, nb);
        const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 2048));
        ProfScope ps("start_frame", s, cap);
        hipLaunchKernelGGL(k_start_frame, dim3(blocks), dim3(256), 0, s, bl, (uint32_t*)g->d_pd, (int)(pd_bytes / 4), f,
                           g->B, g->st, g->fb_count, g->flags, n);
    } else {
        clear_for_build(g, s);
        queue_start(g, Rt_io, px, py, pz, s);
        launch_clear4(g->sh, nb, g->s_status, scan_tiles(nb), g->s_ticket, 4, (uint32_t*)g->sbig, g->B, s);
    }
    {
        ProfScope ps("count_bucket", s, cap, true);
        launch_count_bucket(g->qx, g->qy, g->qz, g->d_pd, g->jobs_q, g->njobs_q, g->hist, g->vox, g->rank, g->err,
                            pj, np, px, py, pz, g->st, g->sh, g->skey, g->srank, g->sbig, g->flags, s);
    }
    {
        ProfScope ps("scan_pair", s, cap, true);
        launch_scan_pair(g->hist, Vt, g->off, g->vm, g->dir, g->scan_status, g->scan_ticket, g->sh, nb, g->soff,
                         g->s_status, g->s_ticket, s);
    }
    {
        ProfScope ps("place_pair", s, cap, true);
        launch_place_pair(g->d_pd, g->jobs_q, g->njobs_q, g->vox, g->rank, g->off, g->slots, pj, np, g->skey,
                          g->srank, g->soff, g->sidx, s);
    }
    {
        ProfScope ps("rank_pair", s, cap, true);
        launch_rank_pair(g->qx, g->qy, g->qz, g->d_pd, g->jobs_q, g->njobs_q, g->vox, g->hist, g->off, g->slots,
                         g->vm, g->qs4, g->pyr, pj, np, px, py, pz, g->skey, g->soff, g->sidx, g->sbig, g->ps4, s);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(VICP_ERR_HIP, std::string("grid build: ") + hipGetErrorString(e));
    g->usable = true;
    g->dilated = true;
    g->rings_applied = rings;
    queue_dilate(g, rings, s, cap);
    return register_impl(g, px, py, pz, m_per_pair, o, Rt_io, stats, s, true);
}

}  // namespace

extern "C" {

int vicp_rebuild_register(vicp_grid* g, const float* qx, const float* qy, const float* qz, int32_t rings,
                          const float* px, const float* py, const float* pz, const int64_t* m_per_pair,
                          const vicp_icp_opts* o, double* Rt_io, vicp_icp_stats* stats, hipStream_t s)
{
    (void)hipGetLastError();   // an error left by other code is not ours to report
    return rebuild_register_impl(g, qx, qy, qz, rings, px, py, pz, m_per_pair, o, Rt_io, stats, s);
}

int vicp_register_batched(const vicp_grid* gc, const float* px, const float* py, const float* pz,
                          const int64_t* m_per_pair, const vicp_icp_opts* o, double* Rt_io, vicp_icp_stats* stats,
                          hipStream_t s)
{
    (void)hipGetLastError();   // an error left by other code is not ours to report
    return register_impl(const_cast<vicp_grid*>(gc), px, py, pz, m_per_pair, o, Rt_io, stats, s);
}

int vicp_register(const vicp_grid* g, const float* px, const float* py, const float* pz, int64_t m,
                  const vicp_icp_opts* o, double Rt_io[12], vicp_icp_stats* stats, hipStream_t s)
{
    if (!g) return fail(VICP_ERR_INVALID_ARG, "null grid");
    if (g->B != 1) return fail(VICP_ERR_INVALID_ARG, "vicp_register needs a single-pair grid");
    if (m < 0) return fail(VICP_ERR_INVALID_ARG, "m < 0");
    return vicp_register_batched(g, px, py, pz, &m, o, Rt_io, stats, s);
}

static int p2p_common(vicp_grid* g, const float* px, const float* py, const float* pz, const int64_t* m_per_pair,
                      const double* xi, hipStream_t s)
{
    int rc = check_grid(g);
    if (rc) return rc;
    if (!m_per_pair || !xi) return fail(VICP_ERR_INVALID_ARG, "null pointer");
    rc = ensure_source(g, m_per_pair, 1, s);
    if (rc) return rc;
    if (g->m_total > 0 && (!px || !py || !pz)) return fail(VICP_ERR_INVALID_ARG, "null pointer");
    const bool cap = capturing(s);
    launch_se3(xi, g->B, g->st, g->jl6, g->fb_count, g->flags, s);
    queue_correspondences(g, px, py, pz, g->nn_idx, g->nn_d2, nullptr, s, cap);
    return VICP_OK;
}

int vicp_p2p_loss_fwd(const vicp_grid* gc, const float* px, const float* py, const float* pz,
                      const int64_t* m_per_pair, const double* xi, double* loss, hipStream_t s)
{
    (void)hipGetLastError();   // an error left by other code is not ours to report
    vicp_grid* g = const_cast<vicp_grid*>(gc);
    if (!loss) return fail(VICP_ERR_INVALID_ARG, "null loss");
    int rc = p2p_common(g, px, py, pz, m_per_pair, xi, s);
    if (rc) return rc;
    const bool cap = capturing(s);
    {
        ProfScope ps("loss_terms", s, cap);
        launch_loss_terms(g->d_pd, g->jobs_p[kT256], g->njobs_p[kT256], px, py, pz, g->qx, g->qy, g->qz, g->st, g->nn_idx,
                          nullptr, nullptr, nullptr, nullptr, g->part, g->flags, s);
    }
    launch_loss_finish(g->d_pd, g->B, g->job_begin, g->part, g->jl6, nullptr, loss, nullptr, s);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(VICP_ERR_HIP, std::string("loss fwd: ") + hipGetErrorString(e));
    return VICP_OK;
}

int vicp_p2p_loss_bwd(const vicp_grid* gc, const float* px, const float* py, const float* pz,
                      const int64_t* m_per_pair, const double* xi, const double* gloss, float* dpx, float* dpy,
                      float* dpz, double* dxi, hipStream_t s)
{
    (void)hipGetLastError();   // an error left by other code is not ours to report
    vicp_grid* g = const_cast<vicp_grid*>(gc);
    if (!gloss || !dxi) return fail(VICP_ERR_INVALID_ARG, "null pointer");
    int rc = p2p_common(g, px, py, pz, m_per_pair, xi, s);
    if (rc) return rc;
    if (g->m_total > 0 && (!dpx || !dpy || !dpz)) return fail(VICP_ERR_INVALID_ARG, "null dP");
    const bool cap = capturing(s);
    {
        ProfScope ps("loss_terms", s, cap);
        launch_loss_terms(g->d_pd, g->jobs_p[kT256], g->njobs_p[kT256], px, py, pz, g->qx, g->qy, g->qz, g->st, g->nn_idx,
                          gloss, dpx, dpy, dpz, g->part, g->flags, s);
    }
    launch_loss_finish(g->d_pd, g->B, g->job_begin, g->part, g->jl6, gloss, nullptr, dxi, s);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(VICP_ERR_HIP, std::string("loss bwd: ") + hipGetErrorString(e));
    return VICP_OK;
}

int vicp_grid_describe(const vicp_grid* g, int32_t pair, vicp_grid_desc* out)
{
    (void)hipGetLastError();   // an error left by other code is not ours to report
    int rc = check_grid(g);
    if (rc) return rc;
    if (!out || pair < 0 || pair >= g->B) return fail(VICP_ERR_INVALID_ARG, "bad pair or output");
    const PairHost& h = g->pairs[pair];
    memset(out, 0, sizeof(*out));
    for (int a = 0; a < 3; ++a) {
        out->origin[a] = h.origin[a];
        out->dims[a] = h.dims[a];
    }
    out->inv = h.inv;
    out->voxel = h.voxel;
    out->V = h.V;
    out->n = h.n;
    out->pad_rings = g->pad;
    out->rings_applied = g->rings_applied;
    out->static_bytes = 8 * h.V;
    out->dynamic_bytes = 4 * (h.n + 2 * h.V);
    out->vanicp_bytes = 65536 * h.V;
    out->extra_bytes = g->extra_bytes();
    VICP_HIP(hipDeviceSynchronize());
    unsigned long long* cnt = nullptr;
    VICP_HIP(hipMalloc(&cnt, sizeof(unsigned long long) * 4));
    VICP_HIP(hipMemset(cnt, 0, sizeof(unsigned long long) * 4));
    hipLaunchKernelGGL(k_grid_stats, dim3(std::max<int64_t>(1, std::min<int64_t>((h.V + 255) / 256, 1 << 20))), dim3(256),
                       0, nullptr, g->hist + h.v_base, g->off + h.v_base, g->vm, h.V, cnt);
    unsigned long long hc[4] = {0, 0, 0, 0};
    uint32_t herr = 0;
    hipError_t e1 = hipMemcpy(hc, cnt, sizeof(hc), hipMemcpyDeviceToHost);
    hipError_t e2 = hipMemcpy(&herr, g->err, sizeof(uint32_t), hipMemcpyDeviceToHost);
    (void)hipFree(cnt);
    if (e1 != hipSuccess || e2 != hipSuccess) return fail(VICP_ERR_HIP, "describe readback failed");
    out->occupied = (int64_t)hc[0];
    out->dilated = (int64_t)hc[1];
    out->max_count = (uint32_t)hc[2];
    if (herr) return fail(VICP_ERR_HIP, "internal: a target point fell outside its grid");
    return VICP_OK;
}

int vicp_grid_export(const vicp_grid* g, int32_t pair, uint32_t* hist, uint32_t* off, uint32_t* vm, hipStream_t s)
{
    (void)hipGetLastError();   // an error left by other code is not ours to report
    int rc = check_grid(g);
    if (rc) return rc;
    if (pair < 0 || pair >= g->B) return fail(VICP_ERR_INVALID_ARG, "bad pair");
    const PairHost& h = g->pairs[pair];
    if (hist) VICP_HIP(hipMemcpyAsync(hist, g->hist + h.v_base, sizeof(uint32_t) * h.V, hipMemcpyDeviceToDevice, s));
    if (off)
        hipLaunchKernelGGL(k_export_off, dim3((unsigned)std::min<int64_t>((h.V + 256) / 256, 4096)), dim3(256), 0, s,
                           g->off + h.v_base, h.V + 1, (uint32_t)h.vm_base, off);
    if (vm)
        VICP_HIP(hipMemcpyAsync(vm, g->vm + h.vm_base, sizeof(uint32_t) * (h.n + 2 * h.V), hipMemcpyDeviceToDevice, s));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(VICP_ERR_HIP, std::string("export: ") + hipGetErrorString(e));
    return VICP_OK;
}

int vicp_grid_free(vicp_grid* g)
{
    if (!g) return VICP_OK;
    (void)hipDeviceSynchronize();
    g->drop_graph();
    (void)vicp_direct_free(g);
    if (g->cap_stream) (void)hipStreamDestroy(g->cap_stream);
    g->release(g->ex_bufs, nullptr);
    g->release(g->wv_bufs, nullptr);
    g->release(g->ws_bufs, nullptr);
    g->release(g->vbufs, nullptr);
    g->release(g->owned, nullptr);
    (void)hipDeviceSynchronize();
    if (g->h_res) (void)hipHostFree(g->h_res);
    if (g->h_box) (void)hipHostFree(g->h_box);
    delete g;
    return VICP_OK;
}

}  // extern "C"

// ------------------------------------------------------------------ autotuning
namespace {

// Every schedule choice of a grid (none changes a correspondence, a count or
// a grid word).
struct Sched {
    int count_block, dil_fused, dil_shape, ring_block, nns_block, nns_lpq, sort_src, fb_grid, search_mode;
};

Sched sched_of(const vicp_grid* g)
{
    return Sched{g->count_block, g->dil_fused ? 1 : 0, g->dil_shape, g->ring_block, g->nns_block, g->nns_lpq,
                 g->sort_src ? 1 : 0, g->fb_grid, g->search_mode};
}

void apply_sched(vicp_grid* g, const Sched& c)
{
    g->count_block = c.count_block;
    g->dil_fused = c.dil_fused != 0;
    g->dil_shape = c.dil_shape;
    g->ring_block = c.ring_block;
    g->nns_block = c.nns_block;
    g->nns_lpq = c.nns_lpq;
    g->sort_src = c.sort_src != 0;
    g->fb_grid = c.fb_grid;
    g->search_mode = c.search_mode;
    g->drop_graph();
}

bool sched_valid(const Sched& c)
{
    auto in = [](int v, std::initializer_list<int> ok) { return std::find(ok.begin(), ok.end(), v) != ok.end(); };
    return in(c.count_block, {256, 512, 1024}) && in(c.dil_fused, {0, 1}) && c.dil_shape >= 0 &&
           c.dil_shape < kDilateShapes && in(c.ring_block, {64, 128, 256}) && in(c.nns_block, {128, 256, 512}) &&
           in(c.nns_lpq, {1, 2, 4, 8}) && in(c.sort_src, {0, 1}) && c.fb_grid >= 1 && c.fb_grid <= 65536 &&
           in(c.search_mode, {0, 1});
}

// Stored schedules by shape: in this process, and in the file named by
// VICP_AUTOTUNE_CACHE when set (one line per shape: key, tab, nine numbers).
std::mutex g_tune_mu;
std::map<std::string, Sched> g_tune;
bool g_tune_loaded = false;

void tune_load_locked()
{
    if (g_tune_loaded) return;
    g_tune_loaded = true;
    const char* path = getenv("VICP_AUTOTUNE_CACHE");
    if (!path || !*path) return;
    FILE* f = fopen(path, "r");
    if (!f) return;
    std::string line;
    char buf[4096];
    while (fgets(buf, sizeof buf, f)) {
        line += buf;
        if (line.empty() || line.back() != '\n') continue;   // a key longer than the buffer
        const size_t tab = line.find('\t');
        Sched c{};
        if (tab != std::string::npos &&
            sscanf(line.c_str() + tab + 1, "%d %d %d %d %d %d %d %d %d", &c.count_block, &c.dil_fused, &c.dil_shape,
                   &c.ring_block, &c.nns_block, &c.nns_lpq, &c.sort_src, &c.fb_grid, &c.search_mode) == 9 &&
            sched_valid(c))
            g_tune[line.substr(0, tab)] = c;
        line.clear();
    }
    fclose(f);
}

void tune_store(const std::string& key, const Sched& c)
{
    std::lock_guard<std::mutex> lk(g_tune_mu);
    tune_load_locked();
    g_tune[key] = c;
    const char* path = getenv("VICP_AUTOTUNE_CACHE");
    if (!path || !*path) return;
    if (FILE* f = fopen(path, "a")) {
        fprintf(f, "%s\t%d %d %d %d %d %d %d %d %d\n", key.c_str(), c.count_block, c.dil_fused, c.dil_shape,
                c.ring_block, c.nns_block, c.nns_lpq, c.sort_src, c.fb_grid, c.search_mode);
        fclose(f);
    }
}

bool tune_find(const std::string& key, Sched* out)
{
    std::lock_guard<std::mutex> lk(g_tune_mu);
    tune_load_locked();
    auto it = g_tune.find(key);
    if (it == g_tune.end()) return false;
    *out = it->second;
    return true;
}

// The shape a schedule is stored under: the device's architecture and CU
// count, and per pair the point counts and grid dimensions; the rings, the
// padding, the grid kind and the searches per bucketing pass.
std::string tune_key(const vicp_grid* g, const int64_t* m, int32_t spp)
{
    std::string k;
    int devi = 0;
    hipDeviceProp_t prop{};
    if (hipGetDevice(&devi) == hipSuccess && hipGetDeviceProperties(&prop, devi) == hipSuccess)
        k += std::string(prop.gcnArchName) + "/" + std::to_string(prop.multiProcessorCount);
    else
        (void)hipGetLastError();
    k += " L" + std::to_string(g->rings_applied) + " P" + std::to_string(g->pad) + (g->fixed ? " F" : " B") + " S" +
         std::to_string(spp);
    for (int p = 0; p < g->B; ++p) {
        const PairHost& h = g->pairs[p];
        k += " " + std::to_string(h.n) + "," + std::to_string(m[p]) + "," + std::to_string(h.dims[0]) + "x" +
             std::to_string(h.dims[1]) + "x" + std::to_string(h.dims[2]);
    }
    return k;
}

// A global-search load for timing: the first max(256, m/64) source points of
// each pair listed as unresolved queries.
__global__ void k_synthetic_misses(const PairDev* __restrict__ pd, int npairs, int32_t* __restrict__ fb_count,
                                   uint32_t* __restrict__ fb_list, unsigned long long* __restrict__ fb_key)
{
    const int p = blockIdx.x;
    if (p >= npairs) return;
    const PairDev& P = pd[p];
    const int64_t F = min(P.m, max((int64_t)256, P.m / 64));
    if (threadIdx.x == 0) fb_count[p] = (int32_t)F;
    for (int64_t i = threadIdx.x; i < F; i += blockDim.x) {
        fb_list[P.p_base + i] = (uint32_t)i;
        fb_key[P.p_base + i] = ~0ull;
    }
}

}  // namespace

extern "C" {

// For tests: how long a block of the grid's loop waits (ticks of 10 ns) for a
// block that has not begun, and for any; not part of the interface.
int vicp_test_loop_waits(vicp_grid* g, uint64_t arrive, uint64_t patience)
{
    if (!g) return fail(VICP_ERR_INVALID_ARG, "null grid");
    g->loop_arrive = arrive;
    g->loop_patience = patience;
    return VICP_OK;
}

int vicp_autotune_cache_clear(void)
{
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tune.clear();
    g_tune_loaded = true;   // the file is not read again in this process
    return VICP_OK;
}

// Times the schedule choices on the caller's data and keeps the fastest; see
// the header for what is timed and how.  None of them changes a result, so
// the grid is left as it was (re-running the count or the dilation rewrites
// the same words).
int vicp_autotune(vicp_grid* g, const float* px, const float* py, const float* pz, const int64_t* m_per_pair,
                  int32_t searches_per_plan, hipStream_t s)
{
    (void)hipGetLastError();   // an error left by other code is not ours to report
    int rc = check_grid(g);
    if (rc) return rc;
    if (!m_per_pair) return fail(VICP_ERR_INVALID_ARG, "null pointer");
    if (searches_per_plan < 1) return fail(VICP_ERR_INVALID_ARG, "searches_per_plan must be >= 1");
    // registrations are timed over kTuneIters iterations, single searches alone
    constexpr int kTuneIters = 8;
    const bool registers = searches_per_plan > 1;
    rc = ensure_source(g, m_per_pair, registers ? kTuneIters : 1, s);
    if (rc) return rc;
    if (g->m_total == 0) return VICP_OK;
    if (!px || !py || !pz) return fail(VICP_ERR_INVALID_ARG, "null pointer");
    const std::string key = tune_key(g, m_per_pair, searches_per_plan);
    Sched cached{};
    if (tune_find(key, &cached)) {
        apply_sched(g, cached);
        return VICP_OK;
    }
    std::vector<double> rt(12 * g->B, 0.0);
    for (int p = 0; p < g->B; ++p) rt[12 * p] = rt[12 * p + 4] = rt[12 * p + 8] = 1.0;
    queue_start(g, rt.data(), px, py, pz, s);
    hipEvent_t a, b;
    VICP_HIP(hipEventCreate(&a));
    VICP_HIP(hipEventCreate(&b));
    // one sample is kBurst back-to-back runs (launch jitter averages out);
    // the figure is the best of three samples after one untimed
    constexpr int kBurst = 8;
    auto timed_raw = [&](auto&& work, int burst = kBurst) -> float {
        float best = 1e30f;
        for (int rep = 0; rep < 4; ++rep) {
            (void)hipEventRecord(a, s);
            for (int r = 0; r < burst; ++r) work();
            (void)hipEventRecord(b, s);
            (void)hipEventSynchronize(b);
            float ms = 0.0f;
            (void)hipEventElapsedTime(&ms, a, b);
            if (rep > 0) best = std::min(best, ms / burst);
        }
        return best;
    };
    auto timed = [&](auto&& work) -> float {
        return timed_raw([&] {
            launch_fill_u32((uint32_t*)g->fb_count, 0u, 2 * g->B, s);
            work();
        });
    };
    // a later candidate replaces the best only when it is clearly faster, so
    // that near-ties resolve the same way from run to run
    constexpr float kMargin = 0.99f;
    // (1) the count's block size: the histogram is cleared and recounted (the
    // counts come out the same; the slots it hands out are only used by a
    // build, which recounts)
    if (!g->packed_hash) {
        float best = 1e30f;
        int best_cb = g->count_block;
        for (int cb : {256, 512, 1024}) {
            g->count_block = cb;
            const float t = timed_raw([&] {
                launch_fill_u32(g->hist, 0u, g->V_total, s);
                queue_count(g, g->qx, g->qy, g->qz, false, s);
            });
            if (t < kMargin * best) {
                best = t;
                best_cb = cb;
            }
        }
        g->count_block = best_cb;
    }
    // (2) the dilation, on a grid dilated with 1 to 4 rings (re-running it
    // rewrites the same words)
    const int L = g->rings_applied;
    if (g->dilated && L >= 1 && L <= kFusedRings) {
        float best = 1e30f;
        Sched bs = sched_of(g);
        for (int fused = 1; fused >= 0; --fused)
            for (int v = 0; v < (fused ? kDilateShapes : 3); ++v) {
                g->dil_fused = fused != 0;
                if (fused)
                    g->dil_shape = v;
                else
                    g->ring_block = 64 << v;
                const float t = timed_raw([&] { queue_dilate(g, L, s, true); });
                if (t < kMargin * best) {
                    best = t;
                    bs = sched_of(g);
                }
            }
        g->dil_fused = bs.dil_fused != 0;
        g->dil_shape = bs.dil_shape;
        g->ring_block = bs.ring_block;
    }
    // (3) the search.  Its block size and candidate loop are those whose search in
    // the registration form, alone and at the identity pose, is the fastest, for
    // each number of lanes and order: the launch-per-step form runs under them
    // (large sources, the direct layout, timing on, a loop that gave up), and the
    // resident loop does not use them.  The lanes and the order are then those of
    // the fastest kTuneIters iterations in the form that the registration would
    // run, or for single searches of the fastest search.
    const float plan_ms = timed([&] { queue_plan(g, px, py, pz, s, true); });
    Sched picked = sched_of(g);
    float best = 1e30f;
    int dev = -1;
    std::unique_lock<std::mutex> loop_lock;
    if (registers && hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices && whole_device(s, dev))
        loop_lock = std::unique_lock<std::mutex>(g_loop_mu[dev], std::try_to_lock);
    // the search kernel's own time, the least of five after one untimed: queued
    // back to back, the launches beside it hide differences of a few microseconds
    auto search_alone = [&]() -> float {
        float least = 1e30f;
        for (int rep = 0; rep < 6; ++rep) {
            launch_fill_u32((uint32_t*)g->fb_count, 0u, 2 * g->B, s);
            ExtEvents ext;
            ext.a = a;
            ext.b = b;
            t_ext = &ext;
            queue_search(g, px, py, pz, nullptr, nullptr, s, true);
            t_ext = nullptr;
            (void)hipEventSynchronize(b);
            float ms = 0.0f;
            if (rep > 0 && ext.used && hipEventElapsedTime(&ms, a, b) == hipSuccess) least = std::min(least, ms);
        }
        return least;
    };
    // kTuneIters iterations; gave_up: whether a loop among them did
    auto iterations = [&](int nloop, bool* gave_up) -> float {
        const uint32_t tag0 = g->loop_tag;
        const float t = timed_raw([&] {
            queue_start(g, rt.data(), px, py, pz, s);
            if (nloop > 0) queue_loop(g, px, py, pz, nloop, kTuneIters, 0, 0.0, nullptr, nullptr, s);
            for (int k = 0; k < kTuneIters && nloop == 0; ++k)
                (void)queue_iteration(g, px, py, pz, k, kTuneIters, 0, 0.0, s, true, false, false, nullptr, nullptr);
        }, 1);
        unsigned long long word = 0;
        if (nloop > 0 && hipMemcpy(&word, g->res + g->o_abort, sizeof(word), hipMemcpyDeviceToHost) != hipSuccess)
            word = ~0ull;
        *gave_up = nloop > 0 && ((uint32_t)word - tag0 - 1u < g->loop_tag - tag0 || word == ~0ull);
        return t / (float)kTuneIters;
    };
    for (int sorted = 0; sorted < 2; ++sorted)
        for (int lpq : {1, 2, 4, 8}) {
            g->sort_src = sorted != 0;
            g->nns_lpq = lpq;
            set_step_budget(g);
            float t = 1e30f;
            int bs_best = 256, mode_best = 0;
            for (int bs : {128, 256, 512})
                for (int mode = 0; mode < 2; ++mode) {
                    g->nns_block = bs;
                    g->search_mode = mode;
                    const float ts = search_alone();
                    if (ts < kMargin * t) {
                        t = ts;
                        bs_best = bs;
                        mode_best = mode;
                    }
                }
            g->nns_block = bs_best;
            g->search_mode = mode_best;
            if (registers) {
                // a loop that gives up did not run its iterations
                bool gave_up = false;
                const int nloop = loop_lock.owns_lock() ? loop_plan(g, loop_capacity(dev, lpq, g->sort_src), s) : 0;
                t = iterations(nloop, &gave_up);
                if (gave_up) t = iterations(0, &gave_up);
            }
            t += sorted ? plan_ms / (float)searches_per_plan : 0.0f;
            if (t < kMargin * best) {
                best = t;
                picked = sched_of(g);
            }
        }
    if (loop_lock.owns_lock()) {
        VICP_HIP(hipStreamSynchronize(s));   // no loop is left running when the device's turn passes on
        loop_lock.unlock();
    }
    queue_start(g, rt.data(), px, py, pz, s);
    apply_sched(g, picked);
    set_step_budget(g);
    int best_fg = g->fb_grid;
    // (4) the exhaustive search's blocks: the fold every iteration runs, and on a
    // crowded grid, whose searches list queries, such a load once per bucketing
    // pass (elsewhere none is listed)
    {
        const int tab = table_of(g->nns_block / g->nns_lpq);
        best = 1e30f;
        for (int fg : {64, 128, 256, 512, 1024}) {
            g->fb_grid = fg;
            const float t0 = timed([&] { queue_search(g, px, py, pz, nullptr, nullptr, s, true); });
            const float t1 = !crowded_grid(g) ? 0.0f : timed_raw([&] {
                hipLaunchKernelGGL(k_synthetic_misses, dim3(g->B), dim3(256), 0, s, g->d_pd, g->B, g->fb_count,
                                   g->fb_list, g->fb_key);
                (void)launch_fallback(g->d_pd, g->B, fg, g->qx, g->qy, g->qz, px, py, pz, g->st, g->fb_count,
                                      g->fb_list, g->fb_key, g->fjobs[tab][wpb_index(g->nns_block)],
                                      g->nfjobs[tab][wpb_index(g->nns_block)], g->npart, g->ctr,
                                      g->fpart, g->fctr, s);
            });
            const float t = t0 + t1 / (float)searches_per_plan;
            if (t < kMargin * best) {
                best = t;
                best_fg = fg;
            }
        }
    }
    g->fb_grid = best_fg;
    g->drop_graph();
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    launch_fill_u32((uint32_t*)g->fb_count, 0u, 2 * g->B, s);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(VICP_ERR_HIP, std::string("autotune: ") + hipGetErrorString(e));
    VICP_HIP(hipStreamSynchronize(s));
    tune_store(key, sched_of(g));
    return VICP_OK;
}

int vicp_get_build_schedule(const vicp_grid* g, int32_t* count_block, int32_t* dilate_fused, int32_t* dilate_tile,
                            int32_t* ring_block)
{
    if (!g) return fail(VICP_ERR_INVALID_ARG, "null grid");
    if (count_block) *count_block = g->count_block;
    if (dilate_fused) *dilate_fused = g->dil_fused ? 1 : 0;
    if (dilate_tile) *dilate_tile = g->dil_shape;
    if (ring_block) *ring_block = g->ring_block;
    return VICP_OK;
}

int vicp_set_build_schedule(vicp_grid* g, int32_t count_block, int32_t dilate_fused, int32_t dilate_tile,
                            int32_t ring_block)
{
    if (!g) return fail(VICP_ERR_INVALID_ARG, "null grid");
    Sched c = sched_of(g);
    c.count_block = count_block;
    c.dil_fused = dilate_fused;
    c.dil_shape = dilate_tile;
    c.ring_block = ring_block;
    if (!sched_valid(c))
        return fail(VICP_ERR_INVALID_ARG, "count_block must be 256, 512 or 1024, dilate_fused 0 or 1, dilate_tile "
                                          "0-4, ring_block 64, 128 or 256");
    apply_sched(g, c);
    return VICP_OK;
}

int vicp_get_schedule(const vicp_grid* g, int32_t* nns_block, int32_t* lanes_per_query, int32_t* sort_source,
                      int32_t* fallback_grid, int32_t* search_mode)
{
    if (!g) return fail(VICP_ERR_INVALID_ARG, "null grid");
    if (nns_block) *nns_block = g->nns_block;
    if (lanes_per_query) *lanes_per_query = g->nns_lpq;
    if (sort_source) *sort_source = g->sort_src ? 1 : 0;
    if (fallback_grid) *fallback_grid = g->fb_grid;
    if (search_mode) *search_mode = g->search_mode;
    return VICP_OK;
}

int vicp_set_schedule(vicp_grid* g, int32_t nns_block, int32_t lanes_per_query, int32_t sort_source,
                      int32_t fallback_grid, int32_t search_mode)
{
    if (!g) return fail(VICP_ERR_INVALID_ARG, "null grid");
    if (nns_block != 128 && nns_block != 256 && nns_block != 512)
        return fail(VICP_ERR_INVALID_ARG, "nns_block must be 128, 256 or 512");
    if (lanes_per_query != 1 && lanes_per_query != 2 && lanes_per_query != 4 && lanes_per_query != 8)
        return fail(VICP_ERR_INVALID_ARG, "lanes_per_query must be 1, 2, 4 or 8");
    if (fallback_grid < 1 || fallback_grid > 65536) return fail(VICP_ERR_INVALID_ARG, "fallback_grid out of range");
    if (search_mode < 0 || search_mode > 1) return fail(VICP_ERR_INVALID_ARG, "search_mode must be 0 or 1");
    g->search_mode = search_mode;
    g->nns_block = nns_block;
    g->nns_lpq = lanes_per_query;
    g->sort_src = sort_source != 0;
    g->fb_grid = fallback_grid;
    g->drop_graph();
    return VICP_OK;
}

int vicp_prof_enable(int32_t on)
{
    std::lock_guard<std::mutex> lk(g_prof.mu);
    g_prof.on = on != 0;
    return VICP_OK;
}

int vicp_prof_read(const char* kernel, int64_t* launches, double* total_ms)
{
    std::lock_guard<std::mutex> lk(g_prof.mu);
    prof_flush_locked();
    if (!kernel) return fail(VICP_ERR_INVALID_ARG, "null kernel name");
    auto it = g_prof.acc.find(kernel);
    if (launches) *launches = it == g_prof.acc.end() ? 0 : it->second.first;
    if (total_ms) *total_ms = it == g_prof.acc.end() ? 0.0 : it->second.second;
    return VICP_OK;
}

int vicp_prof_samples(const char* kernel, double* ms, int64_t cap, int64_t* count)
{
    std::lock_guard<std::mutex> lk(g_prof.mu);
    prof_flush_locked();
    if (!kernel || cap < 0 || (cap > 0 && !ms)) return fail(VICP_ERR_INVALID_ARG, "null kernel name or output");
    auto it = g_prof.samples.find(kernel);
    const int64_t n = it == g_prof.samples.end() ? 0 : (int64_t)it->second.size();
    for (int64_t i = 0; i < std::min(n, cap); ++i) ms[i] = it->second[(size_t)i];
    if (count) *count = n;
    return VICP_OK;
}

int vicp_prof_reset(void)
{
    std::lock_guard<std::mutex> lk(g_prof.mu);
    prof_flush_locked();
    g_prof.acc.clear();
    g_prof.samples.clear();
    return VICP_OK;
}

}  // extern "C"
