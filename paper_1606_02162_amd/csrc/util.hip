// Error reporting, device helpers and small ABI functions of libgila.
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <vector>
#include <algorithm>

#include <rocprofiler-sdk-roctx/roctx.h>

#include "device_util.h"
#include "gila_internal.h"

namespace gila {

// ------------------------------------------------------------------ exclusive scan (int64)
constexpr int kScanItems = 8;                  // items per thread
constexpr int kScanTile = kBlock * kScanItems;  // items per workgroup

__device__ __forceinline__ int64_t load_tile(const int64_t* __restrict__ in, int64_t n,
                                             int64_t (&v)[kScanItems]) {
    const int64_t t0 = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int64_t sum = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        v[i] = (t0 + i < n) ? in[t0 + i] : 0;
        sum += v[i];
    }
    return sum;
}

__global__ __launch_bounds__(kBlock) void tile_sums_kernel(const int64_t* __restrict__ in, int64_t n,
                                                           int64_t* __restrict__ tile_sums) {
    __shared__ int64_t s_red[kWaves];
    int64_t v[kScanItems];
    const int64_t total = block_sum<int64_t>(load_tile(in, n, v), s_red);
    if (threadIdx.x == 0) tile_sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(kBlock) void scan_sums_kernel(int64_t* __restrict__ sums, int64_t m) {
    // in place: sums[i] <- sums[0] + ... + sums[i-1] (one workgroup)
    __shared__ int64_t s_red[kWaves];
    int64_t carry = 0;
    for (int64_t b = 0; b < m; b += kBlock) {
        const int64_t i = b + threadIdx.x;
        const int64_t x = i < m ? sums[i] : 0;
        int64_t total;
        const int64_t ex = block_exclusive_scan<int64_t>(x, s_red, total);
        if (i < m) sums[i] = carry + ex;
        carry += total;
    }
}

// The scan of each tile from the sum of the tiles before it: sums[tile] with SCANNED,
// else added up here.
template <bool SCANNED>
__global__ __launch_bounds__(kBlock) void scan_tiles_kernel(const int64_t* __restrict__ in,
                                                            int64_t* __restrict__ out, int64_t n,
                                                            const int64_t* __restrict__ sums) {
    __shared__ int64_t s_red[kWaves];
    int64_t before = 0;
    if constexpr (SCANNED) {
        before = sums[blockIdx.x];
    } else if (blockIdx.x > 0) {
        for (int t = threadIdx.x; t < (int)blockIdx.x; t += kBlock) before += sums[t];
        before = block_sum<int64_t>(before, s_red);
    }
    const int64_t t0 = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int64_t v[kScanItems];
    const int64_t sum = load_tile(in, n, v);
    int64_t total;
    int64_t run = before + block_exclusive_scan<int64_t>(sum, s_red, total);
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        run += v[i];
        if (t0 + i < n) out[t0 + i + 1] = run;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out[0] = 0;
}

int64_t scan_workspace_count(int64_t n) { return n <= 0 ? 1 : (n + kScanTile - 1) / kScanTile; }

// One launch for a tile, two while adding up the tiles before each costs less than the
// launch that scans their sums (up to kDirectTiles: 8 loads per thread), three above.
// The launches are what the builds' scans cost: a small world of 3k vertices takes nine
// (its layout 917 -> 878 us; pruned R-MAT scale 16, 21 scans, 4528 -> 4326).
constexpr int64_t kDirectTiles = 2048;
int enqueue_exclusive_scan_i64(const int64_t* in, int64_t* out, int64_t n, int64_t* ws,
                               hipStream_t s) {
    n = std::max<int64_t>(n, 0);
    const int64_t tiles = scan_workspace_count(n);
    const dim3 grid((unsigned)tiles);
    if (tiles > 1) hipLaunchKernelGGL(tile_sums_kernel, grid, dim3(kBlock), 0, s, in, n, ws);
    if (tiles > kDirectTiles) {
        hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(kBlock), 0, s, ws, tiles);
        hipLaunchKernelGGL(scan_tiles_kernel<true>, grid, dim3(kBlock), 0, s, in, out, n, ws);
    } else {
        hipLaunchKernelGGL(scan_tiles_kernel<false>, grid, dim3(kBlock), 0, s, in, out, n, ws);
    }
    GILA_HIP(hipGetLastError());
    return GILA_OK;
}

int exclusive_scan_i64(const int64_t* in, int64_t* out, int64_t n, hipStream_t s) {
    int64_t* ws = nullptr;
    GILA_TRY(dalloc_t(&ws, (size_t)scan_workspace_count(n)));
    const int rc = enqueue_exclusive_scan_i64(in, out, n, ws, s);
    const hipError_t e2 = hipStreamSynchronize(s);
    dfree_on(ws, s);
    if (rc) return rc;
    if (e2 != hipSuccess) return fail(GILA_EDEVICE, "scan failed: %s", hipGetErrorString(e2));
    return GILA_OK;
}

// ------------------------------------------------------------------ stable counting pass
// One pass of a stable counting sort by the digit (key >> shift) & mask in
// [0, nkeys), in tiles of `tj` consecutive elements.  Element j of the input
// is perm[j] (j itself when perm is null); key is indexed by element.
// The per-tile histogram is stored digit-major (hist[digit * ntiles + tile]),
// so that its exclusive prefix sum is the first output position of each
// (digit, tile).
__global__ __launch_bounds__(kBlock) void count_tiles_kernel(int64_t T, int64_t tj, int64_t ntiles,
                                                             int32_t nkeys,
                                                             const uint32_t* __restrict__ key,
                                                             int shift, uint32_t mask,
                                                             const int32_t* __restrict__ perm,
                                                             int64_t* __restrict__ hist) {
    extern __shared__ int32_t s_count[];
    for (int s = threadIdx.x; s < nkeys; s += kBlock) s_count[s] = 0;
    __syncthreads();
    const int64_t j0 = (int64_t)blockIdx.x * tj;
    const int64_t j1 = j0 + tj < T ? j0 + tj : T;
    for (int64_t j = j0 + threadIdx.x; j < j1; j += kBlock)
        atomicAdd(&s_count[(key[perm ? perm[j] : j] >> shift) & mask], 1);
    __syncthreads();
    for (int s = threadIdx.x; s < nkeys; s += kBlock) hist[(int64_t)s * ntiles + blockIdx.x] = s_count[s];
}

// W wavefronts per tile, each on a quarter (or all) of it in order, 64
// elements a step.  Lanes with equal digits find each other by one ballot per
// digit bit; an element's place is its digit's next one plus its rank among
// the lower lanes.  Latency-bound (a tile is a chain of steps): one wavefront
// per tile with a 64-step readlane ranking took 126 us a pass on 262144
// elements (64 tiles), this 12.5 us (128 tiles of four wavefronts, 11 ballots
// for 2048 digits).  W = 1 where W histograms of nkeys words do not fit in LDS.
template <int W>
__global__ __launch_bounds__(64 * W) void scatter_tiles_kernel(int64_t T, int64_t tj, int64_t ntiles,
                                                               int32_t nkeys, int bits,
                                                               const uint32_t* __restrict__ key,
                                                               int shift, uint32_t mask,
                                                               const int32_t* __restrict__ perm,
                                                               const int64_t* __restrict__ base,
                                                               int32_t* __restrict__ out) {
    extern __shared__ int32_t s_next[];  // [W][nkeys]
    const int lane = lane64(), w = wave_id();
    const int64_t j0 = (int64_t)blockIdx.x * tj;
    const int64_t j1 = j0 + tj < T ? j0 + tj : T;
    const int64_t part = (tj / W + 63) / 64 * 64;  // W * part >= tj
    const int64_t w0 = min(j0 + w * part, j1), w1 = min(w0 + part, j1);
    int32_t* mine = s_next + (size_t)w * nkeys;
    if constexpr (W > 1) {
        for (int s = threadIdx.x; s < nkeys * W; s += 64 * W) s_next[s] = 0;
        __syncthreads();
        for (int64_t j = w0 + lane; j < w1; j += 64)
            atomicAdd(&mine[(key[perm ? perm[j] : j] >> shift) & mask], 1);
        __syncthreads();
    }
    // first place of each digit for each wavefront
    for (int s = threadIdx.x; s < nkeys; s += 64 * W) {
        int32_t at = (int32_t)base[(int64_t)s * ntiles + blockIdx.x];
        for (int q = 0; q < W; ++q) {
            const int32_t c = W > 1 ? s_next[(size_t)q * nkeys + s] : 0;
            s_next[(size_t)q * nkeys + s] = at;
            at += c;
        }
    }
    __syncthreads();
    const uint64_t below = (1ull << lane) - 1ull;
    for (int64_t c = w0; c < w1; c += 64) {
        const int64_t j = c + lane;
        const bool valid = j < w1;
        const int32_t e = valid ? (perm ? perm[j] : (int32_t)j) : 0;
        const uint32_t d = valid ? (key[e] >> shift) & mask : 0u;
        uint64_t same = __ballot(valid);
        for (int b = 0; b < bits; ++b) {
            const uint64_t on = __ballot((d >> b) & 1u);
            same &= ((d >> b) & 1u) ? on : ~on;
        }
        if (valid) {
            const int32_t at = mine[d];
            out[at + __popcll(same & below)] = e;
            // the last lane of each digit moves its next place
            if ((same >> lane) == 1ull) mine[d] = at + __popcll(same);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

int64_t counting_tile(int64_t T, int32_t nkeys) {
    // tiles of 2048, larger where the histogram would exceed 2^24 words
    return std::max<int64_t>(2048, ((T * nkeys + (1 << 24) - 1) >> 24) + 63) / 64 * 64;
}

int stable_counting_pass(int64_t T, int64_t tj, int32_t nkeys, const uint32_t* key, int shift,
                         uint32_t mask, const int32_t* perm, int32_t* out, int64_t* hist,
                         int64_t* hscan, int64_t* ws, hipStream_t s) {
    if (T <= 0) return GILA_OK;
    const int64_t ntiles = (T + tj - 1) / tj;
    const size_t one = sizeof(int32_t) * (size_t)nkeys;
    constexpr size_t kPlain = 48 * 1024;  // more needs the kernel's limit raised
    int bits = 0;
    while ((1 << bits) < nkeys) ++bits;
    if (one > kPlain) {
        (void)quiet(hipFuncSetAttribute((const void*)count_tiles_kernel,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)one));
        (void)quiet(hipFuncSetAttribute((const void*)scatter_tiles_kernel<1>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)one));
    }
    hipLaunchKernelGGL(count_tiles_kernel, dim3((unsigned)ntiles), dim3(kBlock), one, s, T, tj, ntiles,
                       nkeys, key, shift, mask, perm, hist);
    GILA_HIP(hipGetLastError());
    GILA_TRY(enqueue_exclusive_scan_i64(hist, hscan, ntiles * nkeys, ws, s));
    if (4 * one <= kPlain)
        hipLaunchKernelGGL(scatter_tiles_kernel<4>, dim3((unsigned)ntiles), dim3(256), 4 * one, s, T, tj,
                           ntiles, nkeys, bits, key, shift, mask, perm, hscan, out);
    else
        hipLaunchKernelGGL(scatter_tiles_kernel<1>, dim3((unsigned)ntiles), dim3(64), one, s, T, tj,
                           ntiles, nkeys, bits, key, shift, mask, perm, hscan, out);
    GILA_HIP(hipGetLastError());
    return GILA_OK;
}

int stable_order_by_key(int32_t n, const uint32_t* key, uint32_t max_key, int32_t* out,
                        hipStream_t s) {
    if (n <= 0) return GILA_OK;
    constexpr int kDigitBits = 11;
    constexpr uint32_t kMask = (1u << kDigitBits) - 1u;
    int passes = 1;
    while (passes * kDigitBits < 32 && (max_key >> (passes * kDigitBits)) > 0) ++passes;
    const int64_t tj = counting_tile(n, 1 << kDigitBits);
    const int64_t H = (n + tj - 1) / tj * (1 << kDigitBits);
    const size_t hb = ((size_t)H * 8 + 255) & ~(size_t)255;
    const size_t sb = ((size_t)(H + 1) * 8 + 255) & ~(size_t)255;
    const size_t wb = ((size_t)scan_workspace_count(H) * 8 + 255) & ~(size_t)255;
    struct Tmp {
        void* p = nullptr;
        hipStream_t s;
        ~Tmp() { dfree_on(p, s); }
    } mem{nullptr, s};
    GILA_TRY(dalloc(&mem.p, hb + sb + wb + sizeof(int32_t) * (size_t)n));
    char* at = static_cast<char*>(mem.p);
    int64_t* hist = reinterpret_cast<int64_t*>(at);
    int64_t* hscan = reinterpret_cast<int64_t*>(at + hb);
    int64_t* ws = reinterpret_cast<int64_t*>(at + hb + sb);
    int32_t* buf = reinterpret_cast<int32_t*>(at + hb + sb + wb);
    // the last pass writes `out`; earlier ones alternate so that it does
    const int32_t* src = nullptr;
    for (int p = 0; p < passes; ++p) {
        const int shift = p * kDigitBits;
        const int32_t nkeys = (int32_t)std::min<uint64_t>(1u << kDigitBits, ((uint64_t)max_key >> shift) + 1);
        int32_t* dst = ((passes - 1 - p) & 1) ? buf : out;
        GILA_TRY(stable_counting_pass(n, tj, nkeys, key, shift, kMask, src, dst, hist, hscan, ws, s));
        src = dst;
    }
    return GILA_OK;
}

static double wall_s() {
    return std::chrono::duration<double>(std::chrono::steady_clock::now().time_since_epoch())
        .count();
}

TraceRange::TraceRange(const char* name) { roctxRangePushA(name); }
TraceRange::~TraceRange() { roctxRangePop(); }

// A phase timer is also a roctx range of the whole call, with a marker at
// the end of each phase.
PhaseTimer::PhaseTimer(const char* w, hipStream_t s) : what(w), stream(s) {
    roctxRangePushA(w);
    const char* e = getenv("GILA_TIMING");
    on = e && e[0] == '1';
    t0 = last = on ? wall_s() : 0.0;
}

void PhaseTimer::mark(const char* phase) {
    char name[96];
    snprintf(name, sizeof(name), "%s: %s done", what, phase);
    roctxMarkA(name);
    if (!on) return;
    (void)quiet(hipStreamSynchronize(stream));
    const double t = wall_s();
    char buf[128];
    snprintf(buf, sizeof(buf), " %s=%.2f", phase, (t - last) * 1e3);
    log += buf;
    last = t;
}

PhaseTimer::~PhaseTimer() {
    if (on) fprintf(stderr, "[gila timing] %s total=%.2f ms:%s\n", what, (wall_s() - t0) * 1e3,
                    log.c_str());
    roctxRangePop();
}

// A fixed buffer per thread: recording an error never allocates.
static thread_local char t_last_error[1024];

int fail(int code, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(t_last_error, sizeof(t_last_error), fmt, ap);
    va_end(ap);
    return code;
}

void clear_error() { t_last_error[0] = '\0'; }

// ------------------------------------------------------------------ device memory cache
// hipFree synchronises the whole device.  Blocks released with dfree_on() go to
// a cache instead and are reused by a later dalloc() of the same size class
// once the work on the releasing stream has completed (an event marks it), so
// code that runs beside other streams (the layout server's builder, batched
// launches, ticks) never waits for the whole device.  dfree() keeps
// hipFree's semantics.  Cached blocks beyond kCacheLimit are returned to the
// device (oldest first), and all of them when an allocation fails.
//
// An event must not be asked about once the stream it was recorded on is gone (the
// runtime may look at that stream), so no event outlives its stream here: a public call
// settles what it released on the caller's stream before it returns (SettleOnReturn), the
// layout server what was released on its own streams before it destroys them.
namespace {
struct CachedBlock {
    void* p;
    size_t bytes;
    hipEvent_t ev;  // null: reusable at once
    uint64_t seq;
    hipStream_t stream;  // of the event
};
struct LiveBlock {
    int device;
    size_t bytes;
};
std::mutex g_mem_mu;
std::multimap<std::pair<int, size_t>, CachedBlock> g_cache;
std::map<void*, LiveBlock> g_live;
size_t g_cached_bytes = 0;
uint64_t g_seq = 0;
std::atomic<int64_t> g_events{0};  // cached blocks with an event (changed with the lock held)
constexpr size_t kCacheLimit = (size_t)16 << 30;

size_t size_class(size_t b) {
    constexpr size_t kBig = (size_t)64 << 20;
    if (b > kBig) return (b + kBig - 1) / kBig * kBig;
    size_t r = 512;
    while (r < b) r <<= 1;
    return r;
}

// hipEventQuery reports pending work as hipErrorNotReady (and may refuse the
// query, e.g. while another thread captures a stream), which HIP also keeps
// as the thread's last error: it is taken back here, so that the next launch
// check does not report it; a block whose event cannot be queried waits.
bool block_ready(const CachedBlock& c) {
    if (!c.ev) return true;
    return quiet(hipEventQuery(c.ev)) == hipSuccess;
}

void drop_event(CachedBlock& c) {
    if (!c.ev) return;
    (void)quiet(hipEventDestroy(c.ev));
    c.ev = nullptr;
    --g_events;
}

// Returns ready cached blocks to the device until at most `keep` bytes stay
// cached (all ready blocks for keep = 0).  Lock held.
void trim_locked(size_t keep) {
    std::vector<std::multimap<std::pair<int, size_t>, CachedBlock>::iterator> order;
    for (auto it = g_cache.begin(); it != g_cache.end(); ++it) order.push_back(it);
    std::sort(order.begin(), order.end(),
              [](const auto& a, const auto& b) { return a->second.seq < b->second.seq; });
    for (auto it : order) {
        if (g_cached_bytes <= keep) break;
        if (!block_ready(it->second)) continue;
        DeviceGuard dg(it->first.first);
        if (quiet(hipFree(it->second.p)) != hipSuccess) continue;  // kept for a later trim
        drop_event(it->second);
        g_cached_bytes -= it->second.bytes;
        g_cache.erase(it);
    }
}
}  // namespace

int dalloc(void** p, size_t bytes) {
    *p = nullptr;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return fail(GILA_EDEVICE, "no current device");
    const size_t rb = size_class(bytes ? bytes : 16);
    {
        std::lock_guard<std::mutex> lk(g_mem_mu);
        auto range = g_cache.equal_range({dev, rb});
        for (auto it = range.first; it != range.second; ++it) {
            if (!block_ready(it->second)) continue;
            *p = it->second.p;
            drop_event(it->second);
            g_cached_bytes -= rb;
            g_cache.erase(it);
            g_live[*p] = LiveBlock{dev, rb};
            return GILA_OK;
        }
    }
    hipError_t e = hipMalloc(p, rb);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        {
            std::lock_guard<std::mutex> lk(g_mem_mu);
            trim_locked(0);
        }
        e = hipMalloc(p, rb);
    }
    if (e != hipSuccess) {
        *p = nullptr;
        (void)hipGetLastError();
        return fail(e == hipErrorOutOfMemory ? GILA_ENOMEM : GILA_EDEVICE,
                    "hipMalloc(%zu bytes) failed: %s", bytes, hipGetErrorString(e));
    }
    std::lock_guard<std::mutex> lk(g_mem_mu);
    g_live[*p] = LiveBlock{dev, rb};
    return GILA_OK;
}

void dfree(void* p) {
    if (!p) return;
    {
        std::lock_guard<std::mutex> lk(g_mem_mu);
        g_live.erase(p);
    }
    (void)quiet(hipFree(p));
}

void dfree_on(void* p, hipStream_t s, bool idle) {
    if (!p) return;
    std::lock_guard<std::mutex> lk(g_mem_mu);
    auto it = g_live.find(p);
    if (it == g_live.end()) {  // not from dalloc: plain free
        (void)quiet(hipFree(p));
        return;
    }
    CachedBlock c{p, it->second.bytes, nullptr, ++g_seq, s};
    if (!idle) {
        if (hipEventCreateWithFlags(&c.ev, hipEventDisableTiming) != hipSuccess ||
            hipEventRecord(c.ev, s) != hipSuccess) {
            // cannot mark the stream: wait for it instead
            if (c.ev) (void)quiet(hipEventDestroy(c.ev));
            c.ev = nullptr;
            (void)quiet(hipStreamSynchronize(s));
        }
        if (c.ev) ++g_events;
    }
    g_cache.insert({{it->second.device, c.bytes}, c});
    g_cached_bytes += c.bytes;
    g_live.erase(it);
    if (g_cached_bytes > kCacheLimit) trim_locked(kCacheLimit / 2);
}

void settle_released(hipStream_t s) {
    if (!s || g_events == 0) return;  // (the null stream stays)
    uint64_t upto = 0;
    {
        std::lock_guard<std::mutex> lk(g_mem_mu);
        for (const auto& kv : g_cache)
            if (kv.second.ev && kv.second.stream == s) upto = std::max(upto, kv.second.seq);
    }
    if (upto == 0) return;
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (quiet(hipStreamIsCapturing(s, &st)) != hipSuccess || st != hipStreamCaptureStatusNone) return;
    if (quiet(hipStreamSynchronize(s)) != hipSuccess) return;
    std::lock_guard<std::mutex> lk(g_mem_mu);
    for (auto& kv : g_cache) {
        CachedBlock& c = kv.second;
        if (c.ev && c.stream == s && c.seq <= upto) drop_event(c);
    }
}

int64_t release_cached() {
    std::lock_guard<std::mutex> lk(g_mem_mu);
    const size_t before = g_cached_bytes;
    trim_locked(0);
    return (int64_t)(before - g_cached_bytes);
}

Release public_release() {
    if (hipDeviceSynchronize() != hipSuccess) {
        (void)hipGetLastError();
        return Release{};
    }
    return Release{true, nullptr, true};
}

DeviceGuard::DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) prev = -1;
    ok = (prev == dev) || (hipSetDevice(dev) == hipSuccess);
}

DeviceGuard::~DeviceGuard() {
    if (prev >= 0) (void)quiet(hipSetDevice(prev));
}

static std::mutex g_mu;
static std::map<int, DeviceInfo> g_info;

// Capture streams are per thread (captures on one stream from two threads
// would interleave) and are destroyed when the thread exits.
struct CaptureStreams {
    std::map<int, hipStream_t> by_device;
    ~CaptureStreams() {
        for (auto& kv : by_device) (void)quiet(hipStreamDestroy(kv.second));
    }
};
static thread_local CaptureStreams t_capture;

hipStream_t capture_stream(int device) {
    auto it = t_capture.by_device.find(device);
    if (it != t_capture.by_device.end()) return it->second;
    hipStream_t s = nullptr;
    if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) return nullptr;
    t_capture.by_device[device] = s;
    return s;
}

const DeviceInfo& device_info(int device) {
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_info.find(device);
    if (it != g_info.end()) return it->second;
    DeviceInfo di;
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess &&
        v > 0)
        di.cus = v;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, device) ==
            hipSuccess &&
        v > 0)
        di.max_lds_per_block = (size_t)v;
    g_info[device] = di;
    return g_info[device];
}

}  // namespace gila

extern "C" {

const char* gila_strerror(int status) {
    switch (status) {
        case GILA_OK: return "ok";
        case GILA_EINVAL: return "invalid argument or malformed graph";
        case GILA_ENOMEM: return "out of memory";
        case GILA_EDEVICE: return "device error";
        case GILA_EAGAIN: return "not ready";
        case GILA_ECANCELED: return "cancelled";
        case GILA_EUNSUPPORTED: return "unsupported";
        case GILA_ENONFINITE: return "non-finite force";
        default: return "unknown status";
    }
}

const char* gila_last_error(void) { return gila::t_last_error; }

int gila_version(void) { return 10000; }

int64_t gila_release_cached_memory(void) { return gila::release_cached(); }

}  // extern "C"
