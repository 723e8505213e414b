// A stand-in for the HIP runtime, to run the library's host code without a GPU: memory is
// the host's, kernels do nothing -- but for a few whose results the host reads back
// (emulate() below) -- and streams, events and graphs are objects whose lifetimes are
// watched: a call that names a destroyed one, or asks about an event whose stream is gone,
// ends the program with a message.  (A runtime may keep the stream in the event and look at
// it in the query; then such a call reads freed memory.)
//
// An event is done once its stream has been waited for, or at the second time it is asked.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>

typedef int hipError_t;
enum { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorNotReady = 600 };
struct dim3_ {
    uint32_t x, y, z;
};

namespace {
struct Stream {
    uint64_t done = 0;  // events recorded so far count as done up to here
    uint64_t recorded = 0;
    bool capturing = false;
};
struct Event {
    Stream* stream = nullptr;
    uint64_t seq = 0;
    int asked = 0;
};
std::mutex g_mu;
std::set<Stream*> g_streams;
std::set<Event*> g_events;
std::set<void*> g_graphs;
std::map<const void*, std::string> g_kernels;
std::map<std::string, unsigned> g_block;  // threads per workgroup at each kernel's last launch
Stream g_null;
thread_local dim3_ t_grid, t_block;
thread_local size_t t_shm;
thread_local void* t_stream;
int64_t g_fail_after = -1;  // hipMalloc calls until they fail (< 0: none does)
const void* g_watched;      // positions whose writers are looked for (watched_by)
bool g_touched;

[[noreturn]] void violation(const char* call, const char* what) {
    std::printf("VIOLATION %s: %s\n", call, what);
    std::fflush(stdout);
    std::_Exit(3);
}

Stream* stream_of(void* s, const char* call) {  // lock held
    if (!s) return &g_null;
    Stream* p = static_cast<Stream*>(s);
    if (!g_streams.count(p)) violation(call, "the stream was destroyed");
    return p;
}

Event* event_of(void* e, const char* call) {  // lock held
    Event* p = static_cast<Event*>(e);
    if (!g_events.count(p)) violation(call, "the event was destroyed");
    return p;
}

void check_stream(void* s, const char* call) {
    std::lock_guard<std::mutex> lk(g_mu);
    (void)stream_of(s, call);
}

template <class T>
T arg(void** args, int i) {
    return *static_cast<T*>(args[i]);
}

// What the host may read back, once; everything else it reads is zero.
std::map<const void*, size_t> g_written;

void written(const void* p, size_t n) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_written[p] = n;
}

bool was_written(const void* p) {
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_written.upper_bound(p);
    if (it == g_written.begin()) return false;
    --it;
    if (static_cast<const char*>(p) >= static_cast<const char*>(it->first) + it->second) return false;
    g_written.erase(it);
    return true;
}

// The kernels whose results decide what the host does next: the number of non-empty rows
// (rowptr_check_kernel: n, nnz, rp, check, whose second word it is) and the prefix sum of
// the row lengths (internal_rows_kernel: n, perm, rp, counts, iperm, deg, cnt; then
// scan_tiles_kernel: in, out, n, sums).  Every other count is zero.
thread_local const int64_t* t_deg;
thread_local const int64_t* t_rp;

// Which argument of a kernel is the positions it writes (-1: not one of these).
int watched_by(const std::string& name) {
    const auto is = [&](const char* k) { return name.find(k) != std::string::npos; };
    return is("scatter_old_kernel") ? 3 : is("pack_move_kernel") ? 8 : -1;
}

void emulate(const std::string& name, void** a) {
    const auto is = [&](const char* k) { return name.find(k) != std::string::npos; };
    if (is("scan_tiles_kernel")) {
        const int64_t n = arg<int64_t>(a, 2);
        int64_t* out = arg<int64_t*>(a, 1);
        if (arg<const int64_t*>(a, 0) == t_deg) {
            std::memcpy(out, t_rp, sizeof(int64_t) * (size_t)(n + 1));
            written(out, sizeof(int64_t) * (size_t)(n + 1));
            t_deg = nullptr;
        } else {
            std::memset(out, 0, sizeof(int64_t) * (size_t)(n + 1));
        }
    } else if (is("rowptr_check_kernel")) {
        const int32_t n = arg<int32_t>(a, 0);
        const int64_t* rp = arg<const int64_t*>(a, 2);
        int32_t* check = arg<int32_t*>(a, 3);
        for (int32_t v = 0; v < n; ++v) check[1] += rp[v + 1] > rp[v] ? 1 : 0;
        written(check, 8);
    } else if (is("internal_rows_kernel")) {
        t_rp = arg<const int64_t*>(a, 2);
        t_deg = arg<const int64_t*>(a, 5);
    }
}
}  // namespace

extern "C" {

void fake_hip_fail_malloc_after(int64_t calls) { g_fail_after = calls; }
void fake_hip_watch(const void* positions) {
    g_watched = positions;
    g_touched = false;
}
// Threads per workgroup at the last launch of a kernel whose name holds this (0: none), and
// forgotten.
unsigned fake_hip_block_of(const char* name) {
    std::lock_guard<std::mutex> lk(g_mu);
    for (auto it = g_block.begin(); it != g_block.end(); ++it)
        if (it->first.find(name) != std::string::npos) {
            const unsigned b = it->second;
            g_block.erase(it);
            return b;
        }
    return 0;
}
int fake_hip_touched() { return g_touched ? 1 : 0; }

void** __hipRegisterFatBinary(const void*) { return new void*(nullptr); }
void __hipUnregisterFatBinary(void** m) { delete m; }
void __hipRegisterFunction(void**, const void* host, char* name, const char*, unsigned, void*, void*, void*,
                           void*, int*) {
    g_kernels[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3_ grid, dim3_ block, size_t shm, void* s) {
    t_grid = grid;
    t_block = block;
    t_shm = shm;
    t_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3_* grid, dim3_* block, size_t* shm, void** s) {
    *grid = t_grid;
    *block = t_block;
    *shm = t_shm;
    *s = t_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3_ grid, dim3_ block, void** args, size_t, void* s) {
    bool capturing;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        capturing = stream_of(s, "hipLaunchKernel")->capturing;
        g_block[g_kernels[f]] = block.x;
    }
    if (grid.x == 0 || grid.y == 0 || block.x == 0 || block.x > 1024)
        violation(g_kernels[f].c_str(), "launch shape");
    const int w = watched_by(g_kernels[f]);
    if (w >= 0 && arg<const void*>(args, w) == g_watched) g_touched = true;
    if (!capturing) emulate(g_kernels[f], args);
    return hipSuccess;
}

hipError_t hipDeviceGetAttribute(int* v, int, int) { return *v = 0, hipSuccess; }
hipError_t hipDeviceSynchronize() {
    std::lock_guard<std::mutex> lk(g_mu);
    for (Stream* s : g_streams) s->done = s->recorded;
    g_null.done = g_null.recorded;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "fake error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
    static uint64_t scratch[4096];
    return *p = scratch, hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, int, int) { return hipSuccess; }

hipError_t hipMalloc(void** p, size_t n) {
    if (g_fail_after == 0) return hipErrorOutOfMemory;
    if (g_fail_after > 0) --g_fail_after;
    *p = std::calloc(1, n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return *p = std::calloc(1, n), hipSuccess; }
hipError_t hipHostFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipMemGetInfo(size_t* fr, size_t* tot) { return *fr = *tot = (size_t)1 << 33, hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, int kind) {
    const bool to_host = kind == 2;
    if (to_host && !was_written(s)) std::memset(d, 0, n);
    else std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st) {
    check_stream(st, "hipMemcpyAsync");
    return hipMemcpy(d, s, n, kind);
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, void* st) {
    check_stream(st, "hipMemsetAsync");
    return std::memset(d, v, n), hipSuccess;
}

hipError_t hipStreamCreateWithFlags(void** s, unsigned) {
    std::lock_guard<std::mutex> lk(g_mu);
    Stream* p = new Stream();
    g_streams.insert(p);
    return *s = p, hipSuccess;
}
hipError_t hipStreamDestroy(void* s) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_streams.erase(stream_of(s, "hipStreamDestroy"));  // (not freed: the address stays its own)
    return hipSuccess;
}
hipError_t hipStreamSynchronize(void* s) {
    std::lock_guard<std::mutex> lk(g_mu);
    Stream* p = stream_of(s, "hipStreamSynchronize");
    p->done = p->recorded;
    return hipSuccess;
}

hipError_t hipEventCreateWithFlags(void** e, unsigned) {
    std::lock_guard<std::mutex> lk(g_mu);
    Event* p = new Event();
    g_events.insert(p);
    return *e = p, hipSuccess;
}
hipError_t hipEventCreate(void** e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(void* e) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_events.erase(event_of(e, "hipEventDestroy"));
    return hipSuccess;
}
hipError_t hipEventRecord(void* e, void* s) {
    std::lock_guard<std::mutex> lk(g_mu);
    Event* p = event_of(e, "hipEventRecord");
    p->stream = stream_of(s, "hipEventRecord");
    p->seq = ++p->stream->recorded;
    p->asked = 0;
    return hipSuccess;
}
hipError_t hipEventQuery(void* e) {
    std::lock_guard<std::mutex> lk(g_mu);
    Event* p = event_of(e, "hipEventQuery");
    if (p->stream && p->stream != &g_null && !g_streams.count(p->stream))
        violation("hipEventQuery", "the event's stream was destroyed");
    if (!p->stream || p->seq <= p->stream->done || p->asked++ > 0) return hipSuccess;
    return hipErrorNotReady;
}
hipError_t hipEventElapsedTime(float* t, void*, void*) { return *t = 1.0f, hipSuccess; }

hipError_t hipStreamBeginCapture(void* s, int) {
    std::lock_guard<std::mutex> lk(g_mu);
    stream_of(s, "hipStreamBeginCapture")->capturing = true;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(void* s, int* status) {
    std::lock_guard<std::mutex> lk(g_mu);
    *status = stream_of(s, "hipStreamIsCapturing")->capturing ? 1 : 0;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(void* s, void** g) {
    std::lock_guard<std::mutex> lk(g_mu);
    stream_of(s, "hipStreamEndCapture")->capturing = false;
    *g = std::malloc(1);
    g_graphs.insert(*g);
    return hipSuccess;
}
hipError_t hipGraphDestroy(void* g) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!g_graphs.erase(g)) violation("hipGraphDestroy", "the graph was destroyed");
    return hipSuccess;
}
hipError_t hipGraphInstantiate(void** x, void*, void*, void*, size_t) {
    std::lock_guard<std::mutex> lk(g_mu);
    *x = std::malloc(1);
    g_graphs.insert(*x);
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(void* x) { return hipGraphDestroy(x); }
hipError_t hipGraphLaunch(void* x, void* s) {
    std::lock_guard<std::mutex> lk(g_mu);
    (void)stream_of(s, "hipGraphLaunch");
    if (!g_graphs.count(x)) violation("hipGraphLaunch", "the graph was destroyed");
    return hipSuccess;
}

void roctxMarkA(const char*) {}
int roctxRangePushA(const char*) { return 0; }
int roctxRangePop() { return 0; }

}  // extern "C"
