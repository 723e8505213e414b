// Connected components, each laid out on its own, and packing of their
// drawings (Sections 4.6 and 5.1).
//
// Labels: a forest of parent ids, every parent at most its child's id, so a
// tree's root is its smallest id.  Every vertex starts under its smallest
// neighbour; two rounds over the first two neighbours of every vertex hook
// each tree under a smaller one it touches.  Most vertices are then in one
// tree (found by a sample), and only those outside it link their whole rows,
// exactly: the ends' roots are joined with a compare-and-swap, retried from
// the value found there when another link came first.  An edge with one end
// outside is linked from that end, one inside joins nothing, so the trees are
// then the components: the scheme of M. Sutton, T. Ben-Nun and A. Barak,
// "Optimizing Parallel Graph Connectivity Computation via Subgraph Sampling"
// (2018), with atomic minima for hooks in the rounds.  (Exact links of the first neighbours of all vertices
// at once took 0.64 ms on R-MAT 18: each retry climbs one hop of a long chain
// of fresh hooks.)
//
// Order: a stable sort of the vertices by label groups each component
// (ascending ids inside); a stable sort of the components by decreasing size
// (ties: smaller label) gives their ranks, the order of the packing matrix.
// Vertices are renumbered component by component in rank order, so every
// component is a contiguous id range with its own CSR.
//
// Layout (gila_layout_components): each component of at least two vertices
// gets the cap sqrt((n_C / a_C) d) 0.93^h, a_C the height / width of its
// initial drawing's bounding box (1 when degenerate), and runs its own
// halting rule: components of at most kSmallComponent vertices together in
// one batched launch (FR model), larger ones one after another on the whole
// GPU.  Singletons never move.
//
// Packing: component sizes and bounding boxes are reduced per label (no
// sorting of vertices); components, sorted by decreasing size (ties: smaller
// label), fill a matrix of ceil(sqrt(C)) columns row by row; a column is as
// wide as its widest drawing, a row as tall as its tallest, with the gap
// between consecutive ones; each drawing is translated so that its bounding
// box's lower-left corner is its cell's.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

#include "device_util.h"
#include "gila_internal.h"

namespace gila {

constexpr int32_t kSmallComponent = 2048;

namespace {
// Device scratch released into the block cache when its stream is done.
struct Buf {
    hipStream_t st;
    void* p = nullptr;
    explicit Buf(hipStream_t s) : st(s) {}
    ~Buf() { dfree_on(p, st); }
    template <class T>
    int alloc(size_t count) {
        return dalloc(&p, count * sizeof(T) + 64);
    }
    template <class T>
    T* as() const {
        return static_cast<T*>(p);
    }
};

int grid_for(int64_t items) {
    return (int)std::max<int64_t>(1, std::min<int64_t>(8192, (items + kBlock - 1) / kBlock));
}
}  // namespace

// ------------------------------------------------------------------ labels
// Root of x, as far as this thread can see; every vertex walked is moved up
// to its grandparent.  Other workgroups link and move at the same time, and
// the caches of different XCDs are not coherent within a launch: a value read
// may be old, but an old parent is still an ancestor (or, of a vertex hooked
// meanwhile, the vertex itself).  (Reads through the coherence point instead
// put every walk's last hops on the one address of the largest tree's root:
// 1.35 ms on R-MAT 18.)  The moves are atomic minima, as the hooks are
// compare-and-swaps: plain stores of different ancestors to one vertex by two
// XCDs leave their caches disagreeing after the launch, so that the final
// compression sees a root where the memory holds a vertex below it (3 to 15
// labels of 2^20 vertices in paths of 64, in every run).  Atomic or plain, R-MAT
// 18 takes 0.23 ms; without any moves 2^20 vertices whose trees link into one
// long chain take 6 ms, with them 1.1.
__device__ __forceinline__ int32_t cc_root(int32_t* parent, int32_t x) {
    int32_t p = parent[x];
    while (p != x) {
        const int32_t q = parent[p];
        if (q != p) atomicMin(&parent[x], q);
        x = p;
        p = q;
    }
    return x;
}

// Joins the trees of u and v.  Only a root is ever hooked (the atomic compare
// sees the true parent); where it fails it gives that parent, from which the
// walk goes on, and ids fall on every retry, so it ends.
__device__ __forceinline__ void cc_link(int32_t* parent, int32_t u, int32_t v) {
    int32_t a = cc_root(parent, u), b = cc_root(parent, v);
    while (a != b) {
        const int32_t hi = a > b ? a : b, lo = a > b ? b : a;
        const int32_t was = atomicCAS(&parent[hi], hi, lo);
        if (was == hi || was == lo) break;
        a = cc_root(parent, was);  // hooked meanwhile: go on from its parent
        b = cc_root(parent, lo);
    }
}

constexpr int kHookFirst = 2;   // neighbours of every vertex the first rounds look at
constexpr int kHookRounds = 2;

// Every vertex under its smallest neighbour where that is smaller: a forest
// without any atomic.
__global__ __launch_bounds__(kBlock) void cc_init_kernel(int32_t n, const int64_t* __restrict__ rp,
                                                         const int32_t* __restrict__ ci,
                                                         int32_t* __restrict__ parent) {
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kBlock) {
        int32_t p = (int32_t)v;
        if (rp[v + 1] > rp[v]) p = min(p, ci[rp[v]]);
        parent[v] = p;
    }
}

// One round: every tree (paths compressed, so a parent is a root) goes under
// the smallest of the roots its vertices' first neighbours have, if smaller.
// Where it loses a race it loses only that round's edge.  Lanes with the
// wavefront's first lane's two trees share one atomic: few trees are left
// soon, and atomics on one address go one after another.
__global__ __launch_bounds__(kBlock) void cc_hook_kernel(int32_t n, const int64_t* __restrict__ rp,
                                                         const int32_t* __restrict__ ci,
                                                         int32_t* parent) {
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kBlock) {
        const int64_t b = rp[v], e = rp[v + 1];
        for (int64_t j = b; j < e && j < b + kHookFirst; ++j) {
            const int32_t x = parent[v], y = parent[ci[j]];
            const int32_t hi = x > y ? x : y, lo = x > y ? y : x;
            if (hi == lo || parent[hi] <= lo) continue;
            const bool shared = hi == __builtin_amdgcn_readfirstlane(hi) &&
                                lo == __builtin_amdgcn_readfirstlane(lo);
            const uint64_t same = __ballot(shared);
            if (!shared || (same & ((1ull << lane64()) - 1ull)) == 0ull) atomicMin(&parent[hi], lo);
        }
    }
}

// label[v] = v's root; nothing is being hooked.  Each thread moves only its
// own vertex up (a move of another thread's vertex could undo its last one),
// and all climbing together halves the paths.
__global__ __launch_bounds__(kBlock) void cc_compress_kernel(int32_t n, int32_t* parent) {
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kBlock) {
        int32_t p = parent[v];
        for (;;) {
            const int32_t q = parent[p];
            if (q == p) break;  // (roots do not change in this launch)
            parent[v] = q;
            p = q;
        }
    }
}

// The most frequent label of 256 evenly spaced vertices (the smallest such
// label).  One workgroup; any choice is correct, the best one lets the most
// rows be skipped.
constexpr int kSample = 256;
__global__ __launch_bounds__(kSample) void cc_sample_kernel(int32_t n, const int32_t* __restrict__ label,
                                                            int32_t* __restrict__ most) {
    __shared__ int32_t s_label[kSample];
    __shared__ unsigned long long s_best;
    const int count = n < kSample ? n : kSample;
    const int t = threadIdx.x;
    if (t == 0) s_best = 0ull;
    if (t < count) s_label[t] = label[(int64_t)t * n / count];
    __syncthreads();
    if (t < count) {
        const int32_t l = s_label[t];
        unsigned int same = 0;
        for (int i = 0; i < count; ++i) same += s_label[i] == l ? 1u : 0u;
        atomicMax(&s_best, ((unsigned long long)same << 32) | (unsigned int)~(unsigned int)l);
    }
    __syncthreads();
    if (t == 0) *most = (int32_t)~(unsigned int)(s_best & 0xFFFFFFFFull);
}

// Wavefront per 64 vertices: rows outside the component `most` are linked,
// the wavefront's lanes sharing each longer one.
__global__ __launch_bounds__(kBlock) void cc_rest_kernel(int32_t n, const int64_t* __restrict__ rp,
                                                         const int32_t* __restrict__ ci,
                                                         int32_t* parent,
                                                         const int32_t* __restrict__ most) {
    const int lane = lane64();
    const int32_t skip = *most;
    const int64_t waves = (int64_t)gridDim.x * kWaves;
    const int64_t groups = ((int64_t)n + 63) >> 6;
    for (int64_t g = (int64_t)blockIdx.x * kWaves + wave_id(); g < groups; g += waves) {
        const int64_t v = g * 64 + lane;
        int64_t b = 0, e = 0;
        if (v < n && parent[v] != skip) {
            b = rp[v];
            e = rp[v + 1];
        }
        // short rows by their own lane, long ones by the whole wavefront
        constexpr int64_t kOwn = 8;
        if (e - b <= kOwn)
            for (int64_t j = b; j < e; ++j) cc_link(parent, (int32_t)v, ci[j]);
        uint64_t left = __ballot(e - b > kOwn);
        while (left) {
            const int l = __builtin_ctzll(left);
            left &= left - 1ull;
            const int64_t lb = __shfl(b, l, 64), le = __shfl(e, l, 64);
            const int32_t lv = (int32_t)(g * 64 + l);
            for (int64_t j = lb + lane; j < le; j += 64) cc_link(parent, lv, ci[j]);
        }
    }
}

// Roots (label[v] == v) counted per workgroup into partial[blockIdx.x].
__global__ __launch_bounds__(kBlock) void count_roots_kernel(int32_t n,
                                                             const int32_t* __restrict__ label,
                                                             unsigned long long* __restrict__ partial) {
    __shared__ int64_t s_red[kWaves];
    int64_t c = 0;
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kBlock)
        c += label[v] == (int32_t)v ? 1 : 0;
    const int64_t tot = block_sum<int64_t>(c, s_red);
    if (threadIdx.x == 0) partial[blockIdx.x] = (unsigned long long)tot;
}

// total = partial[0] + ... + partial[count - 1] (one workgroup, fixed order).
__global__ __launch_bounds__(kBlock) void sum_partials_kernel(const unsigned long long* __restrict__ partial,
                                                              int count,
                                                              unsigned long long* __restrict__ total) {
    __shared__ int64_t s_red[kWaves];
    int64_t c = 0;
    for (int i = threadIdx.x; i < count; i += kBlock) c += (int64_t)partial[i];
    const int64_t tot = block_sum<int64_t>(c, s_red);
    if (threadIdx.x == 0) *total = (unsigned long long)tot;
}

// Enqueues the labels of a valid graph into label (device, [n]); `most` is one
// word of scratch.  No synchronisation.
static int enqueue_labels(const gila_csr* g, int32_t* label, int32_t* most, hipStream_t s) {
    const int32_t n = g->n;
    if (n == 0) return GILA_OK;
    const dim3 grid((unsigned)grid_for(n));
    hipLaunchKernelGGL(cc_init_kernel, grid, dim3(kBlock), 0, s, n, g->row_ptr, g->col_idx, label);
    GILA_HIP(hipGetLastError());
    if (g->nnz == 0) return GILA_OK;
    hipLaunchKernelGGL(cc_compress_kernel, grid, dim3(kBlock), 0, s, n, label);
    for (int r = 0; r < kHookRounds; ++r) {
        hipLaunchKernelGGL(cc_hook_kernel, grid, dim3(kBlock), 0, s, n, g->row_ptr, g->col_idx, label);
        hipLaunchKernelGGL(cc_compress_kernel, grid, dim3(kBlock), 0, s, n, label);
    }
    hipLaunchKernelGGL(cc_sample_kernel, dim3(1), dim3(kSample), 0, s, n, label, most);
    hipLaunchKernelGGL(cc_rest_kernel, grid, dim3(kBlock), 0, s, n, g->row_ptr, g->col_idx, label,
                       most);
    hipLaunchKernelGGL(cc_compress_kernel, grid, dim3(kBlock), 0, s, n, label);
    GILA_HIP(hipGetLastError());
    return GILA_OK;
}

static int label_components(const gila_csr* g, int32_t* label, hipStream_t s) {
    Buf most(s);
    GILA_TRY(most.alloc<int32_t>(1));
    return enqueue_labels(g, label, most.as<int32_t>(), s);
}

// Enqueues the number of roots of label[n] into *total; partial: at least
// min(kCountPartials, blocks of kBlock vertices) words.
constexpr int kCountPartials = 2040;
static int enqueue_count_roots(int32_t n, const int32_t* label, unsigned long long* partial,
                               unsigned long long* total, hipStream_t s) {
    const int grid = (int)std::min<int64_t>(kCountPartials, ((int64_t)n + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(count_roots_kernel, dim3(grid), dim3(kBlock), 0, s, n, label, partial);
    hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(kBlock), 0, s, partial, grid, total);
    GILA_HIP(hipGetLastError());
    return GILA_OK;
}

// ------------------------------------------------------------------ component order
// gstart[i] = 1 where the label-sorted sequence starts a new component.
__global__ __launch_bounds__(kBlock) void group_start_kernel(int32_t n, const int32_t* __restrict__ label,
                                                             const int32_t* __restrict__ bylabel,
                                                             int64_t* __restrict__ gstart) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock)
        gstart[i] = (i == 0 || label[bylabel[i]] != label[bylabel[i - 1]]) ? 1 : 0;
}

// First position of every group (components in label order).
__global__ __launch_bounds__(kBlock) void group_bounds_kernel(int32_t n, const int64_t* __restrict__ gstart,
                                                              const int64_t* __restrict__ gidx,
                                                              int64_t* __restrict__ gfirst) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock)
        if (gstart[i]) gfirst[gidx[i]] = i;  // gidx: groups starting before i
}

__global__ __launch_bounds__(kBlock) void group_size_kernel(int32_t C, int32_t n, const int64_t* __restrict__ gfirst,
                                                            int32_t* __restrict__ gsize,
                                                            int32_t* __restrict__ gkey) {
    for (int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x; g < C;
         g += (int64_t)gridDim.x * kBlock) {
        const int64_t end = g + 1 < C ? gfirst[g + 1] : n;
        const int32_t sz = (int32_t)(end - gfirst[g]);
        gsize[g] = sz;
        gkey[g] = n - sz;  // larger components first
    }
}

// Rank r holds group byrank[r]: the group's rank and the sizes by rank.
__global__ __launch_bounds__(kBlock) void rank_tables_kernel(int32_t C, const int32_t* __restrict__ byrank,
                                                             const int32_t* __restrict__ gsize,
                                                             int32_t* __restrict__ grank,
                                                             int32_t* __restrict__ rsize,
                                                             int64_t* __restrict__ rsize64) {
    for (int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x; r < C;
         r += (int64_t)gridDim.x * kBlock) {
        const int32_t g = byrank[r];
        grank[g] = (int32_t)r;
        rsize[r] = gsize[g];
        rsize64[r] = gsize[g];
    }
}

// New numbering: component by component in rank order, ascending ids inside.
__global__ __launch_bounds__(kBlock) void renumber_kernel(int32_t n, const int32_t* __restrict__ bylabel,
                                                          const int64_t* __restrict__ gidx,
                                                          const int64_t* __restrict__ gstart,
                                                          const int64_t* __restrict__ gfirst,
                                                          const int32_t* __restrict__ grank,
                                                          const int64_t* __restrict__ roff,
                                                          int32_t* __restrict__ perm,
                                                          int32_t* __restrict__ iperm,
                                                          int32_t* __restrict__ vrank) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock) {
        const int64_t g = gidx[i] + gstart[i] - 1;  // group of position i
        const int32_t r = grank[g];
        const int64_t at = roff[r] + (i - gfirst[g]);
        const int32_t v = bylabel[i];
        perm[at] = v;
        iperm[v] = (int32_t)at;
        vrank[at] = r;
    }
}

// Components of a labelled graph in rank order (device tables) and the
// renumbering of the vertices.
struct CompOrder {
    int32_t C = 0;                   // components
    int32_t C2 = 0;                  // components with at least two vertices: ranks [0, C2)
    std::vector<int32_t> size;       // host, by rank
    std::vector<int64_t> off;        // host, [C + 1] first new id of each rank
    Buf perm, iperm, vrank, roff;    // device: new -> old, old -> new, rank of new id, offsets
    explicit CompOrder(hipStream_t s) : perm(s), iperm(s), vrank(s), roff(s) {}
};

static int order_components(int32_t n, const int32_t* label, hipStream_t s, CompOrder& o) {
    GILA_TRY(o.perm.alloc<int32_t>((size_t)n));
    GILA_TRY(o.iperm.alloc<int32_t>((size_t)n));
    GILA_TRY(o.vrank.alloc<int32_t>((size_t)n));
    if (n == 0) {
        GILA_TRY(o.roff.alloc<int64_t>(1));
        o.off.assign(1, 0);
        return GILA_OK;
    }
    Buf bylabel(s), gstart(s), gidx(s), ws(s);
    GILA_TRY(bylabel.alloc<int32_t>((size_t)n));
    GILA_TRY(gstart.alloc<int64_t>((size_t)n));
    GILA_TRY(gidx.alloc<int64_t>((size_t)n + 1));
    GILA_TRY(ws.alloc<int64_t>((size_t)scan_workspace_count(n)));
    GILA_TRY(stable_order_by_key(n, reinterpret_cast<const uint32_t*>(label), (uint32_t)(n - 1),
                                 bylabel.as<int32_t>(), s));
    hipLaunchKernelGGL(group_start_kernel, dim3(grid_for(n)), dim3(kBlock), 0, s, n, label,
                       bylabel.as<int32_t>(), gstart.as<int64_t>());
    GILA_HIP(hipGetLastError());
    GILA_TRY(enqueue_exclusive_scan_i64(gstart.as<int64_t>(), gidx.as<int64_t>(), n,
                                        ws.as<int64_t>(), s));
    int64_t C = 0;
    GILA_HIP(hipMemcpyAsync(&C, gidx.as<int64_t>() + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    GILA_HIP(hipStreamSynchronize(s));
    o.C = (int32_t)C;
    Buf gfirst(s), gsize(s), gkey(s), byrank(s), grank(s), rsize(s), rsize64(s);
    GILA_TRY(gfirst.alloc<int64_t>((size_t)C));
    GILA_TRY(gsize.alloc<int32_t>((size_t)C));
    GILA_TRY(gkey.alloc<int32_t>((size_t)C));
    GILA_TRY(byrank.alloc<int32_t>((size_t)C));
    GILA_TRY(grank.alloc<int32_t>((size_t)C));
    GILA_TRY(rsize.alloc<int32_t>((size_t)C));
    GILA_TRY(rsize64.alloc<int64_t>((size_t)C));
    GILA_TRY(o.roff.alloc<int64_t>((size_t)C + 1));
    hipLaunchKernelGGL(group_bounds_kernel, dim3(grid_for(n)), dim3(kBlock), 0, s, n,
                       gstart.as<int64_t>(), gidx.as<int64_t>(), gfirst.as<int64_t>());
    hipLaunchKernelGGL(group_size_kernel, dim3(grid_for(C)), dim3(kBlock), 0, s, o.C, n,
                       gfirst.as<int64_t>(), gsize.as<int32_t>(), gkey.as<int32_t>());
    GILA_HIP(hipGetLastError());
    GILA_TRY(stable_order_by_key((int32_t)C, gkey.as<uint32_t>(), (uint32_t)(n - 1),
                                 byrank.as<int32_t>(), s));
    hipLaunchKernelGGL(rank_tables_kernel, dim3(grid_for(C)), dim3(kBlock), 0, s, o.C,
                       byrank.as<int32_t>(), gsize.as<int32_t>(), grank.as<int32_t>(),
                       rsize.as<int32_t>(), rsize64.as<int64_t>());
    GILA_HIP(hipGetLastError());
    Buf ws2(s);
    GILA_TRY(ws2.alloc<int64_t>((size_t)scan_workspace_count(C)));
    GILA_TRY(enqueue_exclusive_scan_i64(rsize64.as<int64_t>(), o.roff.as<int64_t>(), C,
                                        ws2.as<int64_t>(), s));
    hipLaunchKernelGGL(renumber_kernel, dim3(grid_for(n)), dim3(kBlock), 0, s, n,
                       bylabel.as<int32_t>(), gidx.as<int64_t>(), gstart.as<int64_t>(),
                       gfirst.as<int64_t>(), grank.as<int32_t>(), o.roff.as<int64_t>(),
                       o.perm.as<int32_t>(), o.iperm.as<int32_t>(), o.vrank.as<int32_t>());
    GILA_HIP(hipGetLastError());
    o.size.resize((size_t)C);
    o.off.resize((size_t)C + 1);
    GILA_HIP(hipMemcpyAsync(o.size.data(), rsize.p, sizeof(int32_t) * C, hipMemcpyDeviceToHost, s));
    GILA_HIP(hipMemcpyAsync(o.off.data(), o.roff.p, sizeof(int64_t) * (C + 1), hipMemcpyDeviceToHost, s));
    GILA_HIP(hipStreamSynchronize(s));
    o.C2 = 0;
    while (o.C2 < o.C && o.size[o.C2] >= 2) ++o.C2;
    return GILA_OK;
}

// ------------------------------------------------------------------ bounding boxes and packing
// Bounding box of the contiguous new-id range of every rank r < R (positions
// in new order); one workgroup per rank, grid-stride.
template <class V>
__global__ __launch_bounds__(kBlock) void rank_bbox_kernel(int32_t R, const int64_t* __restrict__ roff,
                                                           const V* __restrict__ pos,
                                                           double4* __restrict__ box) {
    __shared__ double s[4][kWaves];
    for (int64_t r = blockIdx.x; r < R; r += gridDim.x) {
        double x0 = INFINITY, y0 = INFINITY, x1 = -INFINITY, y1 = -INFINITY;
        for (int64_t i = roff[r] + threadIdx.x; i < roff[r + 1]; i += kBlock) {
            const double x = (double)pos[i].x, y = (double)pos[i].y;
            x0 = x < x0 ? x : x0;
            y0 = y < y0 ? y : y0;
            x1 = x > x1 ? x : x1;
            y1 = y > y1 ? y : y1;
        }
        for (int off = 32; off >= 1; off >>= 1) {
            double o = __shfl_xor(x0, off, 64);
            x0 = o < x0 ? o : x0;
            o = __shfl_xor(y0, off, 64);
            y0 = o < y0 ? o : y0;
            o = __shfl_xor(x1, off, 64);
            x1 = o > x1 ? o : x1;
            o = __shfl_xor(y1, off, 64);
            y1 = o > y1 ? o : y1;
        }
        if (lane64() == 0) {
            s[0][wave_id()] = x0;
            s[1][wave_id()] = y0;
            s[2][wave_id()] = x1;
            s[3][wave_id()] = y1;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int q = 1; q < kWaves; ++q) {
                x0 = s[0][q] < x0 ? s[0][q] : x0;
                y0 = s[1][q] < y0 ? s[1][q] : y0;
                x1 = s[2][q] > x1 ? s[2][q] : x1;
                y1 = s[3][q] > y1 ? s[3][q] : y1;
            }
            box[r] = make_double4(x0, y0, x1, y1);
        }
        __syncthreads();
    }
}

template <class V>
__global__ __launch_bounds__(kBlock) void gather_new_kernel(int32_t n, const int32_t* __restrict__ perm,
                                                            const V* __restrict__ src,
                                                            V* __restrict__ dst) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock)
        dst[i] = src[perm[i]];
}

template <class V>
__global__ __launch_bounds__(kBlock) void scatter_old_kernel(int32_t n, const int32_t* __restrict__ perm,
                                                             const V* __restrict__ src,
                                                             V* __restrict__ dst) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock)
        dst[perm[i]] = src[i];
}

// Order-preserving integer keys of coordinates, so that bounding boxes are
// kept with integer atomics.
template <class R>
struct Key;
template <>
struct Key<float> {
    using word = unsigned int;
    static constexpr word kTop = 0x80000000u;
    __device__ static word bits(float f) { return __float_as_uint(f); }
    __device__ static float value(word u) { return __uint_as_float(u); }
};
template <>
struct Key<double> {
    using word = unsigned long long;
    static constexpr word kTop = 0x8000000000000000ull;
    __device__ static word bits(double f) { return (word)__double_as_longlong(f); }
    __device__ static double value(word u) { return __longlong_as_double((long long)u); }
};
template <class R>
__device__ __forceinline__ typename Key<R>::word to_key(R f) {
    const auto u = Key<R>::bits(f);
    return (u & Key<R>::kTop) ? ~u : (u | Key<R>::kTop);
}
template <class R>
__device__ __forceinline__ R from_key(typename Key<R>::word k) {
    return Key<R>::value((k & Key<R>::kTop) ? (k & ~Key<R>::kTop) : ~k);
}

// Size and bounding box of the component with label l (entry l; the others
// stay unused).  Boxes hold keys: xmin, ymin (minimum) and the keys of -xmax,
// -ymax (minimum too).
template <class R>
struct LabelBox {
    typename Key<R>::word k[4];
};

template <class R>
__global__ __launch_bounds__(kBlock) void pack_init_kernel(int32_t n, int32_t* __restrict__ size,
                                                           LabelBox<R>* __restrict__ box) {
    using W = typename Key<R>::word;
    const W inf = to_key((R)INFINITY);
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kBlock) {
        size[v] = 0;
        for (int c = 0; c < 4; ++c) box[v].k[c] = inf;
    }
}

// Adds every vertex to its component.  Atomics on one address go one after
// another, so the vertices of the most frequent label of a sample are
// reduced per workgroup before one set of them, and of the others those that
// share the label of a wavefront's first non-root vertex per wavefront.  Also
// the check of the labels: each in [0, n) and naming a vertex labelled with
// itself (*bad otherwise; such a vertex is left out).
template <class V, class R>
__global__ __launch_bounds__(kBlock) void pack_reduce_kernel(int32_t n, const int32_t* __restrict__ label,
                                                             const int32_t* __restrict__ most_p,
                                                             const V* __restrict__ pos,
                                                             int32_t* __restrict__ size,
                                                             LabelBox<R>* __restrict__ box,
                                                             int32_t* __restrict__ bad) {
    using W = typename Key<R>::word;
    const W inf = to_key((R)INFINITY);
    const int32_t most = *most_p;
    const int lane = lane64();
    const auto lower = [](W x, W y) { return x < y ? x : y; };
    int32_t cnt = 0;
    W mk[4] = {inf, inf, inf, inf};
    bool wrong = false;
    for (int64_t v0 = (int64_t)blockIdx.x * kBlock; v0 < n; v0 += (int64_t)gridDim.x * kBlock) {
        const int64_t v = v0 + threadIdx.x;
        int32_t l = -1;
        W k[4] = {inf, inf, inf, inf};
        if (v < n) {
            l = label[v];
            if (l < 0 || l >= n || label[l] != l) {
                wrong = true;
                l = -1;
            } else {
                const V p = pos[v];
                // (a NaN coordinate takes no part in its box)
                if (p.x == p.x) {
                    k[0] = to_key((R)p.x);
                    k[2] = to_key((R)-p.x);
                }
                if (p.y == p.y) {
                    k[1] = to_key((R)p.y);
                    k[3] = to_key((R)-p.y);
                }
            }
        }
        if (l >= 0 && l == most) {
            ++cnt;
            for (int c = 0; c < 4; ++c) mk[c] = lower(mk[c], k[c]);
            l = -1;
        }
        // the wavefront's shared label: of its first vertex that is no root
        const uint64_t member = __ballot(l >= 0 && l != (int32_t)v);
        if (member) {
            const int32_t lead = __shfl(l, __builtin_ctzll(member), 64);
            const uint64_t mine = __ballot(l == lead);
            W g[4];
            for (int c = 0; c < 4; ++c) {
                g[c] = l == lead ? k[c] : inf;
                for (int off = 32; off >= 1; off >>= 1) g[c] = lower(g[c], __shfl_xor(g[c], off, 64));
            }
            if (lane == 0) {
                atomicAdd(&size[lead], (int32_t)__popcll(mine));
                for (int c = 0; c < 4; ++c) atomicMin(&box[lead].k[c], g[c]);
            }
            if (l == lead) l = -1;
        }
        if (l >= 0) {
            atomicAdd(&size[l], 1);
            for (int c = 0; c < 4; ++c) atomicMin(&box[l].k[c], k[c]);
        }
    }
    __shared__ W s_k[4][kWaves];
    __shared__ int32_t s_n[kWaves];
    cnt = wave_sum(cnt);
    for (int c = 0; c < 4; ++c)
        for (int off = 32; off >= 1; off >>= 1) mk[c] = lower(mk[c], __shfl_xor(mk[c], off, 64));
    if (lane == 0) {
        s_n[wave_id()] = cnt;
        for (int c = 0; c < 4; ++c) s_k[c][wave_id()] = mk[c];
    }
    if (__ballot(wrong) && lane == 0) atomicOr(bad, 1);
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < kWaves; ++q) {
            cnt += s_n[q];
            for (int c = 0; c < 4; ++c) mk[c] = lower(mk[c], s_k[c][q]);
        }
        if (cnt > 0) {
            atomicAdd(&size[most], cnt);
            for (int c = 0; c < 4; ++c) atomicMin(&box[most].k[c], mk[c]);
        }
    }
}

__global__ __launch_bounds__(kBlock) void root_flag_kernel(int32_t n, const int32_t* __restrict__ label,
                                                           int64_t* __restrict__ flag) {
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kBlock)
        flag[v] = label[v] == (int32_t)v ? 1 : 0;
}

// Components in ascending label order, with their sort keys (larger first).
__global__ __launch_bounds__(kBlock) void root_list_kernel(int32_t n, const int32_t* __restrict__ label,
                                                           const int64_t* __restrict__ at,
                                                           const int32_t* __restrict__ size,
                                                           int32_t* __restrict__ root,
                                                           uint32_t* __restrict__ key) {
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kBlock)
        if (label[v] == (int32_t)v) {
            root[at[v]] = (int32_t)v;
            key[at[v]] = (uint32_t)(n - size[v]);
        }
}

// Rank r holds component byrank[r]: each root's rank, each rank's box.
template <class R>
__global__ __launch_bounds__(kBlock) void rank_box_kernel(int32_t C, const int32_t* __restrict__ byrank,
                                                          const int32_t* __restrict__ root,
                                                          const LabelBox<R>* __restrict__ lbox,
                                                          int32_t* __restrict__ rank_of,
                                                          double4* __restrict__ box) {
    for (int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x; r < C;
         r += (int64_t)gridDim.x * kBlock) {
        const int32_t v = root[byrank[r]];
        const LabelBox<R> b = lbox[v];
        rank_of[v] = (int32_t)r;
        box[r] = make_double4((double)from_key<R>(b.k[0]), (double)from_key<R>(b.k[1]),
                              -(double)from_key<R>(b.k[2]), -(double)from_key<R>(b.k[3]));
    }
}

// Column widths and row heights, a wavefront for each: the largest extent
// (at least zero) of its components.
__global__ __launch_bounds__(kBlock) void pack_extent_kernel(int32_t C, int32_t cols, int32_t rows,
                                                             const double4* __restrict__ box,
                                                             double* __restrict__ colw,
                                                             double* __restrict__ rowh) {
    const int lane = lane64();
    const int64_t j = (int64_t)blockIdx.x * kWaves + wave_id();
    if (j >= (int64_t)cols + rows) return;
    double m = 0.0;
    if (j < cols) {
        for (int64_t r = j + (int64_t)lane * cols; r < C; r += 64 * (int64_t)cols)
            m = fmax(m, box[r].z - box[r].x);
    } else {
        const int64_t r0 = (j - cols) * cols, r1 = min(r0 + cols, (int64_t)C);
        for (int64_t r = r0 + lane; r < r1; r += 64) m = fmax(m, box[r].w - box[r].y);
    }
    m = wave_max(m);
    if (lane == 0) (j < cols ? colw[j] : rowh[j - cols]) = m;
}

// Cell corners: running sums of widths (workgroup 0) and heights (1) plus the
// gap, added one after another as a plain loop does, the values staged in LDS
// (there are at most 46341 of each).  The chain of additions is what it takes;
// one thread reading its values from global memory took 56 us for 374.
__global__ __launch_bounds__(kBlock) void pack_cells_kernel(int32_t cols, int32_t rows, double gap,
                                                            const double* __restrict__ colw,
                                                            const double* __restrict__ rowh,
                                                            double* __restrict__ colx,
                                                            double* __restrict__ rowy) {
    constexpr int kStage = 1024;
    __shared__ double s_in[kStage], s_out[kStage];
    __shared__ double s_sum;
    const int32_t count = blockIdx.x == 0 ? cols : rows;
    const double* in = blockIdx.x == 0 ? colw : rowh;
    double* out = blockIdx.x == 0 ? colx : rowy;
    if (threadIdx.x == 0) {
        s_sum = 0.0;
        out[0] = 0.0;
    }
    for (int32_t j0 = 0; j0 < count; j0 += kStage) {
        const int32_t c = min(kStage, count - j0);
        for (int i = threadIdx.x; i < c; i += kBlock) s_in[i] = in[j0 + i];
        __syncthreads();
        if (threadIdx.x == 0) {
            double a = s_sum;
#pragma unroll 8
            for (int i = 0; i < c; ++i) {
                a = a + s_in[i] + gap;
                s_out[i] = a;
            }
            s_sum = a;
        }
        __syncthreads();
        for (int i = threadIdx.x; i < c; i += kBlock) out[j0 + i + 1] = s_out[i];
        __syncthreads();
    }
}

template <class V>
__global__ __launch_bounds__(kBlock) void pack_move_kernel(int32_t n, int32_t cols,
                                                           const int32_t* __restrict__ label,
                                                           const int32_t* __restrict__ rank_of,
                                                           const double4* __restrict__ box,
                                                           const double* __restrict__ colx,
                                                           const double* __restrict__ rowy,
                                                           const V* src, V* pos) {
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kBlock) {
        const int32_t r = rank_of[label[v]];
        const double bx = box[r].x, by = box[r].y;
        V p = src[v];
        p.x = (decltype(p.x))((double)p.x + (colx[r % cols] - bx));
        p.y = (decltype(p.y))((double)p.y + (rowy[r / cols] - by));
        pos[v] = p;
    }
}

// Packs the drawings of the labelled components (caller's ids) from src into pos, which
// may be one.  Whatever fails -- EINVAL for labels out of range or not naming a vertex
// labelled with itself, ENOMEM -- fails before pos is written.
template <class V>
static int pack_positions(int32_t n, const int32_t* label, double gap, const V* src, V* pos,
                          hipStream_t s) {
    using R = decltype(V::x);
    if (n == 0) return GILA_OK;
    Buf size(s), lbox(s), flag(s), at(s), ws(s), small(s);
    GILA_TRY(size.alloc<int32_t>((size_t)n));
    GILA_TRY(lbox.alloc<LabelBox<R>>((size_t)n));
    GILA_TRY(flag.alloc<int64_t>((size_t)n));
    GILA_TRY(at.alloc<int64_t>((size_t)n + 1));
    GILA_TRY(ws.alloc<int64_t>((size_t)scan_workspace_count(n)));
    GILA_TRY(small.alloc<int32_t>(2));
    int32_t* most = small.as<int32_t>();
    int32_t* bad = most + 1;
    const dim3 grid((unsigned)grid_for(n));
    GILA_HIP(hipMemsetAsync(bad, 0, sizeof(int32_t), s));
    hipLaunchKernelGGL(cc_sample_kernel, dim3(1), dim3(kSample), 0, s, n, label, most);
    hipLaunchKernelGGL(pack_init_kernel<R>, grid, dim3(kBlock), 0, s, n, size.as<int32_t>(),
                       lbox.as<LabelBox<R>>());
    // (few enough workgroups that each reduces many vertices of the largest component)
    hipLaunchKernelGGL((pack_reduce_kernel<V, R>), dim3((unsigned)std::min(grid_for(n), 512)), dim3(kBlock),
                       0, s, n, label, most, src, size.as<int32_t>(), lbox.as<LabelBox<R>>(), bad);
    hipLaunchKernelGGL(root_flag_kernel, grid, dim3(kBlock), 0, s, n, label, flag.as<int64_t>());
    GILA_HIP(hipGetLastError());
    GILA_TRY(enqueue_exclusive_scan_i64(flag.as<int64_t>(), at.as<int64_t>(), n, ws.as<int64_t>(), s));
    int32_t hbad = 0;
    int64_t C64 = 0;
    GILA_HIP(hipMemcpyAsync(&hbad, bad, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    GILA_HIP(hipMemcpyAsync(&C64, at.as<int64_t>() + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    GILA_HIP(hipStreamSynchronize(s));
    if (hbad) return fail(GILA_EINVAL, "labels must lie in [0, n) and name a vertex labelled with itself");
    const int32_t C = (int32_t)C64;
    int32_t cols = 1;
    while ((int64_t)cols * cols < C) ++cols;
    const int32_t rows = (C + cols - 1) / cols;
    Buf root(s), key(s), byrank(s), rank_of(s), box(s), ext(s);
    GILA_TRY(root.alloc<int32_t>((size_t)C));
    GILA_TRY(key.alloc<uint32_t>((size_t)C));
    GILA_TRY(byrank.alloc<int32_t>((size_t)C));
    GILA_TRY(rank_of.alloc<int32_t>((size_t)n));
    GILA_TRY(box.alloc<double4>((size_t)C));
    GILA_TRY(ext.alloc<double>(2 * ((size_t)cols + rows) + 2));
    double* colw = ext.as<double>();
    double* rowh = colw + cols;
    double* colx = rowh + rows;
    double* rowy = colx + cols + 1;
    hipLaunchKernelGGL(root_list_kernel, grid, dim3(kBlock), 0, s, n, label, at.as<int64_t>(),
                       size.as<int32_t>(), root.as<int32_t>(), key.as<uint32_t>());
    GILA_HIP(hipGetLastError());
    GILA_TRY(stable_order_by_key(C, key.as<uint32_t>(), (uint32_t)(n - 1), byrank.as<int32_t>(), s));
    hipLaunchKernelGGL(rank_box_kernel<R>, dim3((unsigned)grid_for(C)), dim3(kBlock), 0, s, C,
                       byrank.as<int32_t>(), root.as<int32_t>(), lbox.as<LabelBox<R>>(),
                       rank_of.as<int32_t>(), box.as<double4>());
    hipLaunchKernelGGL(pack_extent_kernel, dim3((unsigned)((cols + rows + kWaves - 1) / kWaves)),
                       dim3(kBlock), 0, s, C, cols, rows, box.as<double4>(), colw, rowh);
    hipLaunchKernelGGL(pack_cells_kernel, dim3(2), dim3(kBlock), 0, s, cols, rows, gap, colw, rowh, colx,
                       rowy);
    hipLaunchKernelGGL(pack_move_kernel<V>, grid, dim3(kBlock), 0, s, n, cols, label,
                       rank_of.as<int32_t>(), box.as<double4>(), colx, rowy, src, pos);
    GILA_HIP(hipGetLastError());
    return GILA_OK;
}

// ------------------------------------------------------------------ per-component CSRs
// Row lengths in new order.
__global__ __launch_bounds__(kBlock) void new_len_kernel(int32_t n, const int32_t* __restrict__ perm,
                                                         const int64_t* __restrict__ rp,
                                                         int64_t* __restrict__ len) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock) {
        const int32_t v = perm[i];
        len[i] = rp[v + 1] - rp[v];
    }
}

// Rows in new order with ids local to the component (ascending: the
// renumbering is monotone inside a component), one wavefront per row.
__global__ __launch_bounds__(kBlock) void new_rows_kernel(int32_t n, const int32_t* __restrict__ perm,
                                                          const int32_t* __restrict__ iperm,
                                                          const int32_t* __restrict__ vrank,
                                                          const int64_t* __restrict__ roff,
                                                          const int64_t* __restrict__ rp,
                                                          const int32_t* __restrict__ ci,
                                                          const int64_t* __restrict__ nrp,
                                                          int32_t* __restrict__ nci) {
    const int64_t waves = (int64_t)gridDim.x * kWaves;
    for (int64_t i = (int64_t)blockIdx.x * kWaves + wave_id(); i < n; i += waves) {
        const int32_t v = perm[i];
        const int64_t base = roff[vrank[i]];
        const int64_t b = rp[v], len = rp[v + 1] - b, o = nrp[i];
        for (int64_t e = lane64(); e < len; e += 64) nci[o + e] = (int32_t)(iperm[ci[b + e]] - base);
    }
}

// Rebased row offsets of every component with at least two vertices: the
// rows of rank r (new ids roff[r] .. roff[r+1]) go to crp[roff[r] + r ..],
// starting at 0.
__global__ __launch_bounds__(kBlock) void comp_rp_kernel(int32_t n, int32_t C2,
                                                         const int32_t* __restrict__ vrank,
                                                         const int64_t* __restrict__ roff,
                                                         const int64_t* __restrict__ nrp,
                                                         int64_t* __restrict__ crp) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock) {
        const int32_t r = vrank[i];
        if (r >= C2) continue;
        const int64_t first = roff[r];
        crp[i + r] = nrp[i] - nrp[first];
        if (i + 1 == roff[r + 1]) crp[i + 1 + r] = nrp[i + 1] - nrp[first];
    }
}

template <class V>
static int layout_components(const gila_csr* g, int32_t k, const gila_params* params, V* pos,
                             hipStream_t s, int32_t* components_out, int32_t* iterations_host) {
    const int32_t n = g->n;
    Buf label(s);
    GILA_TRY(label.alloc<int32_t>((size_t)std::max(n, 1)));
    GILA_TRY(label_components(g, label.as<int32_t>(), s));
    CompOrder o(s);
    GILA_TRY(order_components(n, label.as<int32_t>(), s, o));
    if (components_out) *components_out = o.C;
    if (n == 0) return GILA_OK;
    std::vector<int32_t> runs((size_t)o.C, 0);  // iterations run, by rank
    // graph and positions in new order
    Buf nrp(s), nci(s), crp(s), npos(s), ws(s), len(s);
    GILA_TRY(len.alloc<int64_t>((size_t)n));
    GILA_TRY(nrp.alloc<int64_t>((size_t)n + 1));
    GILA_TRY(nci.alloc<int32_t>((size_t)std::max<int64_t>(g->nnz, 1)));
    GILA_TRY(crp.alloc<int64_t>((size_t)n + (size_t)o.C2 + 1));
    GILA_TRY(npos.alloc<V>((size_t)n));
    GILA_TRY(ws.alloc<int64_t>((size_t)scan_workspace_count(n)));
    hipLaunchKernelGGL(new_len_kernel, dim3(grid_for(n)), dim3(kBlock), 0, s, n,
                       o.perm.as<int32_t>(), g->row_ptr, len.as<int64_t>());
    GILA_HIP(hipGetLastError());
    GILA_TRY(enqueue_exclusive_scan_i64(len.as<int64_t>(), nrp.as<int64_t>(), n, ws.as<int64_t>(), s));
    const int rgrid = (int)std::max<int64_t>(1, std::min<int64_t>(16384, ((int64_t)n + kWaves - 1) / kWaves));
    hipLaunchKernelGGL(new_rows_kernel, dim3(rgrid), dim3(kBlock), 0, s, n, o.perm.as<int32_t>(),
                       o.iperm.as<int32_t>(), o.vrank.as<int32_t>(), o.roff.as<int64_t>(), g->row_ptr,
                       g->col_idx, nrp.as<int64_t>(), nci.as<int32_t>());
    hipLaunchKernelGGL(comp_rp_kernel, dim3(grid_for(n)), dim3(kBlock), 0, s, n, o.C2,
                       o.vrank.as<int32_t>(), o.roff.as<int64_t>(), nrp.as<int64_t>(),
                       crp.as<int64_t>());
    hipLaunchKernelGGL(gather_new_kernel<V>, dim3(grid_for(n)), dim3(kBlock), 0, s, n,
                       o.perm.as<int32_t>(), pos, npos.as<V>());
    GILA_HIP(hipGetLastError());
    // initial bounding boxes -> caps
    std::vector<double4> box((size_t)std::max(o.C2, 1));
    std::vector<int64_t> nrp_at((size_t)o.C2 + 1);
    if (o.C2 > 0) {
        Buf dbox(s);
        GILA_TRY(dbox.alloc<double4>((size_t)o.C2));
        hipLaunchKernelGGL(rank_bbox_kernel<V>, dim3((unsigned)std::min<int64_t>(65536, o.C2)),
                           dim3(kBlock), 0, s, o.C2, o.roff.as<int64_t>(), npos.as<V>(),
                           dbox.as<double4>());
        GILA_HIP(hipGetLastError());
        GILA_HIP(hipMemcpyAsync(box.data(), dbox.p, sizeof(double4) * o.C2, hipMemcpyDeviceToHost, s));
        std::vector<int64_t> nrp_host((size_t)n + 1);
        GILA_HIP(hipMemcpyAsync(nrp_host.data(), nrp.p, sizeof(int64_t) * (n + 1), hipMemcpyDeviceToHost, s));
        GILA_HIP(hipStreamSynchronize(s));
        for (int32_t r = 0; r <= o.C2; ++r) nrp_at[r] = nrp_host[o.off[r]];
    }
    const int32_t H = params->iterations;
    const double d = params->ideal_length;
    std::vector<double> temps((size_t)std::max<int64_t>((int64_t)o.C2 * H, 1));
    std::vector<gila_params> cp((size_t)std::max(o.C2, 1));
    std::vector<gila_csr> cg((size_t)std::max(o.C2, 1));
    for (int32_t r = 0; r < o.C2; ++r) {
        const double w = box[r].z - box[r].x, h = box[r].w - box[r].y;
        const double aspect = (w > 0.0 && h > 0.0) ? h / w : 1.0;
        const double base = std::sqrt(((double)o.size[r] / aspect) * d);
        for (int32_t t = 0; t < H; ++t) temps[(size_t)r * H + t] = base * std::pow(0.93, (double)t);
        cp[r] = *params;
        cp[r].temperature = temps.data() + (size_t)r * H;
        cg[r].n = o.size[r];
        cg[r].nnz = nrp_at[r + 1] - nrp_at[r];
        cg[r].row_ptr = crp.as<int64_t>() + o.off[r] + r;
        cg[r].col_idx = nci.as<int32_t>() + nrp_at[r];
    }
    // large components on the whole GPU, one after another
    const bool batchable = params->force_model == GILA_MODEL_FR;
    int32_t small_first = o.C2;
    if (batchable)
        while (small_first > 0 && o.size[small_first - 1] <= kSmallComponent) --small_first;
    for (int32_t r = 0; r < small_first; ++r) {
        gila_khop* kh = nullptr;
        GILA_TRY(build_khop(&cg[r], k, s, &kh, params->precision));
        gila_stats st{};
        int rc;
        {
            std::lock_guard<std::mutex> lk(kh->mu);
            rc = run_iterations(kh, &cp[r], 0, H, npos.as<V>() + o.off[r], s, &st, false);
        }
        free_khop(kh, Release{true, s});
        GILA_TRY(rc);
        runs[r] = st.iterations_run;
    }
    // the small ones in one batched launch
    const int32_t nsmall = o.C2 - small_first;
    if (nsmall > 0) {
        std::vector<int32_t> ks((size_t)nsmall, k);
        std::vector<void*> pp((size_t)nsmall);
        for (int32_t j = 0; j < nsmall; ++j) pp[j] = npos.as<V>() + o.off[small_first + j];
        gila_batch* b = nullptr;
        GILA_TRY(batch_build(cg.data() + small_first, nsmall, ks.data(), s, &b));
        std::vector<gila_stats> st((size_t)nsmall);
        const int rc = batch_run(b, cp.data() + small_first, pp.data(), s, st.data(), false);
        free_batch(b, Release{true, s});
        GILA_TRY(rc);
        for (int32_t j = 0; j < nsmall; ++j) runs[small_first + j] = st[j].iterations_run;
    }
    Buf laid(s);  // the drawing before it is packed: pos stays as it was until nothing can fail
    GILA_TRY(laid.alloc<V>((size_t)n));
    hipLaunchKernelGGL(scatter_old_kernel<V>, dim3(grid_for(n)), dim3(kBlock), 0, s, n,
                       o.perm.as<int32_t>(), npos.as<V>(), laid.as<V>());
    GILA_HIP(hipGetLastError());
    GILA_TRY(pack_positions<V>(n, label.as<int32_t>(), d, laid.as<V>(), pos, s));
    if (iterations_host) {
        std::vector<int32_t> perm((size_t)n);
        GILA_HIP(hipMemcpyAsync(perm.data(), o.perm.p, sizeof(int32_t) * n, hipMemcpyDeviceToHost, s));
        GILA_HIP(hipStreamSynchronize(s));
        for (int32_t r = 0; r < o.C; ++r)
            for (int64_t i = o.off[r]; i < o.off[r + 1]; ++i) iterations_host[perm[i]] = runs[r];
    }
    GILA_HIP(hipStreamSynchronize(s));
    return GILA_OK;
}

// ------------------------------------------------------------------ labels without allocation
// gila_components_noalloc keeps its scratch in a fixed array per device,
// never in allocated memory.  Layout (64-bit words):
//   [0, 3) CSR checks (CsrCheck), [3] most frequent label (int32),
//   [4] number of components, [8, 8 + kNoAllocPartials) per-workgroup root
//   counts.  The counting grid never exceeds kNoAllocPartials workgroups, so
//   no graph needs more than these 16 KiB.
constexpr int kNoAllocHeader = 8;
constexpr int kNoAllocPartials = kCountPartials;
constexpr int kNoAllocWords = kNoAllocHeader + kNoAllocPartials;
static_assert(sizeof(CsrCheck) == 3 * sizeof(unsigned long long), "three words of scratch");
static __device__ __align__(256) unsigned long long scratch[kNoAllocWords];

constexpr int kMaxScratchDevices = 64;
static std::mutex g_scratch_mu;
static unsigned long long* g_scratch_ptr[kMaxScratchDevices];

// Device address of `scratch` on the current device (each device holds its own
// copy); looked up once per device.  In host code the array's name is only a
// stand-in, so kernels and copies must use this address.
static int scratch_address(unsigned long long** out) {
    int dev = 0;
    GILA_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxScratchDevices) return fail(GILA_EUNSUPPORTED, "device %d", dev);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(GILA_EDEVICE, "hipGetSymbolAddress(scratch) failed: %s",
                        hipGetErrorString(e));
        g_scratch_ptr[dev] = static_cast<unsigned long long*>(p);
    }
    *out = g_scratch_ptr[dev];
    return GILA_OK;
}

// Zeroes words [0, count) (a kernel, not a memset node, so the call can sit in
// a captured graph).
__global__ void clear_words_kernel(unsigned long long* w, int count) {
    for (int i = threadIdx.x; i < count; i += blockDim.x) w[i] = 0ull;
}

static int components_noalloc(const gila_csr* g, int32_t* label, int32_t* count_out,
                              hipStream_t s) {
    if (!g) return fail(GILA_EINVAL, "graph is NULL");
    const int32_t n = g->n;
    const int64_t nnz = g->nnz;
    if (n < 0 || nnz < 0) return fail(GILA_EINVAL, "negative n or nnz");
    if (n > 0 && !g->row_ptr) return fail(GILA_EINVAL, "row_ptr is NULL");
    if (nnz > 0 && !g->col_idx) return fail(GILA_EINVAL, "col_idx is NULL");
    if (nnz % 2) return fail(GILA_EINVAL, "nnz must be even for a symmetric CSR");
    if (nnz > (int64_t)n * (int64_t)(n > 0 ? n - 1 : 0))
        return fail(GILA_EINVAL, "nnz exceeds n(n-1)");
    if (n > 0 && !label) return fail(GILA_EINVAL, "label_dev is NULL");
    unsigned long long* w = nullptr;
    GILA_TRY(scratch_address(&w));
    if (n == 0) {
        if (count_out) *count_out = 0;
        return GILA_OK;
    }
    CsrCheck* check = reinterpret_cast<CsrCheck*>(w);
    unsigned long long* partial = w + kNoAllocHeader;
    hipLaunchKernelGGL(clear_words_kernel, dim3(1), dim3(64), 0, s, w, kNoAllocHeader);
    GILA_TRY(launch_rowptr_check(n, nnz, g->row_ptr, check, s));
    GILA_TRY(launch_validate_csr(n, nnz, g->row_ptr, g->col_idx, check, s));
    CsrCheck found;
    GILA_HIP(hipMemcpyAsync(&found, check, sizeof(found), hipMemcpyDeviceToHost, s));
    GILA_HIP(hipStreamSynchronize(s));
    if (found.flag & (16 | 32))
        return fail(GILA_EINVAL, "row_ptr must run from 0 to nnz without decreasing");
    GILA_TRY(entries_status(found, ""));
    GILA_TRY(enqueue_labels(g, label, reinterpret_cast<int32_t*>(w + 3), s));
    if (count_out) {
        // every component has exactly one root (its smallest id)
        GILA_TRY(enqueue_count_roots(n, label, partial, w + 4, s));
        unsigned long long c = 0;
        GILA_HIP(hipMemcpyAsync(&c, w + 4, sizeof(c), hipMemcpyDeviceToHost, s));
        GILA_HIP(hipStreamSynchronize(s));
        *count_out = (int32_t)c;
    }
    GILA_HIP(hipStreamSynchronize(s));
    return GILA_OK;
}

}  // namespace gila

using namespace gila;

extern "C" {

int gila_components_noalloc(const gila_csr* g_dev, int32_t* label_dev, int32_t* count_out,
                            void* stream) {
    clear_error();
    return components_noalloc(g_dev, label_dev, count_out, (hipStream_t)stream);
}

int gila_components(const gila_csr* g_dev, int32_t* label_dev, int32_t* count_out, void* stream) {
    TraceRange trace_range("gila_components");
    clear_error();
    SettleOnReturn settle(stream);
    hipStream_t s = (hipStream_t)stream;
    GILA_TRY(validate_graph(g_dev, s));
    if (g_dev->n > 0 && !label_dev) return fail(GILA_EINVAL, "label_dev is NULL");
    GILA_TRY(label_components(g_dev, label_dev, s));
    if (count_out) {
        *count_out = 0;
        if (g_dev->n > 0) {
            Buf partial(s);
            GILA_TRY(partial.alloc<unsigned long long>(kCountPartials + 1));
            unsigned long long* total = partial.as<unsigned long long>() + kCountPartials;
            GILA_TRY(enqueue_count_roots(g_dev->n, label_dev, partial.as<unsigned long long>(), total, s));
            unsigned long long c = 0;
            GILA_HIP(hipMemcpyAsync(&c, total, sizeof(c), hipMemcpyDeviceToHost, s));
            GILA_HIP(hipStreamSynchronize(s));
            *count_out = (int32_t)c;
        }
    }
    GILA_HIP(hipStreamSynchronize(s));
    return GILA_OK;
}

int gila_pack_components(int32_t n, const int32_t* label_dev, double gap, int32_t precision,
                         void* pos_dev, void* stream) {
    TraceRange trace_range("gila_pack_components");
    clear_error();
    SettleOnReturn settle(stream);
    if (n < 0) return fail(GILA_EINVAL, "n must be >= 0");
    if (n > 0 && (!label_dev || !pos_dev)) return fail(GILA_EINVAL, "label_dev or pos_dev is NULL");
    if (!(gap >= 0.0) || !std::isfinite(gap)) return fail(GILA_EINVAL, "gap must be finite and >= 0");
    if (precision != GILA_FP64 && precision != GILA_FP32 && precision != GILA_FP32_KAHAN)
        return fail(GILA_EINVAL, "unknown precision %d", precision);
    hipStream_t s = (hipStream_t)stream;
    if (n == 0) return GILA_OK;
    if (precision == GILA_FP64) GILA_TRY(pack_positions<double2>(n, label_dev, gap, (double2*)pos_dev, (double2*)pos_dev, s));
    else GILA_TRY(pack_positions<float2>(n, label_dev, gap, (float2*)pos_dev, (float2*)pos_dev, s));
    GILA_HIP(hipStreamSynchronize(s));
    return GILA_OK;
}

int gila_layout_components(const gila_csr* g_dev, int32_t k, const gila_params* params,
                           void* pos_dev, void* stream, int32_t* components_out,
                           int32_t* iterations_host) {
    TraceRange trace_range("gila_layout_components");
    clear_error();
    SettleOnReturn settle(stream);
    if (!params) return fail(GILA_EINVAL, "params is NULL");
    gila_params p = *params;
    p.temperature = nullptr;  // the caps are the components' own
    GILA_TRY(check_params(&p, false));
    if (k < 1) return fail(GILA_EINVAL, "k must be >= 1 (got %d)", k);
    hipStream_t s = (hipStream_t)stream;
    GILA_TRY(validate_graph(g_dev, s));
    if (g_dev->n > 0 && !pos_dev) return fail(GILA_EINVAL, "pos_dev is NULL");
    if (p.precision == GILA_FP64)
        return layout_components<double2>(g_dev, k, &p, (double2*)pos_dev, s, components_out,
                                          iterations_host);
    return layout_components<float2>(g_dev, k, &p, (float2*)pos_dev, s, components_out,
                                     iterations_host);
}

}  // extern "C"
