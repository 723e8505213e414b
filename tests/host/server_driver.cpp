// Over the stand-in runtime (fake_hip.cpp), by the argument: "streams", bursts of layout
// jobs on servers that come and go, and calls on streams of the caller that come and go
// too; "memory", a components' layout at every allocation that can fail; "batch", the route
// of batches whose largest graph just fits a workgroup's LDS.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../../include/gila.h"

extern "C" int hipStreamCreateWithFlags(void**, unsigned);
extern "C" int hipStreamDestroy(void*);
extern "C" int hipStreamSynchronize(void*);
extern "C" int hipMalloc(void**, size_t);
extern "C" int hipFree(void*);
extern "C" void fake_hip_fail_malloc_after(int64_t);
extern "C" void fake_hip_watch(const void*);
extern "C" int fake_hip_touched();
extern "C" unsigned fake_hip_block_of(const char*);

static void need(bool ok, const char* what) {
    if (!ok) {
        std::printf("FAILED %s: %s\n", what, gila_last_error());
        std::fflush(stdout);
        std::_Exit(2);
    }
}

struct Ring {  // every vertex joined to the two on either side
    std::vector<int64_t> rp;
    std::vector<int32_t> ci;
    gila_csr csr{};
    explicit Ring(int32_t n) {
        rp.push_back(0);
        for (int32_t v = 0; v < n; ++v) {
            int32_t u[4] = {(v + n - 2) % n, (v + n - 1) % n, (v + 1) % n, (v + 2) % n};
            for (int i = 0; i < 4; ++i)
                for (int j = i + 1; j < 4; ++j)
                    if (u[j] < u[i]) std::swap(u[i], u[j]);
            ci.insert(ci.end(), u, u + 4);
            rp.push_back((int64_t)ci.size());
        }
        csr.n = n;
        csr.nnz = (int64_t)ci.size();
        csr.row_ptr = rp.data();
        csr.col_idx = ci.data();
    }
};

// A call that fails for want of memory leaves the caller's positions as they were.
static void memory(const gila_csr& g, gila_params p) {
    std::vector<double> pos(2 * (size_t)g.n, 0.5);
    p.precision = GILA_FP64;
    int failed = 0;
    for (int64_t i = 0;; ++i) {
        (void)hipStreamSynchronize(nullptr);
        (void)gila_release_cached_memory();
        fake_hip_watch(pos.data());
        fake_hip_fail_malloc_after(i);
        const int rc = gila_layout_components(&g, 2, &p, pos.data(), nullptr, nullptr, nullptr);
        fake_hip_fail_malloc_after(-1);
        if (rc == GILA_OK) break;
        need(rc == GILA_ENOMEM, "out of memory");
        need(!fake_hip_touched(), "positions written by a call that failed");
        ++failed;
    }
    need(failed > 20 && fake_hip_touched(), "allocations that fail, and one call that does not");
}

// Complete graphs of n vertices: in 64 KB beside the CSR of 4 (n + 1) + 2 n (n - 1) bytes
// and 1 KB of other state, three bitmaps for each of 16 wavefronts fit up to n = 177, for
// each of 8 up to 178.
static void batch() {
    for (int32_t n : {100, 170, 175, 176, 177, 178, 179}) {
        std::vector<int64_t> rp(1, 0);
        std::vector<int32_t> ci;
        for (int32_t v = 0; v < n; ++v) {
            for (int32_t u = 0; u < n; ++u)
                if (u != v) ci.push_back(u);
            rp.push_back((int64_t)ci.size());
        }
        gila_csr g{};
        g.n = n;
        g.nnz = (int64_t)ci.size();
        g.row_ptr = rp.data();
        g.col_idx = ci.data();
        const int32_t k = 2;
        gila_batch* b = nullptr;
        need(gila_batch_build(&g, 1, &k, nullptr, &b) == GILA_OK, "batch");
        gila_batch_free(b);
        const unsigned graph = fake_hip_block_of("batch_khop_kernel"), source = fake_hip_block_of("khop_bfs_kernel");
        const unsigned want = n <= 177 ? 1024 : n <= 178 ? 512 : 0;
        std::printf("n %d: %u threads per graph's workgroup, %u per source's\n", n, graph, source);
        need(graph == want && (source == 0) == (want != 0), "route");
    }
}

int main(int argc, char** argv) {
    setenv("GILA_PATH", "direct", 1);  // (segments are planned from counts that kernels make)
    std::vector<double> temps(70, 1.0);
    gila_params p{};
    p.iterations = (int32_t)temps.size();
    p.temperature = temps.data();
    p.ideal_length = 10.0;
    p.precision = GILA_FP32_KAHAN;
    p.force_model = GILA_MODEL_FR;
    std::vector<Ring> ring;
    for (int32_t n : {100, 137, 400, 1024, 1025, 3000, 7000, 20000}) ring.emplace_back(n);
    if (argc > 1 && !std::strcmp(argv[1], "memory")) {
        memory(ring[0].csr, p);
        std::printf("OK\n");
        return 0;
    }
    if (argc > 1 && !std::strcmp(argv[1], "batch")) {
        batch();
        std::printf("OK\n");
        return 0;
    }
    for (int round = 0; round < 4; ++round) {
        gila_server* s = nullptr;
        need(gila_server_create(0, 0, 16, &s) == GILA_OK, "create");
        std::vector<uint64_t> t(40);
        std::vector<std::vector<double>> out(40);
        for (int i = 0; i < 40; ++i) {
            const Ring& r = ring[i % ring.size()];
            out[i].assign(2 * (size_t)r.csr.n, 0.5);
            p.precision = i % 3 ? GILA_FP32_KAHAN : GILA_FP64;
            need(gila_submit(s, &r.csr, 2, &p, out[i].data(), &t[i]) == GILA_OK, "submit");
        }
        for (int i = 0; i < 40; i += 7) need(gila_cancel(s, t[i]) == GILA_OK, "cancel");
        for (int i = 0; i < 40; ++i) {
            const int rc = gila_wait(s, t[i], out[i].data(), nullptr);
            need(rc == GILA_OK || rc == GILA_ECANCELED, "wait");
        }
        gila_server_destroy(s);
        // the calling thread's own streams, destroyed as soon as the call has returned
        for (const Ring& r : ring) {
            void* st = nullptr;
            need(hipStreamCreateWithFlags(&st, 1) == 0, "stream");
            void* pos = nullptr;
            need(hipMalloc(&pos, 16 * (size_t)r.csr.n) == 0, "positions");
            p.precision = GILA_FP32;
            need(gila_layout(&r.csr, 2, &p, pos, st, nullptr) == GILA_OK, "layout");
            need(hipStreamSynchronize(st) == 0 && hipStreamDestroy(st) == 0, "stream end");
            need(hipFree(pos) == 0, "positions end");
        }
    }
    std::printf("OK\n");
    return 0;
}
