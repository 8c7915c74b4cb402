// A HIP runtime for host tests: memory is host memory (allocated on use, counted against a
// settable size), streams and events are objects whose use after destruction is reported,
// and kernels do nothing except those the host code of a run takes decisions from, which get
// the few values that carry a run through all its phases.  Linked into the test program, whose
// symbols come before those of the real runtime.
#include "fake_hip.hpp"

#include <sys/mman.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <vector>

thread_local int fake_hip_inside = 0;

namespace {

struct Dim3 {
    uint32_t x, y, z;
};
struct Stream {
    bool alive = true, capturing = false;
    std::vector<std::function<void()>> captured;
};
struct Event {
    bool alive = true;
};
struct Graph {
    std::vector<std::function<void()>> nodes;
};

// The runtime's own allocations do not fail with the library's.
struct Inside {
    Inside() { ++fake_hip_inside; }
    ~Inside() { --fake_hip_inside; }
};

// (made on first use: the library registers its kernels before the program's own statics exist)
struct Tables {
    std::mutex mu;
    std::map<char*, size_t> blocks;
    std::map<const void*, std::string> kernels;
    std::set<Stream*> streams;   // never freed, so that a stale handle can be told
    std::set<Event*> events;
    FakeHip state;
};
Tables& t() {
    static Tables* x = new Tables;
    return *x;
}

void fault(const char* what) {
    std::lock_guard<std::mutex> lk(t().mu);
    if (++t().state.faults <= 10) std::fprintf(stderr, "fake hip: %s\n", what);
}
void check(Stream* s, const char* what) {
    bool bad = false;
    if (s) {
        std::lock_guard<std::mutex> lk(t().mu);
        bad = !t().streams.count(s) || !s->alive;
    }
    if (bad) fault(what);
}
void check(Event* e, const char* what) {
    bool bad;
    {
        std::lock_guard<std::mutex> lk(t().mu);
        bad = !t().events.count(e) || !e->alive;
    }
    if (bad) fault(what);
}

template <typename T>
T arg(void** a, int i) {
    T v;
    std::memcpy(&v, a[i], sizeof(T));
    return v;
}
struct Geometry {   // the first fields of the squares' geometry
    double x0, y0, w1;
};
// squares around the shift (level 1: within 1.2 cells) are resolved; of the squares of a
// level those that hold one of a few fixed points are kept
bool holds_point(const Geometry& g, int64_t level, int64_t ix, int64_t iy) {
    const double w = std::ldexp(g.w1, (int)(1 - level));
    for (int k = 0; k < 5; ++k) {
        const double x = g.x0 + g.w1 * (0.31 + 0.77 * k), y = g.y0 + g.w1 * (0.43 + 0.59 * k);
        if (ix == (int64_t)std::floor((x - g.x0) / w) && iy == (int64_t)std::floor((y - g.y0) / w)) return true;
    }
    return false;
}

std::function<void()> kernel_body(const std::string& name, Dim3 grid, void** a) {
    auto is = [&](const char* s) { return name.find(s) != std::string::npos; };
    if (is("k_fill_u64")) {
        auto* p = arg<unsigned long long*>(a, 0);
        const int n = arg<int>(a, 1);
        return [=] { for (int i = 0; i < n; ++i) p[i] = 0; };
    }
    if (is("k_fill_u32")) {
        auto* p = arg<unsigned*>(a, 0);
        const int n = arg<int>(a, 1);
        const unsigned v = arg<unsigned>(a, 2);
        return [=] { for (int i = 0; i < n; ++i) p[i] = v; };
    }
    if (is("k_fill_i32")) {
        auto* p = arg<int*>(a, 0);
        const int v = arg<int>(a, 1);
        return [=] { *p = v; };
    }
    if (is("k_max_jump")) {
        auto* p = arg<int*>(a, 2);
        return [=] { *p = 0; };
    }
    if (is("k_gs_next")) {   // the start vector's norm: hnorm[2] of every space
        struct Batch {
            void* p[32];
            double* hnorm[4];
        };
        const Batch b = arg<Batch>(a, 1);
        const int ny = (int)grid.y;
        return [=] { for (int y = 0; y < ny; ++y) b.hnorm[y][2] = 1.0; };
    }
    if (is("k_hess_schur")) {
        auto* p = arg<int*>(a, 8);
        return [=] { *p = 0; };
    }
    if (is("k_fine_solutions")) {   // residuals of the nodes
        struct Rule {
            const double* p[4];
            int g;
        };
        const int n = 8 * arg<Rule>(a, 2).g;
        auto* rho = arg<double*>(a, 10);
        return [=] { for (int q = 0; rho && q < n; ++q) rho[q] = 0.0; };
    }
    if (is("k_cells_resid")) {
        const double re = arg<double>(a, 4), im = arg<double>(a, 5);
        const int64_t* cells = arg<const int64_t*>(a, 6);
        const Geometry g = arg<Geometry>(a, 8);
        auto* bits = arg<unsigned long long*>(a, 11);
        const int n = (int)grid.x;
        return [=] {
            for (int c = 0; c < n; ++c) {
                const double x = g.x0 + (cells[2 * c] + 0.5) * g.w1, y = g.y0 + (cells[2 * c + 1] + 0.5) * g.w1;
                const double rho = std::hypot(x - re, y - im) <= 1.2 * g.w1 ? 0.0 : 1.0;
                std::memcpy(&bits[c], &rho, sizeof rho);
            }
        };
    }
    if (is("k_indicators")) {
        const bool persist = is("k_indicators_persist");
        const int64_t* rows = arg<const int64_t*>(a, 1);
        const int64_t nreg = persist ? 0 : arg<int64_t>(a, 2);
        const int64_t* nrows = persist ? arg<const int64_t*>(a, 2) : nullptr;
        const Geometry g = persist ? Geometry{} : arg<Geometry>(a, 3);
        const char* geo = persist ? arg<const char*>(a, 3) : nullptr;
        double* out[5];
        for (int q = 0; q < 5; ++q) out[q] = arg<double*>(a, 5 + q);
        auto* dec = arg<uint8_t*>(a, 10);
        std::vector<double*> o(out, out + 5);
        return [=] {
            const int64_t n = persist ? *nrows : nreg, ld = persist ? 5 : 4;
            for (int64_t r = 0; r < n; ++r) {
                const int64_t* q = rows + ld * r;
                Geometry gr = g;
                if (persist) std::memcpy(&gr, geo + q[4] * 48, sizeof gr);
                for (double* p : o)
                    if (p) p[r] = 0.5;
                if (dec) dec[r] = holds_point(gr, q[0], q[1], q[2]) ? 1 : 0;
            }
        };
    }
    return nullptr;
}

thread_local struct {
    Dim3 grid, block;
    size_t lds;
    Stream* st;
} call;

}  // namespace

FakeHip& fake_hip() { return t().state; }

extern "C" {

void** __hipRegisterFatBinary(const void*) {
    static void* h;
    return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    std::lock_guard<std::mutex> lk(t().mu);
    t().kernels[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t lds, void* st) {
    call = {g, b, lds, (Stream*)st};
    return 0;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* lds, void** st) {
    *g = call.grid;
    *b = call.block;
    *lds = call.lds;
    *st = call.st;
    return 0;
}
int hipLaunchKernel(const void* fn, Dim3 grid, Dim3, void** args, size_t, void* st) {
    Inside in;
    Stream* s = (Stream*)st;
    check(s, "launch on a destroyed stream");
    std::function<void()> body;
    {
        std::lock_guard<std::mutex> lk(t().mu);
        body = kernel_body(t().kernels[fn], grid, args);
    }
    if (s && s->capturing) {
        if (body) s->captured.push_back(body);
    } else if (body) {
        body();
    }
    return 0;
}

int hipGetDeviceCount(int* n) { return *n = 1, 0; }
int hipGetDevice(int* d) { return *d = 0, 0; }
int hipSetDevice(int) { return 0; }
const char* hipGetErrorString(int e) { return e == 2 ? "out of memory" : "error"; }
int hipGetLastError() { return 0; }
int hipGetSymbolAddress(void** p, const void*) { return *p = nullptr, 1; }
int hipDeviceSynchronize() { return 0; }

int hipMalloc(void** p, size_t bytes) {
    Inside in;
    std::lock_guard<std::mutex> lk(t().mu);
    t().state.mallocs += 1;
    t().state.watched += bytes == t().state.watch;
    if (t().state.used + bytes > t().state.total) return *p = nullptr, 2;
    void* q = mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (q == MAP_FAILED) return *p = nullptr, 2;
    t().blocks[(char*)q] = bytes;
    t().state.used += bytes;
    t().state.peak = std::max(t().state.peak, t().state.used);
    return *p = q, 0;
}
static int free_block(void* p, bool waits) {
    if (!p) return 0;
    std::unique_lock<std::mutex> lk(t().mu);
    t().state.frees += 1;
    if (waits && pthread_self() != t().state.main_thread) t().state.frees_elsewhere += 1;
    auto it = t().blocks.find((char*)p);
    if (it == t().blocks.end()) {
        lk.unlock();
        fault("free of memory that is not allocated");
        return 1;
    }
    t().state.used -= it->second;
    munmap(p, it->second);
    t().blocks.erase(it);
    return 0;
}
int hipFree(void* p) { return free_block(p, true); }
int hipMallocAsync(void** p, size_t bytes, void* st) {
    check((Stream*)st, "allocation on a destroyed stream");
    return hipMalloc(p, bytes);
}
int hipFreeAsync(void* p, void* st) {
    check((Stream*)st, "free on a destroyed stream");
    return free_block(p, false);
}
int hipDeviceGetDefaultMemPool(void** p, int) {
    static int pool;
    return *p = &pool, 0;
}
int hipMemPoolSetAttribute(void*, int, void*) { return 0; }
int hipMemGetInfo(size_t* f, size_t* all) {
    std::lock_guard<std::mutex> lk(t().mu);
    *f = t().state.total - t().state.used;
    *all = t().state.total;
    return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int) { return std::memcpy(d, s, n), 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void* st) {
    check((Stream*)st, "copy on a destroyed stream");
    std::memcpy(d, s, n);
    return 0;
}
int hipMemsetAsync(void* d, int v, size_t n, void* st) {
    check((Stream*)st, "fill on a destroyed stream");
    std::memset(d, v, n);
    return 0;
}

int hipStreamCreateWithFlags(void** s, unsigned) {
    Inside in;
    std::lock_guard<std::mutex> lk(t().mu);
    auto* q = new Stream;
    t().streams.insert(q);
    t().state.streams_made += 1;
    return *s = q, 0;
}
int hipStreamDestroy(void* s) {
    check((Stream*)s, "second destruction of a stream");
    std::lock_guard<std::mutex> lk(t().mu);
    ((Stream*)s)->alive = false;
    t().state.streams_destroyed += 1;
    return 0;
}
int hipStreamSynchronize(void* s) {
    check((Stream*)s, "wait for a destroyed stream");
    return 0;
}
int hipStreamGetDevice(void* s, int* d) {
    check((Stream*)s, "query of a destroyed stream");
    return *d = 0, 0;
}
int hipStreamWaitEvent(void* s, void* e, unsigned) {
    check((Stream*)s, "wait on a destroyed stream");
    check((Event*)e, "wait for a destroyed event");
    return 0;
}
int hipEventCreateWithFlags(void** e, unsigned) {
    Inside in;
    std::lock_guard<std::mutex> lk(t().mu);
    auto* q = new Event;
    t().events.insert(q);
    return *e = q, 0;
}
int hipEventCreate(void** e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(void* e) {
    check((Event*)e, "second destruction of an event");
    std::lock_guard<std::mutex> lk(t().mu);
    ((Event*)e)->alive = false;
    return 0;
}
int hipEventRecord(void* e, void* s) {
    check((Event*)e, "record of a destroyed event");
    check((Stream*)s, "record on a destroyed stream");
    return 0;
}
int hipEventSynchronize(void* e) {
    check((Event*)e, "wait for a destroyed event");
    return 0;
}
int hipEventElapsedTime(float* ms, void*, void*) { return *ms = 0.1f, 0; }

int hipStreamBeginCapture(void* s, int) {
    ((Stream*)s)->capturing = true;
    ((Stream*)s)->captured.clear();
    return 0;
}
int hipStreamEndCapture(void* s, void** g) {
    Inside in;
    auto* q = new Graph;
    q->nodes.swap(((Stream*)s)->captured);
    ((Stream*)s)->capturing = false;
    return *g = q, 0;
}
int hipGraphInstantiate(void** x, void* g, void*, char*, size_t) {
    Inside in;
    return *x = new Graph(*(Graph*)g), 0;
}
int hipGraphLaunch(void* x, void* s) {
    check((Stream*)s, "graph on a destroyed stream");
    for (auto& f : ((Graph*)x)->nodes) f();
    return 0;
}
int hipGraphDestroy(void* g) { return delete (Graph*)g, 0; }
int hipGraphExecDestroy(void* g) { return delete (Graph*)g, 0; }
}
