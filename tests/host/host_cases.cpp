// Host logic of the library (memory, streams, threads, errors) on the runtime of
// fake_hip.cpp: host_cases CASE, exit status 0 if the case holds.
#include <dlfcn.h>
#include <errno.h>
#include <pthread.h>

#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "fake_hip.hpp"
#include "simm.h"

static std::atomic<int> failed{0};
#define CHECK(c)                                                                      \
    do {                                                                              \
        if (!(c)) {                                                                   \
            std::printf("%s:%d: %s\n", __FILE__, __LINE__, #c);                       \
            ++failed;                                                                 \
        }                                                                             \
    } while (0)

// The library's allocations: the one numbered fail_at fails (none if negative).
static std::atomic<long> allocations{0}, fail_at{-1};
void* operator new(size_t bytes) {
    if (fake_hip_inside == 0 && allocations.fetch_add(1) == fail_at.load()) throw std::bad_alloc();
    if (void* p = std::malloc(bytes ? bytes : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

// Threads: none to be had once threads_left is 0 (no limit if negative).
static std::atomic<long> threads_left{-1};
extern "C" int pthread_create(pthread_t* t, const pthread_attr_t* a, void* (*f)(void*), void* arg) {
    using Create = int (*)(pthread_t*, const pthread_attr_t*, void* (*)(void*), void*);
    static Create create = (Create)dlsym(RTLD_NEXT, "pthread_create");
    if (threads_left.load() == 0) return EAGAIN;
    if (threads_left.load() > 0) threads_left.fetch_sub(1);
    return create(t, a, f, arg);
}

static simm_pencil band(int64_t n, int kl, int ku) {
    std::vector<double> a(2 * (size_t)(kl + ku + 1) * n, 0.5);
    simm_pencil p = nullptr;
    CHECK(simm_pencil_create_banded(n, kl, ku, a.data(), 0, 0, nullptr, SIMM_MEM_HOST, nullptr, &p) == SIMM_OK);
    return p;
}

static simm_params run_params(uint32_t flags, int lookahead) {
    simm_params q;
    simm_params_default(&q);
    q.x0 = q.y0 = -1;
    q.x1 = q.y1 = 1;
    q.n1 = 4;
    q.m = 12;
    q.levels = 4;
    q.flags = flags;
    q.lookahead = lookahead;
    return q;
}

struct Batch {
    std::vector<simm_pencil> pencils;
    std::vector<simm_params> prm;
    std::vector<std::vector<double>> f;
    std::vector<const double*> fp;
    std::vector<simm_result> out;
    Batch(int count, uint32_t flags) {
        for (int i = 0; i < count; ++i) {
            const int64_t n = 300 + 200 * (i % 7);
            pencils.push_back(band(n, 8, 8));
            prm.push_back(run_params(flags, 2));
            f.emplace_back(2 * n, 1.0);
        }
        for (auto& v : f) fp.push_back(v.data());
    }
    simm_status run(int workers) {
        out.assign(pencils.size(), nullptr);
        return simm_run_batch(pencils.data(), prm.data(), fp.data(), SIMM_MEM_HOST, (int32_t)pencils.size(), workers,
                              out.data());
    }
    void drop() {
        for (auto r : out) simm_result_destroy(r);
        out.clear();
    }
    ~Batch() {
        drop();
        for (auto p : pencils) simm_pencil_destroy(p);
    }
};

// A batch takes its memory and streams from the runtime and gives them back: nothing of it
// is kept while a pencil lives, and blocks kept before it are given back first.
static void batch_keeps_nothing() {
    FakeHip& h = fake_hip();
    Batch b(12, SIMM_FLAG_RELEASE_FACTORS | SIMM_FLAG_PROJECT);
    const size_t pencils_only = h.used;
    {   // a run of its own leaves blocks for reuse
        simm_result r = nullptr;
        CHECK(simm_run(b.pencils[0], &b.prm[0], b.fp[0], SIMM_MEM_HOST, nullptr, &r) == SIMM_OK);
        simm_result_destroy(r);
        CHECK(h.used > pencils_only);
    }
    const long made = h.streams_made, gone = h.streams_destroyed;
    CHECK(b.run(4) == SIMM_OK);
    int32_t shifts = 0;
    int64_t clusters = 0;
    CHECK(simm_result_summary(b.out[5], nullptr, &shifts, &clusters, nullptr) == SIMM_OK);
    CHECK(shifts > 1 && clusters > 0);
    CHECK(h.streams_made > made && h.streams_made - made == h.streams_destroyed - gone);
    b.drop();
    CHECK(h.used == pencils_only);
}

static std::vector<double> ones(int64_t count) { return std::vector<double>(2 * (size_t)count, 1.0); }

// A run, its multiplicities and the gradient of one of its squares; the first error.
static simm_status whole_use(simm_pencil p, const std::vector<double>& f) {
    const simm_params q = run_params(SIMM_FLAG_PROJECT, 3);
    simm_result r = nullptr;
    simm_status rc = simm_run(p, &q, f.data(), SIMM_MEM_HOST, nullptr, &r);
    if (rc != SIMM_OK) {
        CHECK(r == nullptr);
        return rc;
    }
    int64_t nc = 0, n = 0;
    int32_t ns = 0, kl = 0, ku = 0;
    simm_result_summary(r, nullptr, &ns, &nc, nullptr);
    simm_pencil_info(p, &n, &kl, &ku);
    CHECK(ns > 1 && nc > 0);
    ++fake_hip_inside;   // (not the library's)
    std::vector<double> F((size_t)(2 * n * 6), 1.0), grad((size_t)(2 * n));
    std::vector<int32_t> mult((size_t)nc);
    --fake_hip_inside;
    rc = simm_multiplicities(r, F.data(), 6, SIMM_MEM_HOST, 1e-6, nullptr, mult.data(), nullptr, nc);
    simm_shift s = nullptr;
    if (rc == SIMM_OK) rc = simm_result_shift(r, 0, &s);
    if (rc == SIMM_OK) {
        const int64_t squares[] = {1, 1, 1, 0, 1, 2, 1, 0, 1, 1, 2, 0, 1, 2, 2, 0, 2, 3, 3, 0};
        double J = 0.0;
        rc = simm_gradient(&s, 1, squares, 5, &q, 0, 0, nullptr, &J, nullptr, grad.data(), SIMM_MEM_HOST, nullptr);
    }
    simm_result_destroy(r);
    return rc;
}

extern "C" int hipMalloc(void** p, size_t bytes);
extern "C" int hipFree(void* p);

// Builds and destroys a shift of order n and half-bandwidth 8.
static void build_one(int64_t n) {
    const std::vector<double> f = ones(n);
    simm_pencil p = band(n, 8, 8);
    simm_shift s = nullptr;
    CHECK(simm_shift_build(p, 0.1, 0.2, f.data(), SIMM_MEM_HOST, 8, SIMM_PREC_FP64, nullptr, &s) == SIMM_OK);
    simm_shift_destroy(s);
    simm_pencil_destroy(p);
}

// Small blocks too are kept only while a quarter of the memory is free.
static void kept_while_a_quarter_is_free() {
    FakeHip& h = fake_hip();
    h.total = (size_t)4 << 30;
    void* ballast = nullptr;
    CHECK(hipMalloc(&ballast, (size_t)3328 << 20) == 0);
    simm_pencil held = band(300, 8, 8);
    const size_t base = h.used;
    size_t most = 0;
    for (int64_t n = 2000; n < 22000; n += 400) {
        build_one(n);
        most = std::max(most, h.used - base);
    }
    std::printf("%.0f MB kept\n", most / 1e6);
    CHECK(most <= ((size_t)64 << 20));
    simm_pencil_destroy(held);
    hipFree(ballast);
}

// Blocks of sizes that are not asked for any more make room for those that are.
static void sizes_in_use_are_kept() {
    FakeHip& h = fake_hip();
    h.total = (size_t)4 << 30;   // 512 MB of blocks at most
    simm_pencil held = band(300, 8, 8);
    for (int64_t n = 2000; n < 40000; n += 800) build_one(n);
    CHECK(h.used <= ((size_t)513 << 20));
    for (int i = 0; i < 3; ++i) build_one(60000);
    const long before = h.mallocs;
    for (int i = 0; i < 3; ++i) build_one(60000);
    std::printf("%ld allocations in three builds\n", h.mallocs - before);
    CHECK(h.mallocs == before);
    simm_pencil_destroy(held);
}

// Factors are computed ahead of a run's order only where a quarter of the free memory holds
// them with the sweep data of the next one (a wide band's: with spikes and reduced inverse).
static void factors_ahead_fit() {
    FakeHip& h = fake_hip();
    const int64_t n = 24000;
    const std::vector<double> f = ones(n);
    simm_pencil p = band(n, 200, 200);
    const size_t base = h.used;
    simm_shift s = nullptr;
    CHECK(simm_shift_build(p, 0.1, 0.2, f.data(), SIMM_MEM_HOST, 2, SIMM_PREC_FP64, nullptr, &s) == SIMM_OK);
    simm_shift_destroy(s);
    const size_t one = h.peak - base;   // a factor and its sweep data, while they are made
    simm_params q = run_params(SIMM_FLAG_RELEASE_FACTORS, 8);
    q.m = 2;
    for (const double quarter : {0.95, 1.9}) {
        simm_pencil_destroy(p);
        p = band(n, 200, 200);
        h.total = base + (size_t)(4 * quarter * (double)one);
        const long made = h.streams_made;
        simm_result r = nullptr;
        CHECK(simm_run(p, &q, f.data(), SIMM_MEM_HOST, nullptr, &r) == SIMM_OK);
        simm_result_destroy(r);
        const long ahead = h.streams_made - made - 1;   // (one for the Schur forms)
        std::printf("a quarter holds %.2f builds: %ld streams for factors ahead\n", quarter, ahead);
        CHECK(quarter < 1 ? ahead == 0 : ahead > 1);
    }
    simm_pencil_destroy(p);
}

// Blocks take what is asked for, so that what fits without a cache fits with it; one that is
// kept serves requests down to eight ninths of its size.
static void blocks_have_the_size_asked_for() {
    FakeHip& h = fake_hip();
    const int64_t n = 33000;
    const std::vector<double> f = ones(n);
    simm_pencil p = band(n, 8, 8);
    h.watch = 16 * (size_t)n * 100;   // the basis
    simm_shift s = nullptr;
    CHECK(simm_shift_build(p, 0.1, 0.2, f.data(), SIMM_MEM_HOST, 99, SIMM_PREC_FP64, nullptr, &s) == SIMM_OK);
    CHECK(h.watched == 1);
    simm_shift_destroy(s);
    build_one(60000);
    const long before = h.mallocs;
    build_one(59900);
    std::printf("%ld allocations\n", h.mallocs - before);
    CHECK(h.mallocs == before);
    simm_pencil_destroy(p);
}

// Scratch of the spikes' columns: of all of them where memory holds it, else of fewer at a
// time, and the factor stays partitioned.
static void spikes_with_less_scratch() {
    FakeHip& h = fake_hip();
    const int64_t n = 1 << 18, w = 128;
    const std::vector<double> f = ones(n);
    const size_t all = h.total;
    auto build = [&](size_t memory, int64_t* block) {
        h.total = memory;
        simm_pencil p = band(n, w / 2, w / 2);
        simm_shift s = nullptr;
        h.peak = 0;
        const simm_status rc = simm_shift_build(p, 0.1, 0.2, f.data(), SIMM_MEM_HOST, 2, SIMM_PREC_FP64, nullptr, &s);
        *block = 0;
        if (rc == SIMM_OK) CHECK(simm_shift_factor_info(s, block, nullptr, nullptr) == SIMM_OK);
        simm_shift_destroy(s);
        simm_pencil_destroy(p);
        return rc;
    };
    int64_t block = 0;
    CHECK(build(all, &block) == SIMM_OK && block > 0);
    const size_t peak = h.peak, scratch = 16 * (size_t)n * w;
    size_t lo = h.peak / 2, hi = h.peak;   // the least memory of a partitioned factor
    while (hi - lo > scratch / 64) {
        const size_t mid = (lo + hi) / 2;
        (build(mid, &block) == SIMM_OK && block > 0 ? hi : lo) = mid;
    }
    std::printf("%.0f MB are enough, %.0f MB taken where there is more, scratch %.0f MB\n", hi / 1e6, peak / 1e6,
                scratch / 1e6);
    CHECK(hi + 9 * scratch / 10 < peak);
}

// A band that is partitioned is factored whole where memory holds only that.
static void whole_factor_where_it_fits() {
    FakeHip& h = fake_hip();
    const int64_t n = 24000;
    const std::vector<double> f = ones(n);
    auto build = [&](size_t memory, int64_t* block, int32_t* fallback) {
        h.total = memory;
        simm_pencil p = band(n, 200, 200);
        simm_shift s = nullptr;
        h.peak = 0;
        const simm_status rc = simm_shift_build(p, 0.1, 0.2, f.data(), SIMM_MEM_HOST, 2, SIMM_PREC_FP64, nullptr, &s);
        if (rc == SIMM_OK) CHECK(simm_shift_factor_info(s, block, fallback, nullptr) == SIMM_OK);
        simm_shift_destroy(s);
        simm_pencil_destroy(p);
        return rc;
    };
    const size_t all = h.total;
    int64_t block = 0;
    int32_t fallback = 0;
    CHECK(build(all, &block, &fallback) == SIMM_OK && block > 0 && fallback == 0);
    setenv("SIMM_LU_PART", "0", 1);
    CHECK(build(all, &block, &fallback) == SIMM_OK && block == 0);
    const size_t whole = h.peak;
    CHECK(build(whole, &block, &fallback) == SIMM_OK);
    unsetenv("SIMM_LU_PART");
    const simm_status rc = build(whole, &block, &fallback);
    std::printf("%.0f MB: %s\n", whole / 1e6, rc == SIMM_OK ? "ok" : simm_last_error());
    CHECK(rc == SIMM_OK && block == 0 && fallback == 1);
}

// Blocks of three right-hand sides: three squares of a shift, three start vectors.
static void three_at_once() {
    const int64_t n = 500;
    const std::vector<double> f = ones(3 * n);
    simm_pencil p = band(n, 8, 8);
    const simm_params q = run_params(0, 1);
    simm_result r = nullptr;
    CHECK(simm_run(p, &q, f.data(), SIMM_MEM_HOST, nullptr, &r) == SIMM_OK);
    int64_t nc = 0;
    simm_result_summary(r, nullptr, nullptr, &nc, nullptr);
    std::vector<int32_t> mult((size_t)nc);
    CHECK(simm_multiplicities(r, f.data(), 3, SIMM_MEM_HOST, 1e-6, nullptr, mult.data(), nullptr, nc) == SIMM_OK);
    simm_shift s = nullptr;
    CHECK(simm_result_shift(r, 0, &s) == SIMM_OK);
    const int64_t squares[] = {1, 1, 1, 0, 1, 2, 1, 0, 1, 1, 2, 0, 1, 2, 2, 0, 2, 3, 3, 0, 2, 3, 4, 0, 2, 4, 4, 0};
    double J = 0.0;
    std::vector<double> grad((size_t)(2 * n));
    for (int64_t count = 1; count <= 7; ++count)
        CHECK(simm_gradient(&s, 1, squares, count, &q, 0, 0, nullptr, &J, nullptr, grad.data(), SIMM_MEM_HOST, nullptr) ==
              SIMM_OK);
    simm_result_destroy(r);
    simm_pencil_destroy(p);
}

// The threads a run starts beside its own free nothing to the device (its memory is large
// enough); what they release is freed by the run's thread.
static void helpers_free_nothing() {
    FakeHip& h = fake_hip();
    const int64_t n = 1 << 20;
    const std::vector<double> f = ones(n);
    simm_pencil p = band(n, 8, 8);
    h.total = (size_t)110 << 30;   // too little is free for blocks to be kept
    simm_params q = run_params(0, 6);
    q.n1 = 8;
    simm_result r = nullptr;
    CHECK(simm_run(p, &q, f.data(), SIMM_MEM_HOST, nullptr, &r) == SIMM_OK);
    std::printf("%ld blocks freed, %ld by other threads, %.1f GB at most\n", h.frees, h.frees_elsewhere, h.peak / 1e9);
    CHECK(h.frees > 0 && h.frees_elsewhere == 0);
    simm_result_destroy(r);
    simm_pencil_destroy(p);
}

// Calls of several threads at once, a batch among them: all memory comes back.
static void threads_side_by_side() {
    std::vector<std::thread> threads;
    for (int i = 0; i < 3; ++i)
        threads.emplace_back([i]() {
            for (int k = 0; k < 6; ++k) {
                const int64_t n = 400 + 100 * i + 37 * k;
                simm_pencil p = band(n, 8, 8);
                CHECK(whole_use(p, ones(n)) == SIMM_OK);
                simm_pencil_destroy(p);
            }
        });
    for (int k = 0; k < 3; ++k) {
        Batch b(4, k % 2 ? SIMM_FLAG_RELEASE_FACTORS : 0);
        CHECK(b.run(2) == SIMM_OK);
    }
    for (auto& t : threads) t.join();
}

// Calls do their work where the system gives them no thread, or fewer than they ask for.
static void no_threads() {
    for (long left : {0L, 1L, 3L, -1L}) {
        threads_left = left;
        simm_pencil p = band(500, 8, 8);
        const simm_status rc = whole_use(p, ones(500));
        if (rc != SIMM_OK) std::printf("%ld threads: %s\n", left, simm_last_error());
        CHECK(rc == SIMM_OK);
        simm_pencil_destroy(p);
        Batch b(5, SIMM_FLAG_RELEASE_FACTORS);
        CHECK(b.run(3) == SIMM_OK);
    }
}

// Where host memory runs out a call returns ENOMEM (or a message cut short), keeps no memory of
// the device and leaves the library fit for the next call.
static void no_host_memory() {
    for (int batch = 0; batch < 2; ++batch) {
        long total = 0, errors = 0;
        for (long k = -1; k < total; k += std::max<long>(1, total / 300)) {
            {
                const std::vector<double> f = ones(500);
                simm_pencil p = band(500, 8, 8);
                Batch b(batch ? 4 : 0, SIMM_FLAG_RELEASE_FACTORS | SIMM_FLAG_PROJECT);
                if (batch) b.out.assign(b.pencils.size(), nullptr);
                allocations = 0;
                fail_at = k;
                const simm_status rc = batch ? simm_run_batch(b.pencils.data(), b.prm.data(), b.fp.data(), SIMM_MEM_HOST,
                                                              4, 3, b.out.data())
                                             : whole_use(p, f);
                fail_at = -1;
                if (k < 0) {
                    total = allocations.load();
                    CHECK(rc == SIMM_OK && total > 100);
                } else if (rc != SIMM_OK) {
                    ++errors;
                }
                simm_pencil_destroy(p);
            }
            CHECK(fake_hip().used == 0);
        }
        CHECK(errors > 50);
    }
}

int main(int argc, char** argv) {
    const std::map<std::string, void (*)()> cases = {
        {"batch_keeps_nothing", batch_keeps_nothing},
        {"kept_while_a_quarter_is_free", kept_while_a_quarter_is_free},
        {"sizes_in_use_are_kept", sizes_in_use_are_kept},
        {"factors_ahead_fit", factors_ahead_fit},
        {"blocks_have_the_size_asked_for", blocks_have_the_size_asked_for},
        {"spikes_with_less_scratch", spikes_with_less_scratch},
        {"whole_factor_where_it_fits", whole_factor_where_it_fits},
        {"three_at_once", three_at_once},
        {"helpers_free_nothing", helpers_free_nothing},
        {"threads_side_by_side", threads_side_by_side},
        {"no_threads", no_threads},
        {"no_host_memory", no_host_memory},
    };
    const auto it = cases.find(argc > 1 ? argv[1] : "");
    if (it == cases.end()) return 2;
    it->second();
    CHECK(fake_hip().faults == 0);
    CHECK(fake_hip().used == 0);   // every case has destroyed its objects
    return failed ? 1 : 0;
}
