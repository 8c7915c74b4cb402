// Host logic of the library (memory, streams, threads, errors) on the runtime of
// fake_hip.cpp: host_cases CASE, exit status 0 if the case holds.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "fake_hip.hpp"
#include "simm.h"

static int failed = 0;
#define CHECK(c)                                                                      \
    do {                                                                              \
        if (!(c)) {                                                                   \
            std::printf("%s:%d: %s\n", __FILE__, __LINE__, #c);                       \
            ++failed;                                                                 \
        }                                                                             \
    } while (0)

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

int main(int argc, char** argv) {
    const std::map<std::string, void (*)()> cases = {
        {"batch_keeps_nothing", batch_keeps_nothing},
    };
    const auto it = cases.find(argc > 1 ? argv[1] : "");
    if (it == cases.end()) return 2;
    it->second();
    CHECK(fake_hip().faults == 0);
    CHECK(fake_hip().used == 0);   // every case has destroyed its objects
    return failed ? 1 : 0;
}
