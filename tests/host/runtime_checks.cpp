// Checks of plan.cpp over a stand-in runtime (runtime.cpp): what a call hands to its
// kernel and what a plan takes of the device's memory.  The check is named by the
// argument; prints one line per failure and exits non-zero if there was one.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <vector>

#include "runtime.h"
#include "slos.h"

static int failures = 0;
#define CHECK(cond, ...)                                  \
    do {                                                  \
        if (!(cond)) {                                    \
            ++failures;                                   \
            std::printf("FAIL %s:%d: ", __FILE__, __LINE__); \
            std::printf(__VA_ARGS__);                     \
            std::printf(" [%s]\n", slos_last_error());    \
        }                                                 \
    } while (0)

// `count` targets of 12 modes and 6 photons, the first `bunched` of them with two
// photons in a mode
static std::vector<int32_t> targets_of(int count, int bunched)
{
    std::vector<int32_t> t((size_t)count * 12, 0);
    for (int i = 0; i < count; ++i) {
        int32_t *s = t.data() + (size_t)i * 12;
        const int two = i < bunched;
        for (int j = 0; j < 6 - two; ++j) s[(i + 2 * j) % 12] = 1;
        if (two) s[i % 12] = 2;
    }
    return t;
}

// every target of the call is dealt to the kernel, each once
static void check_dealt(int count, const char *what)
{
    const SelectParams &sp = fake.select;
    CHECK(sp.start[SLOS_SELECT_CLASSES] == count, "%s: %lld of %d targets dealt", what,
          (long long)sp.start[SLOS_SELECT_CLASSES], count);
    std::vector<char> met(count, 0);
    for (int i = 0; i < count; ++i) {
        const uint64_t row = sp.order[i] >> SLOS_SELECT_PATTERN_BITS;
        if (row >= (uint64_t)count || met[row]) {
            CHECK(false, "%s: place %d holds row %llu", what, i, (unsigned long long)row);
            break;
        }
        met[row] = 1;
    }
}

// Selected outputs when no helper thread can be started, after a call that had some:
// the helpers' state of that call is not taken for this one's.
static void select_without_threads()
{
    std::vector<int32_t> T(12, 0);
    for (int i = 0; i < 6; ++i) T[i] = 1;
    slos_plan_t p = nullptr;
    CHECK(slos_plan(12, 6, T.data(), SLOS_C64, &p) == SLOS_OK, "plan");
    if (!p) return;
    float u[2], out[2];
    // patterns new to the plan, then known ones, then a refused call, each before one without helpers
    std::vector<int32_t> t = targets_of(20000, 7000);
    CHECK(slos_select(p, u, t.data(), 20000, out, nullptr) == SLOS_OK, "new patterns");
    check_dealt(20000, "new patterns");
    CHECK(slos_select(p, u, t.data(), 20000, out, nullptr) == SLOS_OK, "known patterns");
    check_dealt(20000, "known patterns");
    fake.no_threads = true;
    t = targets_of(16384, 5000);
    CHECK(slos_select(p, u, t.data(), 16384, out, nullptr) == SLOS_OK, "without helpers");
    check_dealt(16384, "without helpers");
    fake.no_threads = false;
    t = targets_of(18000, 9000);
    for (int i = 0; i < 18000; ++i) t[(size_t)i * 12 + 11] += 1;  // seven photons: refused by every thread
    CHECK(slos_select(p, u, t.data(), 18000, out, nullptr) == SLOS_ERR_INVALID_ARG, "seven photons accepted");
    fake.no_threads = true;
    t = targets_of(12000, 0);
    CHECK(slos_select(p, u, t.data(), 12000, out, nullptr) == SLOS_OK, "after a refused call");
    check_dealt(12000, "after a refused call");
    fake.no_threads = false;
    slos_plan_destroy(p);
}

// every multiset of `left` photons, each occupation at most the one before, in at most `room` modes
template <typename F> static void multisets(std::vector<int32_t> &q, int left, size_t room, F &&f)
{
    if (left == 0) {
        f();
        return;
    }
    if (q.size() == room) return;
    for (int v = q.empty() ? left : std::min(left, (int)q.back()); v > 0; --v) {
        q.push_back(v);
        multisets(q, left - v, room, f);
        q.pop_back();
    }
}

// The parts of a workgroup's LDS that targets run in, for every multiset of
// occupations beside a small one: each starts at a multiple of 16 bytes and holds
// its target; and the copy of a call's targets is of whole 16-byte units.
static void select_parts()
{
    const struct { int m, n; } sizes[] = {{11, 11}, {13, 13}, {8, 16}, {8, 21}, {4, 30}};
    for (int flags : {SLOS_C64, SLOS_C128})
        for (const auto &z : sizes) {
            const uint64_t es = flags == SLOS_C64 ? 8 : 16;
            std::vector<int32_t> T(z.m, 0);
            for (int i = 0; i < z.n; ++i) ++T[i % z.m];
            slos_plan_t p = nullptr;
            CHECK(slos_plan(z.m, z.n, T.data(), flags, &p) == SLOS_OK, "plan m=%d n=%d", z.m, z.n);
            if (!p) continue;
            std::vector<int32_t> q;
            multisets(q, z.n, (size_t)z.m, [&] {
                uint64_t R = 1;
                for (int v : q) R *= (uint64_t)v + 1;
                if (R * es > SLOS_LDS_DYNAMIC_MAX) return;
                std::vector<int32_t> t(2 * (size_t)z.m, 0);
                std::copy(q.begin(), q.end(), t.begin());
                t[z.m] = z.n;
                float u[2], out[4];
                CHECK(slos_select(p, u, t.data(), 2, out, nullptr) == SLOS_OK, "m=%d n=%d", z.m, z.n);
                const SelectParams &sp = fake.select;
                CHECK(fake.copied % 16 == 0 && fake.copied >= 2 * (z.n + sizeof(uint64_t)), "%zu bytes copied", fake.copied);
                CHECK(sp.lds <= SLOS_LDS_DYNAMIC_MAX && R * es <= sp.lds, "m=%d n=%d: %u bytes", z.m, z.n, sp.lds);
                for (int j = 0; j < SLOS_SELECT_CLASSES; ++j) {
                    if (sp.start[j + 1] == sp.start[j]) continue;
                    const uint32_t part = sp.lds / (SLOS_SELECT_THREADS / 64 >> (SLOS_SELECT_CLASSES - 1 - j));
                    CHECK(part % 16 == 0, "m=%d n=%d, %llu states: parts of %u bytes", z.m, z.n, (unsigned long long)R, part);
                    for (int64_t i = sp.start[j]; i < sp.start[j + 1]; ++i) {
                        const SelectPattern &pt = sp.patterns[sp.order[i] & ((1u << SLOS_SELECT_PATTERN_BITS) - 1)];
                        CHECK(j == 0 || pt.R * es + (uint64_t)z.n * pt.nocc * SLOS_SELECT_ENTRY(flags == SLOS_C64) <= part,
                              "m=%d n=%d: %u states in %u bytes", z.m, z.n, pt.R, part);
                    }
                }
            });
            slos_plan_destroy(p);
        }
}

// device memory that `make` takes, which returns what undoes it
template <typename F> static size_t memory_of(F &&make)
{
    fake.used = fake.peak = 0;
    auto undo = make();
    const size_t used = fake.peak;
    undo();
    CHECK(fake.used == 0, "%zu bytes not given back", fake.used);
    return used;
}

// Plans, batches and sources are made in the memory that they take without tables,
// and a plan's tables stay within their limits.
static void table_memory()
{
    slos_options_t tiled{};
    auto plan = [&](int m, int n, int flags, bool tables) {
        return [=] {
            std::vector<int32_t> T(m, 0);
            for (int i = 0; i < n; ++i) ++T[i % m];
            slos_options_t o{};
            // the default sizes, named: the same kernels and buffers without tables
            o.leaf_max = flags & SLOS_KEEP_LAYERS ? 4096 : flags & SLOS_C64 ? 16384 : 8192;
            slos_plan_t p = nullptr;
            CHECK(slos_plan_ex(m, n, T.data(), flags, tables ? nullptr : &o, &p) == SLOS_OK, "plan m=%d n=%d flags=%x", m,
                  n, flags);
            return [p] { slos_plan_destroy(p); };
        };
    };
    const struct { int m, n, flags; } plans[] = {{6, 3, SLOS_C128},
                                                 {12, 6, SLOS_C64 | SLOS_KEEP_LAYERS},
                                                 {17, 8, SLOS_C64 | SLOS_COMPENSATED},
                                                 {16, 8, SLOS_C128 | SLOS_KEEP_LAYERS},
                                                 {92, 5, SLOS_C64 | SLOS_KEEP_LAYERS}};
    for (const auto &z : plans) {
        const size_t without = memory_of(plan(z.m, z.n, z.flags, false)), with = memory_of(plan(z.m, z.n, z.flags, true));
        CHECK(with <= without + (size_t(922) << 20) + 8 * (size_t)3200000, "m=%d n=%d flags=%x: %zu bytes beside %zu", z.m,
              z.n, z.flags, with - without, without);
        fake.budget = without;
        memory_of(plan(z.m, z.n, z.flags, true));
        fake.budget = ~size_t(0);
    }
    tiled.leaf_max = 1024;
    auto batch = [&](bool tables) {
        return [=] {
            std::vector<int32_t> ms, in;
            for (int m = 6; m < 15; ++m) {
                ms.push_back(m);
                for (int j = 0; j < m; ++j) in.push_back(j < 6);
            }
            slos_batch_t b = nullptr;
            CHECK(slos_batch_plan((int)ms.size(), ms.data(), in.data(), SLOS_C64, tables ? nullptr : &tiled, &b) == SLOS_OK,
                  "batch");
            return [b] { slos_batch_destroy(b); };
        };
    };
    fake.budget = memory_of(batch(false));
    memory_of(batch(true));
    fake.budget = ~size_t(0);
    tiled.leaf_max = 256;
    auto source = [&](bool tables) {
        return [=] {
            std::vector<int32_t> T(12, 0);
            for (int j = 0; j < 6; ++j) T[j] = 1;
            const slos_source_params_t sp{0.9, 0.05, 0.92};
            slos_source_t s = nullptr;
            CHECK(slos_source_plan(12, T.data(), &sp, -1, tables ? nullptr : &tiled, &s) == SLOS_OK, "source");
            return [s] { slos_source_destroy(s); };
        };
    };
    fake.budget = memory_of(source(false));
    memory_of(source(true));
    fake.budget = ~size_t(0);
}

// slos_amplitudes_noalloc takes every plan that its static area holds without tables
// (the call then ends at the stand-in's missing area), and the tables' plan needs no more
// partial sums per instance.
static void noalloc_area()
{
    const struct { int m, n; } sizes[] = {{6, 3}, {12, 6}, {17, 8}, {20, 6}, {255, 3}, {40, 4}, {8, 20}, {3, 32}, {2, 1}};
    int held = 0;
    for (const auto &z : sizes)
        for (int flags : {SLOS_C64, SLOS_C128})
            for (int batch : {1, 64, 2048, 8192}) {
                std::vector<int32_t> T(z.m, 0);
                for (int i = 0; i < z.n; ++i) ++T[i % z.m];
                int64_t M = 0;
                slos_fock_count(z.m, z.n, &M);
                if (M * batch > 40000000) continue;  // more layers than the stand-in's memory
                int rc[2] = {};
                for (int tables : {0, 1}) {
                    slos_options_t o{};
                    o.max_batch = batch;
                    if (!tables) o.leaf_max = flags == SLOS_C64 ? 16384 : 8192;
                    slos_plan_t p = nullptr;
                    fake.used = fake.peak = 0;
                    CHECK(slos_plan_ex(z.m, z.n, T.data(), flags, &o, &p) == SLOS_OK, "plan m=%d n=%d", z.m, z.n);
                    if (!p) return;
                    float u[2], out[2];
                    rc[tables] = slos_amplitudes_noalloc(p, u, out, nullptr, nullptr);
                    slos_plan_destroy(p);
                }
                held += rc[0] != SLOS_ERR_SIZE_OVERFLOW;
                CHECK(rc[1] != SLOS_ERR_SIZE_OVERFLOW || rc[0] == SLOS_ERR_SIZE_OVERFLOW, "m=%d n=%d flags=%x max_batch=%d",
                      z.m, z.n, flags, batch);
            }
    CHECK(held > 10, "only %d plans fit the area", held);
}

// `call` with each of its host allocations failing in turn: it returns OK or OOM (no
// exception crosses the C entry) and, with `clean`, gives the device's memory back.
template <typename F, typename G> static void fail_each(const char *what, F &&call, G &&after)
{
    for (long i = 0;; ++i) {
        fake.news = i;
        int rc = -100;
        try {
            rc = call();
        } catch (...) {
        }
        const bool reached = fake.news.exchange(-1) < 0;
        CHECK(rc == SLOS_OK || rc == SLOS_ERR_OOM, "%s, allocation %ld: %d", what, i, rc);
        after(rc);
        if (!reached || failures > 20) break;
    }
}

static void allocation_failures()
{
    std::vector<int32_t> T(12, 0);
    for (int i = 0; i < 6; ++i) T[i] = 1;
    for (int flags : {SLOS_C64, SLOS_C128 | SLOS_KEEP_LAYERS}) {
        slos_plan_t p = nullptr;
        fake.used = 0;
        fail_each("plan", [&] { return slos_plan(8, 4, T.data() + 2, flags, &p); },
                  [&](int rc) {
                      CHECK((p != nullptr) == (rc == SLOS_OK), "plan: a handle with an error");
                      slos_plan_destroy(p);
                      p = nullptr;
                      CHECK(fake.used == 0, "plan: %zu bytes kept", fake.used);
                  });
    }
    const int32_t ms[3] = {12, 12, 6};
    std::vector<int32_t> in(T);
    in.insert(in.end(), T.begin(), T.end());
    in.insert(in.end(), T.begin() + 3, T.begin() + 9);
    slos_batch_t b = nullptr;
    fail_each("batch", [&] { return slos_batch_plan(3, ms, in.data(), SLOS_C64, nullptr, &b); },
              [&](int) {
                  slos_batch_destroy(b);
                  b = nullptr;
                  CHECK(fake.used == 0, "batch: %zu bytes kept", fake.used);
              });
    const slos_source_params_t sp{0.9, 0.05, 0.92};
    slos_source_t s = nullptr;
    fail_each("source", [&] { return slos_source_plan(6, T.data() + 3, &sp, -1, nullptr, &s); },
              [&](int) {
                  slos_source_destroy(s);
                  s = nullptr;
                  CHECK(fake.used == 0, "source: %zu bytes kept", fake.used);
              });
    // selected outputs on a new plan: after a failure the same call gives all its targets
    const std::vector<int32_t> t = targets_of(4200, 1000);
    float u[2], out[2];
    slos_plan_t p = nullptr;
    fail_each("select",
              [&] {
                  if (!p) {
                      const long news = fake.news.exchange(-1);
                      CHECK(slos_plan(12, 6, T.data(), SLOS_C64, &p) == SLOS_OK, "plan");
                      fake.news = news;
                  }
                  return slos_select(p, u, t.data(), 4200, out, nullptr);
              },
              [&](int) {
                  CHECK(slos_select(p, u, t.data(), 4200, out, nullptr) == SLOS_OK, "select after a failure");
                  check_dealt(4200, "after a failure");
                  for (int i = 0; i < 4200; ++i) {
                      const SelectPattern &pt = fake.select.patterns[fake.select.order[i] & 0xFFFFu];
                      if (pt.off + pt.R > (uint32_t)((const uint16_t *)fake.select.mask - fake.select.state)) {
                          CHECK(false, "a pattern past the pools");
                          break;
                      }
                  }
                  slos_plan_destroy(p);
                  p = nullptr;
              });
}

int main(int argc, char **argv)
{
    const char *what = argc > 1 ? argv[1] : "";
    if (!std::strcmp(what, "select-threads")) select_without_threads();
    else if (!std::strcmp(what, "select-parts")) select_parts();
    else if (!std::strcmp(what, "table-memory")) table_memory();
    else if (!std::strcmp(what, "noalloc-area")) noalloc_area();
    else if (!std::strcmp(what, "allocation-failures")) allocation_failures();
    else {
        std::printf("no check named '%s'\n", what);
        return 2;
    }
    std::printf("%s: %d failure(s)\n", what, failures);
    return failures ? 1 : 0;
}
