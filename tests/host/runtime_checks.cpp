// Checks of plan.cpp over a stand-in runtime (runtime.cpp): what a call hands to its
// kernel and what a plan takes of the device's memory.  The check is named by the
// argument; prints one line per failure and exits non-zero if there was one.
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

int main(int argc, char **argv)
{
    const char *what = argc > 1 ? argv[1] : "";
    if (!std::strcmp(what, "select-threads")) select_without_threads();
    else {
        std::printf("no check named '%s'\n", what);
        return 2;
    }
    std::printf("%s: %d failure(s)\n", what, failures);
    return failures ? 1 : 0;
}
