// csrc/teuk_staging.h without a GPU: transfers are copies by a thread of their own after a delay.
#include <atomic>
#include <chrono>
#include <cstdint>
#include <cstdio>
#include <ctime>
#include <fstream>
#include <future>
#include <string>

#include "teuk_staging.h"

using namespace teuk;
static int failures = 0;
#define CHECK(x) (void)((x) || (++failures, std::printf("line %d: %s\n", __LINE__, #x)))

static double cpu_seconds()
{
    timespec t;
    clock_gettime(CLOCK_PROCESS_CPUTIME_ID, &t);
    return (double)t.tv_sec + 1e-9 * (double)t.tv_nsec;
}

// One copy of `bytes`; a transfer takes `us`, issue number fail_issue and landing number fail_landed fail.
static int copy(size_t bytes, size_t chunk, int buffers, int workers, int us, bool* exact, long long fail_issue = -1,
                long long fail_landed = -1)
{
    std::vector<unsigned char> src(bytes), dst(bytes + 64, 0xee), mem(chunk * (size_t)buffers);
    for (size_t i = 0; i < bytes; ++i) src[i] = (unsigned char)(i * 31 + (i >> 8) * 7 + 1);
    std::vector<std::future<void>> flight((size_t)buffers);
    long long landings = 0;
    bool started = false;
    const int e = move_chunks(
        (char*)dst.data(), (const char*)mem.data(), bytes, chunk, buffers, workers,
        [&](long long c, int b, size_t n) {
            if (c == fail_issue) return 7;
            flight[(size_t)b] = std::async(std::launch::async, [&, c, b, n] {
                if (us) std::this_thread::sleep_for(std::chrono::microseconds(us));
                std::memcpy(mem.data() + (size_t)b * chunk, src.data() + (size_t)c * chunk, n);
            });
            return 0;
        },
        [&](int b) {
            flight[(size_t)b].get();
            return landings++ == fail_landed ? 9 : 0;
        },
        &started);
    for (auto& f : flight)
        if (f.valid()) f.get();
    CHECK(started);
    *exact = std::memcmp(dst.data(), src.data(), bytes) == 0;
    for (int i = 0; i < 64; ++i) CHECK(dst[bytes + (size_t)i] == 0xee);
    return e;
}

struct Set {
    int device;
};

int main(int argc, char** argv)
{
    const std::string dir = argc > 1 ? argv[1] : "/tmp";
    bool exact;
    // sizes around the chunks, fewer and more of them than buffers and workers
    for (size_t bytes : {1, 999, 1000, 1001, 7999, 8000, 8001, 16000, 100003})
        for (int workers : {1, 2, 3, 8}) {
            CHECK(copy(bytes, 1000, 8, workers, 0, &exact) == 0);
            CHECK(exact);
        }
    CHECK(copy(20000, 1000, 2, 3, 0, &exact) == 0 && exact);
    // an error of either kind, early and late, ends the call
    for (long long c : {0, 3, 19}) {
        CHECK(copy(20000, 1000, 8, 4, 0, &exact, c) == 7);
        CHECK(copy(20000, 1000, 8, 4, 0, &exact, -1, c) == 9);
    }
    // while transfers are slow the threads sleep: 40 of 10 ms, four at a time, 0.1 s
    const double cpu = cpu_seconds();
    CHECK(copy(40000, 1000, 8, 8, 10000, &exact) == 0 && exact);
    const double used = cpu_seconds() - cpu;
    std::printf("cpu time of a copy that waits 0.1 s: %.3f s\n", used);
    CHECK(used < 0.1);

    // the pool: at most two sets, kept while there are users, other devices' idle ones given up
    SetPool<Set, 2> pool;
    int alive = 0;
    auto free = [&](Set* s) { --alive; delete s; };
    auto make = [&](int d) { return [&, d] { ++alive; return new Set{d}; }; };
    auto none = [&]() -> Set* { return nullptr; };
    pool.user_made();
    Set* a = pool.take(0, make(0), free);
    Set* b = pool.take(0, make(0), free);
    CHECK(a && b && !pool.take(0, make(0), free) && alive == 2);
    pool.give(a, free);
    CHECK(pool.take(0, make(0), free) == a);
    pool.give(a, free);
    pool.give(b, free);
    Set* c = pool.take(1, make(1), free);
    CHECK(c && c->device == 1 && alive == 2);
    CHECK(!pool.take(2, none, free) && alive == 1);      // device 0's set went, none was made, its place is free
    Set* d = pool.take(2, make(2), free);
    CHECK(d && d->device == 2 && alive == 2);
    pool.give(d, free);
    pool.user_gone(free);
    CHECK(alive == 1);                                   // c is still in use
    pool.give(c, free);
    CHECK(alive == 0);

    // quotas
    auto write = [&](const char* name, const char* text) {
        std::ofstream(dir + "/" + name) << text;
        return dir + "/" + name;
    };
    const std::string no = dir + "/none";
    CHECK(quota_cpus(write("a", "400000 100000\n").c_str(), no.c_str(), no.c_str()) == 4);
    CHECK(quota_cpus(write("b", "max 100000\n").c_str(), no.c_str(), no.c_str()) == 0);
    CHECK(quota_cpus(write("c", "50000 100000\n").c_str(), no.c_str(), no.c_str()) == 1);
    CHECK(quota_cpus(no.c_str(), write("d", "300000\n").c_str(), write("e", "100000\n").c_str()) == 3);
    CHECK(quota_cpus(no.c_str(), write("f", "-1\n").c_str(), write("g", "100000\n").c_str()) == 0);
    CHECK(quota_cpus(no.c_str(), no.c_str(), no.c_str()) == 0);
    CHECK(usable_cpus() >= 1);
    std::printf("failures %d\n", failures);
    return failures != 0;
}
