// Scheduler::wait (paper_2404_01817_amd/csrc/scheduler.h) on the CPU, with an
// executor whose batches end after a fixed time: timeouts from none to the
// largest number, several waiters, launch errors, requests cancelled by a
// shutdown, and a scheduler destroyed under its waiters.  Argument: which
// check to run.  Exit status 0 when it held.
#include <atomic>
#include <chrono>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <limits>
#include <mutex>
#include <thread>
#include <vector>

#include "scheduler.h"

using neat::sched::Executor;
using neat::sched::Result;
using neat::sched::Scheduler;

namespace {

std::atomic<int> g_fail{0};

#define CHECK(c)                                                               \
    do {                                                                       \
        if (!(c)) {                                                            \
            std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #c); \
            g_fail = 1;                                                        \
        }                                                                      \
    } while (0)

double now_ms() {
    return std::chrono::duration<double, std::milli>(
               std::chrono::steady_clock::now().time_since_epoch())
        .count();
}

struct TimedExec : Executor<int> {
    std::mutex m;
    std::vector<double> end;
    const double ms;
    const int fail_every;
    int launches = 0;
    TimedExec(int slots, double ms_, int fail_every_ = 0)
        : end(slots, -1.0), ms(ms_), fail_every(fail_every_) {}
    int launch(int k, const std::vector<const int *> &) override {
        std::lock_guard<std::mutex> lk(m);
        if (fail_every > 0 && ++launches % fail_every == 0) return NEAT_E_HIP;
        end[k] = now_ms() + ms;
        return NEAT_OK;
    }
    bool finished(int k) override {
        std::lock_guard<std::mutex> lk(m);
        return end[k] < now_ms();
    }
    void drain(int) override {}
};

uint64_t submit(Scheduler<int> &s, uint64_t tag) {
    uint64_t tk = 0;
    CHECK(s.submit((int)tag, 1, 1, tag, false, &tk) == NEAT_OK);
    return tk;
}

// Every timeout that is long enough brings the result of a request of 20 ms.
void timeouts() {
    TimedExec ex(1, 20.0);
    Scheduler<int> s(&ex, 1, 1000, 4, 5);
    for (int64_t us : {(int64_t)1000000, (int64_t)1000000000, (int64_t)8000000000000000,
                       std::numeric_limits<int64_t>::max()}) {
        const uint64_t tk = submit(s, 7);
        Result r;
        const int rc = s.wait(tk, us, &r);
        CHECK(rc == NEAT_OK && r.tag == 7 && r.status == NEAT_OK);
        CHECK(s.wait(tk, us, &r) == NEAT_E_UNKNOWN_TICKET);  // forgotten
    }
    TimedExec slow(1, 400.0);
    Scheduler<int> s2(&slow, 1, 1000, 4, 5);
    const uint64_t tk = submit(s2, 8);
    const double t0 = now_ms();
    Result r;
    for (int64_t us : {(int64_t)0, (int64_t)-1, std::numeric_limits<int64_t>::min()})
        CHECK(s2.wait(tk, us, &r) == NEAT_PENDING);
    CHECK(now_ms() - t0 < 200.0);  // at once
    CHECK(s2.wait(tk, 3000, &r) == NEAT_PENDING && now_ms() - t0 >= 3.0);
    CHECK(s2.wait(tk, 10000000, nullptr) == NEAT_OK && now_ms() - t0 < 5000.0);
    CHECK(s2.wait(tk + 99, 1000, &r) == NEAT_E_UNKNOWN_TICKET);
}

// Several threads wait for tickets of their own, some of failed launches, and
// all of them for one ticket, which one of them gets.
void waiters() {
    TimedExec ex(2, 0.5, 5);
    Scheduler<int> s(&ex, 2, 1000, 3, 5, 50, true);
    std::atomic<int> failed{0};
    std::vector<std::thread> th;
    for (int t = 0; t < 8; ++t)
        th.emplace_back([&, t] {
            for (int i = 0; i < 40; ++i) {
                const uint64_t tk = submit(s, (uint64_t)(100 * t + i));
                Result r;
                CHECK(s.wait(tk, std::numeric_limits<int64_t>::max(), &r) == NEAT_OK);
                CHECK(r.tag == (uint64_t)(100 * t + i));
                CHECK(r.status == NEAT_OK || r.status == NEAT_E_HIP);
                failed += r.status == NEAT_E_HIP;
            }
        });
    for (auto &x : th) x.join();
    CHECK(failed.load() > 0);
    th.clear();
    std::atomic<int> got{0}, gone{0};
    uint64_t tk = submit(s, 1);
    for (int t = 0; t < 8; ++t)
        th.emplace_back([&] {
            Result r;
            const int rc = s.wait(tk, 10000000, &r);
            CHECK(rc == NEAT_OK || rc == NEAT_E_UNKNOWN_TICKET);
            (rc == NEAT_OK ? got : gone)++;
        });
    for (auto &x : th) x.join();
    CHECK(got.load() == 1 && gone.load() == 7);
}

// Waiters of running and queued requests when the scheduler is shut down and
// destroyed: each leaves with its result or NEAT_E_SHUTDOWN in it, and before
// the memory goes.
void destroyed() {
    for (int round = 0; round < 8; ++round) {
        constexpr int W = 48;
        TimedExec ex(1, 60.0);
        auto *s = new Scheduler<int>(&ex, 1, 1000, 4, 5);
        std::vector<uint64_t> tk;
        for (int i = 0; i < W; ++i) tk.push_back(submit(*s, (uint64_t)i));
        std::atomic<int> done{0}, cancelled{0};
        std::vector<std::thread> th;
        for (int i = 0; i < W; ++i)
            th.emplace_back([&, i] {
                Result r;
                CHECK(s->wait(tk[i], std::numeric_limits<int64_t>::max(), &r) == NEAT_OK);
                CHECK(r.tag == (uint64_t)i);
                (r.status == NEAT_E_SHUTDOWN ? cancelled : done)++;
            });
        // all of them asleep, or done (the first batches may end meanwhile)
        while (s->waiting() + done.load() < W) std::this_thread::yield();
        delete s;
        for (auto &x : th) x.join();
        CHECK(done.load() + cancelled.load() == W);
    }
}

}  // namespace

int main(int argc, char **argv) {
    const char *what = argc > 1 ? argv[1] : "";
    if (!std::strcmp(what, "timeouts")) timeouts();
    else if (!std::strcmp(what, "waiters")) waiters();
    else if (!std::strcmp(what, "destroyed")) destroyed();
    else return 2;
    if (g_fail.load() == 0) std::printf("%s: checks passed\n", what);
    return g_fail.load();
}
