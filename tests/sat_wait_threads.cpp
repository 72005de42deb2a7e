// The steps of hb_sat2d's grid-wide wait (csrc/sat_wait.hpp, as the kernel compiles them) with threads as workgroups, of which only
// some run at a time.  Arguments: launches | words, workgroups, of the first group, that run at once, wait limit, polls before a
// workgroup offers to clear, seed.
#define __device__
#define __forceinline__ inline
#include "sat_wait.hpp"

#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <mutex>
#include <random>
#include <thread>
#include <vector>

static thread_local std::minstd_rand t_rng;
static bool g_delays = true;

struct HostMem {
    static void delay() {
        if (!g_delays) return;
        const unsigned r = t_rng() % 64;
        if (r == 0) std::this_thread::sleep_for(std::chrono::microseconds(t_rng() % 200));
        else if (r < 8) std::this_thread::yield();
    }
    template <class T> static T load(const T* p) { delay(); return __atomic_load_n(p, __ATOMIC_SEQ_CST); }
    template <class T> static void store(T* p, T v) { delay(); __atomic_store_n(p, v, __ATOMIC_SEQ_CST); }
    static unsigned add(unsigned* p) { delay(); return __atomic_add_fetch(p, 1u, __ATOMIC_SEQ_CST); }
    template <class T> static T exchange(T* p, T v) { delay(); return __atomic_exchange_n(p, v, __ATOMIC_SEQ_CST); }
    static bool claim(unsigned* p) {
        delay();
        unsigned expect = 1u;
        return __atomic_compare_exchange_n(p, &expect, 2u, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST);
    }
    static void performed() { __atomic_thread_fence(__ATOMIC_SEQ_CST); }
    static void pause() { std::this_thread::yield(); }
};
using Wait = hb::SatWait<HostMem>;
using hb::SatSync;

struct Launch {
    SatSync* S;
    int nwg, first, wait_limit, claim_polls;
    unsigned long long call;
    bool alone;                                           // nobody else writes to the words
    std::vector<std::atomic<int>> published, finished;
    std::atomic<int> early{0};
    std::mutex mu;
    std::condition_variable cv;
    int slots;
    Launch(SatSync* s, int n, int f, int slots_, int limit, int claim, unsigned long long c, bool alone_)
        : S(s), nwg(n), first(f), wait_limit(limit), claim_polls(claim), call(c), alone(alone_), published(n), finished(n), slots(slots_) {}
    void finish(int r) {
        for (int q = 0; q < (r < first ? first : nwg); ++q)
            if (!published[q]) early = 1;
        finished[r]++;
    }
    void workgroup(int wg, unsigned seed) {
        t_rng.seed(seed);
        {
            std::unique_lock<std::mutex> lock(mu);
            cv.wait(lock, [&] { return slots > 0; });
            --slots;
        }
        run(wg);
        {
            std::lock_guard<std::mutex> lock(mu);
            ++slots;
        }
        cv.notify_one();
    }
    void run(int wg) {
        if (wg == 0 && Wait::take(S, call)) {
            Wait::clear(S, nwg, 0, 1);
            Wait::set_ready(S, call, 0, 1);
        }
        published[wg] = 1;
        const int state = Wait::arrive(S, wg, nwg, first, call, wait_limit, claim_polls);
        if (state == 0) return;
        const unsigned late = HostMem::load(&S->late[0]);
        finish(wg);
        if (late == 0) return;
        const int nscan = state == 2 ? nwg : first;
        for (bool found = true; found;) {
            found = false;
            for (int r = 0; r < nscan && !found; ++r)
                if (HostMem::load(&S->todo[r]) == 1u && HostMem::claim(&S->todo[r])) {
                    finish(r);
                    found = true;
                }
        }
    }
    void start(std::vector<std::thread>& threads, std::minstd_rand& rng) {
        std::vector<int> order(nwg);
        for (int i = 0; i < nwg; ++i) order[i] = i;
        std::shuffle(order.begin(), order.end(), rng);
        for (int wg : order) threads.emplace_back(&Launch::workgroup, this, wg, (unsigned)rng());
    }
    int check() const {
        if (early) return puts("a region finished before those it reads were published"), 1;
        for (int r = 0; r < nwg; ++r)
            if (!finished[r]) return printf("region %d unfinished\n", r), 1;
        for (int i = 0; i < SatSync::kGo; ++i)
            if (*Wait::ready(S, i) != 0) return puts("ready left behind"), 1;
        if (*Wait::claim(S) != 0) return puts("claim left behind"), 1;
        return 0;
    }
};

int main(int argc, char** argv) {
    if (argc != 8) return 2;
    const int nwg = atoi(argv[2]), first = atoi(argv[3]), slots = atoi(argv[4]), limit = atoi(argv[5]), claim = atoi(argv[6]);
    std::minstd_rand rng(atoi(argv[7]) + 1);
    static SatSync S;
    unsigned* const words = reinterpret_cast<unsigned*>(&S);
    if (!strcmp(argv[1], "launches")) {
        // numbers of their own, replays of one, words as the last launch left them or anything
        for (unsigned long long call : {77ull, 78ull, 78ull, 78ull, 79ull, 78ull}) {
            if (call == 79 || rng() % 2)
                for (size_t i = 0; i < sizeof(S) / 4; ++i) words[i] = rng() % 3 ? (unsigned)rng() : 1u;
            Launch l(&S, nwg, first, slots, limit, claim, call, true);
            std::vector<std::thread> threads;
            l.start(threads, rng);
            for (auto& t : threads) t.join();
            if (int bad = l.check()) return bad;
        }
        return puts("ok"), 0;
    }
    // Words that someone else writes to: `claim` holds this launch's number and `ready` never does.  And two launches at once.
    g_delays = false;
    *Wait::claim(&S) = 5;
    if (Wait::arrive(&S, 1, nwg, first, 5, limit, claim) != 0) return puts("arrived without ready"), 1;
    Launch a(&S, nwg, first, slots, limit, claim, 6, false), b(&S, nwg, first, slots, limit, claim, 7, false);
    std::vector<std::thread> threads;
    a.start(threads, rng);
    b.start(threads, rng);
    for (auto& t : threads) t.join();
    return puts("ok"), 0;
}
