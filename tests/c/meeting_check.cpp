// Threads as the workgroups of a layer, on the meetings of meeting.h with waits of a few polls, so that some of them give up in nearly
// every round: in the end all have made the same decision, and without a decision to give up all counted the same. Every round ends.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <thread>
#include <vector>

#include "meeting.h"

namespace {
struct HostMem {
    static uint32_t load(const uint32_t* p) { return __atomic_load_n(p, __ATOMIC_SEQ_CST); }
    static uint32_t cas(uint32_t* p, uint32_t was, uint32_t v) {
        __atomic_compare_exchange_n(p, &was, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST);
        return was;
    }
    static void add(uint32_t* p, uint32_t v) { __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST); }
    static void pause() { std::this_thread::yield(); }
};

constexpr int GROUPS = 6, PASSES = 3;
struct Layer {
    uint32_t arrived[PASSES], admits[GROUPS], count[PASSES];
};
struct Result {
    bool lost, counted[PASSES];      // given up; the passes it went beyond
    uint32_t before, total, count[PASSES];
};

void workgroup(Layer& L, int part, int polls, unsigned seed, std::atomic<int>& go, Result& r) {
    HostMem mem;
    std::minstd_rand rnd(seed);
    auto dawdle = [&] { for (unsigned i = rnd() % 4 ? 0 : rnd() % 40; i > 0; --i) std::this_thread::yield(); };
    go.fetch_sub(1);
    while (go.load() > 0) std::this_thread::yield();
    r = Result{};
    for (int p = 0; p < PASSES && !r.lost; ++p) {
        dawdle();
        mem.add(&L.count[p], (uint32_t)(part + 1));
        r.lost = !fg_meet(mem, &L.arrived[p], GROUPS, polls);
        if (r.lost) {
            for (int q = p + 1; q < PASSES; ++q) fg_lost_ahead(mem, &L.arrived[q]);
        } else {
            r.counted[p] = true;
            r.count[p] = mem.load(&L.count[p]);
        }
    }
    dawdle();
    fg_publish(mem, &L.admits[part], r.lost ? FG_GIVEN_UP : (uint32_t)(part + 1));
    for (int q = 0; q < GROUPS && !r.lost; ++q) {
        const uint32_t w = fg_settled(mem, &L.admits[q], polls);
        r.lost = !(w & FG_PUBLISHED) || (w & FG_GIVEN_UP) != 0;
        if (q < part) r.before += w & 0xFFFF;
        r.total += w & 0xFFFF;
    }
}
}  // namespace

int main(int argc, char** argv) {
    const int rounds = argc > 1 ? atoi(argv[1]) : 3000;
    int given_up = 0, whole = 0, wrong = 0;
    for (int round = 0; round < rounds; ++round) {
        Layer L{};
        Result r[GROUPS];
        std::atomic<int> go(GROUPS);
        std::vector<std::thread> threads;
        const int polls = round % 3 == 0 ? 1 << 20 : 1 + round % 60;
        for (int g = 0; g < GROUPS; ++g) threads.emplace_back(workgroup, std::ref(L), g, polls, (unsigned)(round * GROUPS + g + 1), std::ref(go), std::ref(r[g]));
        for (auto& t : threads) t.join();
        bool fine = true;
        for (int g = 0; g < GROUPS; ++g) {
            fine = fine && r[g].lost == r[0].lost && (polls < 1 << 20 || !r[g].lost);
            for (int p = 0; p < PASSES; ++p) fine = fine && (!r[g].counted[p] || r[g].count[p] == GROUPS * (GROUPS + 1) / 2);
            if (!r[g].lost) fine = fine && r[g].total == GROUPS * (GROUPS + 1) / 2 && r[g].before == (uint32_t)(g * (g + 1) / 2);
        }
        wrong += !fine;
        r[0].lost ? ++given_up : ++whole;
    }
    printf("%d rounds given up, %d not, %d wrong\n", given_up, whole, wrong);
    return wrong || !whole || !given_up;
}
