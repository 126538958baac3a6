// Host-only model of how an exchange's result passes through LDS (built and run by
// tests/test_result_slots.py; no kernel is launched).  In a round in which a narrow
// slice reads no row, the workgroup has one barrier, that of read_records: wave 0
// stores the result, every wave passes the barrier, and each reads the result when
// its turn comes, wave 0 going straight on to the next exchange.  This program runs
// every order of the two waves' steps over a few exchanges with as many slots as
// SharedSolve holds and checks that a wave always reads the exchange it is at.
#include <cstdio>
#include <type_traits>

#include "solve.h"

using namespace sssp;

constexpr int kExchanges = 5;
constexpr int kSlots =
    std::extent<decltype(SharedSolve<1024>::res)>::value ? std::extent<decltype(SharedSolve<1024>::res)>::value : 1;

// Step of a wave at exchange t: store (wave 0 only), wait at the barrier, read.
enum Step { kStore, kWait, kRead };
struct Wave {
    int t;
    Step step;
};

struct Model {
    int slot[kSlots];
    Wave w[2];
};

static long states = 0;

static bool run(const Model& m) {
    ++states;
    bool ok = true;
    for (int i = 0; i < 2; ++i) {
        const Wave& w = m.w[i];
        if (w.t > kExchanges) continue;
        Model n = m;
        if (w.step == kStore) {
            if (i == 0) n.slot[w.t % kSlots] = w.t;
            n.w[i].step = kWait;
        } else if (w.step == kWait) {
            // the barrier opens when the other wave is there too; it then reads first or second
            const Wave& o = m.w[1 - i];
            if (o.t < w.t || (o.t == w.t && o.step == kStore)) continue;
            n.w[i].step = kRead;
        } else {
            if (m.slot[w.t % kSlots] != w.t) {
                std::fprintf(stderr, "wave %d at exchange %d reads the result of exchange %d\n", i, w.t,
                             m.slot[w.t % kSlots]);
                return false;
            }
            n.w[i] = Wave{w.t + 1, kStore};
        }
        ok = run(n) && ok;
        if (!ok) return false;
    }
    return ok;
}

int main() {
    Model m{};
    m.w[0] = m.w[1] = Wave{1, kStore};
    if (!run(m)) return 1;
    if (std::extent<decltype(SharedSolve<1024>::res_need)>::value != (kSlots > 1 ? kSlots : 0)) {
        std::fprintf(stderr, "res and res_need have different numbers of slots\n");
        return 1;
    }
    std::printf("result slots ok (%d slots, %ld states)\n", kSlots, states);
    return 0;
}
