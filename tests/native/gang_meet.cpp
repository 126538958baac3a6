// Host-only run of gang_meet (built and run by tests/test_gang_meet.py; no kernel is
// launched): threads stand for the workgroups that other work leaves on the GPU.  They
// pull the tickets of gangs larger and smaller than their number, as k_batch does, and
// every item must be solved exactly once, by its whole gang or by its first part alone.
#include <atomic>
#include <chrono>
#include <cstdio>
#include <thread>
#include <vector>

#include "solve.h"

using namespace sssp;

struct Item {
    int members;
    uint32_t word = 0;
    std::atomic<int> arrived{0}, alone{0}, left{0}, strays{0};
};

static bool run(int workers, const std::vector<int>& gangs, long long limit_us, bool late) {
    std::vector<Item> items(gangs.size());
    std::vector<std::pair<int, int>> tickets;
    for (size_t i = 0; i < gangs.size(); ++i) {
        items[i].members = gangs[i];
        for (int p = 0; p < gangs[i]; ++p) tickets.push_back({(int)i, p});
    }
    std::atomic<size_t> next{0};
    auto now = [] {
        return (long long)std::chrono::duration_cast<std::chrono::microseconds>(
                   std::chrono::steady_clock::now().time_since_epoch()).count();
    };
    auto work = [&](int id) {
        for (size_t t; (t = next.fetch_add(1)) < tickets.size();) {
            Item& it = items[tickets[t].first];
            const int part = tickets[t].second;
            if (late && (t * 7 + id) % 5 == 0) std::this_thread::sleep_for(std::chrono::microseconds(3 * limit_us / 2));
            if (gang_meet(&it.word, part, (uint32_t)it.members, limit_us, now, [] { std::this_thread::yield(); })) {
                it.arrived.fetch_add(1);
                while (it.arrived.load() < it.members) std::this_thread::yield();  // the gang's exchanges
            } else if (part == 0) {
                it.alone.fetch_add(1);
            } else {
                it.strays.fetch_add(1);
            }
            it.left.fetch_add(1);
        }
    };
    std::vector<std::thread> pool;
    for (int i = 0; i < workers; ++i) pool.emplace_back(work, i);
    for (auto& th : pool) th.join();
    int together = 0, alone = 0;
    for (const Item& it : items) {
        const bool whole = it.arrived == it.members && it.alone == 0 && it.strays == 0;
        const bool single = it.arrived == 0 && it.alone == 1 && it.strays == it.members - 1;
        if (it.left != it.members || !(whole || single)) {
            std::fprintf(stderr, "a gang of %d: %d together, %d alone, %d strays\n", it.members, it.arrived.load(),
                         it.alone.load(), it.strays.load());
            return false;
        }
        if (it.members > workers && whole) {
            std::fprintf(stderr, "a gang of %d met on %d workgroups\n", it.members, workers);
            return false;
        }
        together += whole;
        alone += single;
    }
    std::printf("%d workers: %d gangs together, %d alone\n", workers, together, alone);
    return true;
}

int main() {
    bool ok = true;
    for (int workers : {1, 2, 3, 5, 8})
        for (bool late : {false, true})
            ok = ok && run(workers, {6, 6, 4, 4, 3, 3, 2, 2, 2, 2, 8, 8, 2, 3}, 2000, late);
    if (!ok) return 1;
    std::printf("gangs ok\n");
    return 0;
}
