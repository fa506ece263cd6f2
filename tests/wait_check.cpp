// Two threads on one core that hand a word to and fro: polled by loads alone
// each handover waits for the end of a time slice, with Polling it does not.
#include <sched.h>

#include <atomic>
#include <chrono>
#include <cstdio>
#include <thread>

#include "../paper_1204_2586_amd/csrc/host/wait.hpp"

struct Loads {
    void pause() {}
};

template <typename P>
static double handovers(int count)
{
    std::atomic<int> word{0};
    auto side = [&](int mine) {
        for (int i = mine; i < 2 * count; i += 2) {
            P poll;
            while (word.load(std::memory_order_relaxed) != i) poll.pause();
            word.store(i + 1, std::memory_order_relaxed);
        }
    };
    const auto t0 = std::chrono::steady_clock::now();
    std::thread other(side, 1);
    side(0);
    other.join();
    return std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
}

int main()
{
    // a core that nothing else uses: the first of a few that shows it
    cpu_set_t all, one;
    sched_getaffinity(0, sizeof(all), &all);
    for (int cpu = 0, tried = 0; cpu < CPU_SETSIZE && tried < 8; cpu++) {
        if (!CPU_ISSET(cpu, &all)) continue;
        tried++;
        CPU_ZERO(&one);
        CPU_SET(cpu, &one);
        if (sched_setaffinity(0, sizeof(one), &one) != 0) return 2;
        const double loads = handovers<Loads>(100), polling = handovers<auxp::Polling>(100);
        std::printf("core %d: %.3f ms by loads, %.3f ms\n", cpu, 1e3 * loads, 1e3 * polling);
        if (polling < loads / 4) return 0;
    }
    return 1;
}
