// Host check of lp_layout_trial.h: set-ups on several threads share one trial, its choice and its
// times, and never run two at once.
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>

#include "lp_layout_trial.h"

#define CHECK(c) \
    do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)

int main() {
    for (int round = 0; round < 20; ++round) {
        lpgpu::SharedLayoutTrial shared;
        std::atomic<int> runs{0}, inside{0}, ready{0};
        constexpr int kThreads = 6;
        std::vector<lpgpu::LayoutTrial> got(kThreads);
        std::vector<std::thread> threads;
        for (int i = 0; i < kThreads; ++i)
            threads.emplace_back([&, i] {
                ready++;
                while (ready < kThreads) std::this_thread::yield();
                const int rc = shared.get(&got[i], [&](lpgpu::LayoutTrial* t) {
                    CHECK(inside++ == 0);
                    const int k = runs++;
                    std::this_thread::sleep_for(std::chrono::milliseconds(2));
                    t->us[0] = 100.0 + 3 * k + round;
                    t->us[1] = 100.0 + 5 * k;
                    t->layout = t->us[1] < t->us[0] ? 1 : 0;
                    inside--;
                    return 0;
                });
                CHECK(rc == 0);
            });
        for (auto& t : threads) t.join();
        CHECK(runs == 1);
        for (const auto& g : got) {
            CHECK(g.layout == (round > 0 ? 1 : 0));
            CHECK(g.us[0] == 100.0 + round && g.us[1] == 100.0);
        }
    }
    // a failed trial is reported and made again by the next set-up
    lpgpu::SharedLayoutTrial shared;
    lpgpu::LayoutTrial out;
    CHECK(shared.get(&out, [](lpgpu::LayoutTrial*) { return 7; }) == 7);
    CHECK(shared.get(&out, [](lpgpu::LayoutTrial* t) { return t->layout = 1, 0; }) == 0 && out.layout == 1);
    std::puts("ok");
    return 0;
}
