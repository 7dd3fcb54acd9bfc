// Checks of LaunchGate on host threads; prints "ok" or what failed.
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>

#include "launch_gate.hpp"

using stag::LaunchGate;
using stag::LaunchPass;

static void check(bool ok, const char *what)
{
    if (!ok) {
        std::printf("failed: %s\n", what);
        std::exit(1);
    }
}

static bool soon(const std::atomic<int> &v, int want)
{
    for (int i = 0; i < 2000 && v.load() != want; ++i)
        std::this_thread::sleep_for(std::chrono::milliseconds(1));
    return v.load() == want;
}

int main()
{
    {  // grids that fit together are in flight together
        LaunchGate g;
        std::atomic<int> in{0}, go{0};
        std::vector<std::thread> t;
        for (int i = 0; i < 16; ++i)
            t.emplace_back([&] {
                LaunchPass p(g, 16, 256);
                in.fetch_add(1);
                while (!go.load())
                    std::this_thread::yield();
            });
        check(soon(in, 16), "16 grids of 16 blocks are admitted together to 256");
        std::atomic<int> late{0};
        std::thread more([&] {
            LaunchPass p(g, 1, 256);
            late = 1;
        });
        std::this_thread::sleep_for(std::chrono::milliseconds(50));
        check(late.load() == 0, "a 17th waits");
        go = 1;
        for (auto &x : t)
            x.join();
        more.join();
        check(late.load() == 1, "... and follows when they have left");
    }
    {  // the limit holds, a large grid is not passed for ever, one beyond the limit runs alone
        LaunchGate g;
        std::atomic<int> used{0}, worst{0}, large{0};
        std::vector<std::thread> t;
        for (int i = 0; i < 8; ++i)
            t.emplace_back([&, i] {
                for (int k = 0; k < 200; ++k) {
                    const int n = i == 7 ? (k % 10 ? 256 : 300) : 40 + 7 * i;
                    LaunchPass p(g, n, 256);
                    const int u = used.fetch_add(n) + n;
                    check(u <= 256 || u == n, "the grids in flight exceed the limit");
                    int w = worst.load();
                    while (u > w && !worst.compare_exchange_weak(w, u)) {}
                    large += i == 7;
                    used.fetch_sub(n);
                }
            });
        for (auto &x : t)
            x.join();
        check(large.load() == 200, "the large grids ran");
    }
    std::puts("ok");
    return 0;
}
