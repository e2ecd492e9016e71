// The formation of CG teams (csrc/cg_team_join.h) with threads in the place of
// workgroups: `cus` of them run at a time, as many as there is room for, and a
// workgroup that has a place holds its room until its whole team has met.
// Checked: every run ends, a team is whole or not there at all, teams form
// wherever there is room for one, and none where there is not.
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstdio>
#include <mutex>
#include <random>
#include <thread>
#include <vector>

#define __host__
#define __device__
#include "cg_team_join.h"

using Clock = std::chrono::steady_clock;

struct Room {   // CUs, given out in the order of the workgroups' numbers
    std::mutex mu;
    std::condition_variable cv;
    int free_cus, next = 0;
    explicit Room(int n) : free_cus(n) {}
    void take(int number) {
        std::unique_lock<std::mutex> lk(mu);
        cv.wait(lk, [&] { return next == number && free_cus > 0; });
        ++next;
        --free_cus;
        cv.notify_all();
    }
    void give() {
        std::lock_guard<std::mutex> lk(mu);
        ++free_cus;
        cv.notify_all();
    }
};

struct Word {
    std::atomic<unsigned>& w;
    Clock::time_point until;
    unsigned load() const { return w.load(std::memory_order_relaxed); }
    unsigned cas(unsigned expected, unsigned desired) {
        w.compare_exchange_strong(expected, desired, std::memory_order_relaxed);
        return expected;
    }
    bool expired() const { return Clock::now() >= until; }
    void pause() const { std::this_thread::yield(); }
};

int main() {
    constexpr int SIZE = 8;
    std::mt19937 rng(7);
    int fails = 0;
    for (int run = 0; run < 400; ++run) {
        const int teams = 1 + rng() % 4, blocks = (teams + rng() % 2) * SIZE, cus = 1 + rng() % 20;
        // long: every team that has room comes together; short: any may be cut off
        const bool patient = run % 2 == 0;
        const int us = patient ? (cus >= SIZE ? 20000000 : 2000) : (int)(rng() % 60);
        Room room(cus);
        std::atomic<unsigned> word{0};
        std::vector<std::atomic<int>> met(teams);
        for (auto& m : met) m = 0;
        std::vector<int> place(blocks, -2);
        std::atomic<int> stuck{0};
        std::vector<std::thread> th;
        for (int b = 0; b < blocks; ++b)
            th.emplace_back([&, b] {
                room.take(b);
                Word m{word, Clock::now() + std::chrono::microseconds(us)};
                place[b] = team_join(m, SIZE, teams * SIZE);
                if (place[b] >= 0) {   // meets its team: no room given back before that
                    auto& k = met[place[b] / SIZE];
                    ++k;
                    const auto end = Clock::now() + std::chrono::seconds(60);
                    while (k < SIZE && Clock::now() < end) std::this_thread::yield();
                    if (k < SIZE) ++stuck;
                }
                room.give();
            });
        for (auto& t : th) t.join();
        std::vector<int> seen(teams * SIZE, 0);
        int whole = 0;
        for (int b = 0; b < blocks; ++b) {
            if (place[b] >= teams * SIZE || place[b] == -2) ++fails;
            else if (place[b] >= 0 && ++seen[place[b]] > 1) ++fails;
        }
        for (int t = 0; t < teams; ++t) {
            if (met[t] != 0 && met[t] != SIZE) ++fails;
            whole += met[t] == SIZE;
        }
        if (stuck) ++fails;
        if (cus < SIZE && whole) ++fails;
        if (patient && cus >= SIZE && whole != teams) ++fails;
    }
    std::printf("team formation: %d failures\n", fails);
    return fails ? 1 : 0;
}
