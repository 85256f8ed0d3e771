// Drives the pool of statistics scratch without a GPU: stat_pool_check <name of a check>; exit code 0: it holds.
#include "../paper_2106_16064_amd/csrc/stat_pool.hpp"

#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>
#include <thread>
#include <vector>

namespace {

struct Area { int words[4]; };
thread_local int t_device = 0;
bool g_no_memory = false;
Area g_areas[dgsp::kMaxDevices][dgsp::kStatSlots];

struct Runtime {
    static bool device(int& d) { d = t_device; return true; }
    static Area* scratch() { return g_areas[t_device]; }
    static void* pinned(size_t bytes) { return g_no_memory ? nullptr : malloc(bytes); }
};
using Pool = dgsp::StatPool<Area, Runtime>;

bool within(int ms, const std::atomic<int>& n, int want) {
    for (int i = 0; i < ms && n < want; ++i) std::this_thread::sleep_for(std::chrono::milliseconds(1));
    return n >= want;
}

// A place that becomes free on one GPU goes to a call that waits for that GPU, whoever else waits.
bool wakes_the_right_gpu() {
    static Pool pool;
    std::vector<Pool::Slot> held[2];
    std::set<const Area*> seen;
    for (int d = 0; d < 2; ++d)
        for (int i = 0; i < dgsp::kStatSlots; ++i) {
            t_device = d;
            Pool::Slot s;
            if (!pool.take(s, false) || s.device != d || !seen.insert(s.scratch).second) return false;
            held[d].push_back(s);
        }
    static std::atomic<int> done[2];
    const auto call = [](int d) {
        t_device = d;
        Pool::Slot s;
        pool.take(s, false);
        ++done[d];
        pool.give_back(s);
    };
    std::vector<std::thread> threads;
    for (int i = 0; i < 8; ++i) threads.emplace_back(call, 0);
    std::this_thread::sleep_for(std::chrono::milliseconds(200));       // these wait first
    threads.emplace_back(call, 1);
    std::this_thread::sleep_for(std::chrono::milliseconds(200));
    pool.give_back(held[1].back());
    const bool ok = within(5000, done[1], 1) && done[0] == 0;
    if (!ok) std::_Exit(1);                                            // a call that is never woken cannot be joined
    for (const auto& s : held[0]) pool.give_back(s);
    for (auto& t : threads) t.join();
    return done[0] == 8;
}

// Pinned memory that one call could not get is asked for again by the next.
bool asks_again_for_host_words() {
    static Pool pool;
    Pool::Slot s;
    g_no_memory = true;
    if (!pool.take(s, true) || s.host) return false;
    pool.give_back(s);
    g_no_memory = false;
    if (!pool.take(s, true) || !s.host || s.host[0] != 0) return false;
    pool.give_back(s);
    return pool.take(s, false) && !s.host;
}

}  // namespace

int main(int argc, char** argv) {
    const char* name = argc > 1 ? argv[1] : "";
    if (!strcmp(name, "wakes_the_right_gpu")) return wakes_the_right_gpu() ? 0 : 1;
    if (!strcmp(name, "asks_again_for_host_words")) return asks_again_for_host_words() ? 0 : 1;
    fprintf(stderr, "unknown check %s\n", name);
    return 2;
}
