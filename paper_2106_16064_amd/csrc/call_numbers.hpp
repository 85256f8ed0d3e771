// Numbers by which calls tell their words in used memory from anybody else's (shared_rows.hpp; host code only).
//
// Even, and no other call's of the process and the copy of the library; those count from a random number on each, so that
// two of them meet with a chance of 2^-62 a word.  Nothing here throws: the callers are C functions.
#pragma once

#include <sys/random.h>
#include <unistd.h>

#include <atomic>
#include <chrono>
#include <cstddef>
#include <cstdint>

#include "shared_rows.hpp"

namespace dgsp {

// `fill(p, bytes)`: random bytes, false if there are none to have.  Then the time, the process and where its memory lies have to do.
template <typename Fill>
RowWord first_call_number(Fill&& fill) noexcept {
    RowWord number = 0;
    if (!fill(&number, sizeof(number))) {
        number = (RowWord)std::chrono::steady_clock::now().time_since_epoch().count() * 0x9e3779b97f4a7c15ull;
        number ^= (RowWord)getpid() << 40 ^ (RowWord)reinterpret_cast<uintptr_t>(&number) << 20;
    }
    return number & ~1ull;
}

inline RowWord next_call_number() noexcept {
    static std::atomic<RowWord> next{first_call_number([](void* p, size_t bytes) { return getrandom(p, bytes, GRND_NONBLOCK) == (ssize_t)bytes; })};
    return next.fetch_add(2, std::memory_order_relaxed);
}

}  // namespace dgsp
