// Places for the statistics calls that are under way on a GPU (host code only, so that it can be tried without one).
//
// A call owns one scratch area from launch to result; further ones wait for a place on their own GPU.
#pragma once

#include <condition_variable>
#include <cstddef>
#include <mutex>

namespace dgsp {

constexpr int kStatSlots = 8;          // per GPU
constexpr int kMaxDevices = 64;

// `Runtime` asks the GPU runtime about the current device: bool device(int&), Scratch* scratch() with kStatSlots areas that
// stay where they are, void* pinned(size_t) with host memory that the GPU writes (nullptr: there is none).
template <typename Scratch, typename Runtime>
class StatPool {
public:
    struct Slot {
        int device = -1, index = -1;
        Scratch* scratch = nullptr;
        unsigned long long* host = nullptr;         // result words the GPU writes (nullptr: not asked for, or no pinned memory)
        unsigned long long ticket = 0;
    };
    // false: no current device, or its scratch has no address
    bool take(Slot& slot, bool with_host) {
        int dev = -1;
        if (!Runtime::device(dev) || dev < 0 || dev >= kMaxDevices) return false;
        std::unique_lock<std::mutex> lock(mu_);
        Device& d = devices_[dev];
        if (!d.scratch) {
            d.scratch = Runtime::scratch();
            if (!d.scratch) return false;
        }
        if (with_host && !d.host) {                 // a refusal may be passing (a capture elsewhere): the next call asks again
            d.host = static_cast<unsigned long long*>(Runtime::pinned(kStatSlots * kHostWords * sizeof(unsigned long long)));
            for (int i = 0; d.host && i < kStatSlots * kHostWords; ++i) d.host[i] = 0;
        }
        d.free.wait(lock, [&] { return d.taken != (1u << kStatSlots) - 1u; });
        int i = 0;
        while (d.taken >> i & 1u) ++i;
        d.taken |= 1u << i;
        slot.device = dev;
        slot.index = i;
        slot.scratch = d.scratch + i;
        slot.host = with_host && d.host ? d.host + i * kHostWords : nullptr;
        slot.ticket = ++ticket_;
        return true;
    }
    void give_back(const Slot& slot) {
        std::lock_guard<std::mutex> lock(mu_);
        Device& d = devices_[slot.device];
        d.taken &= ~(1u << slot.index);
        d.free.notify_one();                        // whoever waits here waits for this GPU
    }

private:
    static constexpr int kHostWords = 16;
    struct Device {
        Scratch* scratch = nullptr;
        unsigned long long* host = nullptr;
        unsigned taken = 0;
        std::condition_variable free;
    };
    std::mutex mu_;
    Device devices_[kMaxDevices];
    unsigned long long ticket_ = 0;
};

}  // namespace dgsp
