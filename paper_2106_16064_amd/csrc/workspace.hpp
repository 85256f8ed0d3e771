// Device memory for one product (host code only, so that it can be tried without a GPU).
#pragma once

#include <cstddef>

namespace dgsp {

// Memory of the stream that the product runs on: given back when the call returns, it is handed out again to work that comes
// later on that stream only.  None while the stream records a graph, whose replays the allocator may not know of, and none
// unless the stream and the operands are on the current GPU: what the allocator hands out is memory of that one.
//
// `Runtime` asks the GPU runtime and the allocator: bool capture_status(Stream, bool& recording), bool device(int&) (the current
// one) and bool device_of(Stream, int&), false on an error that they leave as the runtime's last one; void* allocate(size_t,
// Stream), memory of the current GPU, which may throw; void release(void*); void forget_error().
template <typename Runtime>
class Workspace {
public:
    using Stream = typename Runtime::Stream;
    Workspace(Stream stream, int device) : stream_(stream), device_(device) {}
    Workspace(const Workspace&) = delete;
    Workspace& operator=(const Workspace&) = delete;
    ~Workspace() {
        if (memory_) Runtime::release(memory_);
    }
    static void* get(void* context, size_t bytes) {
        auto* self = static_cast<Workspace*>(context);
        if (self->memory_ || !self->usable()) return nullptr;
        try {
            self->memory_ = Runtime::allocate(bytes, self->stream_);
        } catch (...) {                            // out of memory: the product does without
            Runtime::forget_error();
            self->memory_ = nullptr;
        }
        return self->memory_;
    }

private:
    bool usable() const {
        bool recording = false;
        int current = -1, on = -1;
        if (Runtime::capture_status(stream_, recording) && Runtime::device(current) && Runtime::device_of(stream_, on))
            return !recording && current == on && current == device_;
        Runtime::forget_error();                   // the product's launches ask for the last error
        return false;
    }
    Stream stream_;
    int device_;                                   // of the operands
    void* memory_ = nullptr;
};

}  // namespace dgsp
