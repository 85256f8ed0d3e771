// Drives the memory of one product without a GPU: workspace_check <name of a check>; exit code 0: it holds.
#include "../paper_2106_16064_amd/csrc/workspace.hpp"

#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <new>

namespace {

int g_held = 0, g_error = 0;                          // blocks handed out; the runtime's last error
int g_current = 0;                                    // the current device; stream s is on device s / 10
bool g_recording = false, g_query_fails = false, g_no_memory = false;
char g_memory[64];

struct Runtime {
    using Stream = int;
    static bool capture_status(Stream, bool& recording) {
        if (g_query_fails) { g_error = 1; return false; }
        recording = g_recording;
        return true;
    }
    static bool device(int& d) { d = g_current; return true; }
    static bool device_of(Stream s, int& d) {
        if (g_query_fails) { g_error = 3; return false; }
        d = s / 10;
        return true;
    }
    static void* allocate(size_t, Stream) {
        if (g_no_memory) { g_error = 2; throw std::bad_alloc(); }
        ++g_held;
        return g_memory;
    }
    static void release(void*) { --g_held; }
    static void forget_error() { g_error = 0; }
};
using Workspace = dgsp::Workspace<Runtime>;

// One block a call, given back with it; none while a graph is recorded.
bool one_block_a_call() {
    {
        Workspace w(1, 0);
        if (Workspace::get(&w, 8) != g_memory || Workspace::get(&w, 8) != nullptr || g_held != 1) return false;
    }
    if (g_held != 0) return false;
    g_recording = true;
    Workspace w(1, 0);
    return Workspace::get(&w, 8) == nullptr && g_held == 0;
}

// A call without memory goes on, and its launches ask for the last error: what the refusal left must be gone.
bool leaves_no_error() {
    Workspace w(1, 0);
    g_query_fails = true;
    if (Workspace::get(&w, 8) != nullptr || g_error != 0) return false;
    g_query_fails = false;
    g_no_memory = true;
    return Workspace::get(&w, 8) == nullptr && g_error == 0 && g_held == 0;
}

// The allocator hands out memory of the current device: a product on another one's stream, or with its operands there, has no
// use for it and may not even reach it.
bool only_on_the_products_gpu() {
    Workspace here(1, 0), stream_elsewhere(11, 0), operands_elsewhere(1, 1), all_elsewhere(11, 1);
    if (Workspace::get(&here, 8) != g_memory) return false;
    for (Workspace* w : {&stream_elsewhere, &operands_elsewhere, &all_elsewhere})
        if (Workspace::get(w, 8) != nullptr) return false;
    g_current = 1;
    return Workspace::get(&all_elsewhere, 8) == g_memory && g_held == 2;
}

}  // namespace

int main(int argc, char** argv) {
    const char* name = argc > 1 ? argv[1] : "";
    if (!strcmp(name, "one_block_a_call")) return one_block_a_call() ? 0 : 1;
    if (!strcmp(name, "leaves_no_error")) return leaves_no_error() ? 0 : 1;
    if (!strcmp(name, "only_on_the_products_gpu")) return only_on_the_products_gpu() ? 0 : 1;
    fprintf(stderr, "unknown check %s\n", name);
    return 2;
}
