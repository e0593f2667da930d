// Launches whose workgroups wait for each other need all of them on the chip at once.  A cooperative launch sees to that by
// going through a queue of its own, which costs 11 us of an idle GPU before the kernel and 11 us after it.  Here such launches
// of one device run one after another instead: each waits for the one before it, on whatever stream or thread that was.  On
// one stream that is the order they have anyway.  (A kernel of 30 us between two small ones: 45.5 us for the three launched
// plainly, 65.7 us cooperatively, 47.7 us like this; with an event that also writes back to the host's memory 49.8 us.)
//
// What this does not order is a launch of another process, a replayed graph and a cooperative launch of the program's own, so a
// kernel launched here has to finish with whatever workgroups it gets.
#include "internal.hpp"

#include <hip/hip_ext.h>

#include <mutex>

namespace rnn {
namespace {

struct Turn {
    std::mutex mu;
    hipEvent_t done = nullptr;     // end of the device's last such launch
};
constexpr int MAX_DEVICES = 64;
Turn g_turns[MAX_DEVICES];

}  // namespace

hipError_t launch_gang(const void* fn, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t s) {
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    int dev = 0;
    // a captured launch runs when its graph is replayed, after and beside launches that are not known here
    bool plain = hipStreamIsCapturing(s, &capturing) == hipSuccess && capturing == hipStreamCaptureStatusNone &&
                 hipGetDevice(&dev) == hipSuccess && dev < MAX_DEVICES;
    if (plain) {
        Turn& t = g_turns[dev];
        std::lock_guard<std::mutex> lock(t.mu);
        if (!t.done) plain = hipEventCreateWithFlags(&t.done, hipEventDisableTiming | hipEventDisableSystemFence) == hipSuccess;
        else plain = hipStreamWaitEvent(s, t.done, 0) == hipSuccess;
        if (plain) return hipExtLaunchKernel(fn, grid, block, args, lds, s, nullptr, t.done, 0);
    }
    (void)hipGetLastError();
    return hipLaunchCooperativeKernel(fn, grid, block, args, (unsigned)lds, s);
}

}  // namespace rnn
