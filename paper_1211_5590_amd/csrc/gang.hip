// Launches whose workgroups wait for each other need all of them on the chip at once, so two of them must not share it.  All of the
// library's but the plain one-window launch, whose caller vouches for an idle GPU, therefore take turns on a device: each waits for
// the one before it, on whatever stream or thread that was.  On one stream that is the order they have anyway.
//
// A cooperative launch is sure of its place beside other work too, but goes through a queue of its own, which costs 11 us of an idle
// GPU before the kernel and 11 us after it; it is not ordered with launches that are not cooperative.  A kernel that finishes with
// whatever workgroups it gets is launched plainly instead.  (A kernel of 30 us between two small ones: 45.5 us for the three launched
// plainly, 65.7 us cooperatively, 47.7 us like this; with an event that also writes back to the host's memory 49.8 us.
// The turn costs a cooperative launch 2 us: 50 examples of a classifier 274.9 -> 276.8 us, a stream of 200 windows 3268 -> 3271.)
//
// What this does not order is a launch of another process, a replayed graph and a cooperative launch of the program's own.
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

hipError_t launch_gang(const void* fn, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t s, bool finishes_with_any) {
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    int dev = 0;
    // a captured launch runs when its graph is replayed, after and beside launches that are not known here
    bool turns = hipStreamIsCapturing(s, &capturing) == hipSuccess && capturing == hipStreamCaptureStatusNone &&
                 hipGetDevice(&dev) == hipSuccess && dev < MAX_DEVICES;
    if (turns) {
        Turn& t = g_turns[dev];
        std::lock_guard<std::mutex> lock(t.mu);
        if (!t.done) turns = hipEventCreateWithFlags(&t.done, hipEventDisableTiming | hipEventDisableSystemFence) == hipSuccess;
        else turns = hipStreamWaitEvent(s, t.done, 0) == hipSuccess;
        if (turns) {
            if (finishes_with_any) return hipExtLaunchKernel(fn, grid, block, args, lds, s, nullptr, t.done, 0);
            const hipError_t e = hipLaunchCooperativeKernel(fn, grid, block, args, (unsigned)lds, s);
            return e == hipSuccess ? hipEventRecord(t.done, s) : e;
        }
    }
    (void)hipGetLastError();
    return hipLaunchCooperativeKernel(fn, grid, block, args, (unsigned)lds, s);
}

}  // namespace rnn
