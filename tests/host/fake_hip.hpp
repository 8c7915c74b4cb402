// What the host tests read and set of the HIP runtime they run on.
#pragma once
#include <pthread.h>

#include <cstddef>
#include <cstdint>

struct FakeHip {
    size_t total = (size_t)288 << 30;   // the device's memory
    size_t used = 0, peak = 0;
    long mallocs = 0, frees = 0;
    size_t watch = 0;
    long watched = 0;                   // allocations of `watch` bytes
    long frees_elsewhere = 0;           // hipFree by another thread than main_thread
    long streams_made = 0, streams_destroyed = 0;
    long faults = 0;                    // uses of what is no longer there
    pthread_t main_thread = pthread_self();
};
FakeHip& fake_hip();
extern thread_local int fake_hip_inside;   // calls of the runtime this thread is in
