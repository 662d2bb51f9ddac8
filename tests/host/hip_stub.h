// A stand-in for the HIP runtime and the kernels, for tests of the library's
// host code without a GPU: every stream executes its work on a thread of its
// own, and the host learns of a completed graph launch some milliseconds
// after the device has (a second thread per stream retires the work). What a
// program may not do is recorded as a violation: using an object after its
// destruction, and destroying a stream, an executable graph or a memory pool
// whose work has not been retired.
#pragma once

#include <atomic>
#include <cstddef>
#include <cstdint>
#include <string>

namespace hipstub {

struct Control {
    // faults to inject
    std::atomic<int> fail_graph_launch{0};   // > 0: the launch that counts it down to 0 fails
    std::atomic<int> fail_device_sync{0};    // != 0: hipDeviceSynchronize fails without waiting
    std::atomic<size_t> memory_limit{0};     // device bytes that can be allocated; 0: no limit
    std::atomic<int> resident_gives_up{0};   // the resident kernel's waits run out
    std::atomic<int> bad_links{0};           // the link check finds a link that is not SU(3)
    std::atomic<int> kernel_ms{0};           // how long a resident or operator kernel takes
    // what happened
    std::atomic<size_t> held{0};             // device bytes of hipMalloc and the pools
    std::atomic<size_t> malloc_held{0}, malloc_peak{0};  // of hipMalloc alone
    std::atomic<int> persist{0}, tiny{0}, stage{0};  // launches: resident, one workgroup, per stage
    std::atomic<int> persist_now{0}, persist_most{0};  // resident kernels running, and the most
    std::atomic<int> blocks_now{0}, blocks_most{0};  // their workgroups at one time
    std::atomic<int> paired_queues{0};       // streams 0 and 1, 2 and 3, ... share a hardware queue of four
    std::atomic<int> never_apart{0};         // no two streams are found to run side by side
    std::atomic<unsigned> queues_used{0};    // by graph launches, a bit each
    std::atomic<int> persist_iters{0};               // the most iterations given to one launch
};
extern Control ctl;

void violation(const std::string& what);
int violations();
// Work that has not been retired yet, over all streams.
int in_flight();

}  // namespace hipstub
