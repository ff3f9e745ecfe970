// Which of a launch's work-groups is the last one to arrive.
#pragma once

namespace fscnn {

#ifdef __HIP__
#define FSCNN_DEVICE __device__
#else
#define FSCNN_DEVICE   // (the protocol runs on the CPU with a memory of the test's)
#endif

// Arrivals at one address are counted one after the other, 8 ns each: 4 us of 512 work-groups.  So they meet in sixteen counters
// a line apart, the last ones of which meet in one.
constexpr int kArriveWays = 16, kCounterInts = (kArriveWays + 1) * 32;

// One thread of work-group `group` of `groups`, behind a barrier that all its stores were waited for in front of; true for the last one, and
// then all counters are zero for whoever has them next: mem.count(c, most) adds one to *c, or makes it zero where it is `most`, and
// returns what was there, all in one operation.  (A zero stored by the last one of a way has to be waited for before it counts in
// front: 1 us of a bank's three launches.)
template <class Mem> FSCNN_DEVICE inline bool arrive(const Mem &mem, int *counter, int groups, int group)
{
    const int way = group % kArriveWays, of_way = (groups - way + kArriveWays - 1) / kArriveWays, ways = groups < kArriveWays ? groups : kArriveWays;
    return mem.count(counter + (way + 1) * 32, of_way - 1) == of_way - 1 && mem.count(counter, ways - 1) == ways - 1;
}

}  // namespace fscnn
