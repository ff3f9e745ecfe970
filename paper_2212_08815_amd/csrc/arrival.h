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
// then all counters are zero for whoever has them next.  mem.add() counts and returns what was there, mem.clear() stores a zero that
// may take its time, mem.wait() returns when this thread's stores are done.
template <class Mem> FSCNN_DEVICE inline bool arrive(const Mem &mem, int *counter, int groups, int group)
{
    auto count = [&](int *c, int all) {
        if (mem.add(c) != all - 1) return false;
        mem.clear(c);
        mem.wait();   // (of all these last ones, before the one behind them can be told: another launch may count here next)
        return true;
    };
    const int way = group % kArriveWays;
    return count(counter + (way + 1) * 32, (groups - way + kArriveWays - 1) / kArriveWays) &&
           count(counter, groups < kArriveWays ? groups : kArriveWays);
}

}  // namespace fscnn
