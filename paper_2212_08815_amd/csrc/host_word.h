// Where a kernel leaves a number for the host.
#pragma once
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <chrono>
#include <mutex>
#include <vector>

namespace fscnn {

// A word of pinned memory for one call (copied from the device to pageable memory the same number takes a launch and 20 us of
// the host's time more).  NULL where there is none: then it is copied.
class HostWord {
public:
    HostWord()
    {
        Words &w = words();
        std::lock_guard<std::mutex> lock(w.mu);
        if (!w.made) {
            w.made = true;
            void *p = nullptr;
            if (hipHostMalloc(&p, kWords * 64, hipHostMallocPortable | hipHostMallocMapped) == hipSuccess)
                for (int i = 0; i < kWords; ++i) w.free.push_back((w.first = static_cast<int *>(p)) + i * 16);
            else
                (void)hipGetLastError();
        }
        if (!w.free.empty()) {
            word = w.free.back();
            w.free.pop_back();
        }
    }
    ~HostWord()
    {
        if (!word || in_flight) return;
        Words &w = words();
        std::lock_guard<std::mutex> lock(w.mu);
        w.free.push_back(word);
    }
    HostWord(const HostWord &) = delete;
    HostWord &operator=(const HostWord &) = delete;
    // for a launch.  From here on until wait() has succeeded a kernel may write it: a call that fails in between never gives it back
    int *hand_out()
    {
        in_flight = true;
        if (word) *const_cast<volatile int *>(word) = kNone;
        return word;
    }
    // a number below kWords that no other word in use has, -1: there is no word
    int slot() const { return word ? (int)((word - words().first) / 16) : -1; }
    static constexpr int kWords = 64;    // calls at one time that find a word
    // the number, which is not negative, as soon as a kernel on `st` has written it (store_host): what follows that kernel on the stream
    // need not be done, and the wait is over 4 to 8 us before a wait for the stream would be.  Where the stream has more than a
    // millisecond to do first, and where there is no word, the stream is waited for; from: where the device has the number as well (NULL: it
    // is not wanted).  A negative number: the stream's work is done and there is none.  second: receives the int behind the number, which is
    // written with it or before it
    hipError_t wait(const int *from, hipStream_t st, int *out, int *second = nullptr)
    {
        if (word) {
            const auto until = std::chrono::steady_clock::now() + std::chrono::milliseconds(1);
            for (int i = 1; (*out = *const_cast<volatile int *>(word)) == kNone; ++i) {
                if (i % 64 == 0 && std::chrono::steady_clock::now() > until) break;
#if defined(__x86_64__)
                __builtin_ia32_pause();
#endif
            }
            if (*out != kNone) {
                std::atomic_thread_fence(std::memory_order_acquire);
                in_flight = false;
                if (second) *second = const_cast<volatile int *>(word)[1];
                return hipSuccess;
            }
        }
        hipError_t e = word || !from ? hipSuccess : hipMemcpyAsync(out, from, sizeof(int), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess && !word && from && second) e = hipMemcpyAsync(second, from + 1, sizeof(int), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return e;
        if (word) *out = *const_cast<volatile int *>(word);
        if (word && second) *second = const_cast<volatile int *>(word)[1];
        // (the stream is done and no kernel has written it: none of its launches counted to their end.  Neither the word nor the counters
        // of its slot serve another call, and the caller finds a negative number)
        in_flight = word && *out == kNone;
        return e;
    }

private:
    static constexpr int kNone = -1;     // (what no kernel writes)
    int *word = nullptr;
    bool in_flight = false;
    struct Words {
        std::mutex mu;
        bool made = false;
        int *first = nullptr;
        std::vector<int *> free;
    };
    static Words &words()
    {
        static Words *w = new Words();   // (never destroyed: handles may outlive static objects)
        return *w;
    }
};

}  // namespace fscnn
