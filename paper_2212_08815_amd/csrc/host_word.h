// Where a kernel leaves a number for the host.
#pragma once
#include <hip/hip_runtime_api.h>

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
                for (int i = 0; i < kWords; ++i) w.free.push_back(static_cast<int *>(p) + i * 16);
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
        return word;
    }
    // the number, once the work on `st` is done; from: where the device has it as well
    hipError_t wait(const int *from, hipStream_t st, int *out)
    {
        hipError_t e = word ? hipSuccess : hipMemcpyAsync(out, from, sizeof(int), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return e;
        in_flight = false;
        if (word) *out = *const_cast<volatile int *>(word);
        return e;
    }

private:
    static constexpr int kWords = 64;    // calls at one time that find a word
    int *word = nullptr;
    bool in_flight = false;
    struct Words {
        std::mutex mu;
        bool made = false;
        std::vector<int *> free;
    };
    static Words &words()
    {
        static Words *w = new Words();   // (never destroyed: handles may outlive static objects)
        return *w;
    }
};

}  // namespace fscnn
