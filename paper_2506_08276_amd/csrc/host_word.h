// The word in pinned host memory by which kernels tell a waiting host that their results are there.  Host code without HIP types.
#pragma once
#include <stdint.h>

#include <chrono>

// Every launch that stores to the word gets a number of its own, one after the other over the context's life: a kernel that a call
// left behind (a call may end early with an error) stores a number that no later wait takes for its own.
class HostWord {
    uint32_t issued_ = 0;

public:
    uint32_t next() { return ++issued_; }  // for the next launch

    // Looks at the word until the number issued last (or, with launches in order, a later one) is there: false if that takes long, as where
    // a kernel is slow, has faulted or was not run (stream capture).  The caller then waits for the stream, which reports what is wrong.
    bool arrives(const uint32_t *word) const
    {
        constexpr auto LONG = std::chrono::milliseconds(20);
        const auto begin = std::chrono::steady_clock::now();
        for (;;) {
            for (int i = 0; i < 256; ++i) {
                if ((int32_t)(__atomic_load_n(word, __ATOMIC_ACQUIRE) - issued_) >= 0) return true;
                __builtin_ia32_pause();
            }
            if (std::chrono::steady_clock::now() - begin > LONG) return false;
        }
    }
};
