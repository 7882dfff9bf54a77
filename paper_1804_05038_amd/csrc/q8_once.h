// q8_once.h -- what has to be done once per device before a first use there (a kernel's attributes belong to the kernel
// on one device: what one device was asked for says nothing about the next).
#pragma once

#include <atomic>

class Q8OncePerDevice {
    std::atomic<unsigned long long> done{0};          // bit d: done on device d
public:
    // Runs f (which returns whether it worked) unless it has worked on this device before; threads that come together may
    // all run it.  Devices past the 64th run it every time.  Returns whether it is done.
    template <class F> bool operator()(int device, F f)
    {
        const unsigned long long bit = device >= 0 && device < 64 ? 1ull << device : 0ull;
        if (done.load(std::memory_order_relaxed) & bit) return true;
        if (!f()) return false;
        done.fetch_or(bit, std::memory_order_relaxed);
        return true;
    }
};
