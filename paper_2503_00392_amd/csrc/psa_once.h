// Host only, and free of HIP: something that has to be done once on every GPU a process uses.
#pragma once

#include <stdint.h>

#include <atomic>

namespace psa {

// operator()(device, f) calls f, which returns 0 on success, unless it has succeeded for this device before; a failure is
// handed on and not remembered.  Safe from several threads (which may then both call f); devices beyond 63 always call it.
class OncePerDevice {
  public:
    template <class F>
    auto operator()(int device, F f) -> decltype(f()) {
        const uint64_t bit = device >= 0 && device < 64 ? 1ull << device : 0ull;
        if (done_.load(std::memory_order_acquire) & bit) return decltype(f())(0);
        const auto e = f();
        if (e == 0) done_.fetch_or(bit, std::memory_order_release);
        return e;
    }

  private:
    std::atomic<uint64_t> done_{0};
};

}  // namespace psa
