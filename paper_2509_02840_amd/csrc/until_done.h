// until_done.h -- a preparation that is made once per process, by the first
// caller for whom it succeeds.
#pragma once
#include <mutex>

namespace bdu {

class UntilDone {
public:
    // 0, or what f returned: a failure (no memory for the code object, say) is
    // the caller's, and the next one tries again.
    template <typename F>
    auto operator()(F f) -> decltype(f())
    {
        std::lock_guard<std::mutex> lk(mu_);
        decltype(f()) e{};
        if (!done_) e = f();
        done_ = e == decltype(e){};
        return e;
    }

private:
    std::mutex mu_;
    bool done_ = false;
};

}  // namespace bdu
