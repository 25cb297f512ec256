// Work that is done once for each device of the process: a function attribute, say,
// belongs to the device that was current when it was set, so one flag for the
// process would leave a second device without it.
#pragma once
#include <mutex>
#include <set>

namespace c3 {

class PerDevice {
    std::mutex mu;
    std::set<int> done;

public:
    // init()'s status, or E() (success) where it has succeeded for device dev before;
    // a failure is not kept: the next call tries again.  Concurrent callers wait for it.
    template <typename E, typename F>
    E once(int dev, F &&init) {
        std::lock_guard<std::mutex> lk(mu);
        if (done.count(dev)) return E();
        const E e = init();
        if (e == E()) done.insert(dev);
        return e;
    }
};

}  // namespace c3
