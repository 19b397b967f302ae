// perdev.hpp -- host values that are found once per device.
#pragma once

#include <mutex>

namespace n2v {

// A T for each device, filled by the first caller that asks for it; the others
// wait until it is whole.  (With a "filled" field tested without a lock, a
// thread could read a value that another was still filling.)
template <class T>
class PerDevice {
  public:
    template <class F>
    const T &get(int dev, F fill)
    {
        Entry &e = entries_[dev & (MAX - 1)];
        std::call_once(e.once, [&] { fill(e.value); });
        return e.value;
    }

  private:
    static constexpr int MAX = 64;
    struct Entry {
        std::once_flag once;
        T value{};
    };
    Entry entries_[MAX];
};

}  // namespace n2v
