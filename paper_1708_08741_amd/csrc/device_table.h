// device_table.h -- a value per GPU of the process, formed on the first use on
// that GPU.  What a launch needs to know of a kernel (function attributes set,
// workgroups resident per compute unit) holds for one device; a process may
// hold lattices on several.  Host code only.
#pragma once
#include <mutex>

namespace lbmep {

template <typename T, int N = 64>
class DeviceTable {
  public:
    // make() of the current device, once per device; from several threads at
    // once it runs in one of them and the others wait.  Devices beyond the
    // table form it on every call.
    template <typename F>
    T get(int device, F &&make) {
        if (device < 0 || device >= N) return make();
        std::call_once(once_[device], [&] { value_[device] = make(); });
        return value_[device];
    }

  private:
    std::once_flag once_[N];
    T value_[N] = {};
};

}  // namespace lbmep
