// first_fit.h -- first-fit allocator over a range of bytes: offsets only, the
// memory belongs to the caller.  Frees coalesce.  Host code only.
#pragma once
#include <algorithm>
#include <cstddef>
#include <map>
#include <unordered_map>

namespace lbmep {

class FirstFit {
  public:
    static constexpr size_t kAlign = 4096;
    static constexpr size_t kNone = ~size_t(0);

    explicit FirstFit(size_t bytes = 0) : size_(bytes / kAlign * kAlign) {
        if (size_) free_[0] = size_;
    }
    // offset of a free run of at least `bytes`, kNone without one
    size_t alloc(size_t bytes) {
        const size_t need = std::max<size_t>(kAlign, (bytes + kAlign - 1) / kAlign * kAlign);
        for (auto it = free_.begin(); it != free_.end(); ++it) {
            if (it->second < need) continue;
            const size_t off = it->first, rest = it->second - need;
            free_.erase(it);
            if (rest) free_[off + need] = rest;
            live_[off] = need;
            used_ += need;
            return off;
        }
        return kNone;
    }
    void release(size_t off) {
        auto lv = live_.find(off);
        if (lv == live_.end()) return;
        size_t start = off, len = lv->second;
        live_.erase(lv);
        used_ -= len;
        auto next = free_.lower_bound(start);
        if (next != free_.end() && next->first == start + len) {
            len += next->second;
            next = free_.erase(next);
        }
        if (next != free_.begin()) {
            auto prev = std::prev(next);
            if (prev->first + prev->second == start) {
                start = prev->first;
                len += prev->second;
                free_.erase(prev);
            }
        }
        free_[start] = len;
    }
    size_t used() const { return used_; }
    size_t size() const { return size_; }

  private:
    size_t size_ = 0, used_ = 0;
    std::map<size_t, size_t> free_;            // offset -> length
    std::unordered_map<size_t, size_t> live_;  // offset -> length
};

}  // namespace lbmep
