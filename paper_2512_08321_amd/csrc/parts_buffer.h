// The handle's memory for E' planes of products cut along k, where the workspace has no room
// for them.  A call can do without these planes (whole products, same results), so having
// them costs no other call anything:
//  - the workspace itself is never grown, moved or freed for them;
//  - an outgrown buffer is kept until the workspace moves or the handle goes: calls in flight
//    and captured graphs may still use it.  Sizes at least double, so what is kept stays
//    below the size in use, and its number below the bits of a size;
//  - a size that could not be had is not asked for again until the workspace moves.
#pragma once

#include <cstddef>
#include <cstdint>

namespace ozc {

class PartsBuffer {
    static constexpr size_t kLeast = (size_t)1 << 20;
    void *ptr_ = nullptr;
    size_t bytes_ = 0, refused_ = SIZE_MAX;
    void *kept_[64];
    int nkept_ = 0;

  public:
    bool covers(size_t need) const { return need <= bytes_; }
    // At least `need` bytes, or null.  alloc(size) gives memory or null; it is not called
    // where the buffer suffices or the size has been refused before.
    template <typename Alloc>
    void *get(size_t need, Alloc alloc) {
        if (covers(need)) return ptr_;
        if (need >= refused_) return nullptr;
        const size_t twice = bytes_ <= SIZE_MAX / 2 ? 2 * bytes_ : need;
        const size_t size = need > twice ? (need > kLeast ? need : kLeast) : twice;
        void *p = alloc(size);
        if (!p) {
            refused_ = need;
            return nullptr;
        }
        if (ptr_) kept_[nkept_++] = ptr_;
        ptr_ = p;
        bytes_ = size;
        return p;
    }
    // Gives everything back: free(p) for each buffer.
    template <typename Free>
    void release(Free free) {
        while (nkept_ > 0) free(kept_[--nkept_]);
        if (ptr_) free(ptr_);
        ptr_ = nullptr;
        bytes_ = 0;
        refused_ = SIZE_MAX;
    }
};

}  // namespace ozc
