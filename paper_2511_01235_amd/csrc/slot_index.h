// Arithmetic on entry and slot indices that may reach INT_MAX, where lo + hi
// or j + 8 no longer fit in 32 bits.  Apart from the kernels that use it, so
// that it can be checked on the host at those limits (constexpr functions are
// compiled for both sides).
#pragma once
#include <cstdint>

namespace mf {

// The first entry of lo..hi (sorted keys, hi excluded) whose key is not below k, or hi.
template <class Keys>
constexpr int first_at_least(const Keys& keys, int lo, int hi, unsigned long long k) {
    while (lo < hi) {
        const int mid = lo + (hi - lo) / 2;
        if (keys[mid] < k) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// f(j) for j = beg, beg + step, ... below end
template <class F>
constexpr void strided(int64_t beg, int64_t end, int step, F f) {
    for (int64_t j = beg; j < end; j += step) f((int)j);
}

// Slot j of a row that ends at `end`, or the row's last one.
constexpr int slot_or_last(int64_t j, int end) { return j < end ? (int)j : end - 1; }

// Workgroups of `block` threads for `items` threads of work in a grid-stride
// loop.  A launch takes fewer than 2^32 threads in all.
constexpr unsigned stride_blocks(int64_t items, int block) {
    const int64_t most = (int64_t{1} << 31) / block, want = (items + block - 1) / block;
    return (unsigned)(want < 1 ? 1 : want < most ? want : most);
}

}  // namespace mf
