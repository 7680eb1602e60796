// sj_search.h -- searches in sorted keys and block sizes, in 32-bit positions up to
// 2^32 - 1 (index arithmetic only, for device and host).
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define SJ_HD __host__ __device__ __forceinline__
#else
#define SJ_HD inline
#endif

namespace sjl {

// First position in [lo, hi) whose key, key_at(position), is > key (keys ascending).
template <typename F>
SJ_HD uint32_t first_above(const F &key_at, uint32_t lo, uint32_t hi, uint64_t key)
{
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (key_at(mid) <= key)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// Position after the run of `key` that holds every position from p's predecessor up to
// it (p <= n, keys ascending): doubling steps, then a binary search in the last step.
template <typename F>
SJ_HD uint32_t run_end(const F &key_at, uint32_t p, uint32_t n, uint64_t key)
{
    uint32_t lo = p, step = 1;
    while (step <= n - lo && key_at(lo + step - 1) == key) {
        lo += step;
        step = step < 1u << 31 ? 2 * step : step;
    }
    return first_above(key_at, lo, lo + (step < n - lo ? step : n - lo), key);
}

// Entries of block `blk` of `tile` entries each of n (blk * tile < n).
SJ_HD uint32_t block_entries(uint32_t blk, uint32_t tile, uint32_t n)
{
    const uint32_t left = n - blk * tile;
    return left < tile ? left : tile;
}

}  // namespace sjl
