// The window form's arithmetic on one ranked seed, on its own so that it also runs on the host.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ilre {

struct SeedInterval {
    bool some;             // the seed owns tokens ..
    uint32_t first, last;  // .. these (0, 0 without any)
};

// The tokens of 0 .. len - 1 whose window of `reach` tokens to each side holds the seed at token `at` and nothing that outranks it.
// dominators: how far the nearest such neighbours are, before it in the low half, behind it in the high half.  `there`: false for
// a place behind the last seed, where `at` and `dominators` are whatever lies in memory; no sum is made of them.
__host__ __device__ __forceinline__ SeedInterval seed_interval(bool there, uint32_t at, uint32_t dominators, uint32_t reach, uint32_t len)
{
    auto lower = [](int32_t a, int32_t b) { return a < b ? a : b; };
    const int32_t r = (int32_t)reach, t = there ? (int32_t)at : 0;
    const int32_t l = lower(lower(r, (int32_t)(dominators & 0xFFFFu) - r - 1), t);
    const int32_t e = lower(lower(r, (int32_t)(dominators >> 16) - r - 1), (int32_t)len - 1 - t);
    const bool some = there & (l + e >= 0);
    return {some, some ? (uint32_t)(t - l) : 0u, some ? (uint32_t)(t + e) : 0u};
}

}  // namespace ilre
