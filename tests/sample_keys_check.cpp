// Host driver for the sample-key test: for the distance keys of a tile whose
// first sample has the exact key `first`, every pair of exact keys in reach
// must keep its order, and the first sample must be in reach itself.  Prints
// the first fault and returns 1.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <vector>

#include "eg_sample.h"

// constant expressions: an overflow in them would not compile
static_assert(eg::key_is_exact(int64_t(1) << 24) && eg::key_is_exact(-(int64_t(1) << 24)), "the last exact ones");
static_assert(!eg::key_is_exact((int64_t(1) << 24) + 1) && !eg::key_is_exact(-(int64_t(1) << 24) - 1), "one further");
static_assert(!eg::key_is_exact(INT64_MAX) && !eg::key_is_exact(INT64_MIN), "both ends");

int main()
{
    // values around the ends, the middle and the steps of 2^31 and kKeyTop
    std::vector<uint64_t> v;
    const uint64_t half = uint64_t(1) << 31, top = eg::kKeyTop, mid = uint64_t(1) << 63;
    for (uint64_t at : {uint64_t(0), half, top, 2 * half, half + top, mid, mid - half, mid + half, mid - top, mid + top,
                        uint64_t(0) - half, uint64_t(0) - top, uint64_t(0) - half - top, uint64_t(0) - 2 * half})
        for (int64_t d = -3; d <= 3; ++d) v.push_back(at + (uint64_t)d);
    for (uint64_t first : v) {
        const uint64_t base = eg::near_base(first);
        auto near = [&](uint64_t x) { return x - base - 1u < top - 1u; };
        if (!near(first)) {
            std::printf("first %llx out of its own reach\n", (unsigned long long)first);
            return 1;
        }
        for (uint64_t x : v)
            for (uint64_t y : v)
                if (near(x) && near(y) && (x < y) != ((uint32_t)(x - base) < (uint32_t)(y - base))) {
                    std::printf("first %llx: %llx and %llx change order\n", (unsigned long long)first,
                                (unsigned long long)x, (unsigned long long)y);
                    return 1;
                }
    }
    return 0;
}
