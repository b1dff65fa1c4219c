// Waits of persistent kernels, as far as they can be told without a GPU. (constexpr functions are host and device
// functions alike.)
#pragma once
#include <stdint.h>

// How long a wait goes on that ends by itself as long as the sweep moves: until `limit` polls have passed without a
// change of `progress` (a counter of the sweep). Per poll: if (look(limit)), read the counter and ask over().
struct dg4_patience {
    uint32_t spins = 0;      // polls since the counter was seen to change
    uint32_t mark = 0;       // the counter then
    constexpr bool look(uint32_t limit) { return (++spins & 63u) == 0 || spins > limit; }
    constexpr bool over(uint32_t progress, uint32_t limit)
    {
        if (progress != mark) { mark = progress; spins = 0; }
        return spins > limit;
    }
};
