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

// Groups of `members` workgroups, formed from those that run. A group has a word: the number of workgroups that
// have sat down so far, then one of two marks, each set once: FORMED with the group's number (by whoever completes it;
// numbers are dealt in the order groups form) or CLOSED (nobody waits for it any longer, and nobody ever will). Both
// are decided on the word itself, so all who sat down agree. `polls` looks at the word without the group being
// formed close it, and so does mem.leave().
// Mem: add(p) (returns the value before), load(p), store(p, v), cas(p, expected, v), pause(), leave().
constexpr uint32_t DG4_GROUP_CLOSED = 1u << 31, DG4_GROUP_FORMED = 1u << 30;
struct dg4_seat {
    int group;               // -1: the group was closed
    bool last;               // this workgroup completed it
};
template <typename Mem>
constexpr dg4_seat dg4_sit(Mem& mem, uint32_t* word, uint32_t members, uint32_t* formed, uint32_t polls)
{
    const uint32_t before = mem.add(word);
    if (before & DG4_GROUP_CLOSED) return dg4_seat{-1, false};
    if (before + 1 == members) {
        const uint32_t number = mem.add(formed);
        mem.store(word, DG4_GROUP_FORMED | number);
        return dg4_seat{(int)number, true};
    }
    for (uint32_t spins = 1;; ++spins) {
        const uint32_t w = mem.load(word);
        if (w & DG4_GROUP_CLOSED) return dg4_seat{-1, false};
        if (w & DG4_GROUP_FORMED) return dg4_seat{(int)(w & ~DG4_GROUP_FORMED), false};
        // (complete but not marked yet: it will be)
        if (w < members && (spins > polls || mem.leave()) && mem.cas(word, w, w | DG4_GROUP_CLOSED)) return dg4_seat{-1, false};
        mem.pause();
    }
}
