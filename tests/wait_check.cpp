// Host checks of csrc/dg4_wait.h; prints one line per failed check and returns their number.
#include <cstdio>
#include <initializer_list>

#include "dg4_wait.h"

static int failed = 0;
static void check(bool ok, const char* what, unsigned limit, unsigned every)
{
    if (!ok) { std::printf("FAILED: %s (limit %u, a ticket every %u polls)\n", what, limit, every); ++failed; }
}

// polls until the wait gives up, at most `polls` (then 0); a ticket moves every `every` polls (0: never)
static unsigned gives_up(unsigned limit, unsigned every, unsigned polls)
{
    dg4_patience p;
    unsigned ticket = 0;
    for (unsigned i = 1; i <= polls; ++i) {
        if (every && i % every == 0) ++ticket;
        if (p.look(limit) && p.over(ticket, limit)) return i;
    }
    return 0;
}

int main()
{
    for (unsigned limit : {1u, 63u, 64u, 65u, 4096u, 5000u}) {
        check(gives_up(limit, 0, 4 * limit + 200) == limit + 1, "nothing moves: over after the limit", limit, 0);
        for (unsigned every : {1u, 2u, 3u, limit / 2, limit - 1, limit})
            if (every && every <= limit) check(gives_up(limit, every, 100 * limit + 10000) == 0, "tickets move: never over", limit, every);
        // a ticket that moved once, early, does not count for ever
        dg4_patience p;
        unsigned last = 0;
        for (unsigned i = 1; i <= 4 * limit + 200 && !last; ++i)
            if (p.look(limit) && p.over(i >= 2 ? 7 : 0, limit)) last = i;
        check(last > limit && last <= 2 * limit + 66, "over after the limit from the last movement", limit, 0);
    }
    return failed;
}
