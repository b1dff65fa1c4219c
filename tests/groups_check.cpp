// The group protocol of csrc/dg4_wait.h on host threads, one per workgroup: the workgroups of one or two sweeps start
// when a place on "their" XCD (number % 8) is free and give it back when they end, as on the device. A sweep is a
// list of tickets; a ticket can only be finished by a whole group, and waits for the ticket before it (the
// hardest chain). Prints what failed and returns 1; a sweep that stands still ends by its own patience.
#include <atomic>
#include <condition_variable>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include <mutex>
#include <thread>
#include <vector>

#include "dg4_wait.h"

struct Places {                                     // free places per XCD
    std::mutex mu;
    std::condition_variable cv;
    std::vector<int> free_;
    void take(int x) { std::unique_lock<std::mutex> l(mu); cv.wait(l, [&] { return free_[x] > 0; }); --free_[x]; }
    void give(int x, int k = 1) { std::lock_guard<std::mutex> l(mu); free_[x] += k; cv.notify_all(); }
};

struct Sweep {
    int C, groups, tickets;
    uint32_t limit, polls;
    std::vector<uint32_t> word, regroup;
    std::vector<std::atomic<uint64_t>> mail;        // [group][2]
    std::vector<std::atomic<int>> together;         // [group] members that have finished their part of a ticket
    std::vector<std::atomic<int>> done;             // [ticket] slices finished
    std::vector<std::atomic<int>> slices;           // [group] the seats taken, a bit each
    uint32_t ticket = 0, formed = 0, loose = 0, aborted = 0;
    std::atomic<int> left{0}, wrong{0};
    Sweep(int c, int g, int t, uint32_t lim, uint32_t po)
        : C(c), groups(g), tickets(t), limit(lim), polls(po), word(g), regroup(g), mail(2 * g), together(g), done(t + 1), slices(g) {}
    bool complete() { for (int t = 0; t < tickets; ++t) if (done[t] != C) return false; return !aborted && !wrong && left == groups * C; }
};

struct Mem {
    Sweep& s;
    dg4_patience patience;
    uint32_t add(uint32_t* q) { return __atomic_fetch_add(q, 1u, __ATOMIC_RELAXED); }
    uint32_t load(const uint32_t* q) { return __atomic_load_n(q, __ATOMIC_RELAXED); }
    void store(uint32_t* q, uint32_t v) { __atomic_store_n(q, v, __ATOMIC_RELAXED); }
    bool cas(uint32_t* q, uint32_t expected, uint32_t v) { return __atomic_compare_exchange_n(q, &expected, v, false, __ATOMIC_RELAXED, __ATOMIC_RELAXED); }
    void pause() { std::this_thread::yield(); }
    bool leave()
    {
        const uint32_t drawn = load(&s.ticket);
        if (drawn >= (uint32_t)s.tickets) return true;
        if (patience.look(s.limit)) {
            if (patience.over(drawn + load(&s.loose), s.limit)) store(&s.aborted, 1u);
            if (load(&s.aborted)) return true;
        }
        return false;
    }
};

static void workgroup(Sweep& s, int b)
{
    int slice = 0, group = -1;
    bool last = false;
    for (int stage = 0; stage < 2 && group < 0; ++stage) {
        Mem mem{s, {}};
        slice = b % s.C;
        uint32_t* word = &s.word[b / s.C];
        if (stage) {
            const int place = (int)mem.add(&s.loose);
            slice = place % s.C;
            word = &s.regroup[place / s.C];
        }
        const dg4_seat at = dg4_sit(mem, word, (uint32_t)s.C, &s.formed, stage ? 0xFFFFFFFFu : s.polls);
        group = at.group; last = at.last;
        if (group < 0 && __atomic_load_n(&s.aborted, __ATOMIC_RELAXED)) break;
    }
    if (group >= 0) {
        if (group >= s.groups) { ++s.wrong; return; }
        if (s.slices[group].fetch_or(1 << slice) & (1 << slice)) ++s.wrong;       // two workgroups on one seat
        auto post = [&](uint64_t number) { s.mail[2 * group + (number & 1)] = (number + 1) << 32 | __atomic_fetch_add(&s.ticket, 1u, __ATOMIC_RELAXED); };
        if (last) post(0);
        for (uint64_t number = 0;; ++number) {
            uint64_t w;
            while ((w = s.mail[2 * group + (number & 1)]) >> 32 != number + 1) {
                if (__atomic_load_n(&s.aborted, __ATOMIC_RELAXED)) return;
                std::this_thread::yield();
            }
            const int t = (int)(uint32_t)w;
            if (t >= s.tickets) break;
            while (t > 0 && s.done[t - 1] != s.C) {
                if (__atomic_load_n(&s.aborted, __ATOMIC_RELAXED)) return;
                std::this_thread::yield();
            }
            ++s.together[group];                    // the exchange: everybody's part is in
            while (s.together[group] < s.C * (int)(number + 1)) std::this_thread::yield();
            if (slice == 0) post(number + 1);
            ++s.done[t];
        }
    }
    ++s.left;
}

static bool run(const char* what, std::vector<Sweep*> sweeps, std::vector<int> places, int late_xcd = -1, int late_places = 0)
{
    Places free;
    free.free_ = places;
    std::vector<std::thread> threads;
    for (Sweep* s : sweeps)
        for (int b = 0; b < s->groups * s->C; ++b)
            threads.emplace_back([&free, s, b] { free.take(b % 8); workgroup(*s, b); free.give(b % 8); });
    std::thread other;
    if (late_xcd >= 0) other = std::thread([&] {    // another kernel's work ends only when the sweep has
        for (Sweep* s : sweeps) while (__atomic_load_n(&s->ticket, __ATOMIC_RELAXED) < (uint32_t)s->tickets && !__atomic_load_n(&s->aborted, __ATOMIC_RELAXED)) std::this_thread::yield();
        free.give(late_xcd, late_places);
    });
    for (std::thread& t : threads) t.join();
    if (other.joinable()) other.join();
    bool ok = true;
    for (Sweep* s : sweeps) ok = ok && s->complete();
    if (!ok) std::printf("FAILED: %s\n", what);
    return ok;
}

static const uint32_t PATIENT = 1u << 30;           // (a loaded machine may keep a thread waiting; the caller has a time limit)

int main(int argc, char** argv)
{
    const int rounds = argc > 1 ? std::atoi(argv[1]) : 5;
    bool ok = true;
    for (int r = 0; r < rounds; ++r)
        for (int C : {4, 8}) {
            const int G = 32 / C;
            for (uint32_t polls : {0u, 3u, 50u}) {
                Sweep a(C, G, 40, PATIENT, polls), b(C, G, 1, PATIENT, polls), c(C, G, 30, PATIENT, polls);
                ok = run("every workgroup runs", {&a}, std::vector<int>(8, 4)) && ok;
                ok = run("one ticket: most groups leave", {&b}, std::vector<int>(8, 4)) && ok;
                // no place on one XCD until the tickets have run out: with fixed seats (hidden 256) no group is ever whole
                std::vector<int> without(8, 4);
                without[3] = 0;
                ok = run("an XCD is never free", {&c}, without, 3, 4) && ok;
                // two sweeps, fewer places than workgroups: either may lack any XCD
                Sweep d(C, G, 25, PATIENT, polls), e(C, G, 25, PATIENT, polls);
                ok = run("two sweeps share the device", {&d, &e}, std::vector<int>(8, 4)) && ok;
                // places of one XCD fewer
                Sweep f(C, G, 25, PATIENT, polls);
                std::vector<int> narrow(8, 4);
                narrow[0] = 1; narrow[5] = 2;
                ok = run("few places on some XCDs", {&f}, narrow) && ok;
            }
        }
    // fewer workgroups than a group: the wait ends by its patience
    Sweep g(8, 4, 5, 300, 10);
    std::vector<std::thread> threads;
    for (int b = 0; b < 7; ++b) threads.emplace_back([&g, b] { workgroup(g, b); });
    for (std::thread& t : threads) t.join();
    if (!g.aborted) { std::printf("FAILED: seven workgroups of eight must give up\n"); ok = false; }
    return ok ? 0 : 1;
}
