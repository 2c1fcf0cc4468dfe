// Which workgroup of a launch is done last (host- and device-compilable, so that it can be checked on the
// CPU).
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define AGILE_TICKET_HD __host__ __device__
#else
#define AGILE_TICKET_HD
#endif

namespace agile {

// Workgroups are counted in TICKETS places a memory channel apart (one place takes about 20 ns an atomic, one
// after another), and the places that are full in one more. A word holds a launch's number and its count:
// every workgroup first raises the word to (its launch, 0), which only a launch's first one changes, so
// nothing that an earlier launch left there is counted, whether it ended or was mixed with others on
// another stream. Launches that follow one another use different words, so two of them that overlap do not
// mix either. A launch number is used once: launches that a graph replays are not counted here.
// (Words that each launch leaves at zero, without the first step, save 0.3 us at 1,024 workgroups and 0.7 at
// 2,048, but two launches that once mix leave them out of step for every later one. A gather of 2,048
// workgroups takes 13.2 / 12.6 / 12.7 us with 16 / 32 / 64 places; 14.4 with the first step at its begin.)
constexpr uint32_t TICKETS = 32, TICKET_STRIDE = 32, TICKET_SETS = 4, TICKET_COUNT_BITS = 16;
constexpr uint32_t TICKET_WORDS = TICKET_SETS * (TICKETS + 1) * TICKET_STRIDE;

AGILE_TICKET_HD inline uint64_t* ticket_set(uint64_t* words, uint64_t launch) {
    return words + launch % TICKET_SETS * (TICKETS + 1) * TICKET_STRIDE;
}

// One thread per workgroup: whether its workgroup is the launch's last one. at.raise(w, v): *w = max(*w, v);
// at.add(w): *w += 1, the old value; relaxed, a thread's go to one word in order.
template <class Atomics>
AGILE_TICKET_HD inline bool last_workgroup(const Atomics& at, uint64_t* words, uint64_t launch, uint32_t block,
                                           uint32_t blocks) {
    uint64_t* set = ticket_set(words, launch);
    const uint64_t none = launch << TICKET_COUNT_BITS;
    const uint32_t s = block % TICKETS, full = (blocks - s + TICKETS - 1) / TICKETS;
    const uint32_t places = blocks < TICKETS ? blocks : TICKETS;
    at.raise(set + s * TICKET_STRIDE, none);
    if (at.add(set + s * TICKET_STRIDE) != none + full - 1) return false;
    at.raise(set + TICKETS * TICKET_STRIDE, none);
    return at.add(set + TICKETS * TICKET_STRIDE) == none + places - 1;
}

}  // namespace agile
