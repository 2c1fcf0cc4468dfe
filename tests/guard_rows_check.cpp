// CPU check of row_outside (compiled with g++ by test_guard_rows.py): for random and extreme bindings,
// row sizes and indices, a row is called outside exactly where none of its bytes lies in the
// binding, worked out in 128 bits, except that it may be called inside without being so.
#include <cstdio>
#include <random>

#include "../paper_2606_06697_amd/csrc/guard_arith.h"

using namespace agile;
typedef __int128 i128;

int main() {
    std::mt19937_64 rng(77);
    const auto pick = [&]() -> uint64_t {
        switch (rng() % 6) {
            case 0: return rng() % 4096;
            case 1: return ~0ull - rng() % 4096;
            case 2: return (1ull << 63) + (rng() % 8192) - 4096;
            default: return rng();
        }
    };
    long wrong = 0, missed = 0, outside = 0;
    for (int it = 0; it < 500000; ++it) {
        uint64_t lo = pick(), hi = pick();
        if (lo > hi) std::swap(lo, hi);
        if (rng() % 3 == 0) hi = lo < ~0ull - 6000 ? lo + rng() % 5000 : hi;
        const Bind b = rng() % 12 == 0 ? Bind{0, 0} : Bind{lo, hi};
        const uint64_t rb = rng() % 4 == 0 ? 4 * (1 + rng() % (1ull << 38)) : 4 * (1 + rng() % 600);
        uint64_t base = b.hi > b.lo ? b.lo + rng() % (b.hi - b.lo) : pick();
        if (rng() % 4 == 0) base = b.lo;
        if (rng() % 4 == 0 && b.hi > b.lo) base = b.hi - 1 - rng() % (b.hi - b.lo < 8 ? b.hi - b.lo : 8);
        const RowGuard g = row_guard(b, base, rb);
        const uint64_t ulo = (uint64_t)g.rlo, uhi = (uint64_t)g.rhi;
        const int64_t cands[] = {0, 1, -1, (int64_t)(ulo - 2), (int64_t)(ulo - 1), g.rlo, (int64_t)(ulo + 1),
                                 (int64_t)(uhi - 1), g.rhi, (int64_t)(uhi + 1), (int64_t)(uhi + 2),
                                 INT64_MIN, INT64_MAX, INT64_MIN + 1, INT64_MAX - 1, (int64_t)rng()};
        for (int64_t x : cands) {
            // bytes [s, s + rb) from the base against [-dlo, dhi)
            const i128 s = (i128)x * (i128)rb;
            const bool touches = g.bound && s < (i128)g.dhi && s + (i128)rb > -(i128)g.dlo;
            const bool out = row_outside(g, x);
            outside += out;
            if (out && touches && wrong++ < 5)
                printf("row %lld of %llu bytes called outside\n", (long long)x, (unsigned long long)rb);
            // only the two rows next to the interval may be called inside without touching it
            const bool next = g.bound && ((i128)x == (i128)g.rlo - 1 || (i128)x == (i128)g.rhi + 1);
            if (!out && !touches && !next && missed++ < 5)
                printf("row %lld of %llu bytes not called outside\n", (long long)x, (unsigned long long)rb);
        }
    }
    if (wrong || missed || !outside) return 1;
    printf("ok\n");
    return 0;
}
