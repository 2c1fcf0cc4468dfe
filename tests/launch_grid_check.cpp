// CPU check of a launch's workgroups (compiled with g++ by test_launch_grid.py): never 2^32 threads or more,
// as many as the items need where a grid holds them, at least one, and no more than the cap.
#include <cstdio>

#include "../paper_2606_06697_amd/csrc/launch_grid.h"

using namespace agile;

int main() {
    const uint64_t items[] = {0, 1, 255, 256, 257, 65535, 1u << 20, (1ull << 31) - 1, 1ull << 31, (1ull << 32) - 1,
                              1ull << 32, (1ull << 33) + 5, 1ull << 35, 1ull << 40, 1ull << 62, ~0ull};
    const uint32_t threads[] = {64, 128, 256, 512, 1024};
    const uint64_t per[] = {1, 2, 64, 128, 256, 512, 2048, 4096};
    const uint64_t caps[] = {1, 1024, 1ull << 22, 1ull << 30, ~0ull};
    int bad = 0;
    for (uint64_t n : items)
        for (uint32_t t : threads)
            for (uint64_t p : per)
                for (uint64_t c : caps) {
                    const uint64_t g = workgroups(n, p, t, c);
                    const unsigned __int128 need = n ? ((unsigned __int128)n + p - 1) / p : 1;
                    const bool fits = need * t < ((unsigned __int128)1 << 32) && need <= c;
                    const bool ok = g >= 1 && g <= c && g * t < (1ull << 32) && (fits ? need == g : g < need) &&
                                    (fits || g == c || (g + 1) * t >= (1ull << 32));
                    if (!ok && bad++ < 5)
                        printf("%llu items, %llu a group of %u threads, cap %llu: %llu\n", (unsigned long long)n,
                               (unsigned long long)p, t, (unsigned long long)c, (unsigned long long)g);
                }
    if (bad) return 1;
    printf("ok\n");
    return 0;
}
