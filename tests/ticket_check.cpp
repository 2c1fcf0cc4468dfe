// CPU check of last_workgroup (compiled with g++ by test_ticket.py). One launch after another elects exactly
// one workgroup, after every other one has been counted, whatever earlier launches left behind: launches
// that overlapped on two streams (workgroups of both in any order), that shared their words, and that were
// cut short. Two launches that follow one another each elect one also when they overlap.
#include <algorithm>
#include <atomic>
#include <cstdio>
#include <random>
#include <thread>
#include <vector>

#include "../paper_2606_06697_amd/csrc/ticket.h"

using namespace agile;

struct Cpu {
    void raise(uint64_t* w, uint64_t v) const {
        uint64_t o = __atomic_load_n(w, __ATOMIC_RELAXED);
        while (o < v && !__atomic_compare_exchange_n(w, &o, v, false, __ATOMIC_RELAXED, __ATOMIC_RELAXED)) {
        }
    }
    uint64_t add(uint64_t* w) const { return __atomic_fetch_add(w, (uint64_t)1, __ATOMIC_RELAXED); }
};

static std::vector<uint64_t> words(TICKET_WORDS, 0);
static std::mt19937 rng(9);
static int fails = 0;

struct Wg {
    uint64_t launch;
    uint32_t block, blocks;
};

static bool run(const Wg& w) { return last_workgroup(Cpu{}, words.data(), w.launch, w.block, w.blocks); }

static void add(std::vector<Wg>& v, uint64_t launch, uint32_t blocks) {
    for (uint32_t b = 0; b < blocks; ++b) v.push_back({launch, b, blocks});
}

// Runs a launch by itself, in a random order: the last workgroup to come must be the one elected.
static void ordered(uint64_t launch, uint32_t blocks, const char* after) {
    std::vector<Wg> v;
    add(v, launch, blocks);
    std::shuffle(v.begin(), v.end(), rng);
    long elected = 0, early = 0;
    for (size_t k = 0; k < v.size(); ++k)
        if (run(v[k])) {
            ++elected;
            early += k + 1 != v.size();
        }
    if ((elected != 1 || early) && fails++ < 8)
        printf("launch %llu of %u workgroups after %s: %ld elected, %ld early\n", (unsigned long long)launch, blocks,
               after, elected, early);
}

int main() {
    const uint32_t sizes[] = {2, 3, 31, 32, 33, 63, 64, 65, 512, 1000, 1024, 2048};
    uint64_t launch = 0;
    for (int rep = 0; rep < 20; ++rep)
        for (uint32_t n : sizes) ordered(launch++, n, "ordered ones");
    for (int rep = 0; rep < 60; ++rep) {
        // neighbours on two streams
        const uint32_t a = sizes[rng() % 12], b = sizes[rng() % 12];
        std::vector<Wg> v;
        add(v, launch, a);
        add(v, launch + 1, b);
        int got[2] = {0, 0};
        std::shuffle(v.begin(), v.end(), rng);
        for (const Wg& w : v) got[w.launch - launch] += run(w);
        if ((got[0] != 1 || got[1] != 1) && fails++ < 8) printf("overlap of %u and %u: %d, %d elected\n", a, b, got[0], got[1]);
        launch += 2;
        for (uint32_t n : {512u, 64u, 1024u, 33u, 2u}) ordered(launch++, n, "two that overlapped");
        // many on many streams, which share words; some end early
        v.clear();
        for (int k = 0; k < 9; ++k) add(v, launch++, sizes[rng() % 12]);
        std::shuffle(v.begin(), v.end(), rng);
        v.resize(v.size() - v.size() / (1 + rng() % 4) / 3);
        for (const Wg& w : v) (void)run(w);
        for (uint32_t n : {512u, 64u, 1024u, 33u, 2u, 2048u}) ordered(launch++, n, "nine that overlapped");
    }
    // workgroups that come at the same time
    for (int rep = 0; rep < 30; ++rep) {
        const uint32_t n = sizes[rng() % 12];
        std::atomic<uint32_t> next{0}, elected{0};
        std::vector<std::thread> t;
        for (int k = 0; k < 4; ++k)
            t.emplace_back([&] {
                for (uint32_t b; (b = next++) < n;) elected += run({launch, b, n});
            });
        for (auto& x : t) x.join();
        if (elected != 1 && fails++ < 8) printf("%u at the same time: %u elected\n", n, elected.load());
        ++launch;
    }
    if (fails) return 1;
    printf("ok\n");
    return 0;
}
