// Host check of the workgroup counts (done_slots.hpp): launches of random grids, their workgroups in random order, some
// overlapping by mistake (which is against the interface and may spoil those); every launch that runs by itself
// afterwards finds exactly one last workgroup, and it is the one that ends last.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <random>
#include <vector>

#include <hip/hip_runtime.h>

#include "done_slots.hpp"

using namespace lacache;

static std::vector<uint32_t> words;
static std::mt19937 rng(7);

// Runs the launches with tickets first, first + 1, ... interleaved; returns how many of their workgroups counted last
// before the launch's end, and how many at it.
static void run(uint32_t first, const std::vector<uint32_t>& grids, int* early, int* last) {
    struct Step {
        uint32_t launch, block;
    };
    std::vector<Step> steps;
    for (uint32_t l = 0; l < grids.size(); ++l)
        for (uint32_t b = 0; b < grids[l]; ++b) steps.push_back({l, b});
    std::shuffle(steps.begin(), steps.end(), rng);
    std::vector<uint32_t> ended(grids.size(), 0u);
    *early = *last = 0;
    for (const Step& s : steps) {
        const uint32_t t = first + s.launch;
        const bool l = count_done(done_slot(words.data(), t), s.block, grids[s.launch], [](uint32_t* p) { return (*p)++; });
        if (s.block == 0)
            for (int i = 0; i < kDoneCount; ++i) done_slot(words.data(), t + 1)[i * kDoneStride] = 0u;
        ++ended[s.launch];
        if (l) ++*(ended[s.launch] == grids[s.launch] ? last : early);
    }
}

int main() {
    words.assign(kDoneWords, 0u);
    uint32_t ticket = 0xFFFFFF00u;  // past the wrap of the ticket too
    int spoiled = 0;
    for (int rep = 0; rep < 20000; ++rep) {
        int early, last;
        const bool overlap = rep % 5 == 0;
        std::vector<uint32_t> grids;
        for (uint32_t n = overlap ? 2 + rng() % 4 : 1; n > 0; --n) grids.push_back(1 + rng() % (rep % 3 ? 256 : 12));
        run(ticket, grids, &early, &last);
        ticket += (uint32_t)grids.size();
        if (overlap) {
            spoiled += early != 0 || last != (int)grids.size();
        } else if (early != 0 || last != 1) {
            std::printf("launch %d (%u workgroups): %d early, %d last\n", rep, grids[0], early, last);
            return 1;
        }
    }
    std::printf("ok 20000 rounds, %d overlapping ones spoiled\n", spoiled);
    return 0;
}
