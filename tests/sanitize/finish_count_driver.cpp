// Launches of several sizes counting on one word in every order the seed gives: alone, a launch finds exactly one last
// workgroup and it is the last to count; after launches that overlapped, the next one alone does so again.
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>

#include "tcr_count.hpp"

static std::mt19937 rng(7);
static uint32_t word = 0;

// Lets the workgroups of launches of these sizes count in a random common order: every launch finds its last workgroup,
// and no other.
static bool count(const std::vector<uint32_t>& sizes) {
    std::vector<std::pair<size_t, uint32_t>> order;
    std::vector<uint32_t> left = sizes;
    for (size_t l = 0; l < sizes.size(); ++l)
        for (uint32_t g = 0; g < sizes[l]; ++g) order.push_back({l, g});
    std::shuffle(order.begin(), order.end(), rng);
    uint32_t found = 0;
    bool at_the_end = true;
    for (const auto& [l, g] : order) {
        const uint32_t weight = tcr::finish_weight(g, sizes[l]), before = word;
        word += weight;
        left[l] -= 1;
        if (tcr::finish_is_last(before, weight)) {
            ++found;
            at_the_end = at_the_end && left[l] == 0;
        }
    }
    return found == sizes.size() && at_the_end;
}

int main() {
    std::uniform_int_distribution<uint32_t> size(1, tcr::kFinishCount), launches(2, 4);
    word = 0u - 1000u * tcr::kFinishCount;              // (the word wraps on the way)
    for (uint32_t groups = 1; groups <= tcr::kFinishCount; ++groups)
        if (!count({groups})) return std::printf("alone: %u\n", groups), 1;
    uint32_t spoiled = 0;
    for (int round = 0; round < 2000; ++round) {
        std::vector<uint32_t> sizes(launches(rng));
        for (uint32_t& s : sizes) s = size(rng);
        if (!count(sizes)) ++spoiled;                   // (unsupported: their own results are wrong)
        if (!count({size(rng)})) return std::printf("after an overlap: round %d\n", round), 1;
    }
    std::printf("%u overlaps spoiled themselves alone\nok\n", spoiled);
    return 0;
}
