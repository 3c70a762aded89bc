// The order in which blocks are walked in turns: every block once, those of a chain in their order, and the chains that follow
// each other and are about equally long a block of each, whatever the chains' lengths.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "rose_internal.h"

static void check(bool ok, const char *what) {
    if (!ok) { std::printf("failed: %s\n", what); std::exit(1); }
}

int main() {
    std::mt19937 rng(1);
    for (int round = 0; round < 4000; ++round) {
        const int n = 1 + (int)(rng() % ROSE_MAX_TP);
        const int kind = (int)(rng() % 4), size = 1 + (int)(rng() % 200);
        std::vector<int32_t> first(ROSE_MAX_TP + 1, 0);
        for (int d = 0; d < n; ++d) {
            const int len = kind == 0 ? size : kind == 1 ? size + (int)(rng() % 3) : kind == 2 ? (int)(rng() % (unsigned)(size + 1))
                                                         : (rng() % 3 ? (int)(rng() % 2) : size);
            first[d + 1] = first[d] + len;
        }
        for (int d = n; d < ROSE_MAX_TP; ++d) first[d + 1] = first[n];
        const rose::Turns t = rose::turns_of(first.data(), n);
        std::vector<int32_t> next(first.begin(), first.end());      // the block of each chain that has to come next
        for (int32_t i = 0; i < first[n]; ++i) {
            const rose::WalkedBlock b = rose::walked_block(t, first.data(), i);
            check(b.shard >= 0 && b.shard < n && b.blk < first[b.shard + 1], "a block of the chain");
            check(b.blk == next[b.shard]++, "a chain's blocks in their order");
            const int32_t x = i - first[t.chain];
            if (x >= 0 && x < t.chains * t.each) check(b.shard == t.chain + x % t.chains, "in turn");
        }
        for (int d = 0; d < n; ++d) check(next[d] == first[d + 1], "every block");
        check(kind != 0 || n < 2 || t.chains * t.each == first[n], "equal chains take turns to the end");
    }
    std::printf("ok\n");
    return 0;
}
