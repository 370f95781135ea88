// The rule of the first tiles on the CPU (tests/test_first_tiles_rule.py): lines of "S B T V blocks words wanted" in, numbers of tiles out.  No GPU call.
#include <algorithm>
#include <cstdio>

#include "../paper_1806_00588_amd/csrc/fused.h"

int main() {
    int S, B, T, V, blocks, wanted;
    double words;
    while (std::scanf("%d %d %d %d %d %lf %d", &S, &B, &T, &V, &blocks, &words, &wanted) == 7)
        std::printf("%d\n", lshbeam::first_tiles_count(S, B, T, V, blocks, words, wanted));
    return 0;
}
