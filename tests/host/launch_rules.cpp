// Launch rules of the library that depend on sizes alone, printed for the CPU
// tests.  Built with the host compiler against the library's internal header;
// no GPU code runs.
#include <cstdio>

#include "../../paper_2504_00987_amd/csrc/labs_internal.h"

using namespace liblabs;

int main() {
    for (int first : {6, 7})
        for (int64_t walks : {1, 64, 4095, 4096, 4097, 1 << 20}) {
            const GroupForm f = group2_form(first, walks, 4096);
            std::printf("group2 %d %lld %d %d\n", kClassMaxN[first], (long long)walks, f.lanes,
                        f.neighbours);
        }
    for (int words : {1, 2, 4})
        for (int64_t replicas : {1, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 1 << 22})
            for (int K = 2; K <= LABS_MAX_K; ++K)
                for (int children = 1; children <= LABS_MAX_CHILDREN; ++children)
                    for (int gens : {1, 3, 1 << 20})
                        std::printf("memetic %d %lld %d %d %d %d\n", words, (long long)replicas, K,
                                    children, gens,
                                    memetic_waves(words, replicas, K, children, gens, 256));
    for (int classes = 1; classes < 8; ++classes)
        for (int64_t replicas : {1, 1024, 1025, 4096, 4097, 1 << 22})
            std::printf("init %d %lld %d\n", classes, (long long)replicas,
                        init_waves(replicas, classes, 256));
    // every subset of present classes, as a batch of one walk per present class
    for (int mask = 0; mask < (1 << kWalkClasses); ++mask)
        for (int lanes : {64, 32, 16}) {
            int64_t ce[kWalkClasses];
            int64_t end = 0;
            for (int c = 0; c < kWalkClasses; ++c) ce[c] = end += (mask >> c) & 1;
            const WalkGroups g = tabu_launch_groups(ce, lanes);
            for (int i = 0; i < g.n; ++i)
                std::printf("launch %d %d %d %d %d %d\n", mask, lanes, g.first[i], g.last[i],
                            g.kind[i], kClassMaxN[g.first[i]]);
        }
    return 0;
}
