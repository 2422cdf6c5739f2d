// Which batches a tuned launch serves, printed for the CPU tests: a launch is
// put where tuning on `tuned` walks keeps it, then asked for by batches of
// other sizes.  Built with the host compiler against the library; no GPU code
// runs.
#include <cstdio>

#include "../../paper_2504_00987_amd/csrc/labs_handle.h"

using namespace liblabs;

int main() {
    const labs_launch mark{128, 2, 1, 3, 0};
    for (int n : {12, 16, 24, 32, 33, 64, 200})
        for (int64_t tuned : {1, 1024, 2048, 2049, 4096, 4097, 16384})
            for (int64_t walks : {1, 1024, 2048, 2049, 4096, 4097, 16384}) {
                labs_handle h;
                const labs_launch plain = choose_launch(&h, n, n, walks);
                const labs_launch at_tuned = choose_launch(&h, n, n, tuned);
                h.tuned[tuned_key(n, n, tuned)] = mark;
                const labs_launch got = choose_launch(&h, n, n, walks);
                const bool same_default = plain.group_lanes == at_tuned.group_lanes &&
                                          plain.walks_per_group == at_tuned.walks_per_group;
                std::printf("tuned %d %lld %lld %d %d\n", n, (long long)tuned, (long long)walks,
                            (int)(got.groups_per_cu == mark.groups_per_cu), (int)same_default);
            }
    return 0;
}
