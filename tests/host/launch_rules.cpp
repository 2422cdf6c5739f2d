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
    return 0;
}
