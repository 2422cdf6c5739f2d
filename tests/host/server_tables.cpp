// labs_server_create when its slot tables do not fit in host memory: the call
// returns a status, nothing is thrown across the C boundary.  Allocations of
// one size fail at a time; the sizes are those of tables of max_slots entries.
// No GPU code runs.
#include <cstdio>
#include <cstdlib>
#include <new>

#include "../../paper_2504_00987_amd/csrc/labs_handle.h"

static std::size_t failing = 0;

void *operator new(std::size_t n) {
    void *p = n == failing ? nullptr : std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

int main() {
    labs_memetic_params p{};
    p.K = 2;
    p.chunk = 1;
    const int32_t slots = 1 << 20;
    for (std::size_t entry : {sizeof(int64_t), sizeof(int)}) {
        labs_handle h;
        labs_server *s = nullptr;
        failing = slots * entry;
        const int rc = labs_server_create(&h, &p, slots, &s);
        failing = 0;
        std::printf("%d %d %d\n", rc, (int)(s == nullptr), (int)!h.last_error.empty());
    }
    return 0;
}
