// Which lists have one chunk per workgroup: those where workgroups of four, dealt to 256 compute units in one turn or two, would
// leave a third or more of the places empty.  Every other list keeps four.  Prints the first length that does not.
#include <cstdio>

#include "sl_internal.h"

int main()
{
    sl_plan p{};
    for (int n = 1; n < 20000; ++n) {
        p.n_chunks = n;
        const int groups = (n + 3) / 4, places = groups <= 256 ? 256 : 512;
        const bool spread = 3 * (places - groups) >= places;
        for (int partial : {0, n / 32, n}) {
            p.n_partial = partial;
            const int want = spread && 32 * partial < n ? 1 : 4;
            if (sl_chunks_per_group(&p) != want) {
                std::printf("%d chunks, %d partial: %d per workgroup, want %d\n", n, partial, sl_chunks_per_group(&p), want);
                return 1;
            }
        }
        if (sl_order(&p, (unsigned)n) != 0 && n < 4096) return 1;
    }
    std::puts("ok");
    return 0;
}
