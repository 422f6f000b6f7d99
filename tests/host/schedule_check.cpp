// Host check of the rules that choose a CG iteration's launches.
//
// usage: schedule_check N fp64 pc n...   (pc: preconditioned)
// Prints "n:launches:blocks" for every n: 2, 3 or 4 launches of an iteration
// on a conforming mesh of n local points, and for 3 the blocks of its update.
#include <cstdio>
#include <cstdlib>

#include "../../paper_2108_12188_amd/csrc/sem_internal.h"

int main(int argc, char **argv) {
    const int N = std::atoi(argv[1]);
    const bool fp64 = std::atoi(argv[2]) != 0;
    const bool pc = std::atoi(argv[3]) != 0;
    for (int q = 4; q < argc; ++q) {
        const int64_t n = std::atoll(argv[q]);
        const int launches = n <= sem::direct_max_points(N)            ? 2
                             : sem::takes_inline_scalars(N, n, fp64, pc) ? 3
                                                                     : 4;
        const int vec = (int)((n + 1023) / 1024);      // vec_blocks up to 4096 of them
        std::printf("%lld:%d:%d\n", (long long)n, launches,
                    launches == 3 ? sem::inline_update_blocks(vec, N, fp64) : 0);
    }
    return 0;
}
