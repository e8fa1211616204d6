// Every block shape that resident sweeps accept against the buffer sizes that
// the kernel is built for (paper_2102_12416_amd/csrc/jc_resident.h), host only.
// Built and run by tests/test_resident_limits_cpu.py.  Prints "shapes <n> unfit
// <shapes that no buffer holds> crowded <shapes of which less than two thirds
// of the work-groups share a compute unit that could>" and lists the first.
#include <algorithm>
#include <cstdio>

#include "jc_resident.h"

int main()
{
    const long lds = 160 * 1024, waves_per_cu = 8;     // two waves on each of four SIMDs
    long shapes = 0, unfit = 0, crowded = 0;
    for (int nx = 1; nx <= 1024; ++nx)
        for (int ny = 1; ny <= 512; ++ny)
            for (int nz = 1; nz <= 32; ++nz) {
                if (!jc::resident_fits(nx, ny, nz))
                    continue;
                ++shapes;
                jc::ResidentShape s;
                s.add(nx, ny, nz);
                long region = 0;
                for (int r : jc::kResidentRegions)
                    if (!region && s.region <= r)
                        region = r;
                bool flat = nz > jc::kResidentFlatPlanes;
                for (int r : jc::kResidentFlatRegions)
                    flat = flat || s.region <= r;
                if (!region || !flat) {
                    if (unfit++ < 10)
                        std::fprintf(stderr, "%d x %d x %d: %ld bytes, no buffer\n", nx, ny, nz, (long)s.region);
                    continue;
                }
                const long waves = (s.pairs + 63) / 64, most = std::max(1l, waves_per_cu / waves);
                const long could = std::min(most, lds / (4 * (long)s.region)), held = std::min(most, lds / (4 * region));
                if (3 * held < 2 * could && crowded++ < 10)
                    std::fprintf(stderr, "%d x %d x %d: %ld of %ld work-groups\n", nx, ny, nz, held, could);
            }
    std::printf("shapes %ld unfit %ld crowded %ld\n", shapes, unfit, crowded);
    return unfit || crowded;
}
