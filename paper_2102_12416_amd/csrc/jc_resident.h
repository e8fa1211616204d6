// Shape limits of the resident sweep kernel (libjc, internal): shared by
// the host runtime, which validates contexts and groups against them, and
// the kernel's launcher.
#pragma once

#include <stdint.h>

namespace jc {

// Blocks that one work-group can sweep many times on chip (the resident
// sweep kernel): at most 32 planes, (nx + 1) / 2 * ny <= 512 cell pairs
// (one thread each), and four planes plus the ghost ring of every plane
// within 64 KiB.  This is the interface's limit; the kernel's own buffers
// (below) round both up and hold every shape within it.
constexpr int kResidentMaxPlanes = 32;
constexpr int kResidentMaxPairs = 512;
constexpr int64_t kResidentMaxLds = 65536;

inline constexpr int64_t resident_lds_bytes(int64_t nx, int64_t ny, int64_t nz)
{
    const int64_t pw = 2 * ((nx + 1) / 2);
    return 8 * (4 * ny * pw + 2 * nz * ny + 2 * nz * pw);
}

inline constexpr bool resident_fits(int64_t nx, int64_t ny, int64_t nz)
{
    return nx >= 1 && ny >= 1 && nz >= 1 && nz <= kResidentMaxPlanes && (nx + 1) / 2 * ny <= kResidentMaxPairs &&
           resident_lds_bytes(nx, ny, nz) <= kResidentMaxLds;
}

// Bytes of one of the kernel's four plane buffers with its ghost rings: the
// pairs (rounded up to whole waves) and a quarter of the planes' rings.  The
// largest over all blocks that fit is 24592 (1024 x 1 x 1).
inline constexpr int64_t resident_region_bytes(int64_t nx, int64_t ny, int64_t nz)
{
    const int64_t ep = (nx + 1) / 2;
    return 16 * ((ep * ny + 63) / 64 * 64 + (nz + 3) / 4 * (2 * ep + ny));
}

// Buffer sizes the kernel is built for.  Its registers let 8 waves share a
// compute unit, so these are the largest buffers of which 8, 6, 4 and 2
// work-groups of fewer waves share its 160 KiB, and every shape that fits.  (With
// 16 KiB for every shape above 16^3 two work-groups of 16 x 10 x 32 cells, of two
// waves each, shared a compute unit: 9.7 us per sweep of 1024 of them, 6.3 now,
// with a source 10.9 and 7.1.)
constexpr int kResidentRegions[5] = {5120, 6656, 10240, 20480, 24832};

// Blocks of up to this many planes have a build of their own, and its buffers.
constexpr int kResidentFlatPlanes = 4;
constexpr int kResidentFlatRegions[3] = {5120, 10240, 24832};

// What a launch has to hold: the largest of each over the blocks it sweeps.
struct ResidentShape {
    int pairs = 0, planes = 0;
    int64_t region = 0;
    bool odd = false;           // some nx is odd

    void add(int64_t nx, int64_t ny, int64_t nz)
    {
        const int64_t r = resident_region_bytes(nx, ny, nz);
        pairs = (int)((nx + 1) / 2 * ny) > pairs ? (int)((nx + 1) / 2 * ny) : pairs;
        planes = (int)nz > planes ? (int)nz : planes;
        region = r > region ? r : region;
        odd = odd || (nx & 1);
    }
};

}  // namespace jc
