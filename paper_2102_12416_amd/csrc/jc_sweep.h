// Device helpers shared by the sweep kernels: the work-group order over the
// XCDs, pacing, and the arrays a sweep works on.
#pragma once

#include <hip/hip_runtime.h>

#include "jc_storage.h"
#include "jc_types.h"

namespace jc {

namespace {

// Work-groups are dispatched round-robin over the 8 XCDs of the chip
// (work-group i to XCD i mod 8).  Give each XCD a contiguous range of
// logical tiles so that tiles sharing halo rows run under the same L2.
__device__ __forceinline__ int logical_block(int bid, int nblocks)
{
    const int per = nblocks >> 3;           // nblocks is a multiple of 8
    return (bid & 7) * per + (bid >> 3);
}

// Pacing.  The work-groups of a launch advance at different rates (a tile
// on a Dirichlet face reads its ghosts from a compact column, other tiles
// read their x halo from the neighbour tile's lines, work-groups sit at
// different distances from the memory they stream), and the launch ends
// with the slowest: measured on the 512^3 launch of 256 tiles, they took
// 359-396 us, so the compute units of the fast ones idled through the
// tail.  With a pace, a work-group waits before plane step k until k *
// pace ticks of the chip's constant 100 MHz clock have passed since it
// started: the fast ones are held to the pace and the memory traffic of
// the slow ones runs without their competition, so all finish together.
// The pace is tuned by timing (jc_autotune); 0 = none.  Each wait is
// bounded (4096 short sleeps), and results do not depend on it.
__device__ __forceinline__ void pace_wait(uint64_t due)
{
    for (int i = 0; i < 4096 && __builtin_amdgcn_s_memrealtime() < due; ++i)
        __builtin_amdgcn_s_sleep(1);
}

// Which arrays of a block a sweep works on: the iterate u (with source b)
// or the refinement correction d (with source r_lo).
enum { FIELD_U = 0, FIELD_D = 1 };

template <typename T, int FIELD> struct Fld;

template <typename T> struct Fld<T, FIELD_U> {
    __device__ static const T* src(const BlockDesc* B, int p) { return B->u[p]; }
    __device__ static T* dst(const BlockDesc* B, int p) { return B->u[p ^ 1]; }
    __device__ static const T* source(const BlockDesc* B) { return B->b; }
    __device__ static const T* gin(const BlockDesc* B, int f, int s) { return B->gin[f][s]; }
    __device__ static T* gout(const BlockDesc* B, int f, int s) { return B->gout[f][s]; }
    __device__ static const T* xg(const BlockDesc* B, int f) { return B->xg[f]; }
    __device__ static int64_t pitch(const BlockDesc* B) { return B->pitch; }
    __device__ static int64_t plane(const BlockDesc* B) { return B->plane; }
};

template <typename T> struct Fld<T, FIELD_D> {
    __device__ static const T* src(const BlockDesc* B, int p) { return static_cast<const T*>(B->d[p]); }
    __device__ static T* dst(const BlockDesc* B, int p) { return static_cast<T*>(B->d[p ^ 1]); }
    __device__ static const T* source(const BlockDesc* B) { return static_cast<const T*>(B->rlo); }
    __device__ static const T* gin(const BlockDesc* B, int f, int s)
    {
        return static_cast<const T*>(B->lgin[f][s]);
    }
    __device__ static T* gout(const BlockDesc* B, int f, int s) { return static_cast<T*>(B->lgout[f][s]); }
    __device__ static const T* xg(const BlockDesc* B, int f) { return static_cast<const T*>(B->lxg[f]); }
    __device__ static int64_t pitch(const BlockDesc* B) { return B->lpitch; }
    __device__ static int64_t plane(const BlockDesc* B) { return B->lplane; }
};

}  // namespace

}  // namespace jc
