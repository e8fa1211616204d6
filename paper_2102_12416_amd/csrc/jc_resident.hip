// Resident sweeps: many sweeps of a small block in one launch.
//
// The on-chip small-grid solver for the Jacobi sweep of paper section 4.3
// (not a design of the paper: its blocks are swept once per launch and
// exchange halos between sweeps): one work-group holds a whole block of at
// most 32 planes and (nx + 1) / 2 * ny <= 512 cell pairs and runs any number
// of Jacobi sweeps on it without leaving the compute unit, so a small solve
// costs one launch per window instead of one per sweep (or per two or three),
// and the block's cells cross HBM once per launch.
//
// Each thread owns the z columns of two adjacent x cells of one row, in
// registers.  A sweep walks the columns two planes per step: every thread
// writes its iterate-k pairs of both planes into LDS, the work-group
// synchronises once, and every thread reads its x and y neighbours and forms
// both updates with the same sums in the same order as every other sweep
// kernel, so results are bitwise those of one-sweep launches.
//
// What bounds a step is LDS -- measured per wave: 13.5 cycles to write a plane's
// pairs, 6 to read the pairs of a row, 4.2 to read one cell of each pair, 34 per
// plane in all -- and then vector issue (about 45 instructions of 4 cycles per
// step on each of four SIMDs).  The design follows from that:
//  - Sweeps walk up and down in turn.  Going up, the update of plane p goes to
//    register slot p - 1, whose old plane is no longer needed; going down, back
//    to slot p.  No plane's update waits in extra registers or is copied.
//  - Of the left and right pairs a thread reads only the cell it needs.
//    (First and second cells in separate arrays cost 38 cycles per plane.)
//  - The four plane buffers (plane z in buffer (z - 1) mod 4) lie at a
//    compile-time distance, and each buffer is followed by the ghost rings of
//    its planes, so an address is one register plus an immediate: an inner
//    thread's neighbour always sits at the same place of the plane's buffer,
//    and a thread on the block's edge advances its register by one ring slot
//    every fourth plane.
//  - A phase between two barriers reads the next step's neighbours, writes the
//    planes of the step after it and computes the current step, so LDS works
//    while the vector units do.
// Measured on MI355X, us per sweep without / with a source (before: addresses
// computed per read, each step's LDS, barrier and arithmetic in a row): 32^3
// 6.95 / 9.0 -> 6.05 / 6.8, 16^3 2.60 / 3.24 -> 2.03 / 2.25, 8^3 1.17 / 1.53 ->
// 0.90 / 0.99; 1024 grids of 32^3 822 -> 1017 GLUP/s with a source.  Per step of
// 32^3 LDS works 568 of 920 cycles and each SIMD issues for 420; what is left is
// the chain from a step's first add to its last write and the barrier.
// A buffer is written two steps after it was read, with a barrier between.
// Where a sweep turns, its first two steps' planes are written, a barrier, its
// first neighbours are read, and another barrier protects them from the third
// step's planes: steps + 1 barriers per sweep.
//
// Blocks of up to four planes (FLAT) have their own build, with registers for
// four planes only.  Two steps have no third and need no such barrier; a single
// step takes the two halves of the buffers in turn, one barrier per sweep.  (The
// build for 32 planes has no registers left for these paths: with them 32^3 took
// 15.0 us per sweep instead of 8.1.)  One block, us per sweep without / with a
// source, in the build for 32 planes and here: 32 x 32 x 4 1.09 / 1.14 and 0.91 /
// 0.93; 256 x 2 x 2 0.55 / 0.56 and 0.33 / 0.33; 1024 x 1 x 1 0.57 / 0.59 and
// 0.32 / 0.32.

#include <hip/hip_runtime.h>

#include <type_traits>

#include "jc_div6.h"
#include "jc_kernels.h"
#include "jc_storage.h"

namespace jc {

namespace {

template <int I, int N, typename F>
__device__ __forceinline__ void up_steps(F& f)
{
    if constexpr (I < N) {
        if (f(std::integral_constant<int, I>{}))
            up_steps<I + 1, N>(f);
    }
}

template <int I, typename F>
__device__ __forceinline__ void down_steps(F& f)
{
    if constexpr (I >= 0) {
        f(std::integral_constant<int, I>{});
        down_steps<I - 1>(f);
    }
}

// The neighbours of a thread's pair in the two planes of a step.
struct Around {
    double xm[2], xp[2];
    v2d ym[2], yp[2];
};

// NZM: the most planes of a block.  ODD: some block swept has an odd nx.
// STAGGER: see `early`.  R: bytes of a plane buffer with its ghost rings.
template <int NZM, bool SRC, bool ODD, bool STAGGER, int R>
__global__ void __launch_bounds__(kResidentMaxPairs)
k_resident(const BlockDesc* __restrict__ blocks, const Item* __restrict__ items, int parity, int nsweeps)
{
    constexpr bool FLAT = NZM <= kResidentFlatPlanes;
    constexpr int NBM = (NZM + 1) / 2;
    __shared__ v2d lds[4 * R / 16];
    const int blk = items ? items[blockIdx.x].block : 0;
    const int p0 = parity ^ (items ? items[blockIdx.x].flip : 0);
    const BlockDesc* B = blocks + blk;
    const int nx = B->n[0], ny = B->n[1], nz = B->n[2];
    const int nb = (nz + 1) >> 1;                 // steps per sweep
    const int ep = (nx + 1) >> 1;                 // cell pairs per row
    const int npair = ep * ny;
    // byte offset of a buffer's ring slots (idle lanes write below it); a slot:
    // the pairs of rows y = 0 and y = ny + 1, the columns x = 0 and x = nx + 1
    const int ring = 16 * ((npair + 63) & ~63);
    const int slot = 16 * (2 * ep + ny);
    const int64_t pitch = B->pitch, plane = B->plane;
    const double* __restrict__ u = B->u[p0];
    const int t = threadIdx.x;
    char* const base = reinterpret_cast<char*>(lds);

    for (int i = t; i < nz * ny; i += blockDim.x) {
        const int z = i / ny, y = i % ny;
        const int64_t o = (int64_t)(z + 1) * plane + (int64_t)(y + 1) * pitch;
        double* const r = reinterpret_cast<double*>(base + (z & 3) * R + ring + (z >> 2) * slot + 32 * ep);
        r[y] = u[o];
        r[ny + y] = u[o + nx + 1];
        if (FLAT && nb == 1) {                    // for the sweeps in the other two buffers
            double* const q = r + 2 * R / 8;
            q[y] = u[o];
            q[ny + y] = u[o + nx + 1];
        }
    }
    for (int i = t; i < nz * ep; i += blockDim.x) {
        const int z = i / ep, j = i % ep;
        const int64_t o = (int64_t)(z + 1) * plane + (2 * j + 1);
        v2d* const r = reinterpret_cast<v2d*>(base + (z & 3) * R + ring + (z >> 2) * slot);
        r[j] = *(const v2d JC_GLOBAL*)(u + o);
        r[ep + j] = *(const v2d JC_GLOBAL*)(u + o + (int64_t)(ny + 1) * pitch);
        if (FLAT && nb == 1) {
            v2d* const q = r + 2 * R / 16;
            q[j] = r[j];
            q[ep + j] = r[ep + j];
        }
    }

    // waves without a pair only keep the barriers company
    if (__builtin_amdgcn_readfirstlane(t & ~63) >= npair) {
        __syncthreads();
        const int barriers = FLAT ? nb : nb + 1;      // per sweep
        for (int k = 0; k < nsweeps; ++k)
            for (int i = 0; i < barriers; ++i)
                __syncthreads();
        return;
    }

    const bool live = t < npair;
    const int j = live ? t % ep : 0, y0 = live ? t / ep : 0;
    const bool b_ok = 2 * j + 2 <= nx;            // else the pair's second cell is the x = nx + 1 ghost
    const int64_t own = (int64_t)(y0 + 1) * pitch + 2 * j + 1;

    // byte offsets of the neighbours in the first plane's buffer, and the
    // advance per ring slot
    const bool e_xm = live && j == 0, e_xp = live && j == ep - 1, e_ym = live && y0 == 0, e_yp = live && y0 == ny - 1;
    int r_xm = !live ? 16 * t : e_xm ? ring + 32 * ep + 8 * y0 : 16 * t - 8;
    int r_xp = !live ? 16 * t : e_xp ? ring + 32 * ep + 8 * ny + 8 * y0 : 16 * t + 16;
    int r_ym = !live ? 16 * t : e_ym ? ring + 16 * j : 16 * (t - ep);
    int r_yp = !live ? 16 * t : e_yp ? ring + 16 * (ep + j) : 16 * (t + ep);
    const int i_xm = e_xm ? slot : 0, i_xp = e_xp ? slot : 0, i_ym = e_ym ? slot : 0, i_yp = e_yp ? slot : 0;

    // plane p in slot p before a sweep up, in slot p - 1 before a sweep down;
    // the top ghost plane above them; the bottom ghosts apart
    double ca[NZM + 2], cb[NZM + 2], ga, gb;
    {
        const v2d g = *(const v2d JC_GLOBAL*)(u + own);
        ga = g.x;
        gb = g.y;
    }
    ca[0] = cb[0] = 0.0;
#pragma unroll
    for (int z = 1; z <= NZM + 1; ++z) {
        ca[z] = cb[z] = 0.0;
        if (z <= nz + 1) {
            const v2d v = *(const v2d JC_GLOBAL*)(u + (int64_t)z * plane + own);
            ca[z] = v.x;
            cb[z] = v.y;
        }
    }
    // source of the two planes of step I in slot I & 1, loaded two steps
    // ahead; where a sweep turns, the last two steps' values serve again (the
    // second plane of a one-plane step repeats the first)
    const int own32 = (int)own;
    const double* const src = B->b;
    double qa[2][2] = {}, qb[2][2] = {};
    auto load_src = [&](int step, double* da, double* db) __attribute__((always_inline)) {
        const int z1 = 2 * step + 1, z2 = z1 + 1 <= nz ? z1 + 1 : z1;
        int o = own32;                            // opaque: no step's address is held in registers
        asm volatile("" : "+v"(o));
        const v2d q1 = *(const v2d JC_GLOBAL*)(src + (int64_t)z1 * plane + o);
        const v2d q2 = *(const v2d JC_GLOBAL*)(src + (int64_t)z2 * plane + o);
        da[0] = q1.x;
        db[0] = q1.y;
        da[1] = q2.x;
        db[1] = q2.y;
    };
    if (SRC) {
        load_src(0, qa[0], qb[0]);
        if (nb > 1)
            load_src(1, qa[1], qb[1]);
    }
    __syncthreads();                              // ghost rings written

    // write the pairs of step I's planes (OFF: slot of plane p is p - OFF) into
    // buffers (2 I + 2 HALF) mod 4 and the next
    auto put = [&](auto ic, auto offc, auto halfc) __attribute__((always_inline)) {
        constexpr int I = decltype(ic)::value, OFF = decltype(offc)::value;
        constexpr int Z = 2 * I + 1, B0 = ((2 * I + 2 * decltype(halfc)::value) & 3) * (R / 16);
        v2d w;
        w.x = ca[Z - OFF];
        w.y = cb[Z - OFF];
        lds[t + B0] = w;
        w.x = ca[Z + 1 - OFF];
        w.y = cb[Z + 1 - OFF];
        lds[t + B0 + R / 16] = w;
    };
    auto get = [&](auto ic, Around& n, auto halfc) __attribute__((always_inline)) {
        constexpr int I = decltype(ic)::value, B0 = ((2 * I + 2 * decltype(halfc)::value) & 3) * R;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            n.xm[k] = *reinterpret_cast<const double*>(base + r_xm + (B0 + k * R));
            n.xp[k] = *reinterpret_cast<const double*>(base + r_xp + (B0 + k * R));
            n.ym[k] = *reinterpret_cast<const v2d*>(base + r_ym + (B0 + k * R));
            n.yp[k] = *reinterpret_cast<const v2d*>(base + r_yp + (B0 + k * R));
        }
    };
    // advance the edge threads' ring registers; opaque, or the compiler would
    // hold every step's addresses in registers
    auto ring_up = [&]() __attribute__((always_inline)) {
        r_xm += i_xm;
        r_xp += i_xp;
        r_ym += i_ym;
        r_yp += i_yp;
        asm volatile("" : "+v"(r_xm), "+v"(r_xp), "+v"(r_ym), "+v"(r_yp));
    };
    auto ring_down = [&]() __attribute__((always_inline)) {
        r_xm -= i_xm;
        r_xp -= i_xp;
        r_ym -= i_ym;
        r_yp -= i_yp;
        asm volatile("" : "+v"(r_xm), "+v"(r_xp), "+v"(r_ym), "+v"(r_yp));
    };
    // the updates of step I's planes; going up (OFF 0) plane p's update goes to
    // slot p - 1, going down (OFF 1) to slot p.  TOP: the step may hold the top
    // plane (alone, if nz is odd), and the top ghost plane moves along.
    auto update = [&](auto ic, auto offc, auto topc, int top, const Around& n) __attribute__((always_inline)) {
        constexpr int I = decltype(ic)::value, OFF = decltype(offc)::value;
        constexpr bool TOP = decltype(topc)::value;
        constexpr int Z = 2 * I + 1, P1 = Z - OFF, P2 = P1 + 1;      // slots of planes Z, Z + 1
        constexpr int T1 = OFF ? Z : Z - 1, T2 = T1 + 1;             // slots of their updates
        constexpr int SET = I & 1;
        const double a1 = ca[P1], b1 = cb[P1], a2 = ca[P2], b2 = cb[P2];
        const double za1 = Z == 1 ? ga : ca[Z == 1 ? 0 : P1 - 1], zb1 = Z == 1 ? gb : cb[Z == 1 ? 0 : P1 - 1];
        if (TOP && Z == top) {                    // the top plane alone: below plane nz + 1
            double sa1 = n.xm[0] + b1;
            double sb1 = a1 + n.xp[0];
            sa1 = sa1 + n.ym[0].x;
            sb1 = sb1 + n.ym[0].y;
            sa1 = sa1 + n.yp[0].x;
            sb1 = sb1 + n.yp[0].y;
            sa1 = sa1 + za1;
            sb1 = sb1 + zb1;
            sa1 = sa1 + a2;
            sb1 = sb1 + b2;
            if (SRC) {
                sa1 = sa1 + qa[SET][0];
                sb1 = sb1 + qb[SET][0];
            }
            double va1, vb1;
            div6_pair(sa1, sb1, va1, vb1);
            ca[T2] = a2;
            cb[T2] = b2;
            ca[T1] = va1;
            cb[T1] = ODD && !b_ok ? b1 : vb1;
            return;
        }
        // in rounds of the four cells' independent operations, kept in this
        // order: a binary64 result is ready after about 12 cycles, three
        // operations later
        double sa1 = n.xm[0] + b1, sb1 = a1 + n.xp[0], sa2 = n.xm[1] + b2, sb2 = a2 + n.xp[1];
        __builtin_amdgcn_sched_barrier(0);
        sa1 = sa1 + n.ym[0].x;
        sb1 = sb1 + n.ym[0].y;
        sa2 = sa2 + n.ym[1].x;
        sb2 = sb2 + n.ym[1].y;
        __builtin_amdgcn_sched_barrier(0);
        sa1 = sa1 + n.yp[0].x;
        sb1 = sb1 + n.yp[0].y;
        sa2 = sa2 + n.yp[1].x;
        sb2 = sb2 + n.yp[1].y;
        __builtin_amdgcn_sched_barrier(0);
        sa1 = sa1 + za1;
        sb1 = sb1 + zb1;
        sa2 = sa2 + a1;
        sb2 = sb2 + b1;
        __builtin_amdgcn_sched_barrier(0);
        sa1 = sa1 + a2;
        sb1 = sb1 + b2;
        sa2 = sa2 + ca[P2 + 1];
        sb2 = sb2 + cb[P2 + 1];
        if (SRC) {
            __builtin_amdgcn_sched_barrier(0);
            sa1 = sa1 + qa[SET][0];
            sb1 = sb1 + qb[SET][0];
            sa2 = sa2 + qa[SET][1];
            sb2 = sb2 + qb[SET][1];
        }
        __builtin_amdgcn_sched_barrier(0);
        double va1, vb1, va2, vb2;
        div6_quad(sa1, sb1, sa2, sb2, va1, vb1, va2, vb2);
        if (TOP) {
            constexpr int from = P2 + 1, to = OFF ? P2 + 2 : P2;
            if constexpr (to < NZM + 2) {
                ca[to] = ca[from];
                cb[to] = cb[from];
            }
        }
        ca[T2] = va2;
        cb[T2] = ODD && !b_ok ? b2 : vb2;
        ca[T1] = va1;
        cb[T1] = ODD && !b_ok ? b1 : vb1;
    };
    using Up = std::integral_constant<int, 0>;
    using Down = std::integral_constant<int, 1>;
    using No = std::false_type;
    using Yes = std::true_type;
    using Low = std::integral_constant<int, 0>;
    using High = std::integral_constant<int, 1>;
    using First = std::integral_constant<int, 0>;
    Around around[2];                             // of step I in I & 1
    // nz, opaque to the compiler in every step: it would otherwise hold every
    // step's conditions in registers
    auto opaque = [](int v) __attribute__((always_inline)) {
        asm volatile("" : "+s"(v));
        return v;
    };
    // With two waves on a SIMD (STAGGER: more than 256 pairs) one uses LDS before
    // it computes and the other after: issue is in order, so with all waves at
    // LDS first the vector units would wait for its queue (32^3: 6.1 us per
    // sweep against 7.1).  Fewer waves only lose by it (16^3: 10 %).
    const bool early = !STAGGER || (__builtin_amdgcn_readfirstlane(t) & 256) == 0;
    auto up = [&](auto ic) __attribute__((always_inline)) -> bool {
        constexpr int I = decltype(ic)::value;
        using Next = std::integral_constant<int, I + 1>;
        using Next2 = std::integral_constant<int, I + 2>;
        const int top = opaque(nz);
        if constexpr (I + 1 < NBM) {
            if (2 * I + 2 < top) {
                auto lds_work = [&]() __attribute__((always_inline)) {
                    if constexpr ((Next::value & 1) == 0)
                        ring_up();
                    get(Next{}, around[(I + 1) & 1], Low{});
                    if constexpr (I + 2 < NBM) {
                        if (2 * I + 4 < top)
                            put(Next2{}, Up{}, Low{});
                    }
                };
                if (early)
                    lds_work();
                update(ic, Up{}, No{}, top, around[I & 1]);
                if constexpr (SRC && I + 2 < NBM) {
                    if (2 * I + 4 < top)
                        load_src(I + 2, qa[I & 1], qb[I & 1]);
                }
                if (!early)
                    lds_work();
                __syncthreads();
                return true;
            }
        }
        update(ic, Up{}, Yes{}, top, around[I & 1]);
        return false;
    };
    auto down = [&](auto ic) __attribute__((always_inline)) {
        constexpr int I = decltype(ic)::value;
        using Next = std::integral_constant<int, I - 1>;
        using Next2 = std::integral_constant<int, I - 2>;
        const int top = opaque(nz);
        if (2 * I >= top)
            return;
        auto lds_work = [&]() __attribute__((always_inline)) {
            if constexpr (I >= 1) {
                if constexpr ((I & 1) == 0)
                    ring_down();
                get(Next{}, around[(I - 1) & 1], Low{});
            }
            if constexpr (I >= 2)
                put(Next2{}, Down{}, Low{});
        };
        if (2 * I + 2 >= top) {                   // the sweep's first step
            put(ic, Down{}, Low{});
            if constexpr (I >= 1)
                put(Next{}, Down{}, Low{});
            __syncthreads();
            get(ic, around[I & 1], Low{});
            if constexpr (!FLAT)
                __syncthreads();
            lds_work();
            update(ic, Down{}, Yes{}, top, around[I & 1]);
        } else {
            if (early)
                lds_work();
            update(ic, Down{}, No{}, top, around[I & 1]);
            if (!early)
                lds_work();
        }
        if constexpr (SRC && I >= 2)
            load_src(I - 2, qa[I & 1], qb[I & 1]);
        if constexpr (I >= 1)
            __syncthreads();
    };
    if (FLAT && nb == 1) {
        for (int k = 0; k < nsweeps; k += 2) {
            put(First{}, Up{}, Low{});
            __syncthreads();
            get(First{}, around[0], Low{});
            update(First{}, Up{}, Yes{}, nz, around[0]);
            if (k + 1 < nsweeps) {
                put(First{}, Down{}, High{});
                __syncthreads();
                get(First{}, around[0], High{});
                update(First{}, Down{}, Yes{}, nz, around[0]);
            }
        }
    } else {
        for (int k = 0; k < nsweeps; k += 2) {
            put(First{}, Up{}, Low{});
            if (FLAT || nb > 1)
                put(std::integral_constant<int, 1>{}, Up{}, Low{});
            __syncthreads();
            get(First{}, around[0], Low{});
            if constexpr (!FLAT)
                __syncthreads();
            up_steps<0, NBM>(up);
            if (k + 1 < nsweeps)
                down_steps<NBM - 1>(down);
        }
    }

    double* const dst = B->u[p0 ^ (nsweeps & 1)];
    if (live) {
        const bool shifted = (nsweeps & 1) != 0;  // the last sweep went up
#pragma unroll
        for (int z = 1; z <= NZM; ++z) {
            if (z <= nz) {
                v2d v;
                v.x = shifted ? ca[z - 1] : ca[z];
                v.y = shifted ? cb[z - 1] : cb[z];
                *(v2d JC_GLOBAL*)(dst + (int64_t)z * plane + own) = v;
            }
        }
    }
}

}  // namespace

hipError_t launch_resident(const BlockDesc* blocks, const Item* items, int nitems, const ResidentShape& shape,
                           int parity, int nsweeps, bool src, hipStream_t s)
{
    const int n = items ? nitems : 1;
    if (n <= 0 || nsweeps <= 0)
        return hipSuccess;
    if (shape.pairs < 1 || shape.pairs > kResidentMaxPairs || shape.planes < 1 || shape.planes > kResidentMaxPlanes)
        return hipErrorInvalidValue;
    const dim3 grid(n), block((shape.pairs + 63) / 64 * 64);
#define JC_RESIDENT_LAUNCH(NZM, SRC, ODD, STAGGER, R)                                                            \
    hipLaunchKernelGGL((k_resident<NZM, SRC, ODD, STAGGER, R>), grid, block, 0, s, blocks, items, parity, nsweeps)
    // the smallest buffers that hold every block: small blocks share a compute unit
#define JC_RESIDENT_CASE(NZM, R, STAGGER)                                                                       \
    if (shape.planes <= NZM && shape.region <= R && (!STAGGER || shape.pairs > 256)) {                            \
        if (src && shape.odd)                                                                                   \
            JC_RESIDENT_LAUNCH(NZM, true, true, STAGGER, R);                                                     \
        else if (src)                                                                                           \
            JC_RESIDENT_LAUNCH(NZM, true, false, STAGGER, R);                                                    \
        else if (shape.odd)                                                                                     \
            JC_RESIDENT_LAUNCH(NZM, false, true, STAGGER, R);                                                    \
        else                                                                                                    \
            JC_RESIDENT_LAUNCH(NZM, false, false, STAGGER, R);                                                   \
        return hipGetLastError();                                                                               \
    }
    JC_RESIDENT_CASE(kResidentFlatPlanes, kResidentFlatRegions[0], false)
    JC_RESIDENT_CASE(kResidentFlatPlanes, kResidentFlatRegions[1], false)
    JC_RESIDENT_CASE(kResidentFlatPlanes, kResidentFlatRegions[2], false)
    JC_RESIDENT_CASE(kResidentMaxPlanes, kResidentRegions[0], false)
    JC_RESIDENT_CASE(kResidentMaxPlanes, kResidentRegions[1], false)
    JC_RESIDENT_CASE(kResidentMaxPlanes, kResidentRegions[2], false)
    JC_RESIDENT_CASE(kResidentMaxPlanes, kResidentRegions[3], true)
    JC_RESIDENT_CASE(kResidentMaxPlanes, kResidentRegions[3], false)
    JC_RESIDENT_CASE(kResidentMaxPlanes, kResidentRegions[4], false)
#undef JC_RESIDENT_CASE
#undef JC_RESIDENT_LAUNCH
    return hipErrorInvalidValue;
}

}  // namespace jc
