// HIP kernels of libjc for gfx950 (CDNA4, wave64).
//
// Jacobi3D, paper section 4.3: each block of the decomposition is swept
// with the 7-point stencil after its halo has been exchanged with up to
// six neighbours.  The sweep marches along z through a tile of 64 x cells
// by tile_y rows, staging each plane in LDS and keeping the z-1, z and z+1
// values of its own cells in registers, so that every interior value is
// fetched from HBM once per sweep.  The stencil is not a contraction, so
// no matrix cores are used: the kernel is bound by HBM bandwidth (16 bytes
// per cell update in FP64).
//
// Bit-exactness: the neighbour sum is formed in one fixed order and
// divided by 6, correctly rounded (jc_div6.h); the library is built with
// -ffp-contract=off, so no multiply-add is fused and every block of every
// decomposition computes the same bits for the same cell.

#include <hip/hip_runtime.h>

#include <type_traits>

#include "jc_div6.h"
#include "jc_kernels.h"
#include "jc_sweep.h"

namespace jc {

namespace {

// ---- sweep kernel: begin (its source is fingerprinted with recorded counters) ----
struct NoRlo {};

// Planes of loads a sweep keeps in flight ahead of the plane it computes:
// three.  For binary64 fields at one 16-wave work-group per CU two planes
// of 16-byte loads are too few bytes in flight to cover the memory
// latency; a bfloat16 thread loads only 4 bytes per plane and field, and
// its inner sweep at 1024^3 ran 7 % faster with three planes than with two
// (binary32 the same; four planes gained nothing for either).
template <typename T> constexpr int prefetch_planes() { return 3; }

// One work-group sweeps a tile of 2 TXP x cells (16, 32 or 64; or 96, 128 or
// 256 for binary64 storage) by TY rows of one block, marching along z.  Each thread owns two adjacent x cells of one row
// (one aligned-pair load per plane: cell x = 1 of every row starts a
// 128-byte line).  Per plane the work-group writes the plane -- its cells
// plus a one-cell halo ring -- into an LDS tile, synchronises once (the
// tile is double-buffered by plane parity) and reads its x and y
// neighbours from LDS; the z-1 / z / z+1 values of its own cells stay in
// registers.
//
// Every thread issues the same global loads in every iteration, with
// clamped addresses where it has nothing to fetch, so that the loads of
// the next planes (prefetch_planes<T>()) stay in flight while the current
// one is computed (no divergent branch around a load).  The halo ring is fetched by
// threads with a halo role: the first TXP threads the row above the tile,
// the next TXP the row below, the next TY the column left of it and the
// next TY the column right of it; the rest re-load their own cells.
//
// T / FIELD: the swept field and its storage (binary64 iterate u, or the
// correction d of the refinement stored as binary64, binary32 or
// bfloat16 with binary32 arithmetic).  FUSED: ghost cells of faces that
// have a neighbour block are read from the neighbour's face buffer of the
// input slot (the pairing's pre-posted receive side), ghost cells of
// unpaired x faces from the block's compact Dirichlet ghost columns, and
// every face cell written is also written to this block's face buffer of
// the output slot -- pack, exchange and unpack folded into the sweep.  RES: accumulate r^2
// of the input iterate, r = (b + s) - 6u, into one partial per
// work-group.  STORE: write the new iterate.  SRC: add the source (b for
// u, r_lo for d).  R: also store r rounded to R into the block's r_lo
// array (the outer pass of the refinement).
template <typename T, int FIELD, int TXP, int TY, bool FUSED, bool RES, bool STORE, bool SRC, typename R>
__global__ void __launch_bounds__(TXP * TY)
k_sweep(const BlockDesc* __restrict__ blocks, const Item* __restrict__ items, int nitems,
        int parity, double* __restrict__ partials, uint32_t pace)
{
    static_assert(TY >= 4 && TXP * TY >= 2 * TXP + 2 * TY && (TXP * TY) % 64 == 0,
                  "halo roles need 2 TXP + 2 TY threads; whole waves");
    using C = typename Tr<T>::C;
    using F = Fld<T, FIELD>;
    constexpr bool RLO = !std::is_same<R, NoRlo>::value;
    constexpr int NT = TXP * TY;
    constexpr int W = 2 * TXP;                    // tile width in cells
    constexpr int LW = W + 4;  // LDS row: col 1 = x0, cols 2..W+1 = x0+1..x0+W, up to col W+2
    __shared__ C S[2][TY + 2][LW];
    __shared__ double wsum[NT / 64];

    const int id = logical_block(blockIdx.x, gridDim.x);
    if (id >= nitems)
        return;                                   // uniform over the work-group
    const uint64_t pace_t0 = pace ? __builtin_amdgcn_s_memrealtime() : 0;
    const Item it = items[id];
    const BlockDesc* B = blocks + it.block;
    const int p = parity ^ it.flip;
    const int nx = B->n[0], ny = B->n[1], nz = B->n[2];
    const int t = threadIdx.x;
    const int lx = t % TXP;
    const int ly = t / TXP;
    const int x0 = it.x0, y0 = it.y0;
    const int x_end = min(x0 + W, nx);            // last x cell of the tile
    const int y_end = min(y0 + TY, ny);           // last row of the tile
    const int ly_last = y_end - y0 - 1;
    const int xa = x0 + 2 * lx + 1;               // this thread's cells: xa, xa + 1
    const int y = y0 + ly + 1;
    const bool row_ok = y <= ny;
    const bool a_ok = row_ok && xa <= nx;
    const bool b_ok = row_ok && xa + 1 <= nx;
    const int xlast = (nx - 1) | 1;               // start of the last aligned pair of a row
    const int xa_c = min(xa, xlast);
    const int y_c = min(y, ny);
    const int64_t pitch = F::pitch(B);
    const int64_t plane = F::plane(B);
    const int64_t ldx = face_ld(ny);              // x-face buffers: (z, y) rows
    const int64_t ldy = face_ld(nx);              // y- and z-face buffers: (z, x) / (y, x) rows
    const T* __restrict__ src = F::src(B, p);
    T* __restrict__ dst = F::dst(B, p);
    const C six = C(6);

    // own pair (xa_c, y_c) at plane zz
    const T* own = src + (int64_t)y_c * pitch + xa_c;
    const T* own_lo = own;                                        // plane 0
    const T* own_hi = own + (int64_t)(nz + 1) * plane;            // plane nz + 1
    if (FUSED) {
        const int64_t zi = (int64_t)(y_c - 1) * ldy + (xa_c - 1);
        if (F::gin(B, ZM, p)) own_lo = F::gin(B, ZM, p) + zi;
        if (F::gin(B, ZP, p)) own_hi = F::gin(B, ZP, p) + zi;
    }
    auto own_at = [&](int zz, C& a, C& b) {
        const T* q = own + (int64_t)zz * plane;
        if (FUSED) {
            q = (zz == 0) ? own_lo : q;
            q = (zz == nz + 1) ? own_hi : q;
        }
        Tr<T>::ld(q, a, b);
    };
    const T* sown = SRC ? F::source(B) + (int64_t)y_c * pitch + xa_c : nullptr;

    // halo role: the pair at hbase + zz * hstride
    const int role = t < TXP ? 0 : t < 2 * TXP ? 1 : t < 2 * TXP + TY ? 2 : t < 2 * TXP + 2 * TY ? 3 : 4;
    const T* hbase = own;
    int64_t hstride = plane;
    int hrow = 0, hcol = 0, hcomp = 0;
    bool hv0 = false, hv1 = false;
    if (role <= 1) {
        const int hl = t % TXP;
        const int hx = x0 + 2 * hl + 1;
        const int hx_c = min(hx, xlast);
        const int hy = role == 0 ? y0 : y_end + 1;
        hv0 = hx <= x_end;
        hv1 = hx + 1 <= x_end;
        hbase = src + (int64_t)hy * pitch + hx_c;
        if (FUSED) {
            const T* const gym = F::gin(B, YM, p);    // read uniformly, selected per thread
            const T* const gyp = F::gin(B, YP, p);
            const T* g = (hy == 0) ? gym : (hy == ny + 1) ? gyp : nullptr;
            if (g) {
                hbase = g - ldy + (hx_c - 1);     // value (z - 1, x - 1)
                hstride = ldy;
            }
        }
        hrow = role == 0 ? 0 : ly_last + 2;
        hcol = 2 * hl + 2;
    } else if (role <= 3) {
        const int r = t - 2 * TXP - (role == 3 ? TY : 0);
        const int hy = y0 + r + 1;
        hv0 = hy <= y_end;
        const int hy_c = min(hy, ny);
        const int hx = role == 2 ? x0 : x_end + 1;
        const int ps = (hx & 1) ? hx : hx - 1;    // aligned pair holding hx
        hcomp = (hx & 1) ? 0 : 1;
        hbase = src + (int64_t)hy_c * pitch + ps;
        // Fused: a paired face's ghosts come from the neighbour's face
        // buffer and a Dirichlet face's from its compact ghost column.
        // Staged: from the block's own column, whose 128-byte lines each
        // hold one row's x = 0 ghost and the previous row's x = nx + 1
        // ghost, both read there.  Both faces' pointers are read uniformly
        // and selected per thread (a per-thread pointer load would stall
        // the prologue).
        const T* const gxm = !FUSED ? nullptr : F::gin(B, XM, p) ? F::gin(B, XM, p) : F::xg(B, XM);
        const T* const gxp = !FUSED ? nullptr : F::gin(B, XP, p) ? F::gin(B, XP, p) : F::xg(B, XP);
        const T* g = (hx == 0) ? gxm : (hx == nx + 1) ? gxp : nullptr;
        if (g) {
            const int fi = hy_c - 1;              // value (z - 1, y - 1)
            hbase = g - ldx + (fi & ~1);
            hcomp = fi & 1;
            hstride = ldx;
        }
        hrow = r + 1;
        hcol = role == 2 ? 1 : x_end - x0 + 2;
    }

    // Face stores of the fused epilogue.  Which of this thread's cells lie
    // on an x or y face does not change along z; a tile that touches no
    // paired x or y face (most tiles) skips them with one uniform branch.
    T* const oxm = FUSED ? F::gout(B, XM, p ^ 1) : nullptr;
    T* const oxp = FUSED ? F::gout(B, XP, p ^ 1) : nullptr;
    T* const oym = FUSED ? F::gout(B, YM, p ^ 1) : nullptr;
    T* const oyp = FUSED ? F::gout(B, YP, p ^ 1) : nullptr;
    T* const ozm = FUSED ? F::gout(B, ZM, p ^ 1) : nullptr;
    T* const ozp = FUSED ? F::gout(B, ZP, p ^ 1) : nullptr;
    const bool xy_tile = FUSED && ((x0 == 0 && oxm) || (x_end == nx && oxp) || (y0 == 0 && oym) ||
                                   (y_end == ny && oyp));
    const bool f_xm = a_ok && xa == 1 && oxm;
    const bool f_xpa = a_ok && xa == nx && oxp;
    const bool f_xpb = b_ok && xa + 1 == nx && oxp;
    const bool f_ym = a_ok && y == 1 && oym;
    const bool f_yp = a_ok && y == ny && oyp;

    // LDS slots of this thread's four writes per plane (own x cells, halo
    // values).  A write with nothing to store goes to column 0, which no
    // thread reads, so the writes need no branch.
    const int lds_a = a_ok ? (ly + 1) * LW + 2 * lx + 2 : 0;
    const int lds_b = b_ok ? (ly + 1) * LW + 2 * lx + 3 : 0;
    const int lds_h0 = (role <= 3 && hv0) ? hrow * LW + hcol : 0;
    const int lds_h1 = (role <= 1 && hv1) ? hrow * LW + hcol + 1 : 0;

    const int zf = it.z0 + 1;                     // first plane of the tile
    const int zl = it.z0 + it.zlen;               // last plane of the tile
    // Register rings of RS slots: own cells, halo and source of plane p in
    // slot (p - zf) mod RS.  At step z the loads of plane z + PD are issued
    // (own cells of z - 1 .. z + PD are live), so every value has PD plane
    // steps to arrive.  Every load lands in the slot it is consumed from:
    // no register is copied while its load is in flight (such a copy waits
    // for every outstanding load).  RS is even so that the LDS buffer of a
    // step (its slot's parity) alternates across the unrolled loop.
    constexpr int PD = prefetch_planes<T>();
    static_assert(PD >= 2 && PD <= 4, "prefetch distance 2..4 planes");
    constexpr int RS = (PD + 3) & ~1;
    C ra[RS], rb[RS], ha[RS], hb[RS], sa_[RS], sb_[RS];
    own_at(zf - 1, ra[RS - 1], rb[RS - 1]);
#pragma unroll
    for (int k = 0; k < PD; ++k) {
        own_at(min(zf + k, zl + 1), ra[k], rb[k]);
        Tr<T>::ld(hbase + (int64_t)min(zf + k, zl) * hstride, ha[k], hb[k]);
    }
#pragma unroll
    for (int k = 0; k < RS; ++k)
        sa_[k] = sb_[k] = C(0);
    if (SRC) {
#pragma unroll
        for (int k = 0; k < PD; ++k)
            Tr<T>::ld(sown + (int64_t)min(zf + k, zl) * plane, sa_[k], sb_[k]);
    }

    double acc = 0.0;
    // one plane; K = (z - zf) mod RS, a compile-time slot number
    auto step = [&](int z, auto kc) {
        constexpr int K = decltype(kc)::value;
        constexpr int SM = (K + RS - 1) % RS, SC = K, SP = (K + 1) % RS, SQ = (K + PD) % RS;
        static_assert(K >= 0 && K < RS, "ring slot");
        constexpr int HC = K & 1;                 // LDS buffer of this plane
        if (pace)
            pace_wait(pace_t0 + (uint64_t)(z - zf) * pace);
        // plane z + PD goes in flight first; the last steps re-read planes
        // they already hold (cache hits) instead of branching
        const int zh = min(z + PD, zl);
        own_at(min(z + PD, zl + 1), ra[SQ], rb[SQ]);
        Tr<T>::ld(hbase + (int64_t)zh * hstride, ha[SQ], hb[SQ]);
        if (SRC)
            Tr<T>::ld(sown + (int64_t)zh * plane, sa_[SQ], sb_[SQ]);
        const C c_a = ra[SC], c_b = rb[SC];
        C (*L)[LW] = S[HC];
        C* const Lf = &S[HC][0][0];
        Lf[lds_a] = c_a;
        Lf[lds_b] = c_b;
        Lf[lds_h0] = hcomp ? hb[SC] : ha[SC];
        Lf[lds_h1] = hb[SC];
        __syncthreads();
        const C xm_a = L[ly + 1][2 * lx + 1];
        const C xp_a = b_ok ? c_b : L[ly + 1][2 * lx + 3];
        C sa = xm_a + xp_a;
        sa = sa + L[ly][2 * lx + 2];
        sa = sa + L[ly + 2][2 * lx + 2];
        sa = sa + ra[SM];
        sa = sa + ra[SP];
        C sb = c_a + L[ly + 1][2 * lx + 4];
        sb = sb + L[ly][2 * lx + 3];
        sb = sb + L[ly + 2][2 * lx + 3];
        sb = sb + rb[SM];
        sb = sb + rb[SP];
        const C s_a = sa_[SC], s_b = sb_[SC];
        if (RES) {
            const C r_a = SRC ? (s_a + sa) - six * c_a : sa - six * c_a;
            const C r_b = SRC ? (s_b + sb) - six * c_b : sb - six * c_b;
            acc = acc + (a_ok ? (double)(r_a * r_a) : 0.0);
            acc = acc + (b_ok ? (double)(r_b * r_b) : 0.0);
            // summed here: the compiler would put the sums of all unrolled
            // planes off to the last of them, and hold or spill their terms
            asm("" : "+v"(acc));
            if constexpr (RLO) {
                // r rounded to the refinement's storage, through binary32
                R* o = static_cast<R*>(B->rlo) + (int64_t)z * B->lplane + (int64_t)y * B->lpitch + xa;
                if constexpr (std::is_same<R, double>::value) {
                    if (a_ok) Tr<double>::st(o, r_a, r_b);
                } else {
                    if (a_ok) Tr<R>::st(o, (float)r_a, (float)r_b);
                }
            }
        }
        if (STORE) {
            C va, vb;
            if (SRC)
                div6_pair(sa + s_a, sb + s_b, va, vb);
            else
                div6_pair(sa, sb, va, vb);
            // past the last cell of a row the pair's second slot is the
            // x = nx + 1 ghost: write back the value it already holds
            vb = b_ok ? vb : c_b;
            const auto pk = Tr<T>::pack(va, vb);
            if (a_ok)
                Tr<T>::stpn(dst + (int64_t)z * plane + (int64_t)y * pitch + xa, pk);
            if (FUSED) {
                // a face row's padding slot takes the second value of a
                // pair that ends past the face (ld is even)
                const int64_t zfi = (int64_t)(y - 1) * ldy + (xa - 1);
                if (z == 1 && ozm && a_ok) Tr<T>::stp(ozm + zfi, pk);
                if (z == nz && ozp && a_ok) Tr<T>::stp(ozp + zfi, pk);
                if (xy_tile) {
                    const int64_t xfi = (int64_t)(z - 1) * ldx + (y - 1);
                    const int64_t yfi = (int64_t)(z - 1) * ldy + (xa - 1);
                    if (f_xm) Tr<T>::st1a(oxm + xfi, pk);
                    if (f_xpa) Tr<T>::st1a(oxp + xfi, pk);
                    if (f_xpb) Tr<T>::st1b(oxp + xfi, pk);
                    if (f_ym) Tr<T>::stp(oym + yfi, pk);
                    if (f_yp) Tr<T>::stp(oyp + yfi, pk);
                }
            }
        }
    };
#define JC_STEP(k) step(z + (k), std::integral_constant<int, (k)>{})
    int z = zf;
    if constexpr (RS == 4) {
        for (; z + 3 <= zl; z += 4) {
            JC_STEP(0);
            JC_STEP(1);
            JC_STEP(2);
            JC_STEP(3);
        }
        if (z <= zl) JC_STEP(0);
        if (z + 1 <= zl) JC_STEP(1);
        if (z + 2 <= zl) JC_STEP(2);
    } else {
        static_assert(RS == 6, "ring of 4 or 6 slots");
        for (; z + 5 <= zl; z += 6) {
            JC_STEP(0);
            JC_STEP(1);
            JC_STEP(2);
            JC_STEP(3);
            JC_STEP(4);
            JC_STEP(5);
        }
        if (z <= zl) JC_STEP(0);
        if (z + 1 <= zl) JC_STEP(1);
        if (z + 2 <= zl) JC_STEP(2);
        if (z + 3 <= zl) JC_STEP(3);
        if (z + 4 <= zl) JC_STEP(4);
    }
#undef JC_STEP
    if (RES) {
        const double w = wave_sum(acc);
        if ((t & 63) == 0)
            wsum[t >> 6] = w;
        __syncthreads();
        if (t == 0) {
            double sum = 0.0;
            for (int i = 0; i < NT / 64; ++i)
                sum = sum + wsum[i];
            partials[id] = sum;
        }
    }
}

template <typename T, int FIELD, int TXP, int TY, bool SRC, typename R>
hipError_t sweep_flags(const BlockDesc* blocks, const Item* items, int nitems, int parity, bool fused,
                       bool resid, bool store, double* partials, hipStream_t s, uint32_t pace)
{
    const int grid = ((nitems + 7) / 8) * 8;
    const dim3 bs(TXP * TY);
#define JC_SWEEP_CASE(FU, RE, ST)                                                                         \
    if (fused == FU && resid == RE && store == ST) {                                                     \
        hipLaunchKernelGGL((k_sweep<T, FIELD, TXP, TY, FU, RE, ST, SRC, R>), dim3(grid), bs, 0, s, blocks, \
                           items, nitems, parity, partials, pace);                                       \
        return hipGetLastError();                                                                        \
    }
    if constexpr (std::is_same<R, NoRlo>::value) {
        if constexpr (FIELD == FIELD_U) {
            JC_SWEEP_CASE(false, false, true)
            JC_SWEEP_CASE(false, true, true)
            JC_SWEEP_CASE(false, true, false)
            JC_SWEEP_CASE(true, true, true)
            JC_SWEEP_CASE(true, true, false)
        }
        JC_SWEEP_CASE(true, false, true)
    } else {
        JC_SWEEP_CASE(true, true, false)
    }
#undef JC_SWEEP_CASE
    return hipErrorInvalidValue;
}

template <typename T, int FIELD, int TXP, bool SRC, typename R>
hipError_t sweep_rows(const BlockDesc* blocks, const Item* items, int nitems, int parity, int tile_y,
                      bool fused, bool resid, bool store, double* partials, hipStream_t s, uint32_t pace)
{
    // at most 1024 threads per work-group
    switch (tile_y) {
    case 4:
        // a 16-cell tile needs 8 rows for whole waves
        if constexpr (TXP * 4 >= 64)
            return sweep_flags<T, FIELD, TXP, 4, SRC, R>(blocks, items, nitems, parity, fused, resid, store, partials, s, pace);
        else
            return hipErrorInvalidValue;
    case 8:
        if constexpr (TXP * 8 <= 1024)
            return sweep_flags<T, FIELD, TXP, 8, SRC, R>(blocks, items, nitems, parity, fused, resid, store, partials, s, pace);
        else
            return hipErrorInvalidValue;
    case 16:
        if constexpr (TXP * 16 <= 1024)
            return sweep_flags<T, FIELD, TXP, 16, SRC, R>(blocks, items, nitems, parity, fused, resid, store, partials, s, pace);
        else
            return hipErrorInvalidValue;
    case 32:
        if constexpr (TXP * 32 <= 1024)
            return sweep_flags<T, FIELD, TXP, 32, SRC, R>(blocks, items, nitems, parity, fused, resid, store, partials, s, pace);
        else
            return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
}

template <typename T, int FIELD, bool SRC, typename R>
hipError_t sweep_tiles(const BlockDesc* blocks, const Item* items, int nitems, int parity, int tile_x, int tile_y,
                       bool fused, bool resid, bool store, double* partials, hipStream_t s, uint32_t pace)
{
    switch (tile_x) {
    case 16: return sweep_rows<T, FIELD, 8, SRC, R>(blocks, items, nitems, parity, tile_y, fused, resid, store, partials, s, pace);
    case 32: return sweep_rows<T, FIELD, 16, SRC, R>(blocks, items, nitems, parity, tile_y, fused, resid, store, partials, s, pace);
    case 64: return sweep_rows<T, FIELD, 32, SRC, R>(blocks, items, nitems, parity, tile_y, fused, resid, store, partials, s, pace);
    default: break;
    }
    // Tiles as wide as a whole block row of 96, 128 or 256 cells (binary64
    // storage): the x halo is then the block's ghost column, never a
    // neighbour tile's lines.
    if constexpr (sizeof(T) == 8) {
        switch (tile_x) {
        case 96: return sweep_rows<T, FIELD, 48, SRC, R>(blocks, items, nitems, parity, tile_y, fused, resid, store, partials, s, pace);
        case 128: return sweep_rows<T, FIELD, 64, SRC, R>(blocks, items, nitems, parity, tile_y, fused, resid, store, partials, s, pace);
        case 256: return sweep_rows<T, FIELD, 128, SRC, R>(blocks, items, nitems, parity, tile_y, fused, resid, store, partials, s, pace);
        default: break;
        }
    }
    return hipErrorInvalidValue;
}

// ---- sweep kernel: end ----

}  // namespace

hipError_t launch_sweep(const BlockDesc* blocks, const Item* items, int nitems, int parity,
                        int tile_x, int tile_y, bool fused, bool resid, bool store, bool src, double* partials,
                        hipStream_t s, uint32_t pace)
{
    if (nitems <= 0)
        return hipSuccess;
    return src ? sweep_tiles<double, FIELD_U, true, NoRlo>(blocks, items, nitems, parity, tile_x, tile_y, fused,
                                                             resid, store, partials, s, pace)
               : sweep_tiles<double, FIELD_U, false, NoRlo>(blocks, items, nitems, parity, tile_x, tile_y, fused,
                                                              resid, store, partials, s, pace);
}

hipError_t launch_ir_residual(const BlockDesc* blocks, const Item* items, int nitems, int parity, int tile_x,
                              int tile_y, bool src, int lo_dtype, double* partials, hipStream_t s)
{
    if (nitems <= 0)
        return hipSuccess;
#define JC_IR_RES(RT)                                                                                  \
    return src ? sweep_tiles<double, FIELD_U, true, RT>(blocks, items, nitems, parity, tile_x, tile_y, true,   \
                                                        true, false, partials, s, 0)                        \
               : sweep_tiles<double, FIELD_U, false, RT>(blocks, items, nitems, parity, tile_x, tile_y, true,  \
                                                         true, false, partials, s, 0);
    switch (lo_dtype) {
    case 0: JC_IR_RES(double)
    case 1: JC_IR_RES(float)
    case 2: JC_IR_RES(bf16)
    default: return hipErrorInvalidValue;
    }
#undef JC_IR_RES
}

hipError_t launch_ir_inner(const BlockDesc* blocks, const Item* items, int nitems, int qparity, int tile_x,
                           int tile_y, int lo_dtype, hipStream_t s, uint32_t pace)
{
    if (nitems <= 0)
        return hipSuccess;
    switch (lo_dtype) {
    case 0: return sweep_tiles<double, FIELD_D, true, NoRlo>(blocks, items, nitems, qparity, tile_x, tile_y, true,
                                                             false, true, nullptr, s, pace);
    case 1: return sweep_tiles<float, FIELD_D, true, NoRlo>(blocks, items, nitems, qparity, tile_x, tile_y, true,
                                                            false, true, nullptr, s, pace);
    case 2: return sweep_tiles<bf16, FIELD_D, true, NoRlo>(blocks, items, nitems, qparity, tile_x, tile_y, true,
                                                           false, true, nullptr, s, pace);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace jc
