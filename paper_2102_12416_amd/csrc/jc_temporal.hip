// Temporal blocking: two or three Jacobi sweeps per launch of one-block
// contexts (binary64 iterate or refinement correction), alone or as a work
// list of several (groups).

#include <hip/hip_runtime.h>

#include <type_traits>

#include "jc_div6.h"
#include "jc_kernels.h"
#include "jc_sweep.h"

namespace jc {

namespace {

// ---- two-step sweep (temporal blocking): begin (fingerprinted with recorded counters) ----
// Two Jacobi sweeps of the single block of a context without face pairs
// per launch: iterate k is read from copy p and iterate k + 2 written to
// copy p ^ 1; iterate k + 1 lives only in LDS and registers.  T / FIELD as
// for k_sweep: the binary64 iterate u (source b), or the refinement
// correction d in its storage format (source r_lo, zero ghosts), whose
// iterate k + 1 is rounded to that format as a stored sweep would leave
// it.  Each cell's two updates take the same sums in the same order as
// two one-step sweeps, so the result is bitwise the same; HBM moves one
// read and one write per cell for two sweeps instead of two of each.
//
// A work-group owns a tile of 2 TXP x cells by TY rows and a z range, and
// marches along z as the one-step sweep does.  Iterate k + 1 is needed on
// the tile and on a one-cell ring around it, so iterate k is loaded on a
// two-cell ring: one aligned pair per thread over (TXP + 2) pairs by (TY +
// 4) rows.  The first TXP * TY threads (whole waves) own the tile's pairs,
// the next 4 (TXP + 2) the two rows above and the two rows below it, the
// next 2 TY the pair left and the pair right of each tile row.  At plane
// step s every thread writes iterate k of its pair at plane s into LDS,
// the work-group synchronises once, every thread computes iterate k + 1 of
// its pair at plane s (a ghost cell keeps its value: the context has no
// face pairs, so every ghost is a fixed boundary value) into a second LDS
// plane, and the tile threads compute iterate k + 2 at plane s - 1 from
// the previous step's second plane.  Both LDS planes are double-buffered
// by step parity.  Values at cells two steps out of the block (the
// outermost ring of a tile on the block edge) are clamped loads that only
// feed discarded results.
//
// Work: with items null, the ntiles tiles of `one` numbered from the
// work-group index; otherwise the work list items[0 .. ntiles), whose tiles
// must be 2 TXP cells by TY rows, each with its block and ping-pong flip
// (groups).
// The one block of a single context comes by value: a small launch is a
// chain of latencies, and the table and 64-bit divisions it replaces were
// part of it.  64^3, 16 rows, z chunks of 1, per sweep: two sweeps 2.64 ->
// 2.40 us (2.86 -> 2.57 with a source), three 2.47 -> 2.33.

// A pair of the arithmetic type rounded to the storage format and back:
// iterate k + 1 is stored between the two sweeps of a one-sweep-per-launch
// run, so the second sweep must read it at storage precision.
template <typename T>
__device__ __forceinline__ void storage_round(typename Tr<T>::C& a, typename Tr<T>::C& b)
{
    if constexpr (std::is_same<T, bf16>::value)
        Tr<T>::unpack(Tr<T>::pack(a, b), a, b);
}

// div6_pair of which only the values with ok are kept.  In a correction the
// others -- lanes outside the block -- stay out of the test for the IEEE
// division: they often have zero sums (zero ghosts, zero padding behind a
// ragged row), and every step of such a tile would take it (groups of edges 96
// to 48, three sweeps, binary32 23.8 -> 20.9 us a launch, bfloat16 24.4 ->
// 20.6).  In the iterate the test over all lanes is 1-2 % faster.
template <int FIELD, typename C>
__device__ __forceinline__ void div6_ok(C sa, C sb, bool a_ok, bool b_ok, C& va, C& vb)
{
    if constexpr (FIELD == FIELD_U) {
        div6_pair(sa, sb, va, vb);
    } else {
        va = div6_fast(sa);
        vb = div6_fast(sb);
        const bool ra = a_ok && div6_redo(va), rb = b_ok && div6_redo(vb);
        if (__builtin_expect(ra || rb, 0)) {
            va = ra ? sa / C(6) : va;
            vb = rb ? sb / C(6) : vb;
        }
    }
}

// A pair of arithmetic values as one LDS access (16 bytes in binary64).
template <typename C> struct Pair2;
template <> struct Pair2<double> { using V = v2d; };
template <> struct Pair2<float> { using V = v2f; };

template <typename T, int FIELD, int TXP, int TY, bool SRC>
__global__ void __launch_bounds__(((TXP + 2) * (TY + 4) + 63) / 64 * 64)
k_sweep2(OneBlock one, const BlockDesc* __restrict__ blocks, const Item* __restrict__ items, int parity, int ntiles,
         uint32_t pace)
{
    using C = typename Tr<T>::C;
    using F = Fld<T, FIELD>;
    constexpr int EP = TXP + 2;                   // pairs of an extended row
    constexpr int ER = TY + 4;                    // extended rows
    constexpr int NTILE = TXP * TY;               // tile threads
    static_assert(NTILE % 64 == 0, "tile threads are whole waves");
    using V = typename Pair2<C>::V;
    // LDS row: two pad cells, 2 EP cells, two pad cells, so that every
    // thread's pair is one aligned vector: a pair is written with one
    // access and its neighbours' pairs are read with one access each
    constexpr int LW = 2 * EP + 4;
    constexpr int LN = (ER + 2) * LW;             // LDS plane: pad row, ER rows, pad row
    __shared__ V A[2][LN / 2 + 1];                // iterate k; pair LN / 2: sink of idle lanes
    __shared__ V Bn[2][LN / 2 + 1];               // iterate k + 1

    const int id = logical_block(blockIdx.x, gridDim.x);
    if (id >= ntiles)
        return;                                   // uniform over the work-group
    const uint64_t pace_t0 = pace ? __builtin_amdgcn_s_memrealtime() : 0;
    const T *src, *source;
    T* out;
    int64_t pitch, plane;
    int nx, ny, nz, x0, y0, zf, zl;
    if (items) {
        const Item it = items[id];
        const BlockDesc* B = blocks + it.block;
        const int p = parity ^ it.flip;
        src = F::src(B, p);
        out = F::dst(B, p);
        source = F::source(B);
        pitch = F::pitch(B);
        plane = F::plane(B);
        nx = B->n[0];
        ny = B->n[1];
        nz = B->n[2];
        x0 = it.x0;
        y0 = it.y0;
        zf = it.z0 + 1;
        zl = it.z0 + it.zlen;
    } else {
        src = static_cast<const T*>(one.src);
        out = static_cast<T*>(one.dst);
        source = static_cast<const T*>(one.source);
        pitch = one.pitch;
        plane = one.plane;
        nx = one.nx;
        ny = one.ny;
        nz = one.nz;
        const uint32_t row = (uint32_t)id / (uint32_t)one.tiles_x;
        const int chunk = (int)(row / (uint32_t)one.tiles_y);
        x0 = (int)((uint32_t)id - row * (uint32_t)one.tiles_x) * (2 * TXP);
        y0 = ((int)row - chunk * one.tiles_y) * TY;
        zf = chunk * one.planes + min(chunk, one.rest) + 1;
        zl = zf + one.planes - (chunk < one.rest ? 0 : 1);
    }

    // this thread's pair (j, r) of the extended region
    const int t = threadIdx.x;
    int j = 0, r = 0;
    bool live = true;
    if (t < NTILE) {
        j = 1 + t % TXP;
        r = 2 + t / TXP;
    } else {
        int q = t - NTILE;
        if (q < 2 * EP) {
            j = q % EP;
            r = q / EP;
        } else if ((q -= 2 * EP) < 2 * EP) {
            j = q % EP;
            r = TY + 2 + q / EP;
        } else if ((q -= 2 * EP) < 2 * TY) {
            j = (q & 1) ? EP - 1 : 0;
            r = 2 + (q >> 1);
        } else {
            live = false;
        }
    }
    const bool tile = t < NTILE;                  // uniform over each wave
    const int xs = x0 - 1 + 2 * j;                // cells xs, xs + 1 (xs odd, >= -1)
    const int ye = y0 - 1 + r;
    const int xs_c = min(xs, nx | 1);             // last pair holding a cell <= nx + 1
    const int ye_c = min(max(ye, 0), ny + 1);
    const bool y_in = ye >= 1 && ye <= ny;
    const bool in_a = live && y_in && xs >= 1 && xs <= nx;
    const bool in_b = live && y_in && xs + 1 >= 1 && xs + 1 <= nx;
    const bool a_ok = tile && ye <= ny && xs <= nx;   // tile cells in the block: stored
    const bool b_ok = tile && ye <= ny && xs + 1 <= nx;
    const int64_t rowoff = (int64_t)ye_c * pitch + xs_c;
    const T* __restrict__ col = src + rowoff;
    const T* __restrict__ scol = SRC ? source + rowoff : nullptr;
    T* __restrict__ dst = out + rowoff;

    const int pn = (r + 1) * (LW / 2) + j + 1;    // LDS pair of cells xs, xs + 1
    const int pw = live ? pn : LN / 2;            // the pair this thread writes

    // register rings: iterate k and the source of plane s in slot
    // (s - zf + 1) mod RS, loads issued PD planes ahead; iterate k + 1 of
    // plane s in slot (s - zf + 1) mod 3
    constexpr int PD = 3;
    constexpr int RS = 6;
    const int zhi = min(zl + 2, nz + 1);          // last plane read
    C ua[RS], ub[RS], ba[RS], bb[RS], va[3], vb[3];
#pragma unroll
    for (int k = 0; k < RS; ++k)
        ba[k] = bb[k] = C(0);
    va[0] = vb[0] = va[1] = vb[1] = va[2] = vb[2] = C(0);
    Tr<T>::ld(col + (int64_t)max(zf - 2, 0) * plane, ua[RS - 1], ub[RS - 1]);
#pragma unroll
    for (int k = 0; k < PD; ++k) {
        const int64_t zk = (int64_t)min(zf - 1 + k, zhi) * plane;
        Tr<T>::ld(col + zk, ua[k], ub[k]);
        if (SRC)
            Tr<T>::ld(scol + zk, ba[k], bb[k]);
    }

    const int s_first = zf - 1;
    auto step = [&](int s, auto kc, auto two) {
        constexpr int K = decltype(kc)::value;
        constexpr bool TWO = decltype(two)::value;
        constexpr int SM = (K + RS - 1) % RS, SC = K, SP = (K + 1) % RS, SQ = (K + PD) % RS;
        constexpr int VC = K % 3, VM = (K + 2) % 3, VMM = (K + 1) % 3;
        constexpr int HC = K & 1;
        if (pace)
            pace_wait(pace_t0 + (uint64_t)(s - s_first) * pace);
        const int64_t zq = (int64_t)min(s + PD, zhi) * plane;
        Tr<T>::ld(col + zq, ua[SQ], ub[SQ]);
        if (SRC)
            Tr<T>::ld(scol + zq, ba[SQ], bb[SQ]);
        V* const Ak = A[HC];
        Ak[pw] = V{ua[SC], ub[SC]};
        __syncthreads();
        // iterate k + 1 at plane s
        const V ym = Ak[pn - LW / 2], yp = Ak[pn + LW / 2], xm = Ak[pn - 1], xp = Ak[pn + 1];
        C sa = xm.y + ub[SC];
        sa = sa + ym.x;
        sa = sa + yp.x;
        sa = sa + ua[SM];
        sa = sa + ua[SP];
        C sb = ua[SC] + xp.x;
        sb = sb + ym.y;
        sb = sb + yp.y;
        sb = sb + ub[SM];
        sb = sb + ub[SP];
        C na, nb;
        if (SRC)
            div6_ok<FIELD>(sa + ba[SC], sb + bb[SC], in_a, in_b, na, nb);
        else
            div6_ok<FIELD>(sa, sb, in_a, in_b, na, nb);
        const bool z_in = s >= 1 && s <= nz;
        storage_round<T>(na, nb);
        va[VC] = (in_a && z_in) ? na : ua[SC];
        vb[VC] = (in_b && z_in) ? nb : ub[SC];
        Bn[HC][pw] = V{va[VC], vb[VC]};
        // iterate k + 2 at plane s - 1
        if (TWO && tile) {
            const V* const Bk = Bn[HC ^ 1];
            const V ym2 = Bk[pn - LW / 2], yp2 = Bk[pn + LW / 2], xm2 = Bk[pn - 1], xp2 = Bk[pn + 1];
            C qa = xm2.y + vb[VM];
            qa = qa + ym2.x;
            qa = qa + yp2.x;
            qa = qa + va[VMM];
            qa = qa + va[VC];
            C qb = va[VM] + xp2.x;
            qb = qb + ym2.y;
            qb = qb + yp2.y;
            qb = qb + vb[VMM];
            qb = qb + vb[VC];
            C wa2, wb2;
            if (SRC)
                div6_ok<FIELD>(qa + ba[SM], qb + bb[SM], in_a, in_b, wa2, wb2);
            else
                div6_ok<FIELD>(qa, qb, in_a, in_b, wa2, wb2);
            // past the last cell of a row the pair's second slot is the
            // x = nx + 1 ghost: write back the value it holds
            wb2 = b_ok ? wb2 : ub[SM];
            if (a_ok)
                Tr<T>::stn(dst + (int64_t)(s - 1) * plane, wa2, wb2);
        }
    };
    using F_ = std::false_type;
    using T_ = std::true_type;
#define JC_STEP2(k) step(s + (k), std::integral_constant<int, ((k) + 2) % RS>{}, T_{})
    int s = zf - 1;
    step(s, std::integral_constant<int, 0>{}, F_{});
    step(s + 1, std::integral_constant<int, 1>{}, F_{});
    s += 2;
    const int s_end = zl + 1;
    for (; s + 5 <= s_end; s += 6) {
        JC_STEP2(0);
        JC_STEP2(1);
        JC_STEP2(2);
        JC_STEP2(3);
        JC_STEP2(4);
        JC_STEP2(5);
    }
    if (s <= s_end) JC_STEP2(0);
    if (s + 1 <= s_end) JC_STEP2(1);
    if (s + 2 <= s_end) JC_STEP2(2);
    if (s + 3 <= s_end) JC_STEP2(3);
    if (s + 4 <= s_end) JC_STEP2(4);
#undef JC_STEP2
}
// ---- two-step sweep: end ----

// ---- three-step sweep (temporal blocking): begin ----
// Three Jacobi sweeps per launch: iterate k from copy p, iterate k + 3 to
// copy p ^ 1; iterates k + 1 and k + 2 live only in LDS and registers.
// The construction of k_sweep2 one level deeper.  Iterate k is loaded on
// a three-cell ring around the tile: TXP + 4 pairs (cells x0 - 3 ..
// x0 + 2 TXP + 4) by TY + 6 rows, one aligned pair per thread.  At plane
// step s every thread writes iterate k of its pair at plane s into LDS,
// the work-group synchronises once, and then
//  - every thread computes iterate k + 1 of its pair at plane s (valid on
//    the tile and a two-cell ring; the outermost values, which would need
//    cells further out, are never read) into LDS plane B;
//  - the threads of the tile and of its one-pair / one-row ring ("mid"
//    threads) compute iterate k + 2 at plane s - 1 from B of the previous
//    step into LDS plane C;
//  - the tile threads compute iterate k + 3 at plane s - 2 from C of the
//    previous step and store it.
// A ghost cell keeps its value at every level (the context has no face
// pairs: every ghost is a fixed boundary value), and iterates k + 1 and
// k + 2 are rounded to the storage format as stored sweeps would leave
// them, so each cell takes the same sums in the same order as in three
// one-step sweeps: the result is bitwise the same.  The three LDS planes
// are double-buffered by step parity, so one barrier per step suffices.
// Thread order: tile threads (whole waves), then the mid ring (rows y0 and
// y0 + TY + 1 over pairs 1 .. TXP + 2, then pairs 1 and TXP + 2 of the tile
// rows), then the rest of the two-cell ring (rows y0 - 1 and y0 + TY + 2
// over pairs 1 .. TXP + 2), then the third ring (the outermost rows, then
// pairs 0 and TXP + 3 of the other rows), whose iterate k + 1 is not
// needed.  Work as for k_sweep2 (items null: the
// tiles of `one`; else a work list of 2 TXP x TY tiles).
template <typename T, int FIELD, int TXP, int TY, bool SRC>
__global__ void __launch_bounds__(((TXP + 4) * (TY + 6) + 63) / 64 * 64)
k_sweep3(OneBlock one, const BlockDesc* __restrict__ blocks, const Item* __restrict__ items, int parity, int ntiles,
         uint32_t pace)
{
    using C = typename Tr<T>::C;
    using F = Fld<T, FIELD>;
    constexpr int EP = TXP + 4;                   // pairs of an extended row
    constexpr int ER = TY + 6;                    // extended rows
    constexpr int NTILE = TXP * TY;               // tile threads
    constexpr int NMID = NTILE + 2 * (TXP + 2) + 2 * TY;
    constexpr int NL1 = NMID + 2 * (TXP + 2);
    static_assert(NTILE % 64 == 0, "tile threads are whole waves");
    using V = typename Pair2<C>::V;
    // LDS row: two pad cells, 2 EP cells, two pad cells, so that every
    // thread's pair is one aligned vector: a pair is written with one
    // access and its neighbours' pairs are read with one access each
    constexpr int LW = 2 * EP + 4;
    constexpr int LN = (ER + 2) * LW;             // LDS plane: pad row, ER rows, pad row
    __shared__ V A[2][LN / 2 + 1];                // iterate k; pair LN / 2: sink of idle lanes
    __shared__ V Bn[2][LN / 2 + 1];               // iterate k + 1
    __shared__ V Cn[2][LN / 2 + 1];               // iterate k + 2

    const int id = logical_block(blockIdx.x, gridDim.x);
    if (id >= ntiles)
        return;                                   // uniform over the work-group
    const uint64_t pace_t0 = pace ? __builtin_amdgcn_s_memrealtime() : 0;
    const T *src, *source;
    T* out;
    int64_t pitch, plane;
    int nx, ny, nz, x0, y0, zf, zl;
    if (items) {
        const Item it = items[id];
        const BlockDesc* B = blocks + it.block;
        const int p = parity ^ it.flip;
        src = F::src(B, p);
        out = F::dst(B, p);
        source = F::source(B);
        pitch = F::pitch(B);
        plane = F::plane(B);
        nx = B->n[0];
        ny = B->n[1];
        nz = B->n[2];
        x0 = it.x0;
        y0 = it.y0;
        zf = it.z0 + 1;
        zl = it.z0 + it.zlen;
    } else {
        src = static_cast<const T*>(one.src);
        out = static_cast<T*>(one.dst);
        source = static_cast<const T*>(one.source);
        pitch = one.pitch;
        plane = one.plane;
        nx = one.nx;
        ny = one.ny;
        nz = one.nz;
        const uint32_t row = (uint32_t)id / (uint32_t)one.tiles_x;
        const int chunk = (int)(row / (uint32_t)one.tiles_y);
        x0 = (int)((uint32_t)id - row * (uint32_t)one.tiles_x) * (2 * TXP);
        y0 = ((int)row - chunk * one.tiles_y) * TY;
        zf = chunk * one.planes + min(chunk, one.rest) + 1;
        zl = zf + one.planes - (chunk < one.rest ? 0 : 1);
    }

    // this thread's pair (j, r) of the extended region
    const int t = threadIdx.x;
    int j = 0, r = 0;
    bool live = true;
    if (t < NTILE) {
        j = 2 + t % TXP;
        r = 3 + t / TXP;
    } else {
        int q = t - NTILE;
        if (q < 2 * (TXP + 2)) {                  // mid rows
            j = 1 + q % (TXP + 2);
            r = q < TXP + 2 ? 2 : TY + 3;
        } else if ((q -= 2 * (TXP + 2)) < 2 * TY) {   // mid pairs of the tile rows
            j = (q & 1) ? TXP + 2 : 1;
            r = 3 + (q >> 1);
        } else if ((q -= 2 * TY) < 2 * (TXP + 2)) {   // second ring: rows 1 and ER - 2
            j = 1 + q % (TXP + 2);
            r = q < TXP + 2 ? 1 : ER - 2;
        } else if ((q -= 2 * (TXP + 2)) < 2 * EP) {   // third ring: rows 0 and ER - 1
            j = q % EP;
            r = q < EP ? 0 : ER - 1;
        } else if ((q -= 2 * EP) < 2 * (ER - 2)) {    // third ring: pairs 0 and EP - 1
            j = (q & 1) ? EP - 1 : 0;
            r = 1 + (q >> 1);
        } else {
            live = false;
        }
    }
    const bool tile = t < NTILE;                  // uniform over each wave
    const bool mid = t < NMID;
    // Iterate k + 1 is needed on the tile and its two-cell ring only (the
    // first NL1 threads); the third ring's threads come last and only load
    // iterate k, so the waves holding none of the first NL1 threads skip the
    // first stage (a wave-uniform branch)
    const bool l1 = (t & ~63) < NL1;
    const int xs = x0 - 3 + 2 * j;                // cells xs, xs + 1 (xs odd, >= -3)
    const int ye = y0 - 2 + r;
    const int xs_c = min(xs, nx | 1);             // last pair holding a cell <= nx + 1
    const int ye_c = min(max(ye, 0), ny + 1);
    const bool y_in = ye >= 1 && ye <= ny;
    const bool in_a = live && y_in && xs >= 1 && xs <= nx;
    const bool in_b = live && y_in && xs + 1 >= 1 && xs + 1 <= nx;
    const bool a_ok = tile && ye <= ny && xs <= nx;   // tile cells in the block: stored
    const bool b_ok = tile && ye <= ny && xs + 1 <= nx;
    const int64_t rowoff = (int64_t)ye_c * pitch + xs_c;
    const T* __restrict__ col = src + rowoff;
    const T* __restrict__ scol = SRC ? source + rowoff : nullptr;
    T* __restrict__ dst = out + rowoff;

    const int pn = (r + 1) * (LW / 2) + j + 1;    // LDS pair of cells xs, xs + 1
    const int pw = live ? pn : LN / 2;            // the pair this thread writes

    // register rings: iterate k and the source of plane s in slot
    // (s - zf + 2) mod RS, loads issued PD planes ahead; iterates k + 1 of
    // plane s and k + 2 of plane s - 1 in slot (s - zf + 2) mod 3
    constexpr int PD = 3;
    constexpr int RS = 6;
    const int zlo = max(zf - 3, 0);               // first plane read
    const int zhi = min(zl + 3, nz + 1);          // last plane read
    C ua[RS], ub[RS], ba[RS], bb[RS], va[3], vb[3], wa3[3], wb3[3];
#pragma unroll
    for (int k = 0; k < RS; ++k)
        ba[k] = bb[k] = C(0);
#pragma unroll
    for (int k = 0; k < 3; ++k)
        va[k] = vb[k] = wa3[k] = wb3[k] = C(0);
    Tr<T>::ld(col + (int64_t)zlo * plane, ua[RS - 1], ub[RS - 1]);
    if (SRC)
        Tr<T>::ld(scol + (int64_t)zlo * plane, ba[RS - 1], bb[RS - 1]);
#pragma unroll
    for (int k = 0; k < PD; ++k) {
        const int64_t zk = (int64_t)min(max(zf - 2 + k, 0), zhi) * plane;
        Tr<T>::ld(col + zk, ua[k], ub[k]);
        if (SRC)
            Tr<T>::ld(scol + zk, ba[k], bb[k]);
    }

    // STAGES: 1 = iterate k + 1 only, 2 = also k + 2, 3 = also k + 3
    const int s_first = zf - 2;
    auto step = [&](int s, auto kc, auto stages) {
        constexpr int K = decltype(kc)::value;
        constexpr int ST = decltype(stages)::value;
        constexpr int SM = (K + RS - 1) % RS, SC = K, SP = (K + 1) % RS, SQ = (K + PD) % RS;
        constexpr int S2 = (K + RS - 2) % RS;     // plane s - 2
        constexpr int VC = K % 3, VM = (K + 2) % 3, VMM = (K + 1) % 3;
        constexpr int HC = K & 1;
        if (pace)
            pace_wait(pace_t0 + (uint64_t)(s - s_first) * pace);
        const int64_t zq = (int64_t)min(s + PD, zhi) * plane;
        Tr<T>::ld(col + zq, ua[SQ], ub[SQ]);
        if (SRC)
            Tr<T>::ld(scol + zq, ba[SQ], bb[SQ]);
        V* const Ak = A[HC];
        Ak[pw] = V{ua[SC], ub[SC]};
        __syncthreads();
        // iterate k + 1 at plane s
        if (l1) {
            const V ym = Ak[pn - LW / 2], yp = Ak[pn + LW / 2], xm = Ak[pn - 1], xp = Ak[pn + 1];
            C sa = xm.y + ub[SC];
            sa = sa + ym.x;
            sa = sa + yp.x;
            sa = sa + ua[SM];
            sa = sa + ua[SP];
            C sb = ua[SC] + xp.x;
            sb = sb + ym.y;
            sb = sb + yp.y;
            sb = sb + ub[SM];
            sb = sb + ub[SP];
            C na, nb;
            if (SRC)
                div6_ok<FIELD>(sa + ba[SC], sb + bb[SC], in_a, in_b, na, nb);
            else
                div6_ok<FIELD>(sa, sb, in_a, in_b, na, nb);
            const bool z_in = s >= 1 && s <= nz;
            storage_round<T>(na, nb);
            va[VC] = (in_a && z_in) ? na : ua[SC];
            vb[VC] = (in_b && z_in) ? nb : ub[SC];
            Bn[HC][pw] = V{va[VC], vb[VC]};
        }
        // iterate k + 2 at plane s - 1
        if (ST >= 2 && mid) {
            const V* const Bk = Bn[HC ^ 1];
            const V ym = Bk[pn - LW / 2], yp = Bk[pn + LW / 2], xm = Bk[pn - 1], xp = Bk[pn + 1];
            C qa = xm.y + vb[VM];
            qa = qa + ym.x;
            qa = qa + yp.x;
            qa = qa + va[VMM];
            qa = qa + va[VC];
            C qb = va[VM] + xp.x;
            qb = qb + ym.y;
            qb = qb + yp.y;
            qb = qb + vb[VMM];
            qb = qb + vb[VC];
            C na, nb;
            if (SRC)
                div6_ok<FIELD>(qa + ba[SM], qb + bb[SM], in_a, in_b, na, nb);
            else
                div6_ok<FIELD>(qa, qb, in_a, in_b, na, nb);
            const bool z_in = s - 1 >= 1 && s - 1 <= nz;
            storage_round<T>(na, nb);
            wa3[VC] = (in_a && z_in) ? na : va[VM];
            wb3[VC] = (in_b && z_in) ? nb : vb[VM];
            Cn[HC][pw] = V{wa3[VC], wb3[VC]};
        }
        // iterate k + 3 at plane s - 2
        if (ST >= 3 && tile) {
            const V* const Ck = Cn[HC ^ 1];
            const V ym = Ck[pn - LW / 2], yp = Ck[pn + LW / 2], xm = Ck[pn - 1], xp = Ck[pn + 1];
            C qa = xm.y + wb3[VM];
            qa = qa + ym.x;
            qa = qa + yp.x;
            qa = qa + wa3[VMM];
            qa = qa + wa3[VC];
            C qb = wa3[VM] + xp.x;
            qb = qb + ym.y;
            qb = qb + yp.y;
            qb = qb + wb3[VMM];
            qb = qb + wb3[VC];
            C oa, ob;
            if (SRC)
                div6_ok<FIELD>(qa + ba[S2], qb + bb[S2], a_ok, b_ok, oa, ob);
            else
                div6_ok<FIELD>(qa, qb, a_ok, b_ok, oa, ob);
            // past the last cell of a row the pair's second slot is the
            // x = nx + 1 ghost: write back the value it holds
            ob = b_ok ? ob : ub[S2];
            if (a_ok)
                Tr<T>::stn(dst + (int64_t)(s - 2) * plane, oa, ob);
        }
    };
    using One = std::integral_constant<int, 1>;
    using Two = std::integral_constant<int, 2>;
    using Three = std::integral_constant<int, 3>;
    int s = zf - 2;
    step(s, std::integral_constant<int, 0>{}, One{});
    step(s + 1, std::integral_constant<int, 1>{}, One{});
    step(s + 2, std::integral_constant<int, 2>{}, Two{});
    step(s + 3, std::integral_constant<int, 3>{}, Two{});
    s += 4;
#define JC_STEP3(k) step(s + (k), std::integral_constant<int, ((k) + 4) % RS>{}, Three{})
    const int s_end = zl + 2;
    for (; s + 5 <= s_end; s += 6) {
        JC_STEP3(0);
        JC_STEP3(1);
        JC_STEP3(2);
        JC_STEP3(3);
        JC_STEP3(4);
        JC_STEP3(5);
    }
    if (s <= s_end) JC_STEP3(0);
    if (s + 1 <= s_end) JC_STEP3(1);
    if (s + 2 <= s_end) JC_STEP3(2);
    if (s + 3 <= s_end) JC_STEP3(3);
    if (s + 4 <= s_end) JC_STEP3(4);
#undef JC_STEP3
}
// ---- three-step sweep: end ----

// ---- three sweeps of a correction in quads: begin ----
typedef float v4f __attribute__((ext_vector_type(4)));

// Four cells (an aligned quad: cell x = 1 of a row starts a line) as stored.
template <typename T> struct Quad;

template <> struct Quad<float> {
    __device__ static v4f ld(const float* p) { return *(const v4f JC_GLOBAL*)(p); }
    __device__ static void stn(float* p, v4f v) { __builtin_nontemporal_store(v, (v4f JC_GLOBAL*)(p)); }
    __device__ static v4f round(v4f v) { return v; }
};

template <> struct Quad<bf16> {
    typedef uint32_t W __attribute__((ext_vector_type(2)));
    __device__ static v4f unpack(W w) { return v4f{bf16_lo(w.x), bf16_hi(w.x), bf16_lo(w.y), bf16_hi(w.y)}; }
    __device__ static W pack(v4f v) { return W{bf16_pair(v.x, v.y), bf16_pair(v.z, v.w)}; }
    __device__ static v4f ld(const bf16* p) { return unpack(*(const W JC_GLOBAL*)(p)); }
    __device__ static void stn(bf16* p, v4f v) { __builtin_nontemporal_store(pack(v), (W JC_GLOBAL*)(p)); }
    __device__ static v4f round(v4f v) { return unpack(pack(v)); }
};

// k_sweep3 for the binary32 and bfloat16 correction (with its source r_lo), a
// tile of 4 TXQ cells by TY rows: four cells per thread instead of two.
// k_sweep3 in these formats is bound by instruction issue, a third of it LDS
// accesses; a quad needs one write, two whole neighbours and two single cells
// per level where two pairs need two writes and eight neighbours, shares its
// addresses and masks, and one quad left and right covers the three-cell ring.
// A tile of 32 rows then fits 11 waves and reads 1.33 quads per quad of the
// tile (16 rows: 1.53).  Cells outside the block do not take part in the test
// for the IEEE division: their sums are often zero (zero ghosts, zero padding
// behind a ragged row), which cost every step of such a tile the division.
// Waves whose cells are all inside skip the selection of ghosts.
//
// Per sweep with the outer step, against k_sweep3 in its best shape: 512^3
// binary32 221 -> 190 us, bfloat16 187 -> 175; 385 x 250 x 333 67 -> 57 and 55
// -> 54 (with the test over all cells 64 and 61); 1024^3 binary32 1.89 -> 1.56
// ms.  The launch alone moves 12 bytes a cell in binary32 at 4.7 TB/s, the
// card's copy rate; in bfloat16 it is still bound by issue.  Tiles of 8, 16
// and 24 rows: 222, 203 and 223 us in binary32 at 512^3.
constexpr int quad_threads(int txq, int ty) { return (txq * ty + 6 * txq + 2 * ty + 8 + 63) / 64 * 64; }

template <typename T, int TXQ, int TY>
__global__ void __launch_bounds__(quad_threads(TXQ, TY))
k_sweep3q(OneBlock one, const BlockDesc* __restrict__ blocks, const Item* __restrict__ items, int parity, int ntiles,
          uint32_t pace)
{
    using F = Fld<T, FIELD_D>;
    constexpr int EP = TXQ + 2;                   // quads of an extended row
    constexpr int ER = TY + 6;                    // extended rows
    constexpr int NTILE = TXQ * TY;               // tile threads
    constexpr int NMID = NTILE + 2 * TXQ + 2 * TY;
    constexpr int NL1 = NMID + 2 * TXQ + 4;
    static_assert(NTILE % 64 == 0, "tile threads are whole waves");
    constexpr int LN = ER * EP;                   // quads of an LDS plane; quad LN: sink of idle lanes
    __shared__ v4f A[2][LN + 1];                  // iterate k
    __shared__ v4f Bn[2][LN + 1];                 // iterate k + 1
    __shared__ v4f Cn[2][LN + 1];                 // iterate k + 2

    const int id = logical_block(blockIdx.x, gridDim.x);
    if (id >= ntiles)
        return;                                   // uniform over the work-group
    const uint64_t pace_t0 = pace ? __builtin_amdgcn_s_memrealtime() : 0;
    const T *src, *source;
    T* out;
    int64_t pitch, plane;
    int nx, ny, nz, x0, y0, zf, zl;
    if (items) {
        const Item it = items[id];
        const BlockDesc* B = blocks + it.block;
        const int p = parity ^ it.flip;
        src = F::src(B, p);
        out = F::dst(B, p);
        source = F::source(B);
        pitch = F::pitch(B);
        plane = F::plane(B);
        nx = B->n[0];
        ny = B->n[1];
        nz = B->n[2];
        x0 = it.x0;
        y0 = it.y0;
        zf = it.z0 + 1;
        zl = it.z0 + it.zlen;
    } else {
        src = static_cast<const T*>(one.src);
        out = static_cast<T*>(one.dst);
        source = static_cast<const T*>(one.source);
        pitch = one.pitch;
        plane = one.plane;
        nx = one.nx;
        ny = one.ny;
        nz = one.nz;
        const uint32_t row = (uint32_t)id / (uint32_t)one.tiles_x;
        const int chunk = (int)(row / (uint32_t)one.tiles_y);
        x0 = (int)((uint32_t)id - row * (uint32_t)one.tiles_x) * (4 * TXQ);
        y0 = ((int)row - chunk * one.tiles_y) * TY;
        zf = chunk * one.planes + min(chunk, one.rest) + 1;
        zl = zf + one.planes - (chunk < one.rest ? 0 : 1);
    }

    // this thread's quad (j, r) of the extended region
    const int t = threadIdx.x;
    int j = 1, r = 3;
    bool live = true;
    if (t < NTILE) {
        j = 1 + t % TXQ;
        r = 3 + t / TXQ;
    } else {
        int q = t - NTILE;
        if (q < 2 * TXQ) {                        // the rows next to the tile
            j = 1 + q % TXQ;
            r = q < TXQ ? 2 : TY + 3;
        } else if ((q -= 2 * TXQ) < 2 * TY) {     // the quads left and right of its rows
            j = (q & 1) ? EP - 1 : 0;
            r = 3 + (q >> 1);
        } else if ((q -= 2 * TY) < 2 * TXQ) {     // second ring: rows 1 and ER - 2
            j = 1 + q % TXQ;
            r = q < TXQ ? 1 : ER - 2;
        } else if ((q -= 2 * TXQ) < 4) {          // and the corners of the first
            j = (q & 1) ? EP - 1 : 0;
            r = (q & 2) ? TY + 3 : 2;
        } else if ((q -= 4) < 2 * TXQ) {          // third ring: rows 0 and ER - 1
            j = 1 + q % TXQ;
            r = q < TXQ ? 0 : ER - 1;
        } else if ((q -= 2 * TXQ) < 4) {          // and the corners of the second
            j = (q & 1) ? EP - 1 : 0;
            r = (q & 2) ? ER - 2 : 1;
        } else {
            live = false;
        }
    }
    const bool tile = t < NTILE;                  // uniform over each wave
    const bool mid = t < NMID;
    const bool l1 = (t & ~63) < NL1;              // the waves that hold a thread of the first stage
    const int xs = x0 - 3 + 4 * j;                // cells xs .. xs + 3 (xs = 1 mod 4, >= -3)
    const int ye = y0 - 2 + r;
    const int xs_c = min(xs, (nx & ~3) + 1);      // last quad holding a cell <= nx + 1
    const int ye_c = min(max(ye, 0), ny + 1);
    const bool y_in = live && ye >= 1 && ye <= ny;
    const bool in0 = y_in && xs >= 1 && xs <= nx;
    const bool in1 = y_in && xs + 1 >= 1 && xs + 1 <= nx;
    const bool in2 = y_in && xs + 2 >= 1 && xs + 2 <= nx;
    const bool in3 = y_in && xs + 3 >= 1 && xs + 3 <= nx;
    // a tile quad is stored whole where it ends at nx + 1 or before, else its
    // first pair: what lies behind a row's x = nx + 1 ghost is not its own
    const bool st4 = tile && ye <= ny && xs + 2 <= nx;
    const bool st2 = tile && ye <= ny && xs <= nx && !st4;
    const int64_t rowoff = (int64_t)ye_c * pitch + xs_c;
    const T* __restrict__ col = src + rowoff;
    const T* __restrict__ scol = source + rowoff;
    T* __restrict__ dst = out + rowoff;

    // LDS quads: own, left, right, above, below; at the rim of the region
    // (results not used) its own instead of one outside
    const int pn = r * EP + j;
    const int pw = live ? pn : LN;                // the quad this thread writes
    const int pl = j > 0 ? pn - 1 : pn, pr = j < EP - 1 ? pn + 1 : pn;
    const int pu = r > 0 ? pn - EP : pn, pd = r < ER - 1 ? pn + EP : pn;

    // register rings as in k_sweep3
    constexpr int PD = 3;
    constexpr int RS = 6;
    const int zlo = max(zf - 3, 0);               // first plane read
    const int zhi = min(zl + 3, nz + 1);          // last plane read
    v4f u[RS], b[RS], v[3], w[3];
#pragma unroll
    for (int k = 0; k < RS; ++k)
        b[k] = v4f(0.0f);
#pragma unroll
    for (int k = 0; k < 3; ++k)
        v[k] = w[k] = v4f(0.0f);
    u[RS - 1] = Quad<T>::ld(col + (int64_t)zlo * plane);
    b[RS - 1] = Quad<T>::ld(scol + (int64_t)zlo * plane);
#pragma unroll
    for (int k = 0; k < PD; ++k) {
        const int64_t zk = (int64_t)min(max(zf - 2 + k, 0), zhi) * plane;
        u[k] = Quad<T>::ld(col + zk);
        b[k] = Quad<T>::ld(scol + zk);
    }

    // the update of `c` from its plane P of the level below, its z neighbours
    // and source
    auto update = [&](const v4f* P, v4f c, v4f zm, v4f zp, v4f s) {
        const v4f ym = P[pu], yp = P[pd];
        const float* const Pf = reinterpret_cast<const float*>(P);
        const float xm = Pf[4 * pl + 3], xp = Pf[4 * pr];
        v4f a{xm + c.y, c.x + c.z, c.y + c.w, c.z + xp};
        a = a + ym;
        a = a + yp;
        a = a + zm;
        a = a + zp;
        a = a + s;
        v4f n{div6_fast(a.x), div6_fast(a.y), div6_fast(a.z), div6_fast(a.w)};
        const bool r0 = in0 && div6_redo(n.x), r1 = in1 && div6_redo(n.y);
        const bool r2 = in2 && div6_redo(n.z), r3 = in3 && div6_redo(n.w);
        if (__builtin_expect(r0 || r1 || r2 || r3, 0)) {
            n.x = r0 ? a.x / 6.0f : n.x;
            n.y = r1 ? a.y / 6.0f : n.y;
            n.z = r2 ? a.z / 6.0f : n.z;
            n.w = r3 ? a.w / 6.0f : n.w;
        }
        return Quad<T>::round(n);
    };
    const bool inner = __all(in0 && in1 && in2 && in3);
    auto keep = [&](v4f n, v4f o, bool z_in) {
        if (inner && z_in)                        // uniform over the wave
            return n;
        return v4f{in0 && z_in ? n.x : o.x, in1 && z_in ? n.y : o.y, in2 && z_in ? n.z : o.z, in3 && z_in ? n.w : o.w};
    };
    // STAGES: 1 = iterate k + 1 only, 2 = also k + 2, 3 = also k + 3
    const int s_first = zf - 2;
    auto step = [&](int s, auto kc, auto stages) {
        constexpr int K = decltype(kc)::value;
        constexpr int ST = decltype(stages)::value;
        constexpr int SM = (K + RS - 1) % RS, SC = K, SP = (K + 1) % RS, SQ = (K + PD) % RS;
        constexpr int S2 = (K + RS - 2) % RS;     // plane s - 2
        constexpr int VC = K % 3, VM = (K + 2) % 3, VMM = (K + 1) % 3;
        constexpr int HC = K & 1;
        if (pace)
            pace_wait(pace_t0 + (uint64_t)(s - s_first) * pace);
        const int64_t zq = (int64_t)min(s + PD, zhi) * plane;
        u[SQ] = Quad<T>::ld(col + zq);
        b[SQ] = Quad<T>::ld(scol + zq);
        A[HC][pw] = u[SC];
        __syncthreads();
        // iterate k + 1 at plane s
        if (l1) {
            v[VC] = keep(update(A[HC], u[SC], u[SM], u[SP], b[SC]), u[SC], s >= 1 && s <= nz);
            Bn[HC][pw] = v[VC];
        }
        // iterate k + 2 at plane s - 1
        if (ST >= 2 && mid) {
            w[VC] = keep(update(Bn[HC ^ 1], v[VM], v[VMM], v[VC], b[SM]), v[VM], s - 1 >= 1 && s - 1 <= nz);
            Cn[HC][pw] = w[VC];
        }
        // iterate k + 3 at plane s - 2
        if (ST >= 3 && tile) {
            const v4f n = update(Cn[HC ^ 1], w[VM], w[VMM], w[VC], b[S2]);
            // the x = nx + 1 ghost behind a row's last cell keeps its value
            const v4f o = keep(n, u[S2], true);
            if (st4)
                Quad<T>::stn(dst + (int64_t)(s - 2) * plane, o);
            else if (st2)
                Tr<T>::stn(dst + (int64_t)(s - 2) * plane, o.x, o.y);
        }
    };
    using One = std::integral_constant<int, 1>;
    using Two = std::integral_constant<int, 2>;
    using Three = std::integral_constant<int, 3>;
    int s = zf - 2;
    step(s, std::integral_constant<int, 0>{}, One{});
    step(s + 1, std::integral_constant<int, 1>{}, One{});
    step(s + 2, std::integral_constant<int, 2>{}, Two{});
    step(s + 3, std::integral_constant<int, 3>{}, Two{});
    s += 4;
#define JC_STEP3(k) step(s + (k), std::integral_constant<int, ((k) + 4) % RS>{}, Three{})
    const int s_end = zl + 2;
    for (; s + 5 <= s_end; s += 6) {
        JC_STEP3(0);
        JC_STEP3(1);
        JC_STEP3(2);
        JC_STEP3(3);
        JC_STEP3(4);
        JC_STEP3(5);
    }
    if (s <= s_end) JC_STEP3(0);
    if (s + 1 <= s_end) JC_STEP3(1);
    if (s + 2 <= s_end) JC_STEP3(2);
    if (s + 3 <= s_end) JC_STEP3(3);
    if (s + 4 <= s_end) JC_STEP3(4);
#undef JC_STEP3
}
// ---- three sweeps of a correction in quads: end ----

// Fills in the tiles of a launch over one block; the work-groups, or 0 where
// there are too many.
int one_block_tiles(OneBlock& one, int tile_y, int z_chunk)
{
    if (one.nx < 1 || one.ny < 1 || one.nz < 1 || z_chunk < 1 || tile_y < 1)
        return 0;
    const int64_t tx = (one.nx + 63) / 64, ty = (one.ny + tile_y - 1) / tile_y;
    const int64_t nch = (one.nz + (int64_t)z_chunk - 1) / z_chunk, n = tx * ty * nch;
    if (n > ((int64_t)1 << 30))
        return 0;
    one.tiles_x = (int32_t)tx;
    one.tiles_y = (int32_t)ty;
    one.planes = (int32_t)(one.nz / nch);
    one.rest = (int32_t)(one.nz % nch);
    return (int)n;
}

template <typename T, int FIELD, int TXP, int TY, bool SRC>
hipError_t sweep2_launch(const OneBlock& one, const BlockDesc* blocks, const Item* items, int parity, int n, hipStream_t s,
                         uint32_t pace)
{
    const int grid = (n + 7) / 8 * 8;
    hipLaunchKernelGGL((k_sweep2<T, FIELD, TXP, TY, SRC>), dim3(grid), dim3(((TXP + 2) * (TY + 4) + 63) / 64 * 64), 0, s,
                       one, blocks, items, parity, n, pace);
    return hipGetLastError();
}

template <typename T, int FIELD, bool SRC>
hipError_t sweep2_rows(const OneBlock& one, const BlockDesc* blocks, const Item* items, int parity, int tile_y, int n,
                       hipStream_t s, uint32_t pace)
{
    switch (tile_y) {
    case 8: return sweep2_launch<T, FIELD, 32, 8, SRC>(one, blocks, items, parity, n, s, pace);
    case 16: return sweep2_launch<T, FIELD, 32, 16, SRC>(one, blocks, items, parity, n, s, pace);
    case 24: return sweep2_launch<T, FIELD, 32, 24, SRC>(one, blocks, items, parity, n, s, pace);
    case 32:
        // a work list of 32-cell tiles: the last two sweeps of a window that a
        // group sweeps three at a time
        if constexpr (sizeof(T) < 8)
            return items ? sweep2_launch<T, FIELD, 16, 32, SRC>(one, blocks, items, parity, n, s, pace)
                         : hipErrorInvalidValue;
        else
            return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
}

template <typename T, int FIELD, int TXP, int TY, bool SRC>
hipError_t sweep3_launch(const OneBlock& one, const BlockDesc* blocks, const Item* items, int parity, int n, hipStream_t s,
                         uint32_t pace)
{
    const int grid = (n + 7) / 8 * 8;
    hipLaunchKernelGGL((k_sweep3<T, FIELD, TXP, TY, SRC>), dim3(grid), dim3(((TXP + 4) * (TY + 6) + 63) / 64 * 64), 0, s,
                       one, blocks, items, parity, n, pace);
    return hipGetLastError();
}

template <typename T, int FIELD, bool SRC>
hipError_t sweep3_rows(const OneBlock& one, const BlockDesc* blocks, const Item* items, int parity, int tile_y, int n,
                       hipStream_t s, uint32_t pace)
{
    switch (tile_y) {
    case 8: return sweep3_launch<T, FIELD, 32, 8, SRC>(one, blocks, items, parity, n, s, pace);
    case 16: return sweep3_launch<T, FIELD, 32, 16, SRC>(one, blocks, items, parity, n, s, pace);
    case 32:
        // a work list of 32-cell tiles
        if constexpr (sizeof(T) < 8)
            return items ? sweep3_launch<T, FIELD, 16, 32, SRC>(one, blocks, items, parity, n, s, pace)
                         : hipErrorInvalidValue;
        else
            return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
}

template <typename T, int TXQ, int TY>
hipError_t quads_launch(const OneBlock& one, const BlockDesc* blocks, const Item* items, int parity, int n, hipStream_t s,
                        uint32_t pace)
{
    const int grid = (n + 7) / 8 * 8;
    hipLaunchKernelGGL((k_sweep3q<T, TXQ, TY>), dim3(grid), dim3(quad_threads(TXQ, TY)), 0, s, one, blocks, items, parity,
                       n, pace);
    return hipGetLastError();
}

// The sweeps of the iterate (with or without a source) and of the correction
// by storage format, `ROWS` = sweep2_rows or sweep3_rows.
#define JC_FIELD_U(ROWS, one, blocks, items, parity, n, pace)                                                   \
    (src ? ROWS<double, FIELD_U, true>(one, blocks, items, parity, tile_y, n, s, pace)                           \
         : ROWS<double, FIELD_U, false>(one, blocks, items, parity, tile_y, n, s, pace))
#define JC_FIELD_D(ROWS, one, blocks, items, parity, n, pace)                                                   \
    (lo_dtype == 0   ? ROWS<double, FIELD_D, true>(one, blocks, items, parity, tile_y, n, s, pace)               \
     : lo_dtype == 1 ? ROWS<float, FIELD_D, true>(one, blocks, items, parity, tile_y, n, s, pace)                \
     : lo_dtype == 2 ? ROWS<bf16, FIELD_D, true>(one, blocks, items, parity, tile_y, n, s, pace)                 \
                     : hipErrorInvalidValue)

}  // namespace

hipError_t launch_sweep2(OneBlock one, int tile_y, int z_chunk, bool src, hipStream_t s, uint32_t pace)
{
    const int n = one_block_tiles(one, tile_y, z_chunk);
    return n < 1 ? hipErrorInvalidValue : JC_FIELD_U(sweep2_rows, one, nullptr, nullptr, 0, n, pace);
}

hipError_t launch_sweep3(OneBlock one, int tile_y, int z_chunk, bool src, hipStream_t s, uint32_t pace)
{
    const int n = one_block_tiles(one, tile_y, z_chunk);
    return n < 1 ? hipErrorInvalidValue : JC_FIELD_U(sweep3_rows, one, nullptr, nullptr, 0, n, pace);
}

hipError_t launch_ir_inner2(OneBlock one, int tile_y, int z_chunk, int lo_dtype, hipStream_t s, uint32_t pace)
{
    const int n = one_block_tiles(one, tile_y, z_chunk);
    return n < 1 ? hipErrorInvalidValue : JC_FIELD_D(sweep2_rows, one, nullptr, nullptr, 0, n, pace);
}

hipError_t launch_ir_inner3(OneBlock one, int tile_y, int z_chunk, int lo_dtype, hipStream_t s, uint32_t pace)
{
    const int n = one_block_tiles(one, tile_y, z_chunk);
    return n < 1 ? hipErrorInvalidValue : JC_FIELD_D(sweep3_rows, one, nullptr, nullptr, 0, n, pace);
}

hipError_t launch_ir_inner3_quads(OneBlock one, int z_chunk, int lo_dtype, hipStream_t s, uint32_t pace)
{
    const int n = one_block_tiles(one, 32, z_chunk);
    if (n < 1)
        return hipErrorInvalidValue;
    return lo_dtype == 1   ? quads_launch<float, 16, 32>(one, nullptr, nullptr, 0, n, s, pace)
           : lo_dtype == 2 ? quads_launch<bf16, 16, 32>(one, nullptr, nullptr, 0, n, s, pace)
                           : hipErrorInvalidValue;
}

hipError_t launch_ir_inner3_quad_items(const BlockDesc* blocks, const Item* items, int nitems, int qparity, int tile_y,
                                       hipStream_t s)
{
    if (nitems <= 0)
        return hipSuccess;
    return tile_y == 16   ? quads_launch<float, 16, 16>(OneBlock{}, blocks, items, qparity, nitems, s, 0)
           : tile_y == 32 ? quads_launch<float, 8, 32>(OneBlock{}, blocks, items, qparity, nitems, s, 0)
                          : hipErrorInvalidValue;
}

hipError_t launch_sweep2_items(const BlockDesc* blocks, const Item* items, int nitems, int parity, int tile_y, bool src,
                               hipStream_t s)
{
    return nitems <= 0 ? hipSuccess : JC_FIELD_U(sweep2_rows, OneBlock{}, blocks, items, parity, nitems, 0u);
}

hipError_t launch_sweep3_items(const BlockDesc* blocks, const Item* items, int nitems, int parity, int tile_y, bool src,
                               hipStream_t s)
{
    return nitems <= 0 ? hipSuccess : JC_FIELD_U(sweep3_rows, OneBlock{}, blocks, items, parity, nitems, 0u);
}

hipError_t launch_ir_inner2_items(const BlockDesc* blocks, const Item* items, int nitems, int qparity, int tile_y,
                                  int lo_dtype, hipStream_t s)
{
    return nitems <= 0 ? hipSuccess : JC_FIELD_D(sweep2_rows, OneBlock{}, blocks, items, qparity, nitems, 0u);
}

hipError_t launch_ir_inner3_items(const BlockDesc* blocks, const Item* items, int nitems, int qparity, int tile_y,
                                  int lo_dtype, hipStream_t s)
{
    return nitems <= 0 ? hipSuccess : JC_FIELD_D(sweep3_rows, OneBlock{}, blocks, items, qparity, nitems, 0u);
}
#undef JC_FIELD_U
#undef JC_FIELD_D

}  // namespace jc
