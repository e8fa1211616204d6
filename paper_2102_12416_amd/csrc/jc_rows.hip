// Passes that touch every cell or face value once: global padded array <->
// blocks, the refinement's first inner sweep and outer update, and the staged
// halo exchange (pack, exchange, unpack; paper section 4.3), all bound by
// memory; and the sums of residual partials.

#include <hip/hip_runtime.h>

#include "jc_div6.h"
#include "jc_kernels.h"
#include "jc_storage.h"

namespace jc {

namespace {

// A pair of cells.  Block arrays hold the pair (x, x + 1), x odd, on a
// 16-byte boundary; rows of the global array start on any 8-byte boundary,
// where the hardware's unaligned 16-byte access costs an extra line at most.
typedef double pair8 __attribute__((ext_vector_type(2), aligned(8)));

__device__ __forceinline__ pair8 ld2(const double* p) { return *(const pair8 JC_GLOBAL*)(p); }
__device__ __forceinline__ void st2(double* p, pair8 v) { *(pair8 JC_GLOBAL*)(p) = v; }
__device__ __forceinline__ double ld1(const double* p) { return *(const double JC_GLOBAL*)(p); }
__device__ __forceinline__ void st1(double* p, double v) { *(double JC_GLOBAL*)(p) = v; }

// Row passes: LX lanes walk a row in 16-byte accesses, 256 / LX rows per
// work-group, one work-group per 256 / LX rows.  LX follows the widest block
// (row_lanes), so that a wave covers several rows of a narrow block and the
// launch has work-groups enough to keep memory busy.  Measured on MI355X
// (read + written bytes; before: one row per work-group, 8-byte accesses):
// the iterate of 125 blocks of up to 64^3 read back in 84 us (4.2 TB/s)
// against 333, of 512^3 in 2 x 2 x 2 blocks in 0.49 ms (4.4 TB/s, as before),
// of 512 x 768 x 1024 in 1.40 ms (4.6 TB/s) against 1.79; a large copy reaches
// 4.8.  Two, four or eight rows in flight per thread were 2 to 20 % slower,
// non-temporal stores up to 6 %.
constexpr int kRowThreads = 256;

// Global padded array -> blocks; blockIdx.y = block.  The iterate: copy 0
// whole (interior and ghosts); of copy 1 the ghosts only, since the first
// sweep writes its interior before anything reads it; and the compact
// Dirichlet ghost columns of unpaired x faces.  The source: whole.
template <int LX>
__global__ void __launch_bounds__(kRowThreads)
k_scatter(const BlockDesc* __restrict__ blocks, const double* __restrict__ g, int64_t gnx, int64_t gny, int which)
{
    constexpr int LY = kRowThreads / LX;
    const BlockDesc& B = blocks[blockIdx.y];
    const int nx = B.n[0], ny = B.n[1], nz = B.n[2];
    const int64_t gpitch = gnx + 2, gplane = (gnx + 2) * (gny + 2);
    const uint32_t rows = (uint32_t)(ny + 2) * (uint32_t)(nz + 2);
    const int lx = threadIdx.x % LX, ly = threadIdx.x / LX;
    const int npair = (nx + 1) / 2;               // pairs (1, 2), (3, 4) .. up to cell nx or nx + 1
    double* const u0 = which == 0 ? B.u[0] : const_cast<double*>(B.b);
    double* const u1 = B.u[1];
    for (uint32_t r = blockIdx.x * LY + ly; r < rows; r += gridDim.x * LY) {
        const int y = (int)(r % (uint32_t)(ny + 2)), z = (int)(r / (uint32_t)(ny + 2));
        const double* const src = g + (B.off[2] + z) * gplane + (B.off[1] + y) * gpitch + B.off[0];
        const int64_t at = (int64_t)z * B.plane + (int64_t)y * B.pitch;
        const bool ghost = y == 0 || y == ny + 1 || z == 0 || z == nz + 1;
        const bool both = which == 0 && ghost;
        for (int k = lx; k < npair; k += LX) {
            const pair8 v = ld2(src + 2 * k + 1);
            st2(u0 + at + 2 * k + 1, v);
            if (both)
                st2(u1 + at + 2 * k + 1, v);
        }
        // the x ghosts: x = 0, and x = nx + 1 (for an odd nx it is also the
        // second cell of the last pair)
        if (lx < 2) {
            const int x = lx == 0 ? 0 : nx + 1;
            const double v = ld1(src + x);
            st1(u0 + at + x, v);
            if (which == 0) {
                st1(u1 + at + x, v);
                double* const col = const_cast<double*>(B.xg[lx == 0 ? XM : XP]);
                if (col && !ghost)
                    st1(col + (int64_t)(z - 1) * face_ld(ny) + (y - 1), v);
            }
        }
    }
}

// Blocks -> global padded array: each block writes its interior, extended
// over the Dirichlet shell on the faces that lie on the global boundary, so
// every element of the global array is written exactly once.
template <int LX>
__global__ void __launch_bounds__(kRowThreads)
k_gather(const BlockDesc* __restrict__ blocks, double* __restrict__ g, int64_t gnx, int64_t gny, int64_t gnz,
         int which, int parity)
{
    constexpr int LY = kRowThreads / LX;
    const BlockDesc& B = blocks[blockIdx.y];
    const int nx = B.n[0], ny = B.n[1], nz = B.n[2];
    const int64_t gpitch = gnx + 2, gplane = (gnx + 2) * (gny + 2);
    const int ylo = B.off[1] == 0 ? 0 : 1, yhi = B.off[1] + ny == gny ? ny + 1 : ny;
    const int zlo = B.off[2] == 0 ? 0 : 1, zhi = B.off[2] + nz == gnz ? nz + 1 : nz;
    const int last = B.off[0] + nx == gnx ? nx + 1 : nx;   // last cell of a row
    const uint32_t ey = (uint32_t)(yhi - ylo + 1), rows = ey * (uint32_t)(zhi - zlo + 1);
    const int lx = threadIdx.x % LX, ly = threadIdx.x / LX;
    const int npair = last / 2;
    const double* const src = which == 0 ? B.u[parity] : B.b;
    for (uint32_t r = blockIdx.x * LY + ly; r < rows; r += gridDim.x * LY) {
        const int y = ylo + (int)(r % ey), z = zlo + (int)(r / ey);
        double* const dst = g + (B.off[2] + z) * gplane + (B.off[1] + y) * gpitch + B.off[0];
        const double* const from = src + (int64_t)z * B.plane + (int64_t)y * B.pitch;
        for (int k = lx; k < npair; k += LX)
            st2(dst + 2 * k + 1, ld2(from + 2 * k + 1));
        // x = 0 on the shell, and the cell that the pairs leave over
        if (lx == 0 && B.off[0] == 0)
            st1(dst, ld1(from));
        if (lx == 1 && (last & 1))
            st1(dst + last, ld1(from + last));
    }
}

// ---- refinement: the passes that touch every cell once ----

// First inner sweep of a refinement step: d_1 = lo((0 + r_lo) / 6) (d_0 = 0,
// so no neighbour is read); writes copy 1 of d and its faces.  Bound by
// memory: reads r_lo, writes d.  A lane takes 16 bytes of a row (2, 4 or 8
// cells); cells past the end of a row are ghosts, padding or the next row's
// x = 0 ghost, all zero for the correction, and are written as zero.
template <typename T, int LX>
__global__ void __launch_bounds__(kRowThreads)
k_ir_first(const BlockDesc* __restrict__ blocks)
{
    using C = typename Tr<T>::C;
    using P = typename Tr<T>::P;
    constexpr int LY = kRowThreads / LX;
    constexpr int NP = 16 / (int)sizeof(P);       // pairs per lane
    constexpr int V = 2 * NP;                     // cells per lane
    typedef uint32_t v4u __attribute__((ext_vector_type(4)));
    const BlockDesc* B = blocks + blockIdx.y;
    const int nx = B->n[0], ny = B->n[1], nz = B->n[2];
    const int64_t ldx = face_ld(ny), ldy = face_ld(nx);
    const T* const rl = static_cast<const T*>(B->rlo);
    T* const d = static_cast<T*>(B->d[1]);
    const int lx = threadIdx.x % LX, ly = threadIdx.x / LX;
    const int nvec = (nx + V - 1) / V;
    const uint32_t rows = (uint32_t)ny * (uint32_t)nz;
    T* const oxm = static_cast<T*>(B->lgout[XM][1]);
    T* const oxp = static_cast<T*>(B->lgout[XP][1]);
    T* const oym = static_cast<T*>(B->lgout[YM][1]);
    T* const oyp = static_cast<T*>(B->lgout[YP][1]);
    T* const ozm = static_cast<T*>(B->lgout[ZM][1]);
    T* const ozp = static_cast<T*>(B->lgout[ZP][1]);
    for (uint32_t r = blockIdx.x * LY + ly; r < rows; r += gridDim.x * LY) {
        const int y = (int)(r % (uint32_t)ny) + 1, z = (int)(r / (uint32_t)ny) + 1;
        const int64_t at = (int64_t)z * B->lplane + (int64_t)y * B->lpitch + 1;
        const bool yz_face = (y == 1 && oym) || (y == ny && oyp) || (z == 1 && ozm) || (z == nz && ozp);
        for (int k = lx; k < nvec; k += LX) {
            union {
                v4u raw;
                P p[NP];
            } v;
            v.raw = *(const v4u JC_GLOBAL*)(rl + at + V * k);
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                C a, b;
                Tr<T>::unpack(v.p[q], a, b);
                const int xa = V * k + 2 * q + 1;
                const C va = xa <= nx ? div6(C(0) + a) : C(0);
                const C vb = xa + 1 <= nx ? div6(C(0) + b) : C(0);
                v.p[q] = Tr<T>::pack(va, vb);
            }
            *(v4u JC_GLOBAL*)(d + at + V * k) = v.raw;
            if (!(yz_face || (k == 0 && oxm) || (V * (k + 1) >= nx && oxp)))
                continue;
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                const int xa = V * k + 2 * q + 1;
                if (xa > nx)
                    break;
                const int64_t xfi = (int64_t)(z - 1) * ldx + (y - 1);
                const int64_t yfi = (int64_t)(z - 1) * ldy + (xa - 1);
                const int64_t zfi = (int64_t)(y - 1) * ldy + (xa - 1);
                if (xa == 1 && oxm) Tr<T>::st1a(oxm + xfi, v.p[q]);
                if (xa == nx && oxp) Tr<T>::st1a(oxp + xfi, v.p[q]);
                if (xa + 1 == nx && oxp) Tr<T>::st1b(oxp + xfi, v.p[q]);
                if (y == 1 && oym) Tr<T>::stp(oym + yfi, v.p[q]);
                if (y == ny && oyp) Tr<T>::stp(oyp + yfi, v.p[q]);
                if (z == 1 && ozm) Tr<T>::stp(ozm + zfi, v.p[q]);
                if (z == nz && ozp) Tr<T>::stp(ozp + zfi, v.p[q]);
            }
        }
    }
}

// Outer update of the refinement: u(copy p) += (double) d(copy q) on the
// interior; the updated face cells go to the u face buffers of slot p.
// Bound by memory: reads u and d, writes u.
template <typename T, int LX>
__global__ void __launch_bounds__(kRowThreads)
k_ir_update(const BlockDesc* __restrict__ blocks, int p, int q)
{
    using C = typename Tr<T>::C;
    constexpr int LY = kRowThreads / LX;
    const BlockDesc* B = blocks + blockIdx.y;
    const int nx = B->n[0], ny = B->n[1], nz = B->n[2];
    const int64_t ldx = face_ld(ny), ldy = face_ld(nx);
    double* const u = B->u[p];
    const T* const d = static_cast<const T*>(B->d[q]);
    const int lx = threadIdx.x % LX, ly = threadIdx.x / LX;
    const int npair = (nx + 1) / 2;
    const uint32_t rows = (uint32_t)ny * (uint32_t)nz;
    double* const oxm = B->gout[XM][p];
    double* const oxp = B->gout[XP][p];
    double* const oym = B->gout[YM][p];
    double* const oyp = B->gout[YP][p];
    double* const ozm = B->gout[ZM][p];
    double* const ozp = B->gout[ZP][p];
    for (uint32_t r = blockIdx.x * LY + ly; r < rows; r += gridDim.x * LY) {
        const int y = (int)(r % (uint32_t)ny) + 1, z = (int)(r / (uint32_t)ny) + 1;
        double* const up = u + (int64_t)z * B->plane + (int64_t)y * B->pitch + 1;
        const T* const dp = d + (int64_t)z * B->lplane + (int64_t)y * B->lpitch + 1;
        for (int j = lx; j < npair; j += LX) {
            const int xa = 2 * j + 1;
            const bool b_ok = xa + 1 <= nx;
            double ua, ub;
            C da, db;
            Tr<double>::ld(up + 2 * j, ua, ub);
            Tr<T>::ld(dp + 2 * j, da, db);
            const double va = ua + (double)da;
            const double vb = b_ok ? ub + (double)db : ub;
            Tr<double>::st(up + 2 * j, va, vb);
            const int64_t xfi = (int64_t)(z - 1) * ldx + (y - 1);
            const int64_t yfi = (int64_t)(z - 1) * ldy + (xa - 1);
            const int64_t zfi = (int64_t)(y - 1) * ldy + (xa - 1);
            if (xa == 1 && oxm) Tr<double>::st1(oxm + xfi, va);
            if (xa == nx && oxp) Tr<double>::st1(oxp + xfi, va);
            if (b_ok && xa + 1 == nx && oxp) Tr<double>::st1(oxp + xfi, vb);
            if (y == 1 && oym) Tr<double>::st(oym + yfi, va, vb);
            if (y == ny && oyp) Tr<double>::st(oyp + yfi, va, vb);
            if (z == 1 && ozm) Tr<double>::st(ozm + zfi, va, vb);
            if (z == nz && ozp) Tr<double>::st(ozp + zfi, va, vb);
        }
    }
}

// Address of the cell (slow, fast) of the plane of face f, at depth
// `ghost` (0: the outermost interior plane, 1: the ghost plane beyond it).
__device__ __forceinline__ int64_t face_cell(const BlockDesc& B, int f, int slow, int fast, int ghost)
{
    const int nx = B.n[0], ny = B.n[1], nz = B.n[2];
    int x, y, z;
    switch (f) {
    case XM: x = ghost ? 0 : 1;            y = fast + 1; z = slow + 1; break;
    case XP: x = ghost ? nx + 1 : nx;      y = fast + 1; z = slow + 1; break;
    case YM: y = ghost ? 0 : 1;            x = fast + 1; z = slow + 1; break;
    case YP: y = ghost ? ny + 1 : ny;      x = fast + 1; z = slow + 1; break;
    case ZM: z = ghost ? 0 : 1;            x = fast + 1; y = slow + 1; break;
    default: z = ghost ? nz + 1 : nz;      x = fast + 1; y = slow + 1; break;
    }
    return (int64_t)z * B.plane + (int64_t)y * B.pitch + x;
}

// Face values in one flat index over the shared plane, one per thread.  An
// x face is a strided gather: a 128-byte line per value, which is what bounds
// the launch (600 faces of up to 64^2: 16 us to pack and 14 to unpack, 19 and
// 20 with one row of the plane per work-group, which idled three lanes of four).
template <bool PACK>
__global__ void __launch_bounds__(256)
k_faces(const BlockDesc* __restrict__ blocks, const PairDesc* __restrict__ pairs, int parity, int slot)
{
    const PairDesc& P = pairs[blockIdx.y];
    const uint32_t n = (uint32_t)P.count, fast = (uint32_t)P.fast;
    const BlockDesc& B = blocks[PACK ? P.src_block : P.dst_block];
    double* const cells = B.u[parity];
    double* const buf = P.buf[slot];
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
        const int s = (int)(i / fast), q = (int)(i % fast);
        double* const cell = cells + face_cell(B, PACK ? P.src_face : P.dst_face, s, q, PACK ? 0 : 1);
        double* const at = buf + s * face_ld(P.fast) + q;
        st1(PACK ? at : cell, ld1(PACK ? cell : at));
    }
}

// The pairing's transfer: every send buffer into the receive buffer
// pre-posted for it.  Buffers are 256-byte aligned with an even number of
// elements: 16-byte vectors.
__global__ void __launch_bounds__(256)
k_exchange(const PairDesc* __restrict__ pairs)
{
    const PairDesc& P = pairs[blockIdx.y];
    const int64_t n2 = P.span >> 1;
    const double2* __restrict__ a = reinterpret_cast<const double2*>(P.buf[0]);
    double2* __restrict__ b = reinterpret_cast<double2*>(P.buf[1]);
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n2; i += (int64_t)gridDim.x * 256)
        b[i] = a[i];
}

// Zero `words` 8-byte words at p (grid-stride).
__global__ void __launch_bounds__(256)
k_zero(uint64_t* __restrict__ p, int64_t words)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < words; i += (int64_t)gridDim.x * 256)
        *(uint64_t JC_GLOBAL*)(p + i) = 0;
}

// Fixed-order sum of one member's partials [ranges[2m], ranges[2m+1]): each
// thread adds a strided subsequence in order (eight loads in flight), then a
// fixed tree over the work-group.  The sums go to `out` in device memory, or
// (`host` not null) straight to pinned host memory, each followed by the
// check's sequence number, which the host waits for: that spares the copy
// and its launch, about 8 us of the 25 that a check of a small grid took.
__global__ void __launch_bounds__(256)
k_reduce(const double* __restrict__ partials, const int32_t* __restrict__ ranges, double* __restrict__ out,
         HostSum* host, uint64_t seq)
{
    const int m = blockIdx.x;
    const int lo = ranges[2 * m], hi = ranges[2 * m + 1];
    double t = 0.0;
    int i = lo + (int)threadIdx.x;
    for (; i + 7 * 256 < hi; i += 8 * 256) {
        double v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            v[k] = partials[i + k * 256];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            t = t + v[k];
    }
    for (; i < hi; i += 256)
        t = t + partials[i];
    __shared__ double w[4];
    t = wave_sum(t);
    if ((threadIdx.x & 63) == 0)
        w[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double sum = ((w[0] + w[1]) + w[2]) + w[3];
        if (host) {
            host[m].sum = sum;
            __hip_atomic_store(&host[m].seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        } else {
            out[m] = sum;
        }
    }
}

// Lanes per row: the power of two in 8 .. 64 that covers the accesses of the
// widest block's row, so that a wave covers several rows of a narrow block.
int row_lanes(int accesses) { return accesses <= 8 ? 8 : accesses <= 16 ? 16 : accesses <= 32 ? 32 : 64; }

// Work-groups of 256 / lanes rows; at most 65536 per block (the kernels
// stride over the rest).
dim3 row_grid(int nblocks, int64_t max_rows, int lanes)
{
    const int64_t per = kRowThreads / lanes;
    int64_t n = (max_rows + per - 1) / per;
    n = n < 1 ? 1 : n > 65536 ? 65536 : n;
    return dim3((unsigned)n, (unsigned)nblocks);
}

dim3 face_grid(int npairs, int64_t max_slow, int64_t max_fast)
{
    const int64_t n = (max_slow * max_fast + 255) / 256;
    return dim3((unsigned)(n < 1 ? 1 : n > 65536 ? 65536 : n), (unsigned)npairs);
}

}  // namespace

hipError_t launch_zero(void* p, size_t bytes, hipStream_t s)
{
    const int64_t words = (int64_t)(bytes / 8);
    if (words <= 0)
        return hipSuccess;
    int64_t blocks = (words + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_zero, dim3((unsigned)blocks), dim3(256), 0, s, static_cast<uint64_t*>(p), words);
    return hipGetLastError();
}

hipError_t launch_reduce(const double* partials, const int32_t* ranges, int nmembers, double* out, HostSum* host,
                         uint64_t seq, hipStream_t s)
{
    if (nmembers <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_reduce, dim3(nmembers), dim3(256), 0, s, partials, ranges, out, host, seq);
    return hipGetLastError();
}

hipError_t launch_pack(const BlockDesc* blocks, const PairDesc* pairs, int npairs, int max_slow, int max_fast,
                       int parity, int slot, hipStream_t s)
{
    if (npairs <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_faces<true>, face_grid(npairs, max_slow, max_fast), dim3(256), 0, s, blocks, pairs, parity,
                       slot);
    return hipGetLastError();
}

hipError_t launch_exchange(const PairDesc* pairs, int npairs, int64_t max_count, hipStream_t s)
{
    if (npairs <= 0)
        return hipSuccess;
    int64_t chunks = (max_count / 2 + 255) / 256;
    if (chunks < 1) chunks = 1;
    if (chunks > 1024) chunks = 1024;
    hipLaunchKernelGGL(k_exchange, dim3((unsigned)chunks, npairs), dim3(256), 0, s, pairs);
    return hipGetLastError();
}

hipError_t launch_unpack(const BlockDesc* blocks, const PairDesc* pairs, int npairs, int max_slow, int max_fast,
                         int parity, hipStream_t s)
{
    if (npairs <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_faces<false>, face_grid(npairs, max_slow, max_fast), dim3(256), 0, s, blocks, pairs, parity,
                       1);
    return hipGetLastError();
}

#define JC_ROW_LANES(K, ...)                                                               \
    switch (lanes) {                                                                      \
    case 8: hipLaunchKernelGGL((K<8>), grid, dim3(kRowThreads), 0, s, __VA_ARGS__); break;   \
    case 16: hipLaunchKernelGGL((K<16>), grid, dim3(kRowThreads), 0, s, __VA_ARGS__); break; \
    case 32: hipLaunchKernelGGL((K<32>), grid, dim3(kRowThreads), 0, s, __VA_ARGS__); break; \
    default: hipLaunchKernelGGL((K<64>), grid, dim3(kRowThreads), 0, s, __VA_ARGS__); break; \
    }
#define JC_ROW_LANES_T(K, T, ...)                                                             \
    switch (lanes) {                                                                         \
    case 8: hipLaunchKernelGGL((K<T, 8>), grid, dim3(kRowThreads), 0, s, __VA_ARGS__); break;   \
    case 16: hipLaunchKernelGGL((K<T, 16>), grid, dim3(kRowThreads), 0, s, __VA_ARGS__); break; \
    case 32: hipLaunchKernelGGL((K<T, 32>), grid, dim3(kRowThreads), 0, s, __VA_ARGS__); break; \
    default: hipLaunchKernelGGL((K<T, 64>), grid, dim3(kRowThreads), 0, s, __VA_ARGS__); break; \
    }

hipError_t launch_ir_first(const BlockDesc* blocks, int nblocks, int64_t max_rows, int64_t max_nx, int lo_dtype,
                           hipStream_t s)
{
    if (nblocks <= 0)
        return hipSuccess;
    // a lane takes 16 bytes: 2, 4 or 8 cells
    const int cells = lo_dtype == 0 ? 2 : lo_dtype == 1 ? 4 : 8;
    const int lanes = row_lanes((int)((max_nx + cells - 1) / cells));
    const dim3 grid = row_grid(nblocks, max_rows, lanes);
    switch (lo_dtype) {
    case 0: JC_ROW_LANES_T(k_ir_first, double, blocks) break;
    case 1: JC_ROW_LANES_T(k_ir_first, float, blocks) break;
    case 2: JC_ROW_LANES_T(k_ir_first, bf16, blocks) break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_ir_update(const BlockDesc* blocks, int nblocks, int64_t max_rows, int64_t max_nx, int p, int q,
                            int lo_dtype, hipStream_t s)
{
    if (nblocks <= 0)
        return hipSuccess;
    const int lanes = row_lanes((int)((max_nx + 1) / 2));
    const dim3 grid = row_grid(nblocks, max_rows, lanes);
    switch (lo_dtype) {
    case 0: JC_ROW_LANES_T(k_ir_update, double, blocks, p, q) break;
    case 1: JC_ROW_LANES_T(k_ir_update, float, blocks, p, q) break;
    case 2: JC_ROW_LANES_T(k_ir_update, bf16, blocks, p, q) break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_scatter(const BlockDesc* blocks, int nblocks, int64_t max_rows, int64_t max_nx,
                          const double* global, int64_t gnx, int64_t gny, int which, hipStream_t s)
{
    if (nblocks <= 0)
        return hipSuccess;
    const int lanes = row_lanes((int)((max_nx + 1) / 2));
    const dim3 grid = row_grid(nblocks, max_rows, lanes);
    JC_ROW_LANES(k_scatter, blocks, global, gnx, gny, which)
    return hipGetLastError();
}

hipError_t launch_gather(const BlockDesc* blocks, int nblocks, int64_t max_rows, int64_t max_nx, double* global,
                         int64_t gnx, int64_t gny, int64_t gnz, int which, int parity, hipStream_t s)
{
    if (nblocks <= 0)
        return hipSuccess;
    const int lanes = row_lanes((int)((max_nx + 1) / 2));
    const dim3 grid = row_grid(nblocks, max_rows, lanes);
    JC_ROW_LANES(k_gather, blocks, global, gnx, gny, gnz, which, parity)
    return hipGetLastError();
}
#undef JC_ROW_LANES
#undef JC_ROW_LANES_T

}  // namespace jc
