// Batched persistent kernel, bandwidth yardsticks (triad, read-only,
// write-only, copy) and the
// per-precision dispatch of the site kernels.
#include "su3_device.h"

namespace su3i {
hipError_t launch_site_p0(int, int, int, int, int, int, size_t, const SiteArgs &, hipStream_t);
hipError_t launch_site_p1(int, int, int, int, int, int, size_t, const SiteArgs &, hipStream_t);
hipError_t launch_site_p2(int, int, int, int, int, int, size_t, const SiteArgs &, hipStream_t);
hipError_t launch_site_p3(int, int, int, int, int, int, size_t, const SiteArgs &, hipStream_t);
hipError_t launch_shift_p0(int, int, int, int, int, size_t, const ShiftArgs &, hipStream_t);
hipError_t launch_shift_p1(int, int, int, int, int, size_t, const ShiftArgs &, hipStream_t);
hipError_t launch_shift_p2(int, int, int, int, int, size_t, const ShiftArgs &, hipStream_t);
hipError_t launch_shift_p3(int, int, int, int, int, size_t, const ShiftArgs &, hipStream_t);
hipError_t launch_site_lds_p0(int, int, int, int, size_t, const SiteArgs &, hipStream_t);
hipError_t launch_site_lds_p1(int, int, int, int, size_t, const SiteArgs &, hipStream_t);
hipError_t launch_site_lds_p2(int, int, int, int, size_t, const SiteArgs &, hipStream_t);
hipError_t launch_site_lds_p3(int, int, int, int, size_t, const SiteArgs &, hipStream_t);
}  // namespace su3i

namespace su3k {

using su3i::BatchItem;

// Evaluate one tile: `count` sites of item `it` from site `first` (a
// multiple of the tile size, hence of S), lanes striding over its groups.
template <int P, int X, int NT, int SCHED>
__device__ __forceinline__ void tile_run(const BatchItem &it, int first,
                                         int count)
{
    constexpr int S = SitesPerLane<P, X>::value;
    const void *const ops[4] = {it.op[0], it.op[1], it.op[2], it.op[3]};
    const int ng = (count + S - 1) / S;
    for (int g = threadIdx.x; g < ng; g += blockDim.x) {
        const uint32_t s0 = uint32_t(first + g * S);
        const uint32_t off = site_offset(it.g, s0);
        const int cnt = first + count - int(s0);
        if (cnt >= S)
            do_group<P, X, S, NT, true, SCHED>(it.z, ops, off, off, it.g.plane, S);
        else
            do_group<P, X, S, NT, false, SCHED>(it.z, ops, off, off, it.g.plane, cnt);
    }
}

template <int P, int NT, int SCHED>
__device__ __forceinline__ void tile_any_expr(const BatchItem &it, int first,
                                              int count)
{
    switch (it.expr) {
    case su3i::MUL: tile_run<P, su3i::MUL, NT, SCHED>(it, first, count); break;
    case su3i::MUL3: tile_run<P, su3i::MUL3, NT, SCHED>(it, first, count); break;
    default:
        if constexpr (P != su3i::C12) {
            switch (it.expr) {
            case su3i::MULADD: tile_run<P, su3i::MULADD, NT, SCHED>(it, first, count); break;
            case su3i::ADD: tile_run<P, su3i::ADD, NT, SCHED>(it, first, count); break;
            case su3i::APB_AB: tile_run<P, su3i::APB_AB, NT, SCHED>(it, first, count); break;
            }
        }
        break;
    }
}

__device__ __forceinline__ uint32_t plane_real_bytes(int prec)
{
    return prec == su3i::F64 ? 8 : prec == su3i::F16 ? 2 : 4;
}

// One tile of the batch: find its item by binary search over the items'
// tile starts -- a small array every workgroup reads, so it stays in the
// scalar cache and no per-tile record has to come from memory before the
// data loads start -- and evaluate it.  The branch on precision and
// expression is uniform across the workgroup.
template <int MODE, int NT, int SCHED>
__device__ __forceinline__ void batch_tile(const BatchItem *items, int nitems, int t,
                                           int T, bool remap)
{
    int lo = 0, hi = nitems - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (items[mid].tile_start <= t)
            lo = mid;
        else
            hi = mid - 1;
    }
    const BatchItem &it = items[lo];
    int local = t - it.tile_start;
    // Entry planes 2 to 16 MiB apart, power-of-two lattices: each XCD takes a
    // range of the item's tiles, as the site kernels' workgroups (items of
    // 32^4 double: 5.6 GB 893 us, dealt one by one 1136).
    const uint32_t plane = it.g.plane * plane_real_bytes(it.prec);
    if (remap && it.g.lg == 31 && (plane & ((2u << 20) - 1)) == 0 && plane <= (16u << 20))
        local = xcd_remap(local, (it.nsites + T - 1) / T);
    const int first = local * T;
    const int count = min(T, it.nsites - first);
    if constexpr (MODE == 0) {
        if (it.prec == su3i::F64)
            tile_run<su3i::F64, su3i::MUL, NT, SCHED>(it, first, count);
        else
            tile_run<su3i::C12, su3i::MUL, NT, SCHED>(it, first, count);
    } else {
        switch (it.prec) {
        case su3i::F64: tile_any_expr<su3i::F64, NT, SCHED>(it, first, count); break;
        case su3i::F32: tile_any_expr<su3i::F32, NT, SCHED>(it, first, count); break;
        case su3i::F16: tile_any_expr<su3i::F16, NT, SCHED>(it, first, count); break;
        case su3i::C12: tile_any_expr<su3i::C12, NT, SCHED>(it, first, count); break;
        }
    }
}

// Batched kernel over the tile table.  Item i owns tiles tile_start_i ..
// tile_start_{i+1} - 1, each of T sites (the item's last tile may be
// shorter).
//   queue == nullptr: one workgroup per tile (a one-shot grid; workgroup b
//     takes tiles b, b + G, ... when the grid is smaller).
//   queue != nullptr: a persistent grid whose workgroups take tiles from a
//     ticket counter in queue[0], in order, until the tiles run out: lane 0
//     draws ticket v and the workgroup takes tile v mod (ntiles + G); a
//     value >= ntiles means no tile is left and the workgroup leaves.  Every
//     workgroup draws once more after its last tile, so a launch draws
//     exactly ntiles + G tickets and leaves the counter at the next
//     multiple of it: the queue never needs resetting between launches of
//     the same batch (it starts at 0; launches must not overlap, which the
//     host sees to).  The next ticket is drawn while the
//     current tile is evaluated, so its latency is hidden.  The ticket goes
//     from lane 0 to the workgroup through the first bytes of the dynamic
//     LDS (the host reserves at least 16).
template <int MODE, int NT, int SCHED>
__global__ __launch_bounds__(256) void k_batch(const BatchItem *items, int nitems,
                                               int ntiles, int T,
                                               unsigned long long *queue)
{
    // dynamic LDS: the ticket of the queued form, and the reserve that
    // caps the workgroups per CU (otherwise never read)
    extern __shared__ char occupancy_reserve[];
    if (!queue) {
        for (int t = blockIdx.x; t < ntiles; t += gridDim.x)
            batch_tile<MODE, NT, SCHED>(items, nitems, t, T, true);
        if (ntiles < 0)
            occupancy_reserve[threadIdx.x] = 0;
        return;
    }
    volatile int *ticket = reinterpret_cast<volatile int *>(occupancy_reserve);
    const unsigned long long m = (unsigned long long)ntiles + gridDim.x;
    unsigned long long next = 0;
    if (threadIdx.x == 0)
        next = atomicAdd(queue, 1ull);
    for (;;) {
        if (threadIdx.x == 0)
            *ticket = (int)(next % m);
        __syncthreads();
        const int t = *ticket;
        __syncthreads();
        if (t >= ntiles)
            break;
        if (threadIdx.x == 0)
            next = atomicAdd(queue, 1ull);
        batch_tile<MODE, NT, SCHED>(items, nitems, t, T, false);
    }
}

// Item records of a batch written from kernel arguments (the allocation-
// free batch: no copy from host memory, so the write can sit in a captured
// graph); with `queue`, also zero the persistent grid's ticket counter.
__global__ __launch_bounds__(64) void k_put_items(BatchItem *dst, su3i::ItemChunk c,
                                                  int count, unsigned long long *queue)
{
    const int i = threadIdx.x;
    if (i < count)
        dst[i] = c.it[i];
    if (queue && i == 0)
        *queue = 0ull;
}

// Stored order <-> canonical host order.  A workgroup handles 64 sites, one
// wave per entry: every wave's access to the stored field is whole lines,
// and the 64 sites' canonical records (9 KB for a matrix), which the waves
// read or write with a stride, stay in the L1 for all of them.  The kernels
// run behind the PCIe copies of the canonical data (48 MB: 1.6 ms) and take
// a few per cent of their time.
__device__ __forceinline__ uint32_t storage_of(const su3i::HostOrder &h, uint32_t s)
{
    if (!h.vnode)
        return s;
    uint32_t osite = 0, lane = 0, ostride = 1, lstride = 1;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const uint32_t x = s % (uint32_t)h.dims[d];
        s /= (uint32_t)h.dims[d];
        const uint32_t n = x / (uint32_t)h.sub[d];
        osite += (x - n * h.sub[d]) * ostride;
        lane += n * lstride;
        ostride *= h.sub[d];
        lstride *= h.simd[d];
    }
    return osite * lstride + lane;
}

// Offset (stored reals) of entry e of storage site q; real scalars hold one
// real per entry, so their offsets are half of a complex entry's.
__device__ __forceinline__ uint32_t entry_offset(const su3i::HostOrder &h, uint32_t q, int e)
{
    return h.ncomp == 1 ? q : site_offset(h.g, q) + (uint32_t)e * h.g.plane;
}

__device__ __forceinline__ void put_stored(const su3i::HostOrder &h, uint32_t at, double v)
{
    if (h.prec == su3i::F64) {
        static_cast<double *>(h.field)[at] = v;
    } else {
        // to half by way of single, each rounding to nearest even (the empty
        // asm keeps the two conversions apart)
        float f = (float)v;
        __asm__ volatile("" : "+v"(f));
        if (h.prec == su3i::F16)
            static_cast<_Float16 *>(h.field)[at] = (_Float16)f;
        else
            static_cast<float *>(h.field)[at] = f;
    }
}

__device__ __forceinline__ double get_stored(const su3i::HostOrder &h, uint32_t at)
{
    if (h.prec == su3i::F64)
        return static_cast<const double *>(h.field)[at];
    if (h.prec == su3i::F16)
        return (double)(float)static_cast<const _Float16 *>(h.field)[at];
    return (double)static_cast<const float *>(h.field)[at];
}

__global__ __launch_bounds__(768) void k_pack(su3i::HostOrder h)
{
    const int e = threadIdx.x / 64;
    const int64_t i = (int64_t)blockIdx.x * 64 + threadIdx.x % 64;  // in the range
    const int64_t s = h.s0 + i;
    const bool site = i < h.count, pad = !site && s >= h.V && s < h.Vpad;
    if (!site && !pad)
        return;
    const uint32_t at = entry_offset(h, site ? storage_of(h, (uint32_t)s) : (uint32_t)s, e);
    const double *v = h.canon + (i * h.canon_entries + e) * h.ncomp;
    for (int c = 0; c < h.ncomp; ++c)
        put_stored(h, at + c, site ? v[c] : 0.0);
}

__global__ __launch_bounds__(768) void k_unpack(su3i::HostOrder h)
{
    const int e = threadIdx.x / 64;
    const int64_t i = (int64_t)blockIdx.x * 64 + threadIdx.x % 64;
    if (i >= h.count)
        return;
    const uint32_t q = storage_of(h, (uint32_t)(h.s0 + i));
    double *v = h.canon + (i * h.canon_entries + e) * h.ncomp;
    if (e < h.E) {
        const uint32_t at = entry_offset(h, q, e);
        for (int c = 0; c < h.ncomp; ++c)
            v[c] = get_stored(h, at + c);
        return;
    }
    // row 2 of the two-row form: conj(row0 x row1) of the stored single
    // values, whose products are exact in double
    const int k = e - 6, p0 = (k + 1) % 3, q0 = (k + 2) % 3;
    const uint32_t a = entry_offset(h, q, p0), b = entry_offset(h, q, 3 + q0);
    const uint32_t c = entry_offset(h, q, q0), d = entry_offset(h, q, 3 + p0);
    const double ar = get_stored(h, a), ai = get_stored(h, a + 1);
    const double br = get_stored(h, b), bi = get_stored(h, b + 1);
    const double cr = get_stored(h, c), ci = get_stored(h, c + 1);
    const double dr = get_stored(h, d), di = get_stored(h, d + 1);
    v[0] = (ar * br - ai * bi) - (cr * dr - ci * di);
    v[1] = -((ar * bi + ai * br) - (cr * di + ci * dr));
}

// Bandwidth yardsticks, one 16-byte element per lane, one-shot grid:
// triad a = b + s*c (doubles), read-only (b and c), write-only (a = s),
// copy (a = b).  The read-only kind writes a[0] only if an element of
// b + c equals (s, -s), which keeps its loads without a store stream.
// With `tail` the triad also covers the double after the last element.
template <int KIND, int NT>
__global__ __launch_bounds__(1024) void k_stream(void *a, const void *b,
                                                 const void *c, double s,
                                                 int64_t n16, int tail)
{
    extern __shared__ char occupancy_reserve[];
    using D2 = VecOf<double, 2>::type;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    D2 *A = static_cast<D2 *>(a);
    const D2 *Bv = static_cast<const D2 *>(b);
    const D2 *C = static_cast<const D2 *>(c);
    if (i < n16) {
        if constexpr (KIND == su3i::STREAM_TRIAD) {
            const D2 bv = vload<NT>(Bv + i);
            const D2 cv = vload<NT>(C + i);
            vstore<NT>(A + i, bv + s * cv);
        } else if constexpr (KIND == su3i::STREAM_READ) {
            const D2 v = vload<NT>(Bv + i) + vload<NT>(C + i);
            if (v[0] == s && v[1] == -s)
                A[0] = v;
        } else if constexpr (KIND == su3i::STREAM_WRITE) {
            D2 v;
            v[0] = s;
            v[1] = s;
            vstore<NT>(A + i, v);
        } else {
            vstore<NT>(A + i, vload<NT>(Bv + i));
        }
    }
    if constexpr (KIND == su3i::STREAM_TRIAD) {
        if (tail && i == 0) {
            const int64_t k = 2 * n16;
            static_cast<double *>(a)[k] = static_cast<const double *>(b)[k] +
                                          s * static_cast<const double *>(c)[k];
        }
    }
    if (n16 < 0)
        occupancy_reserve[threadIdx.x] = 0;
}

}  // namespace su3k

namespace su3i {

hipError_t launch_site(int prec, int expr, int S, int nt, int sched, int block,
                       int grid, size_t shm, const SiteArgs &a, hipStream_t st)
{
    switch (prec) {
    case F64: return launch_site_p0(expr, S, nt, sched, block, grid, shm, a, st);
    case F32: return launch_site_p1(expr, S, nt, sched, block, grid, shm, a, st);
    case F16: return launch_site_p2(expr, S, nt, sched, block, grid, shm, a, st);
    case C12: return launch_site_p3(expr, S, nt, sched, block, grid, shm, a, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_shift(int prec, int mode, int nt, int sched, int block,
                        int grid, size_t shm, const ShiftArgs &a, hipStream_t st)
{
    switch (prec) {
    case F64: return launch_shift_p0(mode, nt, sched, block, grid, shm, a, st);
    case F32: return launch_shift_p1(mode, nt, sched, block, grid, shm, a, st);
    case F16: return launch_shift_p2(mode, nt, sched, block, grid, shm, a, st);
    case C12: return launch_shift_p3(mode, nt, sched, block, grid, shm, a, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_site_lds(int prec, int expr, int nt, int block, int grid,
                           size_t reserve, const SiteArgs &a, hipStream_t st)
{
    switch (prec) {
    case F64: return launch_site_lds_p0(expr, nt, block, grid, reserve, a, st);
    case F32: return launch_site_lds_p1(expr, nt, block, grid, reserve, a, st);
    case F16: return launch_site_lds_p2(expr, nt, block, grid, reserve, a, st);
    case C12: return launch_site_lds_p3(expr, nt, block, grid, reserve, a, st);
    }
    return hipErrorInvalidValue;
}

template <int MODE, int NT, int SCHED>
static void batch_go(const BatchItem *items, int32_t nitems, int32_t ntiles, int32_t T,
                     unsigned long long *queue, int block, int grid, size_t shm,
                     hipStream_t st)
{
    hipLaunchKernelGGL((su3k::k_batch<MODE, NT, SCHED>), dim3(grid), dim3(block), shm, st,
                       items, nitems, ntiles, T, queue);
}

hipError_t launch_batch(int mode, const BatchItem *items, int32_t nitems,
                        int32_t ntiles, int32_t tile_sites, int nt, int sched,
                        int block, int grid, size_t shm, unsigned long long *queue,
                        hipStream_t st)
{
    if (block > 256)
        return hipErrorInvalidValue;
    if (queue && shm < 16)
        shm = 16;  // the ticket
    // nontemporal settings compiled: 0, 3 and 7 (others run as 0 or 3)
    const int ntv = nt == 7 ? 2 : ((nt & 3) == 3 ? 1 : 0);
    const int v = (mode ? 6 : 0) + 2 * ntv + (sched ? 1 : 0);
#define SU3_BATCH(M, N, S) \
    batch_go<M, N, S>(items, nitems, ntiles, tile_sites, queue, block, grid, shm, st)
    switch (v) {
    case 0: SU3_BATCH(0, 0, 0); break;
    case 1: SU3_BATCH(0, 0, 1); break;
    case 2: SU3_BATCH(0, 3, 0); break;
    case 3: SU3_BATCH(0, 3, 1); break;
    case 4: SU3_BATCH(0, 7, 0); break;
    case 5: SU3_BATCH(0, 7, 1); break;
    case 6: SU3_BATCH(1, 0, 0); break;
    case 7: SU3_BATCH(1, 0, 1); break;
    case 8: SU3_BATCH(1, 3, 0); break;
    case 9: SU3_BATCH(1, 3, 1); break;
    case 10: SU3_BATCH(1, 7, 0); break;
    default: SU3_BATCH(1, 7, 1); break;
    }
#undef SU3_BATCH
    return hipGetLastError();
}

hipError_t launch_put_items(BatchItem *dst, const BatchItem *items, int n,
                            unsigned long long *queue, hipStream_t st)
{
    for (int first = 0; first < n; first += kItemChunk) {
        ItemChunk c;
        const int count = n - first < kItemChunk ? n - first : kItemChunk;
        for (int i = 0; i < count; ++i)
            c.it[i] = items[first + i];
        hipLaunchKernelGGL(su3k::k_put_items, dim3(1), dim3(64), 0, st, dst + first, c,
                           count, first == 0 ? queue : nullptr);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

static bool host_order_ok(const HostOrder &h)
{
    return h.count > 0 && h.s0 >= 0 && h.s0 + h.count <= h.V && h.E >= 1 &&
           h.canon_entries <= 12 && h.E <= h.canon_entries;
}

hipError_t launch_pack(const HostOrder &h, hipStream_t st)
{
    if (!host_order_ok(h))
        return hipErrorInvalidValue;
    const int64_t sites = h.s0 + h.count == h.V ? h.Vpad - h.s0 : h.count;
    hipLaunchKernelGGL(su3k::k_pack, dim3((unsigned)((sites + 63) / 64)), dim3(64 * h.E), 0, st,
                       h);
    return hipGetLastError();
}

hipError_t launch_unpack(const HostOrder &h, hipStream_t st)
{
    if (!host_order_ok(h))
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(su3k::k_unpack, dim3((unsigned)((h.count + 63) / 64)),
                       dim3(64 * h.canon_entries), 0, st, h);
    return hipGetLastError();
}

template <int KIND, int NT>
static void stream_go(void *a, const void *b, const void *c, double s,
                      int64_t n16, int tail, int block, int grid, size_t shm,
                      hipStream_t st)
{
    hipLaunchKernelGGL((su3k::k_stream<KIND, NT>), dim3(grid), dim3(block), shm,
                       st, a, b, c, s, n16, tail);
}

template <int KIND>
static hipError_t stream_nt(int nt, void *a, const void *b, const void *c,
                            double s, int64_t n16, int tail, int block,
                            int grid, size_t shm, hipStream_t st)
{
    switch (nt) {
    case 0: stream_go<KIND, 0>(a, b, c, s, n16, tail, block, grid, shm, st); break;
    case 1: stream_go<KIND, 1>(a, b, c, s, n16, tail, block, grid, shm, st); break;
    case 2: stream_go<KIND, 2>(a, b, c, s, n16, tail, block, grid, shm, st); break;
    case 3: stream_go<KIND, 3>(a, b, c, s, n16, tail, block, grid, shm, st); break;
    case 6: stream_go<KIND, 6>(a, b, c, s, n16, tail, block, grid, shm, st); break;
    case 7: stream_go<KIND, 7>(a, b, c, s, n16, tail, block, grid, shm, st); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_stream(int kind, void *a, const void *b, const void *c,
                         double s, int64_t n16, int tail, int nt, int block,
                         size_t shm, hipStream_t st)
{
    if (block < 64 || block > 1024 || block % 64)
        return hipErrorInvalidValue;
    const int64_t g = (n16 + block - 1) / block;
    if (g > ((int64_t)1 << 31) - 1)
        return hipErrorInvalidValue;
    const int grid = g < 1 ? 1 : (int)g;
    switch (kind) {
    case STREAM_TRIAD: return stream_nt<STREAM_TRIAD>(nt, a, b, c, s, n16, tail, block, grid, shm, st);
    case STREAM_READ: return stream_nt<STREAM_READ>(nt, a, b, c, s, n16, tail, block, grid, shm, st);
    case STREAM_WRITE: return stream_nt<STREAM_WRITE>(nt, a, b, c, s, n16, tail, block, grid, shm, st);
    case STREAM_COPY: return stream_nt<STREAM_COPY>(nt, a, b, c, s, n16, tail, block, grid, shm, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace su3i
