// C ABI of the SU(3) streaming library: validation, field handles, host
// pack/unpack, launch planning and tuning, batches.  Declarations and the
// contract of every entry point are in include/su3.h.
#include "su3.h"

#include <hip/hip_runtime.h>

#include <sys/mman.h>
#include <unistd.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <array>
#include <mutex>
#include <string>
#include <thread>
#include <tuple>
#include <vector>

#include "su3_dslash.h"
#include "su3_internal.h"
#include "su3_program.h"

using namespace su3i;

struct su3_field {
    void *ptr;
    size_t bytes;
    int32_t dims[4];
    int64_t V;
    int64_t Vpad;
    int64_t L;  // sites per lane-block (V_pad for SoA)
    int32_t prec;
    int32_t layout;
    int32_t lanes;
    int32_t E;
    int32_t rbytes;
    int32_t owns;
    int32_t device;
    int32_t kind;   // su3_kind
    int32_t canon;  // entries per site on the host (9, 12 or 1)
    int32_t ncomp;  // reals per entry (2 complex, 1 real)
    int32_t simd[4];  // virtual nodes per direction (all 1 unless VNODE)
};

enum { KIND_MATRIX = 0, KIND_SPINOR = 1, KIND_REAL = 2, KIND_COMPLEX = 3 };
static const int kSpinorEntries = 12;

struct su3_batch {
    void *d_mem;       // one allocation: the ticket counter, then the items
    unsigned long long *d_queue;  // persistent grids only, else nullptr
    BatchItem *d_items;
    int32_t nitems;
    int32_t ntiles;
    int32_t mode;
    su3_launch cfg;
    int32_t grid;
    int32_t device;
    // persistent grids: launches draw their tiles from the one counter, so
    // each waits for the one before it
    std::mutex mu;
    hipEvent_t last;  // recorded behind every launch that draws tickets
};

// ------------------------------------------------------------- errors

static thread_local std::string g_last_error;

static su3_status fail(su3_status st, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return st;
}

static su3_status hip_fail(hipError_t e, const char *what)
{
    return fail(SU3_ERR_HIP, "%s: %s (%d)", what, hipGetErrorString(e), (int)e);
}

#define HIP_TRY(call, what)                 \
    do {                                    \
        hipError_t e_ = (call);             \
        if (e_ != hipSuccess)               \
            return hip_fail(e_, what);      \
    } while (0)

// ------------------------------------------------------------- geometry

struct Shape {
    int64_t V, Vpad, L;
    int32_t E, ncomp, rbytes;
    size_t bytes;
};

static su3_status make_shape(const int32_t dims[4], int prec, int layout,
                             int32_t lanes, Shape *out,
                             int kind = KIND_MATRIX,
                             const int32_t *simd = nullptr)
{
    if (!dims)
        return fail(SU3_ERR_INVALID_ARG, "dims is NULL");
    if (prec < SU3_F64 || prec > SU3_C12_F32)
        return fail(SU3_ERR_INVALID_ARG, "unknown precision %d", prec);
    if (kind < KIND_MATRIX || kind > KIND_COMPLEX)
        return fail(SU3_ERR_INVALID_ARG, "unknown field kind %d", kind);
    if (kind != KIND_MATRIX && prec != SU3_F64 && prec != SU3_F32)
        return fail(SU3_ERR_UNSUPPORTED,
                    "spinor and scalar fields are stored in SU3_F64 or SU3_F32");
    if (layout < SU3_LAYOUT_AOS || layout > SU3_LAYOUT_VNODE)
        return fail(SU3_ERR_INVALID_ARG, "unknown layout %d", layout);
    if (layout == SU3_LAYOUT_VNODE && !simd)
        return fail(SU3_ERR_INVALID_ARG,
                    "virtual-node fields are made by su3_vnode_alloc / "
                    "su3_vnode_wrap");
    int64_t V = 1;
    for (int d = 0; d < 4; ++d) {
        if (dims[d] <= 0)
            return fail(SU3_ERR_INVALID_ARG, "dims[%d] = %d must be > 0", d,
                        dims[d]);
        V *= dims[d];
        if (V > ((int64_t)1 << 31))
            return fail(SU3_ERR_INVALID_ARG, "lattice too large");
    }
    Shape s;
    s.V = V;
    s.E = kind == KIND_SPINOR ? kSpinorEntries
          : kind == KIND_MATRIX ? entries_of(prec)
                                : 1;
    s.ncomp = kind == KIND_REAL ? 1 : 2;
    s.rbytes = real_bytes(prec);
    if (layout == SU3_LAYOUT_AOS) {
        s.L = 1;
        s.Vpad = V;
    } else if (layout == SU3_LAYOUT_VNODE) {
        int64_t n = 1;
        for (int d = 0; d < 4; ++d) {
            if (simd[d] < 1 || dims[d] % simd[d] != 0)
                return fail(SU3_ERR_INVALID_ARG,
                            "simd[%d] = %d must be >= 1 and divide dims[%d] = %d",
                            d, simd[d], d, dims[d]);
            n *= simd[d];
        }
        if (n > 256 || (n & (n - 1)) != 0)
            return fail(SU3_ERR_INVALID_ARG,
                        "N_sub = %lld virtual nodes must be a power of two <= 256",
                        (long long)n);
        s.L = n;
        s.Vpad = V;
    } else if (layout == SU3_LAYOUT_SOA) {
        s.Vpad = (V + 63) / 64 * 64;
        s.L = s.Vpad;
    } else {
        if (lanes != 8 && lanes != 16 && lanes != 32 && lanes != 64)
            return fail(SU3_ERR_INVALID_ARG,
                        "AoSoA lanes must be 8, 16, 32 or 64 (got %d)", lanes);
        s.L = lanes;
        s.Vpad = (V + lanes - 1) / lanes * lanes;
    }
    const int64_t reals = s.Vpad * s.E * s.ncomp;
    if (reals >= ((int64_t)1 << 31))
        return fail(SU3_ERR_INVALID_ARG,
                    "field holds %lld reals; the limit is 2^31 - 1",
                    (long long)reals);
    s.bytes = (size_t)reals * s.rbytes;
    *out = s;
    return SU3_OK;
}

// Storage site of lattice site s: s itself, or osite * N_sub + lane in the
// virtual-node layout.
static int64_t storage_site(const su3_field *f, int64_t s)
{
    if (f->layout != SU3_LAYOUT_VNODE)
        return s;
    int64_t osite = 0, lane = 0, ostride = 1, lstride = 1;
    for (int d = 0; d < 4; ++d) {
        const int64_t x = s % f->dims[d];
        s /= f->dims[d];
        const int64_t r = f->dims[d] / f->simd[d];
        osite += (x % r) * ostride;
        lane += (x / r) * lstride;
        ostride *= r;
        lstride *= f->simd[d];
    }
    return osite * f->L + lane;
}

// Whether an entry of a lane-block fills whole 128-byte lines.
static bool whole_lines(const su3_field *f)
{
    return f->layout == SU3_LAYOUT_SOA || f->L * 2 * f->rbytes >= 128;
}

static Geom geom_of(const su3_field *f)
{
    Geom g;
    if (f->layout == SU3_LAYOUT_AOS) {
        g.lg = 0;
        g.mask = 0;
        g.plane = 2;
        g.bstride = 2 * f->E;
    } else if (f->layout == SU3_LAYOUT_SOA) {
        g.lg = 31;
        g.mask = 0x7fffffffu;
        g.plane = (uint32_t)(2 * f->Vpad);
        g.bstride = 0;
    } else {
        uint32_t lg = 0;
        while ((1 << lg) < f->L)
            ++lg;
        g.lg = lg;
        g.mask = (uint32_t)(f->L - 1);
        g.plane = (uint32_t)(2 * f->L);
        g.bstride = (uint32_t)(2 * f->E * f->L);
    }
    return g;
}

// Stored-real index of (site s, entry e, c) -- the host twin of the
// kernels' addressing.
static inline int64_t stored_index(const su3_field *f, int64_t s, int e, int c)
{
    s = storage_site(f, s);
    return ((s / f->L) * f->E + e) * f->ncomp * f->L + (s % f->L) * f->ncomp + c;
}

// ------------------------------------------------------------ fields

static su3_status bytes_of_kind(const int32_t dims[4], int prec, int layout,
                                int32_t lanes, size_t *bytes, int kind)
{
    if (!bytes)
        return fail(SU3_ERR_INVALID_ARG, "bytes is NULL");
    Shape s;
    su3_status st = make_shape(dims, prec, layout, lanes, &s, kind);
    if (st != SU3_OK)
        return st;
    *bytes = s.bytes;
    return SU3_OK;
}

extern "C" su3_status su3_field_bytes(const int32_t dims[4],
                                      su3_precision prec, su3_layout layout,
                                      int32_t lanes, size_t *bytes)
{
    return bytes_of_kind(dims, prec, layout, lanes, bytes, KIND_MATRIX);
}

extern "C" su3_status su3_spinor_bytes(const int32_t dims[4],
                                       su3_precision prec, su3_layout layout,
                                       int32_t lanes, size_t *bytes)
{
    return bytes_of_kind(dims, prec, layout, lanes, bytes, KIND_SPINOR);
}

static std::atomic<int64_t> g_live_fields{0};

static void release_stages();

static su3_field *new_handle(const int32_t dims[4], int prec, int layout,
                             int32_t lanes, const Shape &s, int kind,
                             const int32_t *simd = nullptr)
{
    su3_field *f = new su3_field();
    ++g_live_fields;
    f->ptr = nullptr;
    f->bytes = s.bytes;
    std::memcpy(f->dims, dims, sizeof f->dims);
    f->V = s.V;
    f->Vpad = s.Vpad;
    f->L = s.L;
    f->prec = prec;
    f->layout = layout;
    f->lanes = layout == SU3_LAYOUT_AOSOA ? lanes
               : layout == SU3_LAYOUT_VNODE ? (int32_t)s.L
                                            : 0;
    f->E = s.E;
    f->rbytes = s.rbytes;
    f->owns = 0;
    f->device = -1;
    f->kind = kind;
    f->canon = kind == KIND_SPINOR ? kSpinorEntries : kind == KIND_MATRIX ? 9 : 1;
    f->ncomp = s.ncomp;
    for (int d = 0; d < 4; ++d)
        f->simd[d] = simd ? simd[d] : 1;
    return f;
}

static su3_status alloc_of_kind(su3_field **out, const int32_t dims[4],
                                int prec, int layout, int32_t lanes, int kind,
                                const int32_t *simd = nullptr)
{
    if (!out)
        return fail(SU3_ERR_INVALID_ARG, "out is NULL");
    Shape s;
    su3_status st = make_shape(dims, prec, layout, lanes, &s, kind, simd);
    if (st != SU3_OK)
        return st;
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
    void *p = nullptr;
    hipError_t e = hipMalloc(&p, s.bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        release_stages();  // what the transfers keep
        e = hipMalloc(&p, s.bytes);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(SU3_ERR_OUT_OF_MEMORY, "hipMalloc(%zu bytes): %s", s.bytes,
                    hipGetErrorString(e));
    }
    e = hipMemset(p, 0, s.bytes);
    if (e != hipSuccess) {
        (void)hipFree(p);
        return hip_fail(e, "hipMemset");
    }
    su3_field *f = new_handle(dims, prec, layout, lanes, s, kind, simd);
    f->ptr = p;
    f->owns = 1;
    f->device = dev;
    *out = f;
    return SU3_OK;
}

extern "C" su3_status su3_field_alloc(su3_field **out, const int32_t dims[4],
                                      su3_precision prec, su3_layout layout,
                                      int32_t lanes)
{
    return alloc_of_kind(out, dims, prec, layout, lanes, KIND_MATRIX);
}

extern "C" su3_status su3_spinor_alloc(su3_field **out, const int32_t dims[4],
                                       su3_precision prec, su3_layout layout,
                                       int32_t lanes)
{
    return alloc_of_kind(out, dims, prec, layout, lanes, KIND_SPINOR);
}

static su3_status wrap_of_kind(su3_field **out, void *dev_ptr, size_t bytes,
                               const int32_t dims[4], int prec, int layout,
                               int32_t lanes, int kind,
                               const int32_t *simd = nullptr)
{
    if (!out)
        return fail(SU3_ERR_INVALID_ARG, "out is NULL");
    if (!dev_ptr)
        return fail(SU3_ERR_INVALID_ARG, "dev_ptr is NULL");
    if (((uintptr_t)dev_ptr & 15) != 0)
        return fail(SU3_ERR_INVALID_ARG, "dev_ptr is not 16-byte aligned");
    Shape s;
    su3_status st = make_shape(dims, prec, layout, lanes, &s, kind, simd);
    if (st != SU3_OK)
        return st;
    if (bytes < s.bytes)
        return fail(SU3_ERR_INVALID_ARG,
                    "buffer of %zu bytes is smaller than the field (%zu)",
                    bytes, s.bytes);
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
    hipPointerAttribute_t attr;
    std::memset(&attr, 0, sizeof attr);
    hipError_t e = hipPointerGetAttributes(&attr, dev_ptr);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(SU3_ERR_INVALID_ARG,
                    "dev_ptr is not device memory known to HIP (%s)",
                    hipGetErrorString(e));
    }
    if (attr.type != hipMemoryTypeDevice || attr.device != dev)
        return fail(SU3_ERR_INVALID_ARG,
                    "dev_ptr is not device memory of the current device %d",
                    dev);
    su3_field *f = new_handle(dims, prec, layout, lanes, s, kind, simd);
    f->ptr = dev_ptr;
    f->owns = 0;
    f->device = dev;
    *out = f;
    return SU3_OK;
}

extern "C" su3_status su3_field_wrap(su3_field **out, void *dev_ptr,
                                     size_t bytes, const int32_t dims[4],
                                     su3_precision prec, su3_layout layout,
                                     int32_t lanes)
{
    return wrap_of_kind(out, dev_ptr, bytes, dims, prec, layout, lanes,
                        KIND_MATRIX);
}

extern "C" su3_status su3_spinor_wrap(su3_field **out, void *dev_ptr,
                                      size_t bytes, const int32_t dims[4],
                                      su3_precision prec, su3_layout layout,
                                      int32_t lanes)
{
    return wrap_of_kind(out, dev_ptr, bytes, dims, prec, layout, lanes,
                        KIND_SPINOR);
}

// ---------------------------------------------------- scalar fields

static su3_status check_scalar_kind(int kind)
{
    if (kind != KIND_REAL && kind != KIND_COMPLEX)
        return fail(SU3_ERR_INVALID_ARG,
                    "scalar fields are SU3_KIND_REAL or SU3_KIND_COMPLEX");
    return SU3_OK;
}

extern "C" su3_status su3_scalar_bytes(const int32_t dims[4],
                                       su3_precision prec, su3_layout layout,
                                       int32_t lanes, su3_kind kind,
                                       size_t *bytes)
{
    su3_status st = check_scalar_kind(kind);
    return st != SU3_OK ? st
                        : bytes_of_kind(dims, prec, layout, lanes, bytes, kind);
}

extern "C" su3_status su3_scalar_alloc(su3_field **out, const int32_t dims[4],
                                       su3_precision prec, su3_layout layout,
                                       int32_t lanes, su3_kind kind)
{
    su3_status st = check_scalar_kind(kind);
    return st != SU3_OK ? st
                        : alloc_of_kind(out, dims, prec, layout, lanes, kind);
}

extern "C" su3_status su3_scalar_wrap(su3_field **out, void *dev_ptr,
                                      size_t bytes, const int32_t dims[4],
                                      su3_precision prec, su3_layout layout,
                                      int32_t lanes, su3_kind kind)
{
    su3_status st = check_scalar_kind(kind);
    return st != SU3_OK ? st
                        : wrap_of_kind(out, dev_ptr, bytes, dims, prec, layout,
                                       lanes, kind);
}

// --------------------------------------------- virtual-node fields

static su3_status check_simd(const int32_t *simd)
{
    if (!simd)
        return fail(SU3_ERR_INVALID_ARG, "simd is NULL");
    return SU3_OK;
}

extern "C" su3_status su3_vnode_bytes(const int32_t dims[4],
                                      su3_precision prec, su3_kind kind,
                                      const int32_t simd[4], size_t *bytes)
{
    su3_status st = check_simd(simd);
    if (st != SU3_OK)
        return st;
    if (!bytes)
        return fail(SU3_ERR_INVALID_ARG, "bytes is NULL");
    Shape s;
    st = make_shape(dims, prec, SU3_LAYOUT_VNODE, 0, &s, kind, simd);
    if (st != SU3_OK)
        return st;
    *bytes = s.bytes;
    return SU3_OK;
}

extern "C" su3_status su3_vnode_alloc(su3_field **out, const int32_t dims[4],
                                      su3_precision prec, su3_kind kind,
                                      const int32_t simd[4])
{
    su3_status st = check_simd(simd);
    if (st != SU3_OK)
        return st;
    return alloc_of_kind(out, dims, prec, SU3_LAYOUT_VNODE, 0, kind, simd);
}

extern "C" su3_status su3_vnode_wrap(su3_field **out, void *dev_ptr,
                                     size_t bytes, const int32_t dims[4],
                                     su3_precision prec, su3_kind kind,
                                     const int32_t simd[4])
{
    su3_status st = check_simd(simd);
    if (st != SU3_OK)
        return st;
    return wrap_of_kind(out, dev_ptr, bytes, dims, prec, SU3_LAYOUT_VNODE, 0,
                        kind, simd);
}

extern "C" su3_status su3_field_free(su3_field *f)
{
    if (!f)
        return SU3_OK;
    hipError_t e = hipSuccess;
    const bool owns = f->owns && f->ptr;
    if (owns)
        e = hipFree(f->ptr);
    delete f;
    // a handle on borrowed memory makes no HIP call: its end may come while
    // a stream is captured, which a hipFree would break
    if (--g_live_fields == 0 && owns)
        release_stages();
    if (e != hipSuccess)
        return hip_fail(e, "hipFree");
    return SU3_OK;
}

extern "C" su3_status su3_field_data(const su3_field *f, void **dev_ptr,
                                     size_t *bytes)
{
    if (!f)
        return fail(SU3_ERR_INVALID_ARG, "field is NULL");
    if (dev_ptr)
        *dev_ptr = f->ptr;
    if (bytes)
        *bytes = f->bytes;
    return SU3_OK;
}

// double -> float -> half, each step rounding to nearest even.  The empty
// asm keeps the intermediate float: without it the optimiser folds the two
// conversions into one double -> half rounding, which differs whenever the
// float lands exactly halfway between two halves.
static inline _Float16 half_of(double v)
{
    float f = (float)v;
    __asm__ volatile("" : "+x"(f));
    return (_Float16)f;
}

// Host quantisers: round to nearest even (float: one rounding; half:
// double -> float -> half).
static inline void put_real(void *img, int prec, int64_t idx, double v)
{
    if (prec == SU3_F64)
        static_cast<double *>(img)[idx] = v;
    else if (prec == SU3_F16_F32ACC)
        static_cast<_Float16 *>(img)[idx] = half_of(v);
    else
        static_cast<float *>(img)[idx] = (float)v;
}

static inline double get_real(const void *img, int prec, int64_t idx)
{
    if (prec == SU3_F64)
        return static_cast<const double *>(img)[idx];
    if (prec == SU3_F16_F32ACC)
        return (double)(float)static_cast<const _Float16 *>(img)[idx];
    return (double)static_cast<const float *>(img)[idx];
}

// Device buffers that hold a part of a field's canonical data on its way to
// or from the host.  A transfer holds one for itself until its stream is
// done with it; up to kStagesKept of them wait for the next transfer (any
// thread, any stream).  They go back to the device when the last field is
// freed, if it owns its memory, and when an allocation fails.
struct Stage {
    void *ptr;
    size_t bytes;
    int device;
};
static const size_t kStageBytes = (size_t)16 << 20;
static const size_t kStagesKept = 4;
static std::mutex g_stage_mu;
static Stage g_stages[kStagesKept];
static size_t g_nstages = 0;

static bool acquire_stage(int device, size_t bytes, Stage *out)
{
    {
        std::lock_guard<std::mutex> lk(g_stage_mu);
        for (size_t i = 0; i < g_nstages; ++i)
            if (g_stages[i].device == device && g_stages[i].bytes >= bytes) {
                *out = g_stages[i];
                --g_nstages;
                std::move(g_stages + i + 1, g_stages + g_nstages + 1, g_stages + i);
                return true;
            }
    }
    out->device = device;
    out->bytes = bytes > (size_t)1 << 20 ? kStageBytes : (size_t)1 << 20;
    if (hipMalloc(&out->ptr, out->bytes) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return true;
}

static void give_back_stage(Stage s)
{
    {
        std::lock_guard<std::mutex> lk(g_stage_mu);
        if (g_nstages < kStagesKept) {
            g_stages[g_nstages++] = s;
            return;
        }
        for (Stage &k : g_stages)  // keep the larger ones
            if (k.bytes < s.bytes)
                std::swap(k, s);
    }
    (void)hipFree(s.ptr);
}

static void release_stages()
{
    Stage free_now[kStagesKept];
    size_t n;
    {
        std::lock_guard<std::mutex> lk(g_stage_mu);
        n = g_nstages;
        std::copy(g_stages, g_stages + n, free_now);
        g_nstages = 0;
    }
    for (size_t i = 0; i < n; ++i)
        (void)hipFree(free_now[i].ptr);
}

// Fields of at least this many stored reals are converted on the device;
// below, one thread packs them in less than the extra launch takes.  In and
// out takes 42 us and 0.018 a site on the device; on the host 22 us and 0.06 a
// site in double (equal at 512 sites) and single (550), 0.11 in half (224),
// 0.035 in two-row single (960).
static int64_t device_convert_reals(int prec)
{
    return prec == SU3_F64 ? 9216 : prec == SU3_F32 ? 9900 : prec == SU3_F16_F32ACC ? 4032 : 11520;
}

// Run `part` over the canonical data of a field in pieces that fit a staging
// buffer: part(order of the piece, its first host double, its bytes).
// Returns false, with nothing run, where the device cannot convert (a small
// field, another current device, no memory to stage in); *st is the result
// otherwise.
template <class F>
static bool convert_on_device(const su3_field *f, hipStream_t hs, F part, su3_status *st)
{
    int dev = -1;
    if (f->V * f->E * f->ncomp < device_convert_reals(f->prec) || hipGetDevice(&dev) != hipSuccess ||
        dev != f->device)
        return false;
    const int64_t site_doubles = (int64_t)f->canon * f->ncomp;
    const int64_t per = std::min<int64_t>(f->V, (int64_t)(kStageBytes / 8) / site_doubles);
    Stage stage;
    if (!acquire_stage(dev, (size_t)(per * site_doubles) * 8, &stage))
        return false;
    HostOrder h;
    std::memset(&h, 0, sizeof h);
    h.field = f->ptr;
    h.canon = static_cast<double *>(stage.ptr);
    h.g = geom_of(f);
    h.V = f->V;
    h.Vpad = f->Vpad;
    h.E = f->E;
    h.canon_entries = f->canon;
    h.ncomp = f->ncomp;
    h.prec = f->prec;
    h.vnode = f->layout == SU3_LAYOUT_VNODE;
    for (int d = 0; d < 4; ++d) {
        h.dims[d] = f->dims[d];
        h.sub[d] = f->dims[d] / f->simd[d];
        h.simd[d] = f->simd[d];
    }
    hipError_t e = hipSuccess;
    const char *what = "";
    for (int64_t s0 = 0; s0 < f->V && e == hipSuccess; s0 += per) {
        h.s0 = s0;
        h.count = std::min(per, f->V - s0);
        e = part(h, s0 * site_doubles, (size_t)(h.count * site_doubles) * 8, &what);
    }
    // the buffer is free once the stream has passed its last use
    const hipError_t sync = hipStreamSynchronize(hs);
    give_back_stage(stage);
    if (e == hipSuccess && sync != hipSuccess) {
        e = sync;
        what = "transfer sync";
    }
    *st = e == hipSuccess ? SU3_OK : hip_fail(e, what);
    return true;
}

// Have the kernel map the pages of a large host buffer that is about to be
// written (a fresh one faults on every page: 48 MB takes 11 ms from one
// thread).  Contents stay as they are; the calling thread goes on copying
// meanwhile.
struct Populate {
    std::vector<std::thread> workers;
    std::atomic<size_t> next{0};

    Populate(void *host, size_t bytes)
    {
#ifdef MADV_POPULATE_WRITE
        const size_t piece = (size_t)4 << 20;
        const size_t pieces = bytes / piece;
        if (pieces < 2)
            return;  // before a question to the system: 2.5 us of a small call's 36
        const size_t cpus = std::max(1u, std::thread::hardware_concurrency() / 2);
        const size_t n = std::min(std::min<size_t>(8, cpus), pieces / 2);
        const size_t page = (size_t)sysconf(_SC_PAGESIZE);
        unsigned char *first = reinterpret_cast<unsigned char *>((uintptr_t)host / page * page);
        unsigned char *end = static_cast<unsigned char *>(host) + bytes;
        try {
            for (size_t t = 0; t < n; ++t)
                workers.emplace_back([this, first, end, piece, pieces]() {
                    for (;;) {
                        const size_t i = next++;
                        if (i > pieces)
                            return;
                        unsigned char *p = first + i * piece;
                        if (p >= end)
                            return;
                        (void)madvise(p, std::min<size_t>(piece, (size_t)(end - p)),
                                      MADV_POPULATE_WRITE);
                    }
                });
        } catch (...) {
            // no thread to be had: the copy faults the pages itself
        }
#else
        (void)host;
        (void)bytes;
#endif
    }
    ~Populate()
    {
        for (std::thread &t : workers)
            t.join();
    }
};

extern "C" su3_status su3_field_upload(su3_field *f, const double *host,
                                       void *stream)
{
    if (!f || !host)
        return fail(SU3_ERR_INVALID_ARG, "field or host buffer is NULL");
    hipStream_t st = static_cast<hipStream_t>(stream);
    su3_status done;
    if (convert_on_device(
            f, st,
            [&](const HostOrder &h, int64_t first, size_t bytes, const char **what) {
                *what = "upload copy";
                const hipError_t e = hipMemcpyAsync(h.canon, host + first, bytes,
                                                    hipMemcpyHostToDevice, st);
                if (e != hipSuccess)
                    return e;
                *what = "upload conversion";
                return launch_pack(h, st);
            },
            &done))
        return done;
    std::vector<unsigned char> img(f->bytes, 0);
    for (int64_t s = 0; s < f->V; ++s)
        for (int e = 0; e < f->E; ++e)
            for (int c = 0; c < f->ncomp; ++c)
                put_real(img.data(), f->prec, stored_index(f, s, e, c),
                         host[f->ncomp * (f->canon * s + e) + c]);
    HIP_TRY(hipMemcpyAsync(f->ptr, img.data(), f->bytes,
                           hipMemcpyHostToDevice, st),
            "upload copy");
    HIP_TRY(hipStreamSynchronize(st), "upload sync");
    return SU3_OK;
}

extern "C" su3_status su3_field_download_raw(const su3_field *f, void *host,
                                             size_t bytes, void *stream)
{
    if (!f || !host)
        return fail(SU3_ERR_INVALID_ARG, "field or host buffer is NULL");
    if (bytes < f->bytes)
        return fail(SU3_ERR_INVALID_ARG, "host buffer of %zu bytes < %zu",
                    bytes, f->bytes);
    hipStream_t st = static_cast<hipStream_t>(stream);
    Populate pages(host, f->bytes);
    HIP_TRY(hipMemcpyAsync(host, f->ptr, f->bytes, hipMemcpyDeviceToHost, st),
            "download copy");
    HIP_TRY(hipStreamSynchronize(st), "download sync");
    return SU3_OK;
}

extern "C" su3_status su3_field_download(const su3_field *f, double *host,
                                         void *stream)
{
    if (!f || !host)
        return fail(SU3_ERR_INVALID_ARG, "field or host buffer is NULL");
    {
        hipStream_t hs = static_cast<hipStream_t>(stream);
        su3_status done;
        Populate pages(host, (size_t)(f->V * f->canon * f->ncomp) * 8);
        if (convert_on_device(
                f, hs,
                [&](const HostOrder &h, int64_t first, size_t bytes, const char **what) {
                    *what = "download conversion";
                    const hipError_t e = launch_unpack(h, hs);
                    if (e != hipSuccess)
                        return e;
                    *what = "download copy";
                    return hipMemcpyAsync(host + first, h.canon, bytes,
                                          hipMemcpyDeviceToHost, hs);
                },
                &done))
            return done;
    }
    std::vector<unsigned char> img(f->bytes);
    su3_status st = su3_field_download_raw(f, img.data(), img.size(), stream);
    if (st != SU3_OK)
        return st;
    for (int64_t s = 0; s < f->V; ++s) {
        double *m = host + f->ncomp * f->canon * s;
        for (int e = 0; e < f->E; ++e)
            for (int c = 0; c < f->ncomp; ++c)
                m[f->ncomp * e + c] = get_real(img.data(), f->prec,
                                               stored_index(f, s, e, c));
        if (f->kind == KIND_MATRIX && f->prec == SU3_C12_F32) {
            // row 2 = conj(row0 x row1), in double
            for (int k = 0; k < 3; ++k) {
                const int p = (k + 1) % 3, q = (k + 2) % 3;
                const double ar = m[2 * p], ai = m[2 * p + 1];
                const double br = m[2 * (3 + q)], bi = m[2 * (3 + q) + 1];
                const double cr = m[2 * q], ci = m[2 * q + 1];
                const double dr = m[2 * (3 + p)], di = m[2 * (3 + p) + 1];
                m[2 * (6 + k)] = (ar * br - ai * bi) - (cr * dr - ci * di);
                m[2 * (6 + k) + 1] = -((ar * bi + ai * br) - (cr * di + ci * dr));
            }
        }
    }
    return SU3_OK;
}

// -------------------------------------------------------- device facts

struct DeviceFacts {
    int cus;
    int lds_per_cu;
    int lds_per_block;
};

static DeviceFacts device_facts(int dev)
{
    static std::mutex mu;
    static std::map<int, DeviceFacts> cache;
    std::lock_guard<std::mutex> lk(mu);
    auto it = cache.find(dev);
    if (it != cache.end())
        return it->second;
    DeviceFacts f;
    if (hipDeviceGetAttribute(&f.cus, hipDeviceAttributeMultiprocessorCount,
                              dev) != hipSuccess || f.cus <= 0)
        f.cus = 256;
    if (hipDeviceGetAttribute(&f.lds_per_cu,
                              hipDeviceAttributeMaxSharedMemoryPerMultiprocessor,
                              dev) != hipSuccess || f.lds_per_cu <= 0)
        f.lds_per_cu = 64 * 1024;
    if (hipDeviceGetAttribute(&f.lds_per_block,
                              hipDeviceAttributeMaxSharedMemoryPerBlock,
                              dev) != hipSuccess || f.lds_per_block <= 0)
        f.lds_per_block = 64 * 1024;
    cache[dev] = f;
    return f;
}

static int device_cus(int dev) { return device_facts(dev).cus; }

// LDS to reserve per workgroup so that at most `occupancy` workgroups fit
// on a CU (0: none).  The reserve is never read by the kernels.
static size_t occupancy_reserve(int dev, int occupancy)
{
    if (occupancy <= 0)
        return 0;
    const DeviceFacts f = device_facts(dev);
    size_t r = (size_t)f.lds_per_cu / (size_t)occupancy;
    r = std::min(r, (size_t)f.lds_per_block);
    return r / 256 * 256;
}

// ------------------------------------------------------- launch table

using Key = std::tuple<int, int, int, int, int>;  // expr prec layout lanes vbucket

static int vbucket(int64_t V)
{
    int b = 0;
    while (((int64_t)1 << b) < V)
        ++b;
    return b;
}

static std::mutex g_tune_mu;
static std::map<Key, su3_launch> g_tuned;
static bool g_cache_loaded = false;

// Launch-tuning keys of batches are SU3_EXPR_BATCH + the leading item's
// expression, so that a batch's tuned tile and grid never stand in for a
// single field's launch of the same volume bucket (and the reverse).
static bool is_batch_key(int expr)
{
    return expr >= SU3_EXPR_BATCH && expr <= SU3_EXPR_BATCH + SU3_EXPR_APB_AB;
}

// Bytes a site-local call of V sites reads and writes.
static int64_t site_call_bytes(int expr, int prec, int64_t V)
{
    return V * entries_of(prec) * 2 * real_bytes(prec) * (operands_of(expr) + 1);
}

// Calls of up to this many bytes leave their operands in the 256 MiB
// Infinity Cache, where a program that comes back to its fields finds them.
// Measured with three sets of fields in turn: cached loads win below (FP32
// MUL 24^3 x 48, 143 MB: 23.6 us against 25.7 with nontemporal loads), lose
// above (FP32 MUL3 24^3 x 48, 191 MB: 35.3 against 33.6).  On fields that
// are in no cache cached loads cost up to 5 % (FP32 24^4: 14.3 against 13.6).
static const int64_t kCachedBytes = (int64_t)160 * 1000 * 1000;

// The launch of a call that nothing tuned or set: V sites of the key's
// expression, precision, layout and lanes.
static su3_launch default_launch(int expr, int prec, int layout, int lanes, int64_t V)
{
    su3_launch c;
    c.block = 64;
    c.persistent = 0;
    c.nontemporal = 3;
    c.xcd_remap = 0;
    c.lds_stage = 0;
    c.tile_sites = 4096;
    c.occupancy = layout == SU3_LAYOUT_AOS ? 0 : 5;
    c.schedule = layout == SU3_LAYOUT_AOS ? 0 : 1;
    c.sites_per_lane = 0;
    const bool site = expr >= SU3_EXPR_MUL && expr <= SU3_EXPR_APB_AB;
    // Bytes of an entry in a lane-block.  Where it is shorter than a 128-byte
    // line a nontemporal access takes the line once per piece, so calls on
    // such layouts keep loads, and below 64 bytes stores, cached (N_sub 2 and
    // 4, AoSoA-8).
    const int64_t run = layout == SU3_LAYOUT_AOSOA || layout == SU3_LAYOUT_VNODE
                            ? (int64_t)lanes * 2 * real_bytes(prec)
                            : 1 << 20;
    if (site && layout == SU3_LAYOUT_AOS) {
        // Whole tiles through LDS: FP64 32^4 70 us, against 679 us read
        // directly, site by site.  Calls of up to kCachedBytes keep their
        // loads cached and take every wave that fits (FP32 24^4: 11.4 us
        // against 12.9 with nontemporal loads).  Beyond, double streams best
        // with 6 waves per CU and write-through stores (FP64 40^4: 170 us;
        // 5 waves 173, 8 waves 178; FP64 48^4 358 and 371), the others with
        // 8 (FP32 40^4 85.7 us, uncapped 86.6), four single or double
        // operands with 5 (FP32 MULADD 40^4: 140.9 us, uncapped 152).
        const bool dbl = prec == SU3_F64, four = expr == SU3_EXPR_MULADD;
        c.lds_stage = 1;
        if (site_call_bytes(expr, prec, V) <= kCachedBytes) {
            c.occupancy = 0;
            c.nontemporal = 2;
        } else if (dbl && !four) {
            c.block = 128;
            c.occupancy = 3;
            c.nontemporal = 7;
        } else {
            c.occupancy = four && prec != SU3_F16_F32ACC ? 5 : 8;
        }
    }
    if (site && layout != SU3_LAYOUT_AOS) {
        // Up to kCachedBytes: cached loads, every wave that fits (half MUL3
        // 24^4, 48 MB: 8.8 us against 13.6 with nontemporal loads and 5
        // waves per CU).  Beyond, fewer waves and streaming stores: double
        // 5 waves (48^4 MUL 352 us; 8 waves 382, uncapped 415), single and
        // two-row 8 up to half a GB (FP32 32^4 41.5 us, 5 waves 46.6) and 5
        // from there (FP32 48^4 180 us, 8 waves 188), half 8 (MUL3 48^4
        // 124 us, 5 waves 165).  Write-through stores gain 1-2 % where the
        // call exceeds the cache several times, and lose below.
        const int64_t bytes = site_call_bytes(expr, prec, V);
        const bool dbl = prec == SU3_F64, half = prec == SU3_F16_F32ACC;
        const bool large = bytes > (int64_t)512 * 1000 * 1000;
        if (bytes <= kCachedBytes) {
            c.occupancy = 0;
            c.nontemporal = 2;
            // (half MUL3 7.2 us against 8.3 row by row at 229425 sites;
            // MULADD, with four operands of two sites, the other way round)
            c.schedule = !half || expr == SU3_EXPR_MULADD;
        } else {
            c.occupancy = dbl || (large && !half) ? 5 : 8;
            c.nontemporal = dbl || large ? 7 : 3;
        }
        if (run < 64 && (bytes > kCachedBytes || run < 32 || !half)) {
            // 5 waves per CU (FP32 N_sub 2 48^3 x 24 MUL: 133 us, with
            // nontemporal accesses 419 to 489), 8 in small calls (half N_sub 2
            // 24^4 ADD 11.2 us, 5 waves 12.3, loads cached alone 29.5); small
            // half calls on pieces of 32 bytes take every wave (MUL3 24^4 8.5
            // and 10.2)
            c.occupancy = bytes > kCachedBytes || run == 16 ? 5 : 8;
            c.nontemporal = 0;
            c.schedule = 1;
        } else if (run == 64 && bytes > kCachedBytes) {
            c.occupancy = 5;
            c.nontemporal = 2;
            c.schedule = 1;
        } else if (run < 256 && c.nontemporal == 7) {
            c.nontemporal = 3;
        }
        // Entry planes a multiple of 2 MiB apart (2 to 16 MiB: power-of-two
        // lattices) meet in the same memory channels: there each XCD takes a
        // range of its own (FP64 32^4 73 us against 81, 16^3 x 32 9.0 against
        // 10.8).  Planes of 32 MiB lose by it (FP64 32^3 x 64: 155 against
        // 141), and so does half with 3-4 operands, whose lanes take 8 bytes.
        if (layout == SU3_LAYOUT_SOA) {
            const int64_t plane = (V + 63) / 64 * 64 * 2 * real_bytes(prec);
            c.xcd_remap = plane % (2 << 20) == 0 && plane <= (16 << 20) &&
                          !(half && operands_of(expr) > 2);
        }
    }
    if (is_batch_key(expr)) {
        // One tile per workgroup, one group of sites per lane: a batch of any
        // size fills the chip (four lattices of 8^4 to 24^3 x 48: 18 us
        // against 141 with one wave walking 4096 sites).  Two waves of one
        // double site per lane (32 lattices, 5.6 GB: 893 us; one wave with
        // two sites in turn 991), else one wave, whose lanes take 2 or 4
        // sites (64 lattices: two-row 3.3 GB 554 us, 676 beside an idle
        // wave; single 5.0 GB 818 by rows, 1240; half 2.5 GB 444 with 256
        // sites, 785 with 128).
        const int op = expr - SU3_EXPR_BATCH;
        const bool dbl = prec == SU3_F64;
        c.block = dbl ? 128 : 64;
        c.tile_sites = dbl ? 128 : 64 * natural_sites(prec, op);
        c.occupancy = 0;
        c.schedule = op != SU3_EXPR_MUL || prec == SU3_F32;
        const int64_t bytes = site_call_bytes(expr - SU3_EXPR_BATCH, prec, V);
        c.nontemporal = bytes <= (int64_t)100 * 1000 * 1000 ? 0
                        : bytes <= (int64_t)1000 * 1000 * 1000 ? 3
                                                               : 7;
        // (12 lattices of 32^4, N_sub 4: single 652 us, streamed 1406; half 304
        // and 1301; double 990 and 1155)
        if (run <= 64)
            c.nontemporal = 0;
    }
    if (expr == SU3_EXPR_CSHIFT || expr == SU3_EXPR_MUL_SHIFTED) {
        // One site per lane: 8 (single) or 4 bytes (half) per access instead
        // of 16, so it takes 16 waves per CU to keep as many bytes in flight
        // (FP32 24^3 x 48: 24.7 us against 35.1 with 5; half 48^4 98.6
        // against 220).  Double needs fewer the larger the call (product
        // 48^4: 5 waves 377 us, 10 waves 391; 24^3 x 48: 10 waves 49.8 us, 5
        // waves 52.7; copy 48^4 6 waves 254, 5 waves 262), and stores past L2 too
        // from there on only (30^4 59.2 us, with streaming stores 62.2; 36^4 121
        // and 116).  Stores and loads
        // are cached below 64 to 100 MB (half copy 32^4: 12 us against 19).
        // AoS reads every line once per entry, so its loads always stay
        // cached (FP64 32^4: 103 us against 452).
        const bool product = expr == SU3_EXPR_MUL_SHIFTED, dbl = prec == SU3_F64;
        const int64_t bytes = V * entries_of(prec) * 2 * real_bytes(prec) * (product ? 3 : 2);
        const int64_t MB = 1000 * 1000;
        c.schedule = dbl || prec == SU3_C12_F32;
        c.block = 256;
        c.occupancy = 4;
        c.nontemporal = bytes <= 100 * MB ? 0 : prec == SU3_F32 ? 7 : 3;
        if (layout == SU3_LAYOUT_AOS) {
            c.block = dbl || prec == SU3_F32 ? 128 : 256;
            c.occupancy = dbl || prec == SU3_F32 ? 3 : prec == SU3_F16_F32ACC ? 0 : 4;
            c.nontemporal = 0;
        } else if (dbl && product && bytes > 100 * MB) {
            c.block = bytes > 200 * MB && bytes <= 512 * MB ? 128 : 64;
            c.occupancy = bytes > 200 * MB ? 5 : 0;
            c.nontemporal = bytes > 512 * MB ? 7 : 3;
        } else if (dbl && !product) {
            c.block = 128;
            c.occupancy = bytes <= 64 * MB ? 5 : 3;
            c.nontemporal = bytes <= 64 * MB ? 0 : bytes <= 200 * MB ? 3 : 7;
        }
        if (run < 64 && bytes > 100 * MB) {
            // (FP32 N_sub 2 48^3 x 24 copy 91 us, nontemporal loads 215 to 379)
            c.block = product && run == 32 ? 128 : 256;
            c.occupancy = product && run == 32 ? 3 : 4;
            c.nontemporal = 2;
            c.schedule = 0;
        } else if (run <= 64 && dbl && bytes > 64 * MB) {
            c.nontemporal = 2;
        }
        // Power-of-two planes, as for the site-local calls (FP64 32^4 product
        // 73 us against 87, copy 50 against 63; FP32 38 against 42; half copy
        // 11.8 against 14.3, but its product 21.2 against 20.9).
        if (layout == SU3_LAYOUT_SOA) {
            const int64_t plane = (V + 63) / 64 * 64 * 2 * real_bytes(prec);
            c.xcd_remap = plane % (2 << 20) == 0 && plane <= (16 << 20) &&
                          !(product && prec == SU3_F16_F32ACC);
        }
    }
    if (expr == SU3_EXPR_PROGRAM || expr == SU3_EXPR_PROGRAM_SCALAR) {
        c.block = 128;
        c.occupancy = 0;
        c.schedule = 0;
        // Power-of-two planes, as for the site-local calls (FP64 32^4
        // a*b-adj(b)*adj(a) 75.8 us against 80.6, FP32 16^2 x 32^2 a*b+c*d 18.5
        // against 22.8; planes of 32 MiB neither gain nor lose).
        if (layout == SU3_LAYOUT_SOA && V > 0) {
            const int64_t plane = (V + 63) / 64 * 64 * 2 * real_bytes(prec);
            c.xcd_remap = plane % (2 << 20) == 0 && plane <= (16 << 20);
        }
    }
    if (expr == SU3_EXPR_DSLASH) {
        // cached loads (neighbours re-read each spinor), nontemporal stores;
        // default_dslash plans the rest from the lattice's extents
        c.block = 256;
        c.nontemporal = 2;
        c.occupancy = 0;
        c.schedule = prec == SU3_F64 ? 17 : 16;
        c.tile_sites = prec == SU3_F64 ? 8 : 7;
    }
    return c;
}

static bool nt_valid(int nt, bool streaming)
{
    return (nt >= 0 && nt <= 3) || (streaming && (nt == 6 || nt == 7));
}

static su3_status check_launch(const su3_launch &c, int layout, int expr)
{
    const bool lds_walk = expr == SU3_EXPR_DSLASH && c.schedule >= 4;
    const bool site = expr >= SU3_EXPR_MUL && expr <= SU3_EXPR_APB_AB;
    const bool batch = is_batch_key(expr);
    const bool streaming = site || batch || expr == SU3_EXPR_CSHIFT ||
                           expr == SU3_EXPR_MUL_SHIFTED;
    const bool wide = site && (c.nontemporal & 3) == 3 && !c.lds_stage;
    if (c.block != 64 && c.block != 128 && c.block != 256 &&
        !(lds_walk && c.block == 512) &&
        !(wide && (c.block == 512 || c.block == 1024)))
        return fail(SU3_ERR_INVALID_ARG,
                    "block %d not in {64, 128, 256}%s", c.block,
                    lds_walk ? " or 512"
                    : site   ? " (512 or 1024 need nontemporal 3 or 7)"
                             : "");
    if (!nt_valid(c.nontemporal, streaming))
        return fail(SU3_ERR_INVALID_ARG, "nontemporal %d not in %s",
                    c.nontemporal, streaming ? "{0, 1, 2, 3, 6, 7}" : "[0, 3]");
    if (c.sites_per_lane != 0 && c.sites_per_lane != 1 &&
        c.sites_per_lane != 2 && c.sites_per_lane != 4 &&
        c.sites_per_lane != 8)
        return fail(SU3_ERR_INVALID_ARG,
                    "sites_per_lane %d not in {0, 1, 2, 4, 8}",
                    c.sites_per_lane);
    if (c.persistent < 0 || c.persistent > 64)
        return fail(SU3_ERR_INVALID_ARG, "persistent %d not in [0, 64]",
                    c.persistent);
    if (c.xcd_remap < 0 || c.xcd_remap > (lds_walk ? 2 : 1))
        return fail(SU3_ERR_INVALID_ARG, "xcd_remap must be 0 or 1%s",
                    lds_walk ? " or 2" : "");
    if (c.lds_stage < 0 || c.lds_stage > 1 ||
        (c.lds_stage && layout != SU3_LAYOUT_AOS))
        return fail(SU3_ERR_INVALID_ARG, "lds_stage is for the AoS layout only");
    if (c.lds_stage && c.block > 128)
        return fail(SU3_ERR_INVALID_ARG, "lds_stage needs block <= 128");
    if (expr == SU3_EXPR_DSLASH) {
        if (c.tile_sites < 1 || c.tile_sites > 4096)
            return fail(SU3_ERR_INVALID_ARG,
                        "Dslash tile_sites (t-slices per lane) must be in "
                        "[1, 4096]");
    } else if (c.tile_sites < 64 || c.tile_sites % 64 != 0 ||
               c.tile_sites > (1 << 24)) {
        return fail(SU3_ERR_INVALID_ARG,
                    "tile_sites must be a positive multiple of 64");
    }
    if (c.occupancy < 0 || c.occupancy > 64)
        return fail(SU3_ERR_INVALID_ARG, "occupancy %d not in [0, 64]",
                    c.occupancy);
    if (expr == SU3_EXPR_DSLASH) {
        LdsShape sh;
        if (c.schedule < 0 || c.schedule > 28)
            return fail(SU3_ERR_INVALID_ARG,
                        "Dslash schedule (site tile) must be in [0, 28]");
        if (lds_walk && c.schedule <= 8 && !lds_shape(c.schedule, c.block, 8, 0, 1, sh))
            return fail(SU3_ERR_INVALID_ARG,
                        "the LDS-tiled Dslash (schedule %d) has no tile for "
                        "block %d", c.schedule, c.block);
    } else if (c.schedule < 0 || c.schedule > 1) {
        return fail(SU3_ERR_INVALID_ARG, "schedule must be 0 or 1");
    }
    return SU3_OK;
}

static void load_cache_locked();

// The tuned or set launch of a key, if there is one.
static bool tuned_launch(int expr, int prec, int layout, int lanes, int64_t V,
                         su3_launch *c)
{
    std::lock_guard<std::mutex> lk(g_tune_mu);
    load_cache_locked();
    auto it = g_tuned.find(Key(expr, prec, layout, lanes, vbucket(V)));
    if (it == g_tuned.end())
        return false;
    *c = it->second;
    return true;
}

// Program keys hold two settings: that of the form of their own program (a*b,
// trace(a*adj(b)): by rows, on AoS fields the trace and large products on one lane
// per site), and, under kOtherForm, that of the other form.
static const int kOtherForm = 1 << 16;

static bool is_program_key(int expr)
{
    return expr == SU3_EXPR_PROGRAM || expr == SU3_EXPR_PROGRAM_SCALAR;
}

// AoS matrices up to which one product runs by rows, and their bytes.
static const int64_t kAosRowBytes = (int64_t)50 * 1000 * 1000;

static int64_t aos_bytes(const su3_field *z, int arith)
{
    return z->V * 18 * real_bytes(arith);
}

static bool row_product_aos(const su3_field *z, int arith)
{
    return aos_bytes(z, arith) <= kAosRowBytes;
}

// The setting of a program's key (form: PF_*, by_rows) that holds for it.  A
// setting of schedule 0 holds for every program of the key, as a caller sets it;
// the tuner's, of schedule 1, for the form it was timed on: the caps that suit
// one form cost the other up to half (FP32 48^4 a*b+c*d on one lane per site,
// with the cap that is best for a*b by rows 481 us, with its own 318).
// Nor does the cap that suits one product suit longer programs by rows (FP64 48^4
// c*a*b+0.5: with a*b's 399 us, uncapped 368).
static bool tuned_program(int expr, int prec, const su3_field *z, int form, const RowCode *rows,
                          su3_launch *c)
{
    const bool own_rows = z->layout != SU3_LAYOUT_AOS ||
                          (expr == SU3_EXPR_PROGRAM && row_product_aos(z, prec));
    const bool own = (rows != nullptr) == own_rows;
    if (tuned_launch(expr, prec, z->layout, z->lanes, z->V, c) &&
        (c->schedule == 0 || (form == PF_MATRIX && own))) {
        if (c->schedule == 1 && rows && rows->n > 1)
            c->occupancy = 0;
        return true;
    }
    return form == PF_MATRIX && !own &&
           tuned_launch(expr + kOtherForm, prec, z->layout, z->lanes, z->V, c);
}

static su3_launch lookup_launch(int expr, int prec, int layout, int lanes,
                                int64_t V)
{
    su3_launch c;
    return tuned_launch(expr, prec, layout, lanes, V, &c)
               ? c
               : default_launch(expr, prec, layout, lanes, V);
}

// Workgroups of a walk that a CU holds.
static int dslash_per_cu(const LdsShape &sh, int prec)
{
    const bool dbl = prec == SU3_F64;
    const int wave_slots = dbl ? 8 : prec == SU3_F32 ? 16 : 12;
    const int lanes = sh.nsub * sh.tx * sh.ty * sh.tz;
    return std::max(1, std::min((int)(160 * 1024 / lds_shape_bytes(sh, dbl ? 16 : 8)),
                                wave_slots / ((lanes + 63) / 64)));
}

// Estimated microseconds of an LDS-tiled Dslash walk of `walk` t-slices over
// (outer) extents o: the rounds of workgroups the CUs need, each walking its
// slices and a start-up, at a slice time that is the larger of a latency floor
// (barriers, LDS and a slice's dependent loads) and the tile's bytes at a CU's
// share of the memory rate.  The last walk of each tile may be shorter; those
// run last, beside the remaining long ones.  The constants are fitted to 44
// measured lattices (24^4 to 64 x 32^3, odd extents, virtual nodes; up to 13
// row tiles with up to 12 walks each) and checked on 12 more in eight layouts
// and three precisions: the planned launch takes 0.88 of the time of one fixed
// schedule (double 17 in walks of 8, single 16 in walks of 7) on average and at
// most 1.05.
static double dslash_walk_us(const LdsShape &sh, int prec, const int32_t o[4],
                             int walk, int cus)
{
    const bool dbl = prec == SU3_F64;
    const double spinor = dbl ? 192 : 96, link = dbl ? 144 : prec == SU3_F32 ? 72 : 48;
    const double floor_us = dbl ? 12.0 : sh.nb == 1 ? 13.0 : sh.nsub == 1 ? 10.4 : 10.2;
    const double start = 0.5, cu_bytes_per_us = 28e3;
    // bytes per site: links, input, output, and the share of the face sites'
    // second reads that miss (in double a halo saves some of those of a
    // square tile, and costs a 2 x 4 one, with more faces per row, what it
    // saves: 3 x 3 FP64 48^4 968 us against 1004, 2 x 4 FP64 32^4 219 against
    // 211)
    const double miss = dbl ? 0.5 : 1.0;
    const double x_cut = sh.tx < o[0] ? 0.5 / sh.tx : 0.0;
    const double yz_cut = miss * (1.0 / sh.ty + 1.0 / sh.tz);
    const double site_bytes = 2 * spinor + 4 * link + (2 * spinor + link) *
                              (x_cut + yz_cut * (dbl && sh.halo && sh.ty == sh.tz ? 0.85 : 1.0));
    const int lanes = sh.nsub * sh.tx * sh.ty * sh.tz, per_cu = dslash_per_cu(sh, prec);
    const int64_t tiles = (int64_t)((o[0] + sh.tx - 1) / sh.tx) *
                          ((o[1] + sh.ty - 1) / sh.ty) * ((o[2] + sh.tz - 1) / sh.tz);
    const int chunks = (o[3] + walk - 1) / walk, last = o[3] - (chunks - 1) * walk;
    const int64_t slots = (int64_t)cus * per_cu;
    const auto walk_us = [&](int slices, int64_t resident) {
        return (slices + start) *
               std::max(floor_us, (double)resident * lanes * site_bytes / cu_bytes_per_us);
    };
    const auto rounds_us = [&](int64_t groups, int slices) {
        const int64_t rest = groups % slots;
        return (double)(groups / slots) * walk_us(slices, per_cu) +
               (rest ? walk_us(slices, (rest + cus - 1) / cus) : 0.0);
    };
    if (last == walk)
        return rounds_us(tiles * chunks, walk);
    const int64_t rest = tiles * (chunks - 1) % slots;
    double us = (double)(tiles * (chunks - 1) / slots) * walk_us(walk, per_cu);
    if (rest == 0)
        return us + rounds_us(tiles, last);
    const int64_t resident = rest + tiles >= slots ? per_cu : (rest + tiles + cus - 1) / cus;
    const double lng = walk_us(walk, resident), shrt = walk_us(last, resident);
    const int64_t beside = (slots - rest) * (int64_t)(lng / shrt);
    us += lng;
    if (tiles > beside)
        us += (double)((tiles - beside + slots - 1) / slots) * shrt;
    return us;
}

// Whether a walk's workgroups go to the XCDs in ranges of tiles rather than
// one by one: tiles that run on one XCD at the same t read each other's faces
// from its L2.  Ranges share whole rows of tiles (FP64 32^4, 2 x 4 rows: 211 us
// against 237; FP32 64 x 32^3 230 against 270; FP64 48^4 968 against 984), dealt
// singly the tiles share a face only where eight divides their distance.
// Counted per face, weighted by the faces per site; where both share alike
// ranges read memory in longer pieces (FP32 32^4, 4 x 4 rows: 115 us against
// 127).  Not where rounding the ranges up to whole tiles takes an XCD one more
// round (81 tiles in 3 walks: 257 us against 152).
static bool dslash_ranges(const LdsShape &sh, const int32_t o[4], int walk, int cus, int per_cu)
{
    const int nx = (o[0] + sh.tx - 1) / sh.tx, ny = (o[1] + sh.ty - 1) / sh.ty,
              nz = (o[2] + sh.tz - 1) / sh.tz, n = nx * ny * nz, t8 = (n + 7) / 8;
    const int64_t chunks = (o[3] + walk - 1) / walk;
    const int64_t xcd = std::max(1, cus / 8 * per_cu), slots = std::max(1, cus * per_cu);
    if ((t8 * chunks + xcd - 1) / xcd > (n * chunks + slots - 1) / slots)
        return false;
    // nor where it gives some CU one more workgroup (100 tiles in 5 walks, 65
    // for the 32 CUs of an XCD: FP32 20 x 40^3 198 us, singly 141)
    const int64_t cus_xcd = std::max(1, cus / 8), cus_all = std::max(1, cus);
    if ((t8 * chunks + cus_xcd - 1) / cus_xcd > (n * chunks + cus_all - 1) / cus_all)
        return false;
    double singly = 0, ranges = 0;
    for (int z = 0; z < nz; ++z)
        for (int y = 0; y < ny; ++y)
            for (int x = 0; x < nx; ++x) {
                const int t = x + nx * (y + ny * z);
                const int ty = x + nx * ((y + 1) % ny + ny * z), tz = x + nx * (y + ny * ((z + 1) % nz));
                if (n % 8 == 0)
                    singly += (t % 8 == ty % 8) / (double)sh.ty + (t % 8 == tz % 8) / (double)sh.tz;
                ranges += (t / t8 == ty / t8) / (double)sh.ty + (t / t8 == tz / t8) / (double)sh.tz;
            }
    return ranges >= singly - 0.01 * n;
}

// The untuned launch of the Wilson hopping term on lattice dims (virtual
// nodes simd, L sites per lane-block).
static su3_launch plan_dslash(int prec, int layout, int64_t L, const int32_t dims[4],
                              const int32_t simd[4], int cus)
{
    const bool dbl = prec == SU3_F64, vn = layout == SU3_LAYOUT_VNODE;
    const int cbytes = dbl ? 16 : 8, nsub = vn ? (int)L : 1;
    int32_t o[4];
    int64_t V = 1;
    for (int mu = 0; mu < 4; ++mu) {
        o[mu] = dims[mu] / simd[mu];
        V *= dims[mu];
    }
    su3_launch c = default_launch(SU3_EXPR_DSLASH, prec, layout, 0, V);
    // One wave per hop where the lattice cannot fill the chip otherwise (16^3
    // x 32, two-row links: 12.7 us, walks 46.8, one lane per site 15.8) and
    // as long as its second reads of each spinor come from the caches: to
    // 24^4 (FP64 79 us, best walk 76) on whole lines, less where a wave's
    // entry is shorter than a line (N_sub < 8 FP64 24^4: 101 against 84) or
    // double spinors lie site after site (174 against 148).
    // Single AoS spinors keep it at any size: the walks store nontemporally,
    // which AoS pays for (FP32 32^4: 238 us against 434).
    const bool aos = layout == SU3_LAYOUT_AOS, pairs = vn && nsub < 4;
    const int64_t most = aos && !dbl ? ((int64_t)1 << 31) : (aos || (vn && nsub < 8)) ? 150000 : 360000;
    su3_launch hops = c;
    hops.schedule = 0;
    hops.tile_sites = 1;
    hops.sites_per_lane = 8;
    hops.xcd_remap = 1;
    hops.nontemporal = aos || (vn && nsub < 8) ? 0 : 2;
    if (V <= most)
        return hops;
    double best = 1e300;
    // of equals the first: two buffers where the links are two-row (48^4 16/7
    // 454 us, 12/7 466), one otherwise (FP32 26 x 30 x 34 x 28 100 us, 103)
    static const int by_tile[] = {9, 10, 11, 12, 16, 17, 18, 20, 21, 22, 26, 27, 28};
    static const int by_buffers[] = {16, 18, 26, 28, 9, 10, 11, 12, 17, 20, 21, 22, 27};
    LdsShape rows;
    const int aos_rows = lds_shape(18, 256, cbytes, o[0], 1, rows) ? 18 : 17;
    // Outer rows that no tile holds and that divide badly are cut into many
    // pieces, whose walks the model takes for too fast: there 4 x 4 rows with
    // two buffers and walks of 7 (N_sub 8 FP32 34^4, pieces of 2: 195 us, the
    // model's 17/9 264).
    const bool small = !dbl && V <= 700000 && !(pairs && prec == SU3_F32);
    if (vn && !dbl && lds_shape(16, 256, cbytes, o[0], nsub, rows) && 12 * rows.tx < o[0])
        return small ? hops : c;
    for (int sched : prec == SU3_C12_F32 ? by_buffers : by_tile) {
        LdsShape sh;
        // Where a lane's line holds more of other entries than of its own,
        // only two buffers, which read a slice ahead: double AoS in 3 x 3 rows
        // (32^4 18/16 447 us, 22/8 512, 17/8 488), single with N_sub 2 (48^4
        // 18/24 848 us, 17/24 1066, 16/7 986).
        if ((aos && sched != aos_rows && sched != aos_rows + 10) ||
            (pairs && !dbl && sched != 16 && sched != 18))
            continue;
        if (!lds_shape(sched, 256, cbytes, o[0], nsub, sh))
            continue;
        // Walks of equal length, the last one shorter; virtual nodes halve the
        // t extent, which leaves few of those, so there every length counts
        // (two-row links 40^2 x 32^2 in 16 nodes: walks of 7 175 us, the best
        // of 6 188; lexicographic fields lose by it, FP64 40^4 577 against 529).
        for (int walk = std::min(o[3], 4096); walk > 0; --walk) {
            const int chunks = (o[3] + walk - 1) / walk;
            if (!vn && walk != (o[3] + chunks - 1) / chunks)
                continue;
            const double us = dslash_walk_us(sh, prec, o, walk, cus);
            if (us < best) {
                best = us;
                c.schedule = sched;
                c.tile_sites = walk;
                // (singly where lines hold several entries: N_sub 2 FP64 48^4
                // 1334 us, in ranges 1417; N_sub 4 44^4 830 and 871)
                c.xcd_remap = !(vn && nsub < 8) &&
                                      dslash_ranges(sh, o, walk, cus, dslash_per_cu(sh, prec))
                                  ? 2
                                  : 0;
            }
        }
    }
    // Single spinors to 24^3 x 48 take one wave per hop where the walks suffer
    // from the lattice's extents: a site's hops take 0.092 ns with two-row
    // links and 0.108 with three rows (N_sub 16 28^4 55 us, walk 99; FP32 66
    // and 82; FP32 26^4 49.5 and 65.6), but with N_sub 2 0.19 (28^4 119, 92).
    // With virtual nodes, and on few t-slices, where a tile needs few walks,
    // the model takes the walks for slower than they are.
    const double hop_us = (prec == SU3_C12_F32 ? 0.092e-3 : 0.108e-3) * (double)V;
    const double margin = vn || o[3] <= 16 ? 1.16 : 1.05;
    return small && best > margin * hop_us ? hops : c;
}

// plan_dslash, remembered per lattice (a few microseconds of host time
// each); a bounded table of plain values, shared by all threads.
static su3_launch default_dslash(int prec, int layout, int64_t L, const int32_t dims[4],
                                 const int32_t simd[4], int cus)
{
    struct Plan {
        int32_t key[11];  // zero: none (no extent is)
        su3_launch c;
    };
    static std::mutex mu;
    static Plan plans[256];  // by a hash of the key, the newest kept
    const int32_t key[11] = {prec,    layout,  cus,     dims[0], dims[1], dims[2],
                             dims[3], simd[0], simd[1], simd[2], simd[3]};
    uint32_t h = 0;
    for (int32_t v : key)
        h = (h ^ (uint32_t)v) * 2654435761u;
    std::lock_guard<std::mutex> lk(mu);
    Plan &p = plans[h >> 24];
    if (std::memcmp(p.key, key, sizeof key) != 0) {
        p.c = plan_dslash(prec, layout, L, dims, simd, cus);
        std::memcpy(p.key, key, sizeof key);
    }
    return p.c;
}

// JSON cache: one object per line with integer fields.
static std::string device_tag()
{
    int dev = 0;
    hipDeviceProp_t p;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipGetDeviceProperties(&p, dev) != hipSuccess)
        return "unknown";
    char buf[300];
    snprintf(buf, sizeof buf, "%s:%d", p.gcnArchName, p.multiProcessorCount);
    return buf;
}

static bool parse_int(const std::string &line, const char *key, int *v)
{
    std::string pat = std::string("\"") + key + "\":";
    size_t pos = line.find(pat);
    if (pos == std::string::npos)
        return false;
    *v = atoi(line.c_str() + pos + pat.size());
    return true;
}

static void load_cache_locked()
{
    if (g_cache_loaded)
        return;
    g_cache_loaded = true;
    const char *path = getenv("SU3_TUNE_CACHE");
    if (!path || !*path)
        return;
    FILE *fp = fopen(path, "r");
    if (!fp)
        return;
    const std::string tag = device_tag();
    char buf[1024];
    while (fgets(buf, sizeof buf, fp)) {
        std::string line(buf);
        if (line.find("\"device\":\"" + tag + "\"") == std::string::npos)
            continue;
        int ex, pr, la, ln, vb;
        su3_launch c;
        if (!parse_int(line, "expr", &ex) || !parse_int(line, "prec", &pr) ||
            !parse_int(line, "layout", &la) || !parse_int(line, "lanes", &ln) ||
            !parse_int(line, "vbucket", &vb) ||
            !parse_int(line, "block", &c.block) ||
            !parse_int(line, "persistent", &c.persistent) ||
            !parse_int(line, "nontemporal", &c.nontemporal) ||
            !parse_int(line, "xcd_remap", &c.xcd_remap) ||
            !parse_int(line, "lds_stage", &c.lds_stage) ||
            !parse_int(line, "tile_sites", &c.tile_sites) ||
            !parse_int(line, "occupancy", &c.occupancy) ||
            !parse_int(line, "schedule", &c.schedule))
            continue;
        if (!parse_int(line, "sites_per_lane", &c.sites_per_lane))
            c.sites_per_lane = 0;
        if (check_launch(c, la, ex) != SU3_OK)
            continue;
        if (is_program_key(ex)) {
            // lines that name no form are from before there were two
            if (c.schedule == 0)
                continue;
            int other = 0;
            (void)parse_int(line, "other_form", &other);
            ex += other ? kOtherForm : 0;
        }
        g_tuned[Key(ex, pr, la, ln, vb)] = c;
    }
    fclose(fp);
}

static void append_cache(const Key &k, const su3_launch &c, double us)
{
    const char *path = getenv("SU3_TUNE_CACHE");
    if (!path || !*path)
        return;
    FILE *fp = fopen(path, "a");
    if (!fp)
        return;
    fprintf(fp,
            "{\"device\":\"%s\",\"expr\":%d,\"prec\":%d,\"layout\":%d,"
            "\"lanes\":%d,\"vbucket\":%d,\"block\":%d,\"persistent\":%d,"
            "\"nontemporal\":%d,\"xcd_remap\":%d,\"lds_stage\":%d,"
            "\"tile_sites\":%d,\"occupancy\":%d,\"schedule\":%d,"
            "\"sites_per_lane\":%d,%s\"us\":%.3f}\n",
            device_tag().c_str(), std::get<0>(k) & ~kOtherForm, std::get<1>(k),
            std::get<2>(k), std::get<3>(k), std::get<4>(k), c.block,
            c.persistent, c.nontemporal, c.xcd_remap, c.lds_stage,
            c.tile_sites, c.occupancy, c.schedule, c.sites_per_lane,
            std::get<0>(k) & kOtherForm ? "\"other_form\":1," : "", us);
    fclose(fp);
}

// --------------------------------------------------------- validation

static bool same_geometry(const su3_field *a, const su3_field *b)
{
    return a->layout == b->layout && a->lanes == b->lanes &&
           std::memcmp(a->dims, b->dims, sizeof a->dims) == 0 &&
           std::memcmp(a->simd, b->simd, sizeof a->simd) == 0 &&
           a->device == b->device;
}

static bool same_shape(const su3_field *a, const su3_field *b)
{
    return a->kind == b->kind && a->prec == b->prec && same_geometry(a, b);
}

static bool overlaps(const su3_field *a, const su3_field *b)
{
    const uintptr_t a0 = (uintptr_t)a->ptr, a1 = a0 + a->bytes;
    const uintptr_t b0 = (uintptr_t)b->ptr, b1 = b0 + b->bytes;
    return a0 < b1 && b0 < a1;
}

static su3_status validate_item(const su3_field *z, int expr,
                                const su3_field *const *ops, int32_t n_ops)
{
    if (!z)
        return fail(SU3_ERR_INVALID_ARG, "output field is NULL");
    if (z->kind != KIND_MATRIX)
        return fail(SU3_ERR_MISMATCH,
                    "a spinor field where an SU(3) matrix field is expected");
    if (expr < SU3_EXPR_MUL || expr > SU3_EXPR_APB_AB)
        return fail(SU3_ERR_INVALID_ARG, "unknown expression %d", expr);
    if (!ops)
        return fail(SU3_ERR_INVALID_ARG, "operand list is NULL");
    if (n_ops != operands_of(expr))
        return fail(SU3_ERR_INVALID_ARG, "expression %d takes %d operands, got %d",
                    expr, operands_of(expr), n_ops);
    for (int k = 0; k < n_ops; ++k) {
        if (!ops[k])
            return fail(SU3_ERR_INVALID_ARG, "operand %d is NULL", k);
        if (!same_shape(z, ops[k]))
            return fail(SU3_ERR_MISMATCH,
                        "operand %d differs from the output in dims, "
                        "precision, layout, lanes or device", k);
    }
    if (z->prec == SU3_C12_F32 && expr != SU3_EXPR_MUL &&
        expr != SU3_EXPR_MUL3)
        return fail(SU3_ERR_UNSUPPORTED,
                    "the two-row compressed form supports MUL and MUL3 only "
                    "(sums leave SU(3))");
    for (int k = 0; k < n_ops; ++k)
        if (overlaps(z, ops[k]) &&
            !(z->ptr == ops[k]->ptr && z->bytes == ops[k]->bytes))
            return fail(SU3_ERR_ALIAS,
                        "output partially overlaps operand %d", k);
    return SU3_OK;
}

// ------------------------------------------------------------ compute

// What a staged launch may count, a tile per operand.  The kernel passes all of
// them through one tile; settings beyond the limit stay refused all the same.
static const size_t kLdsStageMaxBytes = 65536;

static su3_status launch_item(su3_field *z, int expr,
                              const su3_field *const *ops, int32_t n_ops,
                              const su3_launch &c, hipStream_t st)
{
    SiteArgs a;
    std::memset(&a, 0, sizeof a);
    a.z = z->ptr;
    for (int k = 0; k < n_ops; ++k)
        a.op[k] = ops[k]->ptr;
    a.g = geom_of(z);
    a.nsites = (int32_t)z->V;
    a.xcd_remap = c.xcd_remap;
    hipError_t e;
    if (z->layout == SU3_LAYOUT_AOS && c.lds_stage) {
        const size_t shm = (size_t)n_ops * c.block * z->E * 2 * z->rbytes;
        if (shm > kLdsStageMaxBytes)
            return fail(SU3_ERR_UNSUPPORTED,
                        "LDS staging of %d operands x %d sites counts %zu bytes "
                        "(limit %zu)", n_ops, c.block, shm,
                        kLdsStageMaxBytes);
        const int64_t tiles = (z->V + c.block - 1) / c.block;
        int64_t grid = tiles;
        if (c.persistent)
            grid = std::min<int64_t>(grid, (int64_t)c.persistent *
                                               device_cus(z->device));
        a.ngroups = (int32_t)z->V;
        e = launch_site_lds(z->prec, expr, c.nontemporal, c.block, (int)grid,
                            occupancy_reserve(z->device, c.occupancy), a, st);
    } else {
        // S sites per lane must sit in one lane-block: the natural count
        // (or 1 where the blocks are shorter), or the launch's own count
        int S = natural_sites(z->prec, expr);
        if (c.sites_per_lane > 0) {
            S = c.sites_per_lane;
            if (!sites_compiled(z->prec, expr, S) ||
                (S > 1 && (z->layout == SU3_LAYOUT_AOS || z->L % S != 0)))
                return fail(SU3_ERR_INVALID_ARG,
                            "sites_per_lane %d is not offered for this "
                            "expression, precision and lane-block", S);
        } else if (z->layout == SU3_LAYOUT_AOS || z->L % S != 0) {
            S = 1;
        }
        a.ngroups = (int32_t)((z->V + S - 1) / S);
        int64_t grid = (a.ngroups + c.block - 1) / c.block;
        if (c.persistent)
            grid = std::min<int64_t>(grid, (int64_t)c.persistent *
                                               device_cus(z->device));
        e = launch_site(z->prec, expr, S, c.nontemporal, c.schedule, c.block,
                        (int)grid, occupancy_reserve(z->device, c.occupancy), a,
                        st);
    }
    if (e != hipSuccess)
        return hip_fail(e, "kernel launch");
    return SU3_OK;
}

extern "C" su3_status su3_fused_eval(su3_field *z, su3_expr expr,
                                     const su3_field *const *ops,
                                     int32_t n_ops, void *stream)
{
    su3_status st = validate_item(z, expr, ops, n_ops);
    if (st != SU3_OK)
        return st;
    const su3_launch c =
        lookup_launch(expr, z->prec, z->layout, z->lanes, z->V);
    return launch_item(z, expr, ops, n_ops, c,
                       static_cast<hipStream_t>(stream));
}

extern "C" su3_status su3_mult(su3_field *z, const su3_field *x,
                               const su3_field *y, void *stream)
{
    const su3_field *ops[2] = {x, y};
    return su3_fused_eval(z, SU3_EXPR_MUL, ops, 2, stream);
}

// ----------------------------------------------------- shifted operands

// Launch of the shifted-operand kernels: the tuned (or default) setting of
// the key (SU3_EXPR_CSHIFT or SU3_EXPR_MUL_SHIFTED, precision, layout,
// lanes, volume); one site per lane, one-shot grid.
static su3_status launch_shift_op(int mode, su3_field *z, const su3_field *x,
                                  const su3_field *y, int32_t mu,
                                  int32_t shift, void *stream,
                                  const su3_launch *forced = nullptr)
{
    const su3_launch c =
        forced ? *forced
               : lookup_launch(mode ? SU3_EXPR_MUL_SHIFTED : SU3_EXPR_CSHIFT,
                               z->prec, z->layout, z->lanes, z->V);
    ShiftArgs a;
    std::memset(&a, 0, sizeof a);
    a.z = z->ptr;
    a.x = x ? x->ptr : nullptr;
    a.y = y->ptr;
    a.g = geom_of(z);
    a.nsites = (int32_t)z->V;
    // outer stride (storage sites) and extent along mu; lane stride and
    // count along mu (1 lane outside the virtual-node layout)
    int64_t ostride = z->layout == SU3_LAYOUT_VNODE ? z->L : 1;
    int64_t lstride = 1;
    for (int d = 0; d < mu; ++d) {
        ostride *= z->dims[d] / z->simd[d];
        lstride *= z->simd[d];
    }
    const int64_t L = z->dims[mu];
    a.stride = (uint32_t)ostride;
    a.extent = (uint32_t)(L / z->simd[mu]);
    a.nlanes = (uint32_t)z->simd[mu];
    a.lstride = (uint32_t)lstride;
    a.lmask = z->layout == SU3_LAYOUT_VNODE ? (uint32_t)(z->L - 1) : 0u;
    a.shift = (uint32_t)(((int64_t)shift % L + L) % L);
    a.xcd_remap = c.xcd_remap;
    const int64_t grid = (z->V + c.block - 1) / c.block;
    hipError_t e = launch_shift(z->prec, mode, c.nontemporal, c.schedule,
                                c.block, (int)grid,
                                occupancy_reserve(z->device, c.occupancy), a,
                                static_cast<hipStream_t>(stream));
    if (e != hipSuccess)
        return hip_fail(e, "shift kernel launch");
    return SU3_OK;
}

extern "C" su3_status su3_cshift(su3_field *dst, const su3_field *src,
                                 int32_t mu, int32_t shift, void *stream)
{
    if (!dst || !src)
        return fail(SU3_ERR_INVALID_ARG, "field is NULL");
    if (mu < 0 || mu > 3)
        return fail(SU3_ERR_INVALID_ARG, "direction %d not in [0, 3]", mu);
    if (dst->kind != KIND_MATRIX || src->kind != KIND_MATRIX)
        return fail(SU3_ERR_MISMATCH,
                    "a spinor field where an SU(3) matrix field is expected");
    if (!same_shape(dst, src))
        return fail(SU3_ERR_MISMATCH, "dst and src differ in dims, precision, "
                                      "layout, lanes or device");
    if (overlaps(dst, src))
        return fail(SU3_ERR_ALIAS, "dst overlaps src (a shift is a gather: "
                                   "it cannot run in place)");
    return launch_shift_op(0, dst, nullptr, src, mu, shift, stream);
}

extern "C" su3_status su3_mult_shifted(su3_field *z, const su3_field *x,
                                       const su3_field *y, int32_t mu,
                                       int32_t shift, void *stream)
{
    if (!z || !x || !y)
        return fail(SU3_ERR_INVALID_ARG, "field is NULL");
    if (mu < 0 || mu > 3)
        return fail(SU3_ERR_INVALID_ARG, "direction %d not in [0, 3]", mu);
    if (z->kind != KIND_MATRIX)
        return fail(SU3_ERR_MISMATCH,
                    "a spinor field where an SU(3) matrix field is expected");
    if (!same_shape(z, x) || !same_shape(z, y))
        return fail(SU3_ERR_MISMATCH, "operands differ in dims, precision, "
                                      "layout, lanes or device");
    if (overlaps(z, y))
        return fail(SU3_ERR_ALIAS, "z overlaps the shifted operand y");
    if (overlaps(z, x) && !(z->ptr == x->ptr && z->bytes == x->bytes))
        return fail(SU3_ERR_ALIAS, "z partially overlaps x");
    return launch_shift_op(1, z, x, y, mu, shift, stream);
}

// ------------------------------------------------------ Wilson hopping

// Site tiles of the one-site Dslash kernel by `schedule` (1..3) and block
// B: 8 x 4 x 2 x B/64, 4 x 4 x 4 x B/64, 8 x 2 x 2 x B/32.
static void dslash_tile(int schedule, int block, uint32_t t[4])
{
    static const uint32_t shape[3][3] = {{8, 4, 2}, {4, 4, 4}, {8, 2, 2}};
    const uint32_t *sh = shape[(schedule - 1) % 3];
    t[0] = sh[0];
    t[1] = sh[1];
    t[2] = sh[2];
    t[3] = (uint32_t)block / (sh[0] * sh[1] * sh[2]);
}

static int spinor_prec_of_links(int link_prec)
{
    return link_prec == SU3_F64 ? SU3_F64 : SU3_F32;
}

// One site per lane, one-shot grid, the tuned (or default) block and
// occupancy of the key (SU3_EXPR_DSLASH, link precision, layout, lanes,
// volume).
static su3_status launch_dslash_op(su3_field *out, su3_field *const links[4],
                                   const su3_field *in, void *stream,
                                   const su3_launch *forced = nullptr)
{
    const su3_field *u0 = links[0];
    su3_launch c;
    if (forced)
        c = *forced;
    else if (!tuned_launch(SU3_EXPR_DSLASH, u0->prec, u0->layout, u0->lanes, u0->V, &c))
        c = default_dslash(u0->prec, u0->layout, u0->L, u0->dims, u0->simd,
                           device_cus(u0->device));
    const int cbytes = 2 * out->rbytes;  // one complex spinor entry
    const bool vn = out->layout == SU3_LAYOUT_VNODE;
    const int nsub = vn ? (int)out->L : 1;
    const int lx = (int)(out->dims[0] / out->simd[0]);  // (outer) x extent
    LdsShape sh = {0, 0, 0, 0, 1};
    // LDS-tiled walks: schedules 4.. on lexicographic fields, the row tiles
    // (9..18) on virtual-node fields
    bool lds = c.schedule >= (vn ? 9 : 4);
    if (lds && c.schedule >= 19 && !lds_shape(c.schedule, c.block, cbytes, lx, nsub, sh)) {
        // a halo walk that does not fit: its rows with one buffer and a
        // halo, else the same rows without a halo (and their fallbacks)
        const int rows = c.schedule - 10;
        const int one_buffer = rows == 18 ? 17 : rows >= 13 && rows <= 16 ? rows - 4 : 0;
        c.schedule = one_buffer && lds_shape(one_buffer + 10, 0, cbytes, lx, nsub, sh)
                         ? one_buffer + 10
                         : rows;
    }
    if (lds && !lds_shape(c.schedule, c.block, cbytes, lx, nsub, sh)) {
        // buffers too large: the same rows with one buffer, else rows of
        // 2 x 2; a fixed tile too large for double spinors: the schedule's
        // smallest; else 16 x 4 x 4 (virtual nodes: one site per lane)
        const int one_buffer = c.schedule == 18                         ? 17
                               : c.schedule >= 13 && c.schedule <= 16 ? c.schedule - 4
                                                                      : 0;
        if (one_buffer && lds_shape(one_buffer, 0, cbytes, lx, nsub, sh)) {
            c.schedule = one_buffer;
        } else if (c.schedule >= 9 && lds_shape(9, 0, cbytes, lx, nsub, sh)) {
            c.schedule = 9;
        } else if (vn) {
            lds = false;
        } else {
            if (c.schedule >= 9)
                c.schedule = 8;
            c.block = c.schedule >= 7 ? 256 : 128;
            lds_shape(c.schedule, c.block, cbytes, lx, 1, sh);
        }
    }
    if (lds)
        c.block = sh.nsub * sh.tx * sh.ty * sh.tz;
    else if (c.block > 256)
        c.block = 256;  // the one-site and walk kernels take at most 256
    DslashArgs a;
    std::memset(&a, 0, sizeof a);
    a.out = out->ptr;
    a.in = in->ptr;
    for (int mu = 0; mu < 4; ++mu)
        a.u[mu] = links[mu]->ptr;
    a.gs = geom_of(out);
    a.gl = geom_of(u0);
    a.nsites = (int32_t)out->V;
    a.xcd_remap = c.xcd_remap;
    // outer extents and strides (storage sites), lane counts and strides
    int64_t ostride = vn ? out->L : 1, lstride = 1;
    uint32_t lg = 0;
    while (vn && ((int64_t)1 << lg) < out->L)
        ++lg;
    a.lg = lg;
    a.lmask = vn ? (uint32_t)(out->L - 1) : 0u;
    for (int mu = 0; mu < 4; ++mu) {
        a.dims[mu] = (uint32_t)(out->dims[mu] / out->simd[mu]);
        a.stride[mu] = (uint32_t)ostride;
        a.nlanes[mu] = (uint32_t)out->simd[mu];
        a.lstride[mu] = (uint32_t)lstride;
        ostride *= a.dims[mu];
        lstride *= out->simd[mu];
    }
    // lanes: one per site, or (lexicographic site order only) one per
    // (x, y, z) site and chunk of `walk` t-slices
    const int64_t Lt = a.dims[3];  // (outer) t extent
    a.walk = vn ? 1u : (uint32_t)std::min<int64_t>(std::max(c.tile_sites, 1), Lt);
    const int64_t lanes = a.walk <= 1 ? out->V
                                      : a.stride[3] * ((Lt + a.walk - 1) / a.walk);
    int64_t grid = (lanes + c.block - 1) / c.block;
    if (lds) {
        // LDS-tiled walk: tiles of (x, y, z) sites walking t
        // (not in calls that the Infinity Cache holds from one to the next: two-
        // row links 32^3 x 24, 302 MB, 60.2 us bypassed, 56.9 cached; FP32 28^4,
        // 295 MB, 64.4 and 61.8; FP32 32^3 x 24, 377 MB, 70.0 and 76.6)
        a.t_bypass = whole_lines(u0) && 4 * u0->bytes + 2 * out->bytes > (size_t)330 * 1000 * 1000;
        a.lds_tile = (uint32_t)c.schedule;
        a.lds_tx = (uint32_t)sh.tx;
        a.walk = (uint32_t)std::min<int64_t>(std::max(c.tile_sites, 1), Lt);
        const uint32_t tdim[3] = {(uint32_t)sh.tx, (uint32_t)sh.ty, (uint32_t)sh.tz};
        grid = (Lt + a.walk - 1) / a.walk;
        int64_t ntiles = 1;
        for (int mu = 0; mu < 3; ++mu) {
            a.ntile[mu] = (a.dims[mu] + tdim[mu] - 1) / tdim[mu];
            ntiles *= a.ntile[mu];
        }
        grid *= ntiles;
        if (c.xcd_remap == 2)  // XCD slabs: 8 ranges of ceil(ntiles / 8) tiles
            grid = (Lt + a.walk - 1) / a.walk * 8 * ((ntiles + 7) / 8);
        if (c.persistent > 0) {
            // k workgroups per CU, each an equal share of the (tile, slice)
            // pairs: no tail of partly filled rounds, few walk starts
            const int64_t pairs = ntiles * Lt;
            const int64_t g = std::min<int64_t>(
                pairs, (int64_t)device_cus(out->device) * c.persistent);
            a.span = (uint32_t)((pairs + g - 1) / g);
            grid = (pairs + a.span - 1) / a.span;
        }
    } else if (a.walk <= 1 && !vn && c.schedule > 0) {
        dslash_tile(c.schedule, c.block, a.tile);
        grid = 1;
        for (int mu = 0; mu < 4; ++mu) {
            a.ntile[mu] = (uint32_t)((out->dims[mu] + a.tile[mu] - 1) / a.tile[mu]);
            grid *= a.ntile[mu];
        }
    }
    size_t shm = occupancy_reserve(out->device, c.occupancy);
    if (a.lds_tile)  // the tile's slice buffers (no occupancy cap)
        shm = lds_shape_bytes(sh, cbytes);
    if (!lds && a.walk <= 1 && c.schedule == 0 && c.sites_per_lane == 8) {
        a.hop_waves = 1;
        c.block = kDslashHopBlock;
        grid = (out->V + kDslashHopSites - 1) / kDslashHopSites;
        shm = (size_t)kDslashHopComplex * cbytes;
    }
    hipError_t e = launch_dslash(out->prec, u0->prec, c.nontemporal, c.block,
                                 (int)grid, shm, a,
                                 static_cast<hipStream_t>(stream));
    if (e != hipSuccess)
        return hip_fail(e, "Dslash kernel launch");
    return SU3_OK;
}

extern "C" su3_status su3_dslash(su3_field *out, su3_field *const links[4],
                                 const su3_field *in, void *stream)
{
    if (!out || !in || !links)
        return fail(SU3_ERR_INVALID_ARG, "field or link list is NULL");
    for (int mu = 0; mu < 4; ++mu)
        if (!links[mu])
            return fail(SU3_ERR_INVALID_ARG, "links[%d] is NULL", mu);
    if (out->kind != KIND_SPINOR || in->kind != KIND_SPINOR)
        return fail(SU3_ERR_MISMATCH, "in and out must be spinor fields");
    if (!same_shape(out, in))
        return fail(SU3_ERR_MISMATCH, "in and out differ in dims, precision, "
                                      "layout, lanes or device");
    for (int mu = 0; mu < 4; ++mu) {
        const su3_field *u = links[mu];
        if (u->kind != KIND_MATRIX)
            return fail(SU3_ERR_MISMATCH, "links[%d] is not a matrix field", mu);
        if (!same_shape(u, links[0]))
            return fail(SU3_ERR_MISMATCH,
                        "links[%d] differs from links[0] in dims, precision, "
                        "layout, lanes or device", mu);
        if (!same_geometry(u, out))
            return fail(SU3_ERR_MISMATCH,
                        "links[%d] differs from the spinors in dims, layout, "
                        "lanes, virtual nodes or device", mu);
    }
    const int lp = links[0]->prec;
    if (lp == SU3_F16_F32ACC || spinor_prec_of_links(lp) != out->prec)
        return fail(SU3_ERR_UNSUPPORTED,
                    "precision pair (spinor %d, links %d) not supported: "
                    "F64 spinors take F64 links, F32 spinors F32 or C12 links",
                    out->prec, lp);
    if (overlaps(out, in))
        return fail(SU3_ERR_ALIAS, "out overlaps in (a stencil gathers "
                                   "neighbours: it cannot run in place)");
    for (int mu = 0; mu < 4; ++mu)
        if (overlaps(out, links[mu]))
            return fail(SU3_ERR_ALIAS, "out overlaps links[%d]", mu);
    return launch_dslash_op(out, links, in, stream);
}

// ------------------------------------------------ expression programs

struct su3_program {
    ProgCode code;
    int32_t kinds[kProgMaxOps];
};

static const char *kind_name(int k)
{
    switch (k) {
    case KIND_MATRIX: return "matrix";
    case KIND_SPINOR: return "spinor";
    case KIND_REAL: return "real";
    case KIND_COMPLEX: return "complex";
    }
    return "unknown";
}

extern "C" su3_status su3_program_create(su3_program **out, const char *expr,
                                         int32_t n_ops, const su3_kind *kinds)
{
    if (!out || !expr)
        return fail(SU3_ERR_INVALID_ARG, "out or expression is NULL");
    if (n_ops < 0 || n_ops > kProgMaxOps)
        return fail(SU3_ERR_INVALID_ARG, "n_ops %d not in [0, %d]", n_ops,
                    kProgMaxOps);
    if (n_ops > 0 && !kinds)
        return fail(SU3_ERR_INVALID_ARG, "kinds is NULL");
    int k32[kProgMaxOps] = {0};
    for (int k = 0; k < n_ops; ++k) {
        if (kinds[k] < KIND_MATRIX || kinds[k] > KIND_COMPLEX)
            return fail(SU3_ERR_INVALID_ARG, "unknown kind %d of operand %d",
                        (int)kinds[k], k);
        if (kinds[k] == KIND_SPINOR)
            return fail(SU3_ERR_UNSUPPORTED,
                        "expressions take matrix, real and complex fields");
        k32[k] = kinds[k];
    }
    su3_program *p = new su3_program();
    char err[256];
    if (!compile_program(expr, n_ops, k32, &p->code, err, sizeof err)) {
        delete p;
        return fail(SU3_ERR_INVALID_ARG, "expression \"%s\": %s", expr, err);
    }
    for (int k = 0; k < kProgMaxOps; ++k)
        p->kinds[k] = k < n_ops ? k32[k] : -1;
    *out = p;
    return SU3_OK;
}

extern "C" su3_status su3_program_info(const su3_program *p,
                                       su3_kind *result_kind,
                                       int32_t *n_instr, int32_t *n_regs)
{
    if (!p)
        return fail(SU3_ERR_INVALID_ARG, "program is NULL");
    if (result_kind)
        *result_kind = (su3_kind)p->code.result_kind;
    if (n_instr)
        *n_instr = p->code.ninstr;
    if (n_regs)
        *n_regs = p->code.nregs;
    return SU3_OK;
}

extern "C" su3_status su3_program_destroy(su3_program *p)
{
    delete p;
    return SU3_OK;
}

static int row_sites_per_lane(const su3_field *z, int arith)
{
    return arith == SU3_F32 && z->L % 2 == 0 ? 2 : 1;
}

// The code of a matrix program in the row form, or null for the one-lane
// kernel.
static const RowCode *row_code(const su3_program *p, const su3_field *z, int arith)
{
    const ProgCode &pc = p->code;
    const bool aos = z->layout == SU3_LAYOUT_AOS;
    if (pc.rows.n == 0)  // more slots than there are: no known expression
        return nullptr;
    // AoS matrices without a matrix to store: the one-lane kernel's cached
    // loads reach the rest of a site's record in the same lines (FP64 32^4
    // trace(a*adj(b)): 58 us against 88 through LDS).
    if (aos && pc.result_kind != FK_MATRIX)
        return nullptr;
    const DeviceFacts f = device_facts(z->device);
    const int spl = row_sites_per_lane(z, arith);
    const int64_t groups = (z->V + 64 * spl - 1) / (64 * spl);
    const int64_t slots = (int64_t)pc.rows.nslots * kRowSlotVecs * spl * 2 * real_bytes(arith);
    const int64_t at_once = f.cus * (f.lds_per_cu / slots);
    // AoS with a matrix to store: the one-lane kernel's cached stores reach the
    // rest of the record likewise.  By rows go a product of fields in the caches
    // (FP64 16^4 a*adj(b) 6.5 us against 8.0, 24^4 28.3 both, 48^4 494 against 450;
    // FP32 24^4 20.1 and 23.0, 32^4 in turn 71 and 68), programs of three slots, in
    // double of smaller ones (c*a*b+0.5 in turn 22^4 27.3 and 30.3, 24^4 50 and 40;
    // FP32 28^4 44.7 and 48.3), and of more than four in one round (force term
    // FP32 16^4 13.3 and 16.8, FP64 16^4, two rounds, 32.8 and 25.1; four slots,
    // FP64 a*b+c*d, 12^4 8.2 and 7.1, 48^4 1391 and 731).
    if (aos) {
        const bool cached = row_product_aos(z, arith);
        const bool small = arith == SU3_F32 || 10 * aos_bytes(z, arith) <= 7 * kAosRowBytes;
        return (pc.rows.nslots <= 2   ? cached
                : pc.rows.nslots == 3 ? cached && small
                                      : pc.rows.nslots > 4 && groups <= at_once)
                   ? &pc.rows
                   : nullptr;
    }
    // every workgroup resident at once: nothing to gain from smaller ones
    // (force term, six slots, FP64 12^4: 12.1 us, with registers 14.3)
    if (groups <= at_once)
        return &pc.rows;
    // Up to four slots of 9 KB the registers cost more than the waves they
    // make room for (FP64 48^4 a*b+c*d: 630 us, with registers 646); beyond,
    // values that stay with their wave move there (force term FP64 48^4: 1679
    // us in slots, 1090 with registers, 1437 on the one-lane kernel; FP32 855,
    // 517 and 560).
    if (pc.rows.nslots > 4)
        return &pc.rows_held;
    // Four slots: 12 waves per CU with the loads of 16 bytes per lane and row
    // are too few in single (FP32 20^4 a*b+c*d: 14.7 us against 11.5 on the
    // one-lane kernel, 48^4 trace(a*b*adj(c)*adj(d)) 283 against 259).
    if (pc.rows.nslots == 4 && arith == SU3_F32)
        return nullptr;
    // Three slots in single, 5 workgroups per CU, gain 4 to 10 % where they take
    // no more rounds than the one-lane kernel with its 12 waves per CU, and lose
    // more in calls of a few rounds where they take one more (c*a*b+0.5, 20^3 x
    // 24, two rounds, 11.5 us against 8.7 in one; 25, two and two, 11.5 and 12.6;
    // 24^4, three and two, 16.9 and 15.2).
    const int64_t lane_groups = (z->V + 63) / 64, lanes_at_once = 12 * (int64_t)f.cus;
    if (pc.rows.nslots == 3 && arith == SU3_F32 && groups < 3 * at_once &&
        (groups + at_once - 1) / at_once > (lane_groups + lanes_at_once - 1) / lanes_at_once)
        return nullptr;
    return &pc.rows;
}

// The launch of a program that nothing tuned or set (rows: its row form).
// Stores are nontemporal, loads too, except
// - where a lane-block's entry is less than a 128-byte line (FP32 AoSoA-8 32^4
//   a*b+c*d: 66.6 us against 72.9), and for AoS sites read entry by entry; below
//   64 bytes stores stay cached too (FP32 N_sub 2 22^4 a*adj(b): 13.3 us, with
//   nontemporal stores 35.4);
// - by rows from 80 to 150 MB (FP64 22^4 a*adj(b), 101 MB, three sets of fields
//   in turn: 17.4 us against 20.4).  Below, the loads of a call that is repeated
//   on the same fields are faster past the L2s (FP64 16^4 a*b+c*d, 47 MB, 8.5
//   us, cached 10.3), and as fast with sets in turn; above, the Infinity Cache
//   no longer holds them (FP64 26^4 a*adj(b) 35.4 and 33.1).  The one-lane kernel
//   never gains by it (FP32 20^4 a*b+c*d 10.1, cached 11.7);
// - AoS records, and programs without a matrix value, to 150 MB (FP64 48^3 x 24
//   a+b+a*b on real fields, 64 MB: 11.9 us against 12.6; FP32 36^4 a*conj(b)+a on
//   AoS complex ones 9.6 and 12.4; but in single 48^4 real ones, 64 MB: 13.0 us,
//   past the caches 10.4).
// One product alone streams best with 5 workgroups per CU beyond 600 MB (FP64
// 48^4 a*adj(b): 361 us, uncapped 405; 36^4 117 and 119; FP32 36^4, 363 MB, 59.7
// and 57.4); longer programs want them all.
static su3_launch program_launch(const su3_program *p, const su3_field *z,
                                 const su3_field *const *ops, int arith, const RowCode *rows,
                                 int form)
{
    su3_launch c = default_launch(SU3_EXPR_PROGRAM, arith, z->layout, z->lanes, z->V);
    int64_t bytes = (int64_t)z->bytes;
    for (int k = 0; k < p->code.nops; ++k)
        if (p->code.used >> k & 1)
            bytes += (int64_t)ops[k]->bytes;
    const int64_t MB = 1000 * 1000;
    const bool aos = z->layout == SU3_LAYOUT_AOS;
    const int64_t run = z->L * 2 * (int64_t)real_bytes(arith);
    const bool split = form == PF_MATRIX && (aos ? !rows : run < 128);
    const bool resident = bytes <= 150 * MB &&
                          (form != PF_MATRIX ? form == PF_SCALAR || arith == SU3_F64
                                             : aos || (rows && bytes > 80 * MB));
    c.nontemporal = split && !aos && run < 64 ? 0 : resident || split ? 2 : 3;
    if (aos && split && p->code.result_kind == FK_MATRIX) {
        // stores cached too (FP64 32^4 a*adj(b) 108 us, nontemporal 439); few
        // waves, whose records stay in the caches until they are done (93 us with
        // 4 per CU, and no program slower; FP32 48^4 a*b+c*d 442 with 8, uncapped
        // 501, but 24^4 32.5 and 29.9)
        c.nontemporal = 0;
        c.block = 64;
        c.occupancy = arith == SU3_F64 ? 4 : aos_bytes(z, arith) > kAosRowBytes ? 8 : 0;
    }
    if (rows && rows->n == 1 && bytes > 600 * MB && !aos)
        c.occupancy = 5;
    return c;
}

static su3_status launch_program_op(const su3_program *p, su3_field *z,
                                    const su3_field *const *ops, int arith,
                                    hipStream_t st,
                                    const su3_launch *forced = nullptr)
{
    const int form = p->code.real_only ? PF_REAL
                     : p->code.scalar_only ? PF_SCALAR
                                           : PF_MATRIX;
    // matrix-valued programs with a real or complex result (a trace) read
    // far more than they write, and are tuned under their own key
    const su3_expr key = form == PF_MATRIX && p->code.result_kind != FK_MATRIX
                             ? SU3_EXPR_PROGRAM_SCALAR
                             : SU3_EXPR_PROGRAM;
    const RowCode *rows = form == PF_MATRIX ? row_code(p, z, arith) : nullptr;
    su3_launch c;
    if (forced)
        c = *forced;
    else if (!tuned_program(key, arith, z, form, rows, &c))
        c = program_launch(p, z, ops, arith, rows, form);
    if (!forced && form != PF_MATRIX) {
        // the block and occupancy cap are the matrix kernel's (a wave of it
        // keeps up to 18 KB of loads in flight); a scalar-valued wave keeps
        // 2-4 KB per operand, so it runs in full workgroups, uncapped
        c.block = 256;
        c.occupancy = 0;
    }
    ProgArgs a;
    std::memset(&a, 0, sizeof a);
    a.z = z->ptr;
    a.gz = geom_of(z);
    a.zkind = (uint8_t)z->kind;
    a.zprec = (uint8_t)z->prec;
    for (int k = 0; k < p->code.nops; ++k) {
        a.op[k] = ops[k]->ptr;
        a.g[k] = geom_of(ops[k]);
        a.kind[k] = (uint8_t)ops[k]->kind;
        a.prec[k] = (uint8_t)ops[k]->prec;
    }
    a.xcd_remap = c.xcd_remap != 0;
    a.nops = (uint8_t)p->code.nops;
    a.ninstr = (uint8_t)p->code.ninstr;
    a.result = (uint8_t)p->code.result;
    a.used = (uint8_t)p->code.used;
    a.nsites = (int32_t)z->V;
    for (int t = 0; t < p->code.ninstr; ++t)
        a.ins[t] = p->code.ins[t];
    for (int k = 0; k < p->code.nimm; ++k) {
        a.imm[k][0] = p->code.imm[k][0];
        a.imm[k][1] = p->code.imm[k][1];
    }
    hipError_t e;
    if (rows) {
        RowArgs r;
        std::memset(&r, 0, sizeof r);
        r.z = a.z;
        r.gz = a.gz;
        r.zkind = a.zkind;
        r.zprec = a.zprec;
        std::memcpy(r.op, a.op, sizeof r.op);
        std::memcpy(r.g, a.g, sizeof r.g);
        std::memcpy(r.kind, a.kind, sizeof r.kind);
        std::memcpy(r.prec, a.prec, sizeof r.prec);
        std::memcpy(r.slot, rows->slot, sizeof r.slot);
        std::memcpy(r.imm, a.imm, sizeof r.imm);
        std::memcpy(r.ins, rows->ins, sizeof r.ins);
        r.nops = a.nops;
        r.used = a.used;
        r.ninstr = (uint8_t)rows->n;
        r.nslots = (uint8_t)rows->nslots;
        r.held = rows->held;
        r.aos = z->layout == SU3_LAYOUT_AOS;
        r.xcd_remap = a.xcd_remap;
        r.nsites = a.nsites;
        e = launch_program_rows(arith, row_sites_per_lane(z, arith), c.nontemporal,
                                occupancy_reserve(z->device, c.occupancy), r, st);
        if (e != hipSuccess)
            return hip_fail(e, "program kernel launch");
        return SU3_OK;
    }
    const int64_t per = program_sites_per_lane(arith, form);
    const int64_t lanes = (z->V + per - 1) / per;
    const int64_t grid = (lanes + c.block - 1) / c.block;
    e = launch_program(arith, form, p->code.nregs,
                                  c.nontemporal, c.block, (int)grid,
                                  occupancy_reserve(z->device, c.occupancy), a,
                                  st);
    if (e != hipSuccess)
        return hip_fail(e, "program kernel launch");
    return SU3_OK;
}

extern "C" su3_status su3_program_eval(const su3_program *p, su3_field *z,
                                       const su3_field *const *ops,
                                       int32_t n_ops, void *stream)
{
    if (!p || !z)
        return fail(SU3_ERR_INVALID_ARG, "program or output is NULL");
    if (n_ops != p->code.nops)
        return fail(SU3_ERR_INVALID_ARG, "the program takes %d operands, got %d",
                    p->code.nops, n_ops);
    if (n_ops > 0 && !ops)
        return fail(SU3_ERR_INVALID_ARG, "operand list is NULL");
    if (z->kind != p->code.result_kind)
        return fail(SU3_ERR_MISMATCH,
                    "the expression is %s-valued, the output a %s field",
                    kind_name(p->code.result_kind), kind_name(z->kind));
    if (z->prec == SU3_F16_F32ACC)
        return fail(SU3_ERR_UNSUPPORTED, "expressions take F64, F32 or C12 fields");
    const int arith = z->prec == SU3_F64 ? SU3_F64 : SU3_F32;
    for (int k = 0; k < n_ops; ++k) {
        const su3_field *o = ops[k];
        if (!o)
            return fail(SU3_ERR_INVALID_ARG, "operand %d is NULL", k);
        if (o->kind != p->kinds[k])
            return fail(SU3_ERR_MISMATCH,
                        "operand %d is a %s field, the program declared %s", k,
                        kind_name(o->kind), kind_name(p->kinds[k]));
        if (!same_geometry(o, z))
            return fail(SU3_ERR_MISMATCH,
                        "operand %d differs from the output in dims, layout, "
                        "lanes, virtual nodes or device", k);
        if (o->prec == SU3_F16_F32ACC)
            return fail(SU3_ERR_UNSUPPORTED,
                        "expressions take F64, F32 or C12 fields");
        if ((o->prec == SU3_F64) != (arith == SU3_F64))
            return fail(SU3_ERR_MISMATCH,
                        "operand %d: an expression is evaluated in one precision "
                        "(all fields F64, or all F32/C12)", k);
        if (overlaps(z, o) && !(z->ptr == o->ptr && z->bytes == o->bytes))
            return fail(SU3_ERR_ALIAS, "output partially overlaps operand %d", k);
    }
    if (z->prec == SU3_C12_F32 && !p->code.su3_closed)
        return fail(SU3_ERR_UNSUPPORTED,
                    "a compressed output needs an SU(3)-valued expression "
                    "(products, adjoints, transposes, conjugates of matrices)");
    return launch_program_op(p, z, ops, arith, static_cast<hipStream_t>(stream));
}

// ------------------------------------------------------- launch tuning

// The virtual-node split a tuning key of N_sub = lanes stands for: factors
// of two handed to t, z, y, x in turn where the extent allows.
static su3_status default_simd(const int32_t dims[4], int32_t lanes,
                               int32_t simd[4])
{
    if (!dims)
        return fail(SU3_ERR_INVALID_ARG, "dims is NULL");
    if (lanes < 1 || lanes > 256 || (lanes & (lanes - 1)) != 0)
        return fail(SU3_ERR_INVALID_ARG,
                    "virtual-node lanes %d must be a power of two <= 256",
                    lanes);
    for (int d = 0; d < 4; ++d)
        simd[d] = 1;
    int left = lanes;
    for (int round = 0; left > 1 && round < 64; ++round)
        for (int d = 3; d >= 0 && left > 1; --d)
            if (dims[d] > 0 && dims[d] % (2 * simd[d]) == 0) {
                simd[d] *= 2;
                left /= 2;
            }
    if (left > 1)
        return fail(SU3_ERR_INVALID_ARG,
                    "dims cannot be split into %d virtual nodes", lanes);
    return SU3_OK;
}

static su3_status key_of(su3_expr expr, su3_precision prec, su3_layout layout,
                         int32_t lanes, const int32_t dims[4], Key *k,
                         Shape *shape)
{
    if ((expr < SU3_EXPR_MUL || expr > SU3_EXPR_PROGRAM_SCALAR) && !is_batch_key(expr))
        return fail(SU3_ERR_INVALID_ARG, "unknown expression %d", expr);
    const int base = is_batch_key(expr) ? expr - SU3_EXPR_BATCH : (int)expr;
    if ((expr == SU3_EXPR_PROGRAM || expr == SU3_EXPR_PROGRAM_SCALAR) && prec != SU3_F64 &&
        prec != SU3_F32)
        return fail(SU3_ERR_UNSUPPORTED,
                    "expression programs evaluate in F64 or F32");
    if (expr == SU3_EXPR_DSLASH && prec == SU3_F16_F32ACC)
        return fail(SU3_ERR_UNSUPPORTED,
                    "Dslash links are stored in F64, F32 or C12");
    int32_t simd[4] = {1, 1, 1, 1};
    if (layout == SU3_LAYOUT_VNODE) {
        su3_status st = default_simd(dims, lanes, simd);
        if (st != SU3_OK)
            return st;
    }
    Shape s;
    su3_status st = make_shape(dims, prec, layout, lanes, &s, KIND_MATRIX,
                               layout == SU3_LAYOUT_VNODE ? simd : nullptr);
    if (st != SU3_OK)
        return st;
    if (prec == SU3_C12_F32 &&
        (base == SU3_EXPR_MULADD || base == SU3_EXPR_ADD ||
         base == SU3_EXPR_APB_AB))
        return fail(SU3_ERR_UNSUPPORTED,
                    "the two-row compressed form supports MUL and MUL3 only");
    *k = Key(expr, prec, layout,
             layout == SU3_LAYOUT_AOSOA || layout == SU3_LAYOUT_VNODE ? lanes : 0,
             vbucket(s.V));
    if (shape)
        *shape = s;
    return SU3_OK;
}

extern "C" su3_status su3_launch_get(su3_expr expr, su3_precision prec,
                                     su3_layout layout, int32_t lanes,
                                     const int32_t dims[4], su3_launch *out)
{
    if (!out)
        return fail(SU3_ERR_INVALID_ARG, "out is NULL");
    Key k;
    Shape s;
    su3_status st = key_of(expr, prec, layout, lanes, dims, &k, &s);
    if (st != SU3_OK)
        return st;
    if (tuned_launch(expr, prec, layout, std::get<3>(k), s.V, out))
        return SU3_OK;
    *out = default_launch(expr, prec, layout, std::get<3>(k), s.V);
    if (expr == SU3_EXPR_DSLASH) {
        int32_t simd[4] = {1, 1, 1, 1};
        if (layout == SU3_LAYOUT_VNODE)
            (void)default_simd(dims, lanes, simd);  // checked by key_of
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess)
            dev = 0;
        *out = default_dslash(prec, layout, s.L, dims, simd, device_cus(dev));
    }
    return SU3_OK;
}

extern "C" su3_status su3_launch_set(su3_expr expr, su3_precision prec,
                                     su3_layout layout, int32_t lanes,
                                     const int32_t dims[4],
                                     const su3_launch *cfg)
{
    if (!cfg)
        return fail(SU3_ERR_INVALID_ARG, "cfg is NULL");
    Key k;
    su3_status st = key_of(expr, prec, layout, lanes, dims, &k, nullptr);
    if (st != SU3_OK)
        return st;
    st = check_launch(*cfg, layout, expr);
    if (st != SU3_OK)
        return st;
    std::lock_guard<std::mutex> lk(g_tune_mu);
    load_cache_locked();
    g_tuned[k] = *cfg;
    std::get<0>(k) += kOtherForm;
    g_tuned.erase(k);
    return SU3_OK;
}

extern "C" su3_status su3_launch_reset(void)
{
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tuned.clear();
    g_cache_loaded = true;  // do not reload the file
    return SU3_OK;
}

// Candidate launches of the autotuner's sweep for a site-local expression
// (or a shift: expr CSHIFT / MUL_SHIFTED, one site per lane, blocks up to
// 256).  Persistent grid-stride launches are kept as a few samples only: on
// this hardware one-shot grids stream writes far better.
static std::vector<su3_launch> candidates(int layout, int expr, int prec)
{
    std::vector<su3_launch> out;
    su3_launch c;
    c.persistent = 0;
    c.xcd_remap = 0;
    c.lds_stage = 0;
    c.tile_sites = 4096;
    c.sites_per_lane = 0;
    if (layout == SU3_LAYOUT_AOS) {
        for (int b : {64, 128, 256})
            for (int nt : {0, 2, 3, 7})
                for (int lds = 0; lds < 2; ++lds)
                    for (int occ : {0, 3, 5, 8}) {
                        if (lds ? b > 128 : occ || nt == 2)
                            continue;
                        c.block = b;
                        c.nontemporal = nt;
                        c.lds_stage = lds;
                        c.occupancy = occ;
                        c.schedule = 0;
                        out.push_back(c);
                    }
        return out;
    }
    const bool site = expr >= SU3_EXPR_MUL && expr <= SU3_EXPR_APB_AB;
    // sites per lane: the natural count, and twice it for the product
    std::vector<int> spl = {0};
    if (expr == SU3_EXPR_MUL && prec != SU3_F16_F32ACC)
        spl.push_back(2 * natural_sites(prec, expr));
    for (int S : spl)
        for (int b : {64, 128, 256})
            for (int occ : {0, 2, 3, 4, 5, 6, 8})
                for (int sched : {0, 1})
                    for (int nt : {0, 2, 3, 7})
                        for (int x : {0, 1}) {
                            if (S && (nt != 7 || x))
                                continue;  // wide lanes: streaming stores only
                            c.block = b;
                            c.occupancy = occ;
                            c.schedule = sched;
                            c.nontemporal = nt;
                            c.xcd_remap = x;
                            c.sites_per_lane = S;
                            out.push_back(c);
                        }
    c.xcd_remap = 0;
    c.sites_per_lane = 0;
    // 512- and 1024-lane workgroups (streaming stores), at most 32 waves
    // per compute unit
    if (site)
        for (int b : {512, 1024})
            for (int occ : {0, 1, 2, 3, 4})
                for (int sched : {0, 1}) {
                    if (occ * (b / 64) > 32)
                        continue;
                    c.block = b;
                    c.occupancy = occ;
                    c.schedule = sched;
                    c.nontemporal = 7;
                    out.push_back(c);
                }
    for (int b : {64, 256})
        for (int p : {2, 4})
            for (int sched : {0, 1}) {
                c.block = b;
                c.persistent = p;
                c.occupancy = 0;
                c.schedule = sched;
                c.nontemporal = 7;
                out.push_back(c);
            }
    return out;
}

// Candidates for the Wilson hopping kernel: t-slices per lane (1: one
// site per lane, in index order or in site tiles), block, occupancy cap,
// XCD remapping (nontemporal stores, cached spinor loads); LDS-tiled
// walks of every tile that fits the precision (cbytes per complex entry)
// and the lattice's x extent lx (whole-row tiles).
static std::vector<su3_launch> dslash_candidates(int cbytes, int lx, int nsub)
{
    std::vector<su3_launch> out;
    su3_launch c = default_launch(SU3_EXPR_DSLASH, SU3_F64, SU3_LAYOUT_SOA, 0, 0);
    c.nontemporal = 2;
    // virtual nodes: one site per lane in index order, or row tiles
    for (int walk : {1, 4, 8})
        for (int sched = 0; sched <= (walk == 1 && nsub == 1 ? 3 : 0); ++sched)
            for (int b : {64, 128, 256})
                for (int occ : {0, 2, 3, 4, 6})
                    for (int x : {0, 1}) {
                        if (nsub > 1 && walk > 1)
                            continue;
                        c.tile_sites = walk;
                        c.schedule = sched;
                        c.block = b;
                        c.occupancy = occ;
                        c.xcd_remap = x;
                        out.push_back(c);
                    }
    // one wave per hop
    c.tile_sites = 1;
    c.schedule = 0;
    c.block = 64;
    c.occupancy = 0;
    c.sites_per_lane = 8;
    for (int x : {0, 1}) {
        c.xcd_remap = x;
        out.push_back(c);
    }
    c.sites_per_lane = 0;
    // LDS-tiled walks: every tile shape that fits this spinor precision and
    // lattice (cached loads; nontemporal stores), with and without a halo
    for (int sched = 4; sched <= 28; ++sched)
        for (int b : {128, 256, 512}) {
            LdsShape sh;
            if (!lds_shape(sched, b, cbytes, lx, nsub, sh) || (sched >= 9 && b != 256))
                continue;
            for (int walk : {4, 5, 6, 7, 8, 12, 16, 48})
                for (int x : {0, 1, 2}) {
                    c.tile_sites = walk;
                    c.schedule = sched;
                    c.block = b;
                    c.occupancy = 0;
                    c.xcd_remap = x;
                    out.push_back(c);
                }
            // k workgroups per CU, equal shares of the (tile, slice) pairs
            for (int k : {1, 2, 3}) {
                c.tile_sites = 1;
                c.schedule = sched;
                c.block = b;
                c.occupancy = 0;
                c.xcd_remap = 0;
                c.nontemporal = 2;
                c.persistent = k;
                out.push_back(c);
                c.persistent = 0;
            }
        }
    return out;
}

// Candidates for a program: occupancy cap and nontemporal bits, and on one
// lane per site the block (workgroups by rows are three waves).
static std::vector<su3_launch> program_candidates(bool by_rows)
{
    std::vector<su3_launch> out;
    su3_launch c = default_launch(SU3_EXPR_PROGRAM, SU3_F64, SU3_LAYOUT_SOA, 0, 0);
    for (int b : {64, 128, 256})
        for (int occ : {0, 2, 3, 4, 5, 6, 8})
            for (int nt : {0, 2, 3}) {
                if (by_rows && b != 128)
                    continue;
                c.block = b;
                c.occupancy = occ;
                c.nontemporal = nt;
                out.push_back(c);
            }
    return out;
}

// Median time (microseconds) of `reps` launches after `warm` warm-ups, each
// launch bracketed by its own events.
template <class F>
static su3_status time_launch(F launch, hipStream_t st, int warm, int reps,
                              double *us)
{
    for (int i = 0; i < warm; ++i) {
        su3_status s = launch();
        if (s != SU3_OK)
            return s;
    }
    std::vector<hipEvent_t> ev(2 * reps);
    for (auto &e : ev)
        HIP_TRY(hipEventCreate(&e), "hipEventCreate");
    su3_status result = SU3_OK;
    for (int i = 0; i < reps && result == SU3_OK; ++i) {
        (void)hipEventRecord(ev[2 * i], st);
        result = launch();
        (void)hipEventRecord(ev[2 * i + 1], st);
    }
    hipError_t e = hipStreamSynchronize(st);
    std::vector<double> t;
    for (int i = 0; i < reps && result == SU3_OK && e == hipSuccess; ++i) {
        float ms = 0;
        if (hipEventElapsedTime(&ms, ev[2 * i], ev[2 * i + 1]) == hipSuccess)
            t.push_back(ms * 1000.0);
    }
    for (auto &x : ev)
        (void)hipEventDestroy(x);
    if (result != SU3_OK)
        return result;
    if (e != hipSuccess)
        return hip_fail(e, "autotune sync");
    if (t.empty())
        return fail(SU3_ERR_HIP, "no timing recorded");
    std::sort(t.begin(), t.end());
    *us = t[t.size() / 2];
    return SU3_OK;
}

static su3_status autotune_impl(su3_expr expr, su3_precision prec,
                                su3_layout layout, int32_t lanes,
                                const int32_t dims[4], void *stream,
                                su3_launch *best, double *best_us)
{
    if (is_batch_key(expr))
        return fail(SU3_ERR_INVALID_ARG,
                    "batch keys are tuned by su3_batch_autotune");
    Key k;
    Shape s;
    su3_status st = key_of(expr, prec, layout, lanes, dims, &k, &s);
    if (st != SU3_OK)
        return st;
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const bool dslash = expr == SU3_EXPR_DSLASH;
    // Dslash: f[0] out, f[1] in (spinors), f[2..5] links
    const int nops = expr == SU3_EXPR_CSHIFT ? 1
                     : dslash              ? 5
                                           : operands_of(expr);
    int32_t simd[4] = {1, 1, 1, 1};
    if (layout == SU3_LAYOUT_VNODE)
        (void)default_simd(dims, lanes, simd);  // checked by key_of
    // Operand sets: one, or -- when a set of 64 to 512 MiB fits twice into
    // the 256 MiB Infinity Cache -- as many as make 1 GiB, launched in
    // rotation, so that each timed launch finds its operands in HBM (tuning
    // on one cache-resident set picked launches up to 23 % slower cold at
    // 32^4).  Below 64 MiB launches are short enough that per-launch timing
    // of rotating sets misleads (16^4: the hot choice is faster hot and
    // cold), so they keep one set.
    std::vector<std::array<su3_field *, 6>> sets(1);
    sets[0].fill(nullptr);
    for (size_t n = 0; n < sets.size() && st == SU3_OK; ++n) {
        su3_field **f = sets[n].data();
        size_t set_bytes = 0;
        for (int i = 0; i <= nops && st == SU3_OK; ++i) {
            const bool spinor = dslash && i < 2;
            const int fp = spinor ? spinor_prec_of_links(prec) : prec;
            const int kind = spinor                                          ? KIND_SPINOR
                             : i == 0 && expr == SU3_EXPR_PROGRAM_SCALAR ? KIND_COMPLEX
                                                                          : KIND_MATRIX;
            if (layout == SU3_LAYOUT_VNODE)
                st = alloc_of_kind(&f[i], dims, fp, layout, 0, kind, simd);
            else
                st = alloc_of_kind(&f[i], dims, fp, layout, lanes, kind);
            if (st == SU3_OK) {
                set_bytes += f[i]->bytes;
                // a non-zero bit pattern (finite in every precision)
                hipError_t e = hipMemsetD32Async((hipDeviceptr_t)f[i]->ptr,
                                                 0x3c003c00u, f[i]->bytes / 4, hs);
                if (e != hipSuccess)
                    st = hip_fail(e, "fill");
            }
        }
        if (n == 0 && st == SU3_OK && set_bytes < ((size_t)512 << 20) &&
            set_bytes >= ((size_t)64 << 20)) {
            const size_t want = (((size_t)1 << 30) + set_bytes - 1) / set_bytes;
            sets.resize(std::max<size_t>(2, want));
            for (size_t m = 1; m < sets.size(); ++m)
                sets[m].fill(nullptr);
        }
    }
    size_t turn = 0;
    // the call's own launch is the first candidate
    su3_launch win = dslash ? default_dslash(prec, layout, s.L, dims, simd,
                                             device_cus(sets[0][0] ? sets[0][0]->device : 0))
                            : default_launch(expr, prec, layout, std::get<3>(k), s.V);
    double win_us = 1e300;
    // expression programs are timed on the streaming product a*b, those
    // with a scalar result on the trace of a product; where programs of four
    // operands run in the other form, on one lane per site, these too
    const bool program = is_program_key(expr), traced = expr == SU3_EXPR_PROGRAM_SCALAR;
    su3_program prog, prog4;
    const int kinds[4] = {KIND_MATRIX, KIND_MATRIX, KIND_MATRIX, KIND_MATRIX};
    char err[128];
    if (st == SU3_OK && program &&
        (!compile_program(traced ? "trace(a*adj(b))" : "a*b", 2, kinds, &prog.code, err,
                          sizeof err) ||
         !compile_program(traced ? "trace(a*b*adj(c)*adj(d))" : "a*b+c*d", 4, kinds,
                          &prog4.code, err, sizeof err)))
        st = fail(SU3_ERR_HIP, "internal program: %s", err);
    const auto sweep = [&](const std::vector<su3_launch> &list, const su3_program *pr,
                           su3_launch *win, double *win_us) {
        const su3_field *f0 = sets[0][0];
        for (su3_launch c : list) {
            if (program || expr == SU3_EXPR_CSHIFT || expr == SU3_EXPR_MUL_SHIFTED)
                c.xcd_remap = default_launch(expr, prec, layout, f0->lanes, f0->V).xcd_remap;
            double us = 0;
            su3_status r = time_launch(
                [&]() {
                    su3_field *const *f = sets[turn++ % sets.size()].data();
                    const su3_field *ops[4] = {f[1], f[2], f[3], f[4]};
                    su3_field *links[4] = {f[2], f[3], f[4], f[5]};
                    if (dslash)
                        return launch_dslash_op(f[0], links, f[1], stream, &c);
                    if (program)
                        return launch_program_op(pr, f[0], ops, prec, hs, &c);
                    if (expr == SU3_EXPR_CSHIFT)
                        return launch_shift_op(0, f[0], nullptr, f[1], 1, 1,
                                               stream, &c);
                    if (expr == SU3_EXPR_MUL_SHIFTED)
                        return launch_shift_op(1, f[0], f[1], f[2], 1, 1,
                                               stream, &c);
                    return launch_item(f[0], expr, ops, nops, c, hs);
                },
                hs, 3, 10, &us);
            if (r != SU3_OK) {
                (void)hipGetLastError();
                continue;  // a launch shape the device refused
            }
            if (us < *win_us) {
                *win_us = us;
                *win = c;
            }
        }
    };
    // the candidates of a program, its untuned launch first
    const auto program_list = [&](const su3_program *pr) {
        su3_field *const *f = sets[0].data();
        const su3_field *ops[4] = {f[1], f[2], f[3], f[4]};
        const RowCode *rows = row_code(pr, f[0], prec);
        std::vector<su3_launch> list = program_candidates(rows != nullptr);
        list.insert(list.begin(), program_launch(pr, f[0], ops, prec, rows, PF_MATRIX));
        for (su3_launch &c : list)
            c.schedule = 1;  // for its form only
        return list;
    };
    if (st == SU3_OK) {
        const su3_field *f0 = sets[0][0];
        std::vector<su3_launch> list =
            dslash ? dslash_candidates(2 * f0->rbytes, f0->dims[0] / f0->simd[0],
                                       layout == SU3_LAYOUT_VNODE ? (int)f0->L : 1)
            : program ? program_list(&prog)
                      : candidates(layout, expr, prec);
        if (expr == SU3_EXPR_CSHIFT)  // a copy has no row phases
            list.erase(std::remove_if(list.begin(), list.end(),
                                      [](const su3_launch &c) { return c.schedule != 0; }),
                       list.end());
        if (!program)
            list.insert(list.begin(), win);
        sweep(list, &prog, &win, &win_us);
        if (win_us >= 1e300)
            st = fail(SU3_ERR_HIP, "no candidate launch ran");
    }
    // the other form needs two operands more; without room for them it keeps
    // its untuned launch
    su3_launch win4 = win;
    double win4_us = 1e300;
    if (st == SU3_OK && program && row_code(&prog, sets[0][0], prec) &&
        !row_code(&prog4, sets[0][0], prec)) {
        bool room = true;
        for (auto &set : sets)
            for (int i = 3; i <= 4 && room; ++i) {
                room = (layout == SU3_LAYOUT_VNODE
                            ? alloc_of_kind(&set[i], dims, prec, layout, 0, KIND_MATRIX, simd)
                            : alloc_of_kind(&set[i], dims, prec, layout, lanes, KIND_MATRIX)) ==
                           SU3_OK &&
                       hipMemsetD32Async((hipDeviceptr_t)set[i]->ptr, 0x3c003c00u,
                                         set[i]->bytes / 4, hs) == hipSuccess;
            }
        if (room)
            sweep(program_list(&prog4), &prog4, &win4, &win4_us);
        else
            (void)hipGetLastError();
    }
    for (auto &set : sets)
        for (su3_field *fi : set)
            su3_field_free(fi);
    if (st != SU3_OK)
        return st;
    Key k4 = k;
    std::get<0>(k4) += kOtherForm;
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        load_cache_locked();
        g_tuned[k] = win;
        if (win4_us < 1e300)
            g_tuned[k4] = win4;
        else if (program)
            g_tuned.erase(k4);
    }
    append_cache(k, win, win_us);
    if (win4_us < 1e300)
        append_cache(k4, win4, win4_us);
    if (best)
        *best = win;
    if (best_us)
        *best_us = win_us;
    return SU3_OK;
}

extern "C" su3_status su3_autotune(su3_expr expr, su3_precision prec,
                                   su3_layout layout, int32_t lanes,
                                   const int32_t dims[4], void *stream,
                                   su3_launch *best)
{
    return autotune_impl(expr, prec, layout, lanes, dims, stream, best, nullptr);
}

extern "C" su3_status su3_layout_recommend(su3_expr expr, su3_precision prec,
                                           const int32_t dims[4], void *stream,
                                           su3_layout *layout, int32_t *lanes,
                                           su3_launch *best, double *us)
{
    if (expr < SU3_EXPR_MUL || expr > SU3_EXPR_APB_AB)
        return fail(SU3_ERR_INVALID_ARG,
                    "layouts are recommended for the site-local expressions");
    if (!layout || !lanes)
        return fail(SU3_ERR_INVALID_ARG, "layout or lanes is NULL");
    // the candidates: SoA and AoSoA with every lane count; each tuned (and
    // its launch kept, as su3_autotune does); the fastest tuned time wins,
    // ties to the earlier (larger contiguous runs first)
    const struct { su3_layout lay; int32_t L; } cand[] = {
        {SU3_LAYOUT_SOA, 0}, {SU3_LAYOUT_AOSOA, 64}, {SU3_LAYOUT_AOSOA, 32},
        {SU3_LAYOUT_AOSOA, 16}, {SU3_LAYOUT_AOSOA, 8}};
    double win_us = 1e300;
    for (const auto &c : cand) {
        su3_launch l;
        double t = 0;
        su3_status st = autotune_impl(expr, prec, c.lay, c.L, dims, stream, &l, &t);
        if (st != SU3_OK)
            return st;
        if (t < win_us) {
            win_us = t;
            *layout = c.lay;
            *lanes = c.L;
            if (best)
                *best = l;
        }
    }
    if (us)
        *us = win_us;
    return SU3_OK;
}

// ------------------------------------------------------------ batches

// The items of a batch as the kernel reads them, validated (each item by
// su3_fused_eval's rules; batch-level rules here), with the tile table
// of the launch `cfg`: forced (the autotuner), else the tuned (or default)
// setting of the batch key (SU3_EXPR_BATCH + leading expression, leading
// item's precision, layout, lanes) at the total volume; the default is that
// of the precision of most bytes, double's where it has three quarters of them
// (64 lattices of two-row links with half their bytes in double: 953 us with
// one wave per tile, 1041 with two; three quarters in double 763 and 740).
struct BatchPlan {
    std::vector<BatchItem> items;
    int mode;
    int device;
    int64_t ntiles;
    su3_launch cfg;
};

static su3_launch default_batch(const su3_expr *exprs, su3_field *const *z, int32_t n)
{
    int64_t sites = 0, bytes[4] = {0, 0, 0, 0}, all = 0;
    for (int i = 0; i < n; ++i) {
        const int64_t b = site_call_bytes(exprs[i], z[i]->prec, z[i]->V);
        sites += z[i]->V;
        bytes[z[i]->prec] += b;
        all += b;
    }
    int prec = SU3_F64;
    if (4 * bytes[SU3_F64] < 3 * all) {
        prec = SU3_F32;
        for (int q : {SU3_F16_F32ACC, SU3_C12_F32})
            if (bytes[q] > bytes[prec])
                prec = q;
    }
    return default_launch(SU3_EXPR_BATCH + exprs[0], prec, z[0]->layout, z[0]->lanes, sites);
}

static su3_status plan_batch(const su3_expr *exprs, su3_field *const *z,
                             const su3_field *const *ops, int32_t n,
                             const su3_launch *forced, BatchPlan *plan)
{
    if (!exprs || !z || !ops)
        return fail(SU3_ERR_INVALID_ARG, "NULL argument");
    if (n <= 0)
        return fail(SU3_ERR_INVALID_ARG, "batch needs at least one item");
    std::vector<BatchItem> &items = plan->items;
    items.assign(n, BatchItem());
    int mode = 0;
    int64_t total_sites = 0;
    int dev = -1;
    for (int i = 0; i < n; ++i) {
        const int nops = (exprs[i] >= SU3_EXPR_MUL && exprs[i] <= SU3_EXPR_APB_AB)
                             ? operands_of(exprs[i])
                             : 0;
        su3_status st = validate_item(z[i], exprs[i], ops + 4 * i, nops);
        if (st != SU3_OK)
            return fail(st, "batch item %d: %s", i, g_last_error.c_str());
        for (int k = nops; k < 4; ++k)
            if (ops[4 * i + k])
                return fail(SU3_ERR_INVALID_ARG,
                            "batch item %d: unused operand slot %d not NULL",
                            i, k);
        if (dev < 0)
            dev = z[i]->device;
        else if (z[i]->device != dev)
            return fail(SU3_ERR_MISMATCH, "batch items on different devices");
        if (z[i]->layout == SU3_LAYOUT_AOS ||
            (z[i]->layout == SU3_LAYOUT_VNODE && z[i]->L < 4))
            return fail(SU3_ERR_UNSUPPORTED,
                        "batch item %d: batches take SoA, AoSoA or "
                        "virtual-node fields with N_sub >= 4", i);
        BatchItem &it = items[i];
        std::memset(&it, 0, sizeof it);
        it.z = z[i]->ptr;
        for (int k = 0; k < nops; ++k)
            it.op[k] = ops[4 * i + k]->ptr;
        it.g = geom_of(z[i]);
        it.nsites = (int32_t)z[i]->V;
        it.prec = z[i]->prec;
        it.expr = exprs[i];
        if (!(exprs[i] == SU3_EXPR_MUL &&
              (z[i]->prec == SU3_F64 || z[i]->prec == SU3_C12_F32)))
            mode = 1;
        total_sites += z[i]->V;
    }
    su3_launch cfg;
    if (forced) {
        cfg = *forced;
    } else if (!tuned_launch(SU3_EXPR_BATCH + exprs[0], z[0]->prec, z[0]->layout, z[0]->lanes,
                             total_sites, &cfg)) {
        cfg = default_batch(exprs, z, n);
    }
    const int T = cfg.tile_sites;
    // tile table: item i owns ceil(V_i / T) tiles starting at the exclusive
    // prefix sum of its predecessors' counts
    int64_t ntiles = 0;
    for (int i = 0; i < n; ++i) {
        items[i].tile_start = (int32_t)ntiles;
        ntiles += (z[i]->V + T - 1) / T;
        if (ntiles >= ((int64_t)1 << 31))
            return fail(SU3_ERR_INVALID_ARG, "too many tiles");
    }
    plan->mode = mode;
    plan->device = dev;
    plan->ntiles = ntiles;
    plan->cfg = cfg;
    return SU3_OK;
}

// Workgroups of a batch launch: k per CU for a persistent grid (at most one
// per tile), else one per tile.
static int32_t batch_grid(const BatchPlan &p)
{
    return p.cfg.persistent > 0
               ? (int32_t)std::min<int64_t>(p.ntiles, (int64_t)p.cfg.persistent *
                                                          device_cus(p.device))
               : (int32_t)p.ntiles;
}

static su3_status batch_create(su3_batch **out, const su3_expr *exprs,
                               su3_field *const *z, const su3_field *const *ops,
                               int32_t n, void *stream, const su3_launch *forced)
{
    if (!out)
        return fail(SU3_ERR_INVALID_ARG, "NULL argument");
    BatchPlan plan;
    su3_status pst = plan_batch(exprs, z, ops, n, forced, &plan);
    if (pst != SU3_OK)
        return pst;
    const std::vector<BatchItem> &items = plan.items;
    const int mode = plan.mode, dev = plan.device;
    const int64_t ntiles = plan.ntiles;
    const su3_launch cfg = plan.cfg;
    su3_batch *b = new su3_batch();
    b->nitems = n;
    b->ntiles = (int32_t)ntiles;
    b->mode = mode;
    b->cfg = cfg;
    b->device = dev;
    // persistent k > 0: k workgroups per CU draw the tiles from a ticket
    // counter; 0: one workgroup per tile
    b->grid = batch_grid(plan);
    hipStream_t hs = static_cast<hipStream_t>(stream);
    // the counter (16 bytes, zero) and the item table in one allocation
    const size_t bytes = 16 + sizeof(BatchItem) * n;
    std::vector<unsigned char> image(bytes, 0);
    std::memcpy(image.data() + 16, items.data(), sizeof(BatchItem) * n);
    hipError_t e = hipMalloc(&b->d_mem, bytes);
    if (e == hipSuccess) {
        b->d_queue = cfg.persistent > 0 ? static_cast<unsigned long long *>(b->d_mem)
                                        : nullptr;
        b->d_items = reinterpret_cast<BatchItem *>(static_cast<unsigned char *>(b->d_mem) + 16);
        e = hipMemcpyAsync(b->d_mem, image.data(), bytes, hipMemcpyHostToDevice, hs);
    }
    if (e == hipSuccess)
        e = hipStreamSynchronize(hs);
    if (e == hipSuccess && b->d_queue)
        e = hipEventCreateWithFlags(&b->last, hipEventDisableTiming);
    if (e != hipSuccess) {
        su3_status r = hip_fail(e, "batch create");
        su3_batch_destroy(b);
        return r;
    }
    *out = b;
    return SU3_OK;
}

extern "C" su3_status su3_batch_create(su3_batch **out, const su3_expr *exprs,
                                       su3_field *const *z,
                                       const su3_field *const *ops, int32_t n,
                                       void *stream)
{
    return batch_create(out, exprs, z, ops, n, stream, nullptr);
}

// ------------------------------------------- allocation-free batches

// Scratch of su3_batch_run: the persistent grid's ticket counter (bytes
// 0..15) and up to kRunMaxItems item records (from byte 256).  A
// file-scope device array: every device the library runs on holds one
// copy for the life of the process, at its own address, which host code
// reaches only through run_scratch() (the array's name is a host-side
// stand-in, not a device address).
static const int kRunMaxItems = 1024;
static const size_t kRunScratchBytes = 256 + sizeof(BatchItem) * kRunMaxItems;
static __device__ __align__(256) unsigned char scratch[kRunScratchBytes];

// Device address of `scratch` on device `dev` (the current device),
// looked up once per device.
static su3_status run_scratch(int dev, unsigned char **out)
{
    static std::mutex mu;
    static unsigned char *ptrs[64];
    if (dev < 0 || dev >= 64)
        return fail(SU3_ERR_UNSUPPORTED, "device %d beyond the 64 the library serves", dev);
    std::lock_guard<std::mutex> lk(mu);
    if (!ptrs[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess)
            return hip_fail(e, "hipGetSymbolAddress(scratch)");
        if (!p)
            return fail(SU3_ERR_HIP, "no device address for the batch scratch");
        ptrs[dev] = static_cast<unsigned char *>(p);
    }
    *out = ptrs[dev];
    return SU3_OK;
}

extern "C" su3_status su3_batch_run(const su3_expr *exprs, su3_field *const *z,
                                    const su3_field *const *ops, int32_t n,
                                    void *stream)
{
    if (n > kRunMaxItems)
        return fail(SU3_ERR_INVALID_ARG,
                    "su3_batch_run takes at most %d items (got %d); "
                    "su3_batch_create takes any number", kRunMaxItems, n);
    BatchPlan plan;
    su3_status st = plan_batch(exprs, z, ops, n, nullptr, &plan);
    if (st != SU3_OK)
        return st;
    int cur = -1;
    HIP_TRY(hipGetDevice(&cur), "hipGetDevice");
    if (cur != plan.device)
        return fail(SU3_ERR_MISMATCH,
                    "the batch's fields are on device %d, the current device is %d",
                    plan.device, cur);
    unsigned char *sp = nullptr;
    st = run_scratch(plan.device, &sp);
    if (st != SU3_OK)
        return st;
    unsigned long long *queue =
        plan.cfg.persistent > 0 ? reinterpret_cast<unsigned long long *>(sp) : nullptr;
    BatchItem *items = reinterpret_cast<BatchItem *>(sp + 256);
    hipStream_t hs = static_cast<hipStream_t>(stream);
    hipError_t e = launch_put_items(items, plan.items.data(), n, queue, hs);
    if (e == hipSuccess)
        e = launch_batch(plan.mode, items, n, (int32_t)plan.ntiles,
                         plan.cfg.tile_sites, plan.cfg.nontemporal, plan.cfg.schedule,
                         plan.cfg.block, batch_grid(plan),
                         occupancy_reserve(plan.device, plan.cfg.occupancy), queue, hs);
    if (e != hipSuccess)
        return hip_fail(e, "batch run launch");
    return SU3_OK;
}

extern "C" su3_status su3_batch_launch(su3_batch *b, void *stream)
{
    if (!b)
        return fail(SU3_ERR_INVALID_ARG, "batch is NULL");
    hipStream_t hs = static_cast<hipStream_t>(stream);
    unsigned long long *queue = b->d_queue;
    if (queue) {
        // nothing orders a captured launch against others of this batch when
        // its graph runs: it strides over the tiles without the counter
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(hs, &capture) != hipSuccess) {
            (void)hipGetLastError();
            queue = nullptr;
        } else if (capture != hipStreamCaptureStatusNone) {
            queue = nullptr;
        }
    }
    std::unique_lock<std::mutex> lock(b->mu, std::defer_lock);
    if (queue) {
        lock.lock();
        HIP_TRY(hipStreamWaitEvent(hs, b->last, 0), "batch order");
    }
    // one kernel: launched directly it costs 2.8 us of a stream's time, as a
    // graph of one node 15.3 us (either replayed back to back)
    hipError_t e =
        launch_batch(b->mode, b->d_items, b->nitems, b->ntiles, b->cfg.tile_sites,
                     b->cfg.nontemporal, b->cfg.schedule, b->cfg.block, b->grid,
                     occupancy_reserve(b->device, b->cfg.occupancy), queue, hs);
    if (e == hipSuccess && queue)
        e = hipEventRecord(b->last, hs);
    if (e != hipSuccess)
        return hip_fail(e, "batch launch");
    return SU3_OK;
}

extern "C" su3_status su3_batch_destroy(su3_batch *b)
{
    if (!b)
        return SU3_OK;
    if (b->last)
        (void)hipEventDestroy(b->last);
    if (b->d_mem)
        (void)hipFree(b->d_mem);
    delete b;
    return SU3_OK;
}

// Candidate launches of the batch autotuner: for each tile size, one-shot
// grids (one workgroup per tile: blocks of 64 or 128, occupancy caps,
// schedules, cached, nontemporal or streaming) and persistent grids drawing
// the tiles from the ticket counter (blocks of 64 or 256, 2-8 workgroups
// per CU, streaming stores).
static std::vector<su3_launch> batch_candidates()
{
    std::vector<su3_launch> out;
    su3_launch c;
    c.xcd_remap = 0;
    c.lds_stage = 0;
    c.sites_per_lane = 0;
    for (int tile : {64, 128, 256, 512, 2048, 8192}) {
        c.tile_sites = tile;
        c.persistent = 0;
        for (int b : {64, 128})
            for (int occ : {0, 4, 6})
                for (int sched : {0, 1})
                    for (int nt : {0, 3, 7}) {
                        c.block = b;
                        c.occupancy = occ;
                        c.schedule = sched;
                        c.nontemporal = nt;
                        out.push_back(c);
                    }
        c.occupancy = 0;
        c.nontemporal = 7;
        for (int b : {64, 256})
            for (int k : {2, 4, 8})
                for (int sched : {0, 1}) {
                    c.block = b;
                    c.persistent = k;
                    c.schedule = sched;
                    out.push_back(c);
                }
    }
    return out;
}

extern "C" su3_status su3_batch_autotune(const su3_expr *exprs,
                                         su3_field *const *z,
                                         const su3_field *const *ops,
                                         int32_t n, void *stream,
                                         su3_launch *best)
{
    if (!exprs || !z || !ops || n <= 0 || !z[0])
        return fail(SU3_ERR_INVALID_ARG, "NULL argument or empty batch");
    hipStream_t hs = static_cast<hipStream_t>(stream);
    std::vector<su3_launch> list = batch_candidates();
    BatchPlan plan;
    su3_status valid = plan_batch(exprs, z, ops, n, &list[0], &plan);
    if (valid != SU3_OK)
        return valid;  // nothing tuned
    int64_t total = 0;
    for (int i = 0; i < n; ++i)
        total += z[i]->V;
    // the batch's own launch is the first candidate
    su3_launch win = default_batch(exprs, z, n);
    list.insert(list.begin(), win);
    double win_us = 1e300;
    for (const su3_launch &c : list) {
        su3_batch *b = nullptr;
        su3_status st = batch_create(&b, exprs, z, ops, n, stream, &c);
        if (st != SU3_OK)
            return st;
        double us = 0;
        st = time_launch([&]() { return su3_batch_launch(b, stream); }, hs, 2,
                         5, &us);
        su3_batch_destroy(b);
        if (st != SU3_OK)
            return st;
        if (us < win_us) {
            win_us = us;
            win = c;
        }
    }
    const Key k(SU3_EXPR_BATCH + exprs[0], z[0]->prec, z[0]->layout,
                z[0]->lanes, vbucket(total));
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        load_cache_locked();
        g_tuned[k] = win;
    }
    append_cache(k, win, win_us);
    if (best)
        *best = win;
    return SU3_OK;
}

extern "C" su3_status su3_batch_tiles(const su3_batch *b, int32_t *rows,
                                      int64_t cap, int64_t *n_tiles)
{
    if (!b || !n_tiles)
        return fail(SU3_ERR_INVALID_ARG, "NULL argument");
    *n_tiles = b->ntiles;
    if (!rows || cap < b->ntiles)
        return SU3_OK;
    // expand the table from the items the kernel reads (tile starts, sizes)
    std::vector<BatchItem> items(b->nitems);
    HIP_TRY(hipMemcpy(items.data(), b->d_items, sizeof(BatchItem) * b->nitems,
                      hipMemcpyDeviceToHost),
            "batch items copy");
    const int64_t T = b->cfg.tile_sites;
    for (int i = 0; i < b->nitems; ++i) {
        const int64_t end = i + 1 < b->nitems ? items[i + 1].tile_start : b->ntiles;
        for (int64_t t = items[i].tile_start; t < end; ++t) {
            const int64_t first = (t - items[i].tile_start) * T;
            rows[4 * t + 0] = i;
            rows[4 * t + 1] = (int32_t)first;
            rows[4 * t + 2] = (int32_t)std::min<int64_t>(T, items[i].nsites - first);
            rows[4 * t + 3] = items[i].prec;
        }
    }
    return SU3_OK;
}

// ------------------------------------------------------ yardsticks

// Default launch of each yardstick kind (the fastest of its sweep at 2.29
// GB on MI355X): 64-lane workgroups, 20 per compute unit for the triad,
// 16 for read-only, no cap for copy; 128-lane workgroups, 12 per compute
// unit, for the write-only stream; write-through streaming stores and
// nontemporal loads.
static su3_launch stream_default(int kind)
{
    su3_launch c;
    std::memset(&c, 0, sizeof c);
    c.block = kind == SU3_STREAM_WRITE ? 128 : 64;
    c.occupancy = kind == SU3_STREAM_TRIAD  ? 20
                  : kind == SU3_STREAM_READ ? 16
                  : kind == SU3_STREAM_WRITE ? 12
                                             : 0;
    c.nontemporal = 7;
    c.tile_sites = 4096;
    return c;
}

static su3_status stream_launch(int kind, void *a, const void *b,
                                const void *c, double s, int64_t n16,
                                int tail, const su3_launch &cfg,
                                hipStream_t st)
{
    if (kind < SU3_STREAM_TRIAD || kind > SU3_STREAM_COPY)
        return fail(SU3_ERR_INVALID_ARG, "unknown yardstick kind %d", kind);
    const bool reads_b = kind != SU3_STREAM_WRITE;
    const bool reads_c = kind == SU3_STREAM_TRIAD || kind == SU3_STREAM_READ;
    if (!a || (reads_b && !b) || (reads_c && !c))
        return fail(SU3_ERR_INVALID_ARG, "NULL array");
    if (n16 < 0 || (n16 == 0 && !tail))
        return fail(SU3_ERR_INVALID_ARG, "empty arrays");
    if (((uintptr_t)a | (uintptr_t)(reads_b ? b : a) |
         (uintptr_t)(reads_c ? c : a)) & 15)
        return fail(SU3_ERR_INVALID_ARG, "arrays must be 16-byte aligned");
    if (cfg.block < 64 || cfg.block > 1024 || cfg.block % 64)
        return fail(SU3_ERR_INVALID_ARG,
                    "block %d not a multiple of 64 in [64, 1024]", cfg.block);
    if (!nt_valid(cfg.nontemporal, true))
        return fail(SU3_ERR_INVALID_ARG, "nontemporal %d not in {0, 1, 2, 3, 6, 7}",
                    cfg.nontemporal);
    if (cfg.occupancy < 0 || cfg.occupancy > 64)
        return fail(SU3_ERR_INVALID_ARG, "occupancy %d not in [0, 64]",
                    cfg.occupancy);
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
    hipError_t e = launch_stream(kind, a, b, c, s, n16, tail,
                                 cfg.nontemporal, cfg.block,
                                 occupancy_reserve(dev, cfg.occupancy), st);
    if (e != hipSuccess)
        return hip_fail(e, "yardstick launch");
    return SU3_OK;
}

extern "C" su3_status su3_stream(su3_stream_kind kind, void *a, const void *b,
                                 const void *c, double s, size_t bytes,
                                 const su3_launch *cfg, void *stream)
{
    if (bytes == 0 || bytes % 16)
        return fail(SU3_ERR_INVALID_ARG,
                    "bytes must be a positive multiple of 16");
    const su3_launch l = cfg ? *cfg : stream_default(kind);
    return stream_launch(kind, a, b, c, s, (int64_t)(bytes / 16), 0, l,
                         static_cast<hipStream_t>(stream));
}

extern "C" su3_status su3_stream_autotune(su3_stream_kind kind, void *a,
                                          const void *b, const void *c,
                                          size_t bytes, void *stream,
                                          su3_launch *best, double *us_out)
{
    if (bytes == 0 || bytes % 16)
        return fail(SU3_ERR_INVALID_ARG,
                    "bytes must be a positive multiple of 16");
    hipStream_t hs = static_cast<hipStream_t>(stream);
    su3_launch win = stream_default(kind);
    double win_us = 1e300;
    su3_launch l = win;
    for (int blk : {64, 128, 256, 512, 1024})
        for (int occ : {0, 1, 2, 3, 4, 6, 8, 12, 16, 20, 24, 32})
            for (int nt : {0, 2, 3, 6, 7}) {
                if (occ * (blk / 64) > 32 || (occ == 0 && blk > 256) ||
                    (occ == 1 && blk < 512))
                    continue;
                l.block = blk;
                l.occupancy = occ;
                l.nontemporal = nt;
                double us = 0;
                su3_status st = time_launch(
                    [&]() {
                        return stream_launch(kind, a, b, c, 3.0,
                                             (int64_t)(bytes / 16), 0, l, hs);
                    },
                    hs, 3, 10, &us);
                if (st != SU3_OK && win_us >= 1e300)
                    return st;  // invalid arguments: nothing tuned
                if (st != SU3_OK) {
                    (void)hipGetLastError();
                    continue;
                }
                if (us < win_us) {
                    win_us = us;
                    win = l;
                }
            }
    if (best)
        *best = win;
    if (us_out)
        *us_out = win_us;
    return SU3_OK;
}

extern "C" su3_status su3_triad(double *a, const double *b, const double *c,
                                double s, int64_t n, void *stream)
{
    if (n <= 0)
        return fail(SU3_ERR_INVALID_ARG, "n must be > 0");
    return stream_launch(SU3_STREAM_TRIAD, a, b, c, s, n / 2, (int)(n & 1),
                         stream_default(SU3_STREAM_TRIAD),
                         static_cast<hipStream_t>(stream));
}

extern "C" su3_status su3_copy(void *dst, const void *src, size_t bytes,
                               void *stream)
{
    if (bytes == 0 || bytes % 16)
        return fail(SU3_ERR_INVALID_ARG,
                    "bytes must be a positive multiple of 16");
    return stream_launch(SU3_STREAM_COPY, dst, src, nullptr, 0.0,
                         (int64_t)(bytes / 16), 0,
                         stream_default(SU3_STREAM_COPY),
                         static_cast<hipStream_t>(stream));
}

// ------------------------------------------------------------ misc

extern "C" su3_status su3_sync(void *stream)
{
    HIP_TRY(hipStreamSynchronize(static_cast<hipStream_t>(stream)),
            "hipStreamSynchronize");
    HIP_TRY(hipGetLastError(), "pending error");
    return SU3_OK;
}

extern "C" const char *su3_status_string(su3_status s)
{
    switch (s) {
    case SU3_OK: return "SU3_OK";
    case SU3_ERR_INVALID_ARG: return "SU3_ERR_INVALID_ARG";
    case SU3_ERR_MISMATCH: return "SU3_ERR_MISMATCH";
    case SU3_ERR_UNSUPPORTED: return "SU3_ERR_UNSUPPORTED";
    case SU3_ERR_OUT_OF_MEMORY: return "SU3_ERR_OUT_OF_MEMORY";
    case SU3_ERR_ALIAS: return "SU3_ERR_ALIAS";
    case SU3_ERR_HIP: return "SU3_ERR_HIP";
    }
    return "SU3_ERR_UNKNOWN";
}

extern "C" const char *su3_last_error(void)
{
    return g_last_error.c_str();
}
