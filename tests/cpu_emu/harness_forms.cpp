// Forms of the calls that only some sizes, layouts or launches reach, run on
// the CPU (see harness.cpp): programs by rows (in place, eight slots, ragged
// lattices), the hopping term with one wave per hop and on rows too long for
// their tiles, overlapping launches of a batch.  Prints "fails 0" on success.
#include "su3.h"
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <new>
#include <sstream>
#include <string>
#include <vector>
#include <hip/hip_runtime.h>
extern "C" {
void su3gen_field(uint64_t seed, uint64_t field_id, int64_t s_begin, int64_t count, double *out);
void su3gen_spinor(uint64_t seed, uint64_t field_id, int64_t s_begin, int64_t count, double *out);
int oracle_roundtrip(int prec, const double *in, double *out, int64_t V);
int oracle_dslash(const double *const *u, const double *in, double *out, const int32_t dims[4]);
int oracle_eval_expr(const char *text, int nops, const int *kinds, const double *const *fields, double *out, int64_t V);
}

void *operator new(size_t n)
{
    void *p = emu_failing_new ? nullptr : std::malloc(n ? n : 1);
    if (!p)
        throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

static int fails = 0;
#define CHECK(cond, ...)         \
    do {                         \
        if (!(cond)) {           \
            std::printf(__VA_ARGS__); \
            std::printf("\n");   \
            ++fails;             \
        }                        \
    } while (0)

struct Lay {
    int layout, lanes;  // lanes: AoSoA; virtual nodes: simd of t
};
static int64_t volume(const int *d) { return (int64_t)d[0] * d[1] * d[2] * d[3]; }
static int reals_of(int kind) { return kind == SU3_KIND_MATRIX ? 18 : kind == SU3_KIND_SPINOR ? 24 : kind == SU3_KIND_COMPLEX ? 2 : 1; }

static su3_field *make(const int *d, int prec, int kind, Lay l, const double *host)
{
    su3_field *f = nullptr;
    su3_status st;
    if (l.layout == SU3_LAYOUT_VNODE) {
        const int simd[4] = {1, 1, 1, l.lanes};
        st = su3_vnode_alloc(&f, d, (su3_precision)prec, (su3_kind)kind, simd);
    } else if (kind == SU3_KIND_MATRIX) {
        st = su3_field_alloc(&f, d, (su3_precision)prec, (su3_layout)l.layout, l.lanes);
    } else if (kind == SU3_KIND_SPINOR) {
        st = su3_spinor_alloc(&f, d, (su3_precision)prec, (su3_layout)l.layout, l.lanes);
    } else {
        st = su3_scalar_alloc(&f, d, (su3_precision)prec, (su3_layout)l.layout, l.lanes, (su3_kind)kind);
    }
    CHECK(st == SU3_OK, "alloc: %s", su3_last_error());
    if (host)
        CHECK(su3_field_upload(f, host, nullptr) == SU3_OK, "upload: %s", su3_last_error());
    return f;
}

static std::vector<double> host_values(int64_t V, int kind, int id)
{
    std::vector<double> h(18 * V);
    su3gen_field(21, 30 + id, 0, V, h.data());
    h.resize(reals_of(kind) * V);
    return h;
}

static std::vector<double> stored(const std::vector<double> &h, int64_t V, int kind, int prec)
{
    std::vector<double> q(h);
    if (kind == SU3_KIND_MATRIX)
        oracle_roundtrip(prec, h.data(), q.data(), V);
    else if (prec != SU3_F64)
        for (double &x : q)
            x = (double)(float)x;
    return q;
}

static const int M = SU3_KIND_MATRIX, R = SU3_KIND_REAL, C = SU3_KIND_COMPLEX;

// Programs by rows: against the oracle, and in place (over operand 0) bit for
// bit as out of place.
static void programs()
{
    struct Ex { const char *text; int n; int kinds[8]; };
    static const Ex exs[] = {
        {"a*b", 2, {M, M}}, {"a*adj(b) - conj(a)", 2, {M, M}}, {"transpose(a)", 1, {M}},
        {"(a*b+c*d)*(a*c+b*d)+(a-b)*(c-d)", 4, {M, M, M, M}},
        {"a*b+c*d+e*f+g*h", 8, {M, M, M, M, M, M, M, M}},  // eight slots
        {"a*b + c*a - d*b + 0.5", 4, {M, M, C, R}}, {"trace(a*b*adj(c)*adj(d))", 4, {M, M, M, M}},
        {"real(trace(a*adj(b)))*c", 3, {M, M, R}}};
    static const int lattices[][4] = {{3, 3, 3, 7}, {4, 4, 4, 2}, {5, 1, 1, 1}, {3, 5, 7, 9}};
    static const Lay lays[] = {{SU3_LAYOUT_AOS, 0}, {SU3_LAYOUT_SOA, 0}, {SU3_LAYOUT_AOSOA, 8}, {SU3_LAYOUT_VNODE, 2}};
    for (const auto &d : lattices)
        for (const Lay &l : lays) {
            if (l.layout == SU3_LAYOUT_VNODE && d[3] % l.lanes)
                continue;
            const int64_t V = volume(d);
            for (int arith : {(int)SU3_F64, (int)SU3_F32, (int)SU3_C12_F32})
                for (const Ex &ex : exs) {
                    su3_program *p;
                    su3_kind kinds[8], rk;
                    for (int k = 0; k < ex.n; ++k) kinds[k] = (su3_kind)ex.kinds[k];
                    if (su3_program_create(&p, ex.text, ex.n, kinds) != SU3_OK) { CHECK(false, "%s: %s", ex.text, su3_last_error()); continue; }
                    su3_program_info(p, &rk, nullptr, nullptr);
                    std::vector<su3_field *> f;
                    std::vector<std::vector<double>> q;
                    std::vector<const double *> qp;
                    for (int k = 0; k < ex.n; ++k) {
                        const int prec = ex.kinds[k] == M || arith == SU3_F64 ? arith : (int)SU3_F32;
                        const std::vector<double> h = host_values(V, ex.kinds[k], k);
                        f.push_back(make(d, prec, ex.kinds[k], l, h.data()));
                        q.push_back(stored(h, V, ex.kinds[k], prec));
                    }
                    for (auto &x : q) qp.push_back(x.data());
                    const int zprec = arith == SU3_F64 ? (int)SU3_F64 : (int)SU3_F32;
                    su3_field *z = make(d, zprec, rk, l, nullptr);
                    const int n = reals_of(rk);
                    std::vector<double> want(18 * V), got(n * V), over(n * V);
                    oracle_eval_expr(ex.text, ex.n, ex.kinds, qp.data(), want.data(), V);
                    CHECK(su3_program_eval(p, z, f.data(), ex.n, nullptr) == SU3_OK, "%s: %s", ex.text, su3_last_error());
                    if (l.layout != SU3_LAYOUT_AOS) {
                        const bool rows = blockDim.x == 192;  // three waves
                        // (single with four slots: one lane per site)
                        CHECK(rows || arith != SU3_F64, "%s, %lld sites: not by rows", ex.text, (long long)V);
                    }
                    su3_field_download(z, got.data(), nullptr);
                    double err = 0, mag = 0;
                    for (int64_t i = 0; i < n * V; ++i) { err = std::max(err, std::fabs(got[i] - want[i])); mag = std::max(mag, std::fabs(want[i])); }
                    CHECK(err <= (arith == SU3_F64 ? 1e-13 : 2e-6) * (1 + mag), "%s arith %d layout %d V %lld: err %.3e", ex.text, arith, l.layout, (long long)V, err);
                    if (rk == ex.kinds[0] && (arith != SU3_C12_F32 || rk != SU3_KIND_MATRIX)) {
                        CHECK(su3_program_eval(p, f[0], f.data(), ex.n, nullptr) == SU3_OK, "%s in place: %s", ex.text, su3_last_error());
                        su3_field_download(f[0], over.data(), nullptr);
                        CHECK(std::memcmp(over.data(), got.data(), sizeof(double) * n * V) == 0, "%s arith %d layout %d: differs in place", ex.text, arith, l.layout);
                    }
                    su3_field_free(z);
                    for (auto *x : f) su3_field_free(x);
                    su3_program_destroy(p);
                }
        }
    std::printf("programs by rows done\n");
}

// Traces of negatives and conjugates: each term changes its sign before the
// sum, so sums that cancel keep the zero's sign.
// Which launch an untuned program takes: by rows where that needs no more
// rounds of workgroups than one lane per site (3 slots in single: 15 workgroups
// of 128 sites at once on the three emulated compute units, 18 of the one-lane
// kernel's), and which loads of operand 0 bypass the caches.
static void program_launches()
{
    struct Case { const char *text; int kinds[4]; int n; int prec; Lay l; int d[4]; bool rows, bypass; };
    static const Lay soa = {SU3_LAYOUT_SOA, 0}, aos = {SU3_LAYOUT_AOS, 0};
    static const char *const update = "c*a*b+0.5";
    static const Case cases[] = {
        {update, {M, M, R}, 3, SU3_F32, soa, {8, 4, 4, 15}, true, true},   // 1 round, 1
        {update, {M, M, R}, 3, SU3_F32, soa, {8, 4, 4, 16}, false, true},  // 2, 1
        {update, {M, M, R}, 3, SU3_F32, soa, {8, 4, 4, 18}, false, true},  // 2, 1
        {update, {M, M, R}, 3, SU3_F32, soa, {8, 4, 4, 19}, true, true},   // 2, 2
        {update, {M, M, R}, 3, SU3_F32, soa, {8, 4, 4, 31}, false, true},  // 3, 2
        {update, {M, M, R}, 3, SU3_F32, soa, {8, 4, 4, 37}, true, true},   // 3, 3
        {update, {M, M, R}, 3, SU3_F64, soa, {8, 4, 4, 31}, true, true},
        {"a*adj(b)", {M, M}, 2, SU3_F64, soa, {24, 24, 24, 13}, true, true},   // 78 MB
        {"a*adj(b)", {M, M}, 2, SU3_F64, soa, {24, 24, 24, 14}, true, false},  // 84 MB
        {"a*adj(b)", {M, M}, 2, SU3_F64, soa, {24, 24, 24, 26}, true, true},   // 155 MB
        {"a*b+c*d", {M, M, M, M}, 4, SU3_F32, soa, {24, 24, 24, 18}, false, true},  // 90 MB
        {"a*b+c*d", {M, M, M, M}, 4, SU3_F32, {SU3_LAYOUT_AOSOA, 8}, {8, 8, 8, 8}, false, false},
        {"a*adj(b)", {M, M}, 2, SU3_F32, {SU3_LAYOUT_VNODE, 2}, {4, 4, 4, 4}, true, false},
        // AoS: products of up to 50 MB per field, three slots in double of up to 35 MB
        {"a*adj(b)", {M, M}, 2, SU3_F64, aos, {24, 24, 24, 25}, true, false},
        {"a*adj(b)", {M, M}, 2, SU3_F64, aos, {24, 24, 24, 26}, false, false},
        {update, {M, M, R}, 3, SU3_F64, aos, {24, 24, 24, 17}, true, false},  // 34 MB
        {update, {M, M, R}, 3, SU3_F64, aos, {24, 24, 24, 18}, false, false},
        {"a*b+c*d", {M, M, M, M}, 4, SU3_F64, aos, {4, 4, 4, 4}, false, false},
        {"(a*b+c*d)*(a*c+b*d)+(a-b)*(c-d)", {M, M, M, M}, 4, SU3_F64, aos, {4, 4, 4, 6}, true, false},  // 6 of 6 at once
        {"(a*b+c*d)*(a*c+b*d)+(a-b)*(c-d)", {M, M, M, M}, 4, SU3_F64, aos, {4, 4, 4, 7}, false, false},
        {"a+b+a*b", {R, R}, 2, SU3_F32, soa, {8, 8, 8, 8}, false, true},
        {"a+b+a*b", {R, R}, 2, SU3_F64, soa, {8, 8, 8, 8}, false, false}};
    for (const Case &c : cases) {
        su3_program *p;
        su3_kind kinds[4], rk;
        std::vector<su3_field *> f;
        for (int k = 0; k < c.n; ++k) {
            kinds[k] = (su3_kind)c.kinds[k];
            f.push_back(make(c.d, c.prec, c.kinds[k], c.l, nullptr));
        }
        if (su3_program_create(&p, c.text, c.n, kinds) != SU3_OK) { CHECK(false, "%s: %s", c.text, su3_last_error()); continue; }
        su3_program_info(p, &rk, nullptr, nullptr);
        su3_field *z = make(c.d, c.prec, rk, c.l, nullptr);
        void *q;
        size_t n;
        su3_field_data(f[0], &q, &n);
        emu_watch_lo = (const char *)q;
        emu_watch_hi = emu_watch_lo + n;
        emu_watched = 0;
        CHECK(su3_program_eval(p, z, f.data(), c.n, nullptr) == SU3_OK, "%s: %s", c.text, su3_last_error());
        CHECK((blockDim.x == 192) == c.rows, "%s prec %d layout %d/%d t %d: %u lanes", c.text, c.prec, c.l.layout, c.l.lanes, c.d[3], blockDim.x);
        CHECK((emu_watched > 0) == c.bypass, "%s prec %d layout %d/%d t %d: %ld loads bypass the caches", c.text, c.prec, c.l.layout, c.l.lanes, c.d[3], emu_watched);
        emu_watch_lo = emu_watch_hi = nullptr;
        for (su3_field *x : f) su3_field_free(x);
        su3_field_free(z);
        su3_program_destroy(p);
    }
    std::printf("program launches done\n");
}

// Settings of a program key: one that a caller sets holds for every program of
// the key, the tuner's (schedule 1) for the form it was timed on; saved settings
// that name no form are left out.
static void program_settings()
{
    const int d[4] = {8, 4, 4, 16};  // 16 workgroups of 128 sites, 12 of four slots at once
    const Lay l = {SU3_LAYOUT_SOA, 0};
    const auto get = [&](su3_expr e, su3_precision prec) {
        su3_launch c;
        std::memset(&c, 0, sizeof c);
        CHECK(su3_launch_get(e, prec, SU3_LAYOUT_SOA, 0, d, &c) == SU3_OK, "get: %s", su3_last_error());
        return c;
    };
    const auto line = [&](int expr, int prec, int block, int schedule, const char *more) {
        std::ostringstream o;
        o << "{\"device\":\"emu:3\",\"expr\":" << expr << ",\"prec\":" << prec << ",\"layout\":1,\"lanes\":0,\"vbucket\":11,\"block\":" << block
          << ",\"persistent\":0,\"nontemporal\":3,\"xcd_remap\":0,\"lds_stage\":0,\"tile_sites\":4096,\"occupancy\":0,\"schedule\":" << schedule
          << ",\"sites_per_lane\":0," << more << "\"us\":1.0}\n";
        return o.str();
    };
    char path[] = "/tmp/su3_forms_XXXXXX";
    const int fd = mkstemp(path);
    CHECK(fd >= 0, "mkstemp");
    std::ofstream(path) << line(SU3_EXPR_PROGRAM, SU3_F64, 256, 0, "") << line(SU3_EXPR_PROGRAM_SCALAR, SU3_F32, 256, 1, "\"other_form\":1,")
                        << line(SU3_EXPR_PROGRAM, SU3_F32, 64, 1, "");
    setenv("SU3_TUNE_CACHE", path, 1);
    CHECK(get(SU3_EXPR_PROGRAM, SU3_F64).block == 128, "a line without a form holds");
    CHECK(get(SU3_EXPR_PROGRAM_SCALAR, SU3_F32).block == 128, "the other form's line holds for the first");
    CHECK(get(SU3_EXPR_PROGRAM, SU3_F32).block == 64, "a line is lost");

    // the programs: by rows, on one lane per site, without a matrix
    struct Ex { const char *text; int n, kind; su3_program *p; su3_field *f[4], *z; };
    Ex ex[] = {{"a*b", 2, M, nullptr, {}, nullptr}, {"a*b+c*d", 4, M, nullptr, {}, nullptr}, {"a+b", 2, R, nullptr, {}, nullptr},
               {"trace(a*b*adj(c)*adj(d))", 4, M, nullptr, {}, nullptr}};
    for (Ex &e : ex) {
        su3_kind kinds[4], rk;
        for (int k = 0; k < e.n; ++k) {
            kinds[k] = (su3_kind)e.kind;
            const std::vector<double> h = host_values(volume(d), e.kind, k);
            e.f[k] = make(d, SU3_F32, e.kind, l, h.data());
        }
        CHECK(su3_program_create(&e.p, e.text, e.n, kinds) == SU3_OK, "%s: %s", e.text, su3_last_error());
        su3_program_info(e.p, &rk, nullptr, nullptr);
        e.z = make(d, SU3_F32, rk, l, nullptr);
    }
    // loads past the caches?  And the lanes of the launch
    const auto run = [&](const Ex &e, unsigned *lanes) {
        void *q;
        size_t n;
        su3_field_data(e.f[0], &q, &n);
        emu_watch_lo = (const char *)q;
        emu_watch_hi = emu_watch_lo + n;
        emu_watched = 0;
        CHECK(su3_program_eval(e.p, e.z, e.f, e.n, nullptr) == SU3_OK, "%s: %s", e.text, su3_last_error());
        emu_watch_lo = emu_watch_hi = nullptr;
        *lanes = blockDim.x;
        return emu_watched > 0;
    };
    unsigned lanes;
    CHECK(!(run(ex[3], &lanes), lanes != 256), "the trace on one lane per site: %u lanes, not as saved", lanes);
    su3_launch_reset();
    for (int schedule = 0; schedule < 2; ++schedule) {
        su3_launch c = {64, 0, 0, 0, 0, 4096, 0, schedule, 0};
        CHECK(su3_launch_set(SU3_EXPR_PROGRAM, SU3_F32, SU3_LAYOUT_SOA, 0, d, &c) == SU3_OK, "set: %s", su3_last_error());
        const su3_launch g = get(SU3_EXPR_PROGRAM, SU3_F32);
        CHECK(std::memcmp(&g, &c, sizeof c) == 0, "another setting than was set");
        CHECK(!run(ex[0], &lanes) && lanes == 192, "schedule %d: not for a*b", schedule);
        CHECK(run(ex[1], &lanes) == (schedule == 1) && lanes == (schedule ? 128u : 64u), "schedule %d: a*b+c*d in %u lanes", schedule, lanes);
        CHECK(run(ex[2], &lanes) == (schedule == 1), "schedule %d: a+b", schedule);
    }
    // tuned where blocks of 256 lanes are fastest: the four operands' programs
    // run in those, a*b by rows as untuned (all launches by rows took alike)
    su3_launch_reset();
    emu_launch_ms = [] { return blockDim.x == 256 ? 0.5f : 1.0f; };
    for (su3_expr e : {SU3_EXPR_PROGRAM, SU3_EXPR_PROGRAM_SCALAR}) {
        su3_launch best, was = get(e, SU3_F32);
        CHECK(su3_autotune(e, SU3_F32, SU3_LAYOUT_SOA, 0, d, nullptr, &best) == SU3_OK, "autotune: %s", su3_last_error());
        CHECK(best.schedule == 1, "the tuner's setting names no form");
        was.schedule = 1;
        CHECK(std::memcmp(&was, &best, sizeof was) == 0, "by rows: nontemporal %d, cap %d", best.nontemporal, best.occupancy);
        const su3_launch g = get(e, SU3_F32);
        CHECK(std::memcmp(&g, &best, sizeof g) == 0, "another setting than the tuner's");
    }
    emu_launch_ms = nullptr;
    CHECK((run(ex[1], &lanes), lanes == 256), "a*b+c*d tuned: %u lanes", lanes);
    CHECK((run(ex[3], &lanes), lanes == 256), "trace tuned: %u lanes", lanes);
    std::stringstream saved;
    saved << std::ifstream(path).rdbuf();
    size_t others = 0;
    for (size_t at = 0; (at = saved.str().find("\"other_form\":1", at)) != std::string::npos; ++at) ++others;
    CHECK(others == 3, "%zu lines of the other form", others);
    su3_launch_reset();
    unsetenv("SU3_TUNE_CACHE");
    std::remove(path);
    for (Ex &e : ex) {
        for (su3_field *f : e.f) su3_field_free(f);
        su3_field_free(e.z);
        su3_program_destroy(e.p);
    }
    std::printf("program settings done\n");
}

// Where every candidate takes alike, a tuner keeps the call's own launch.
static void tuners()
{
    struct Case { su3_expr e; su3_precision prec; Lay l; };
    const Lay soa = {SU3_LAYOUT_SOA, 0}, aos = {SU3_LAYOUT_AOS, 0}, short_runs = {SU3_LAYOUT_AOSOA, 8}, vn = {SU3_LAYOUT_VNODE, 4};
    const Case cases[] = {
        {SU3_EXPR_MUL, SU3_F64, soa}, {SU3_EXPR_MULADD, SU3_F32, soa}, {SU3_EXPR_MUL, SU3_F64, aos}, {SU3_EXPR_MUL, SU3_F16_F32ACC, short_runs},
        {SU3_EXPR_MUL, SU3_F32, vn}, {SU3_EXPR_CSHIFT, SU3_F64, soa}, {SU3_EXPR_MUL_SHIFTED, SU3_F64, aos}, {SU3_EXPR_MUL_SHIFTED, SU3_F32, vn},
        {SU3_EXPR_DSLASH, SU3_F64, soa}, {SU3_EXPR_DSLASH, SU3_F32, vn}, {SU3_EXPR_PROGRAM, SU3_F64, aos}, {SU3_EXPR_PROGRAM_SCALAR, SU3_F64, aos}};
    const int d[4] = {2, 2, 2, 4};
    for (const Case &c : cases) {
        su3_launch was, best, now;
        su3_launch_reset();
        CHECK(su3_launch_get(c.e, c.prec, (su3_layout)c.l.layout, c.l.lanes, d, &was) == SU3_OK, "get: %s", su3_last_error());
        CHECK(su3_autotune(c.e, c.prec, (su3_layout)c.l.layout, c.l.lanes, d, nullptr, &best) == SU3_OK, "autotune: %s", su3_last_error());
        CHECK(su3_launch_get(c.e, c.prec, (su3_layout)c.l.layout, c.l.lanes, d, &now) == SU3_OK, "get: %s", su3_last_error());
        CHECK(std::memcmp(&best, &now, sizeof now) == 0, "expr %d: the table holds another launch", c.e);
        if (c.e == SU3_EXPR_PROGRAM || c.e == SU3_EXPR_PROGRAM_SCALAR) {
            CHECK(best.schedule == 1, "expr %d: no form", c.e);
            best.schedule = was.schedule;
            was.nontemporal = best.nontemporal;  // by the operands' bytes
        }
        CHECK(std::memcmp(&best, &was, sizeof was) == 0, "expr %d prec %d layout %d/%d: block %d nontemporal %d cap %d schedule %d, untuned %d %d %d %d", c.e, c.prec, c.l.layout, c.l.lanes,
              best.block, best.nontemporal, best.occupancy, best.schedule, was.block, was.nontemporal, was.occupancy, was.schedule);
    }
    for (const Lay &l : {soa, short_runs}) {
        su3_field *z = make(d, SU3_F32, M, l, nullptr), *x = make(d, SU3_F32, M, l, nullptr), *y = make(d, SU3_F32, M, l, nullptr);
        const su3_expr e = SU3_EXPR_MUL;
        const su3_field *ops[4] = {x, y, nullptr, nullptr};
        su3_launch was, best;
        su3_launch_reset();
        CHECK(su3_launch_get((su3_expr)(SU3_EXPR_BATCH + SU3_EXPR_MUL), SU3_F32, (su3_layout)l.layout, l.lanes, d, &was) == SU3_OK, "get: %s", su3_last_error());
        CHECK(su3_batch_autotune(&e, &z, ops, 1, nullptr, &best) == SU3_OK, "batch autotune: %s", su3_last_error());
        CHECK(std::memcmp(&best, &was, sizeof was) == 0, "batch layout %d: tile %d nontemporal %d, untuned %d %d", l.layout, best.tile_sites, best.nontemporal, was.tile_sites, was.nontemporal);
        for (su3_field *f : {z, x, y}) su3_field_free(f);
    }
    su3_launch_reset();
    std::printf("tuners done\n");
}

static void traces()
{
    static const char *const texts[] = {"trace(-a)", "trace(conj(a))", "trace(adj(-a))", "trace(transpose(-conj(a)))", "-trace(a)"};
    const int d[4] = {3, 3, 3, 3};
    const int64_t V = volume(d);
    std::vector<double> h(18 * V), got(2 * V);
    for (int64_t i = 0; i < 18 * V; ++i) h[i] = (double)((i * 7 + i / 18) % 3 - 1);  // -1, 0, 1
    for (int prec : {(int)SU3_F64, (int)SU3_F32})
        for (Lay l : {Lay{SU3_LAYOUT_SOA, 0}, Lay{SU3_LAYOUT_AOSOA, 16}})
            for (const char *text : texts) {
                su3_field *a = make(d, prec, M, l, h.data()), *z = make(d, prec, C, l, nullptr);
                su3_program *p;
                const su3_kind kind = SU3_KIND_MATRIX;
                su3_program_create(&p, text, 1, &kind);
                CHECK(su3_program_eval(p, z, &a, 1, nullptr) == SU3_OK, "%s: %s", text, su3_last_error());
                su3_field_download(z, got.data(), nullptr);
                const bool outside = text[0] == '-', neg = std::strchr(text, '-') && !outside;
                const bool conj = std::strstr(text, "conj") || std::strstr(text, "adj");
                int bad = 0;
                for (int64_t s = 0; s < V; ++s)
                    for (int c = 0; c < 2; ++c) {
                        const double sign = neg != (conj && c == 1) ? -1.0 : 1.0;
                        const double *m = &h[18 * s + c];
                        double t = (sign * m[0] + sign * m[8]) + sign * m[16];
                        if (outside) t = -t;
                        bad += std::memcmp(&t, &got[2 * s + c], sizeof t) != 0;
                    }
                CHECK(bad == 0, "%s prec %d layout %d: %d reals differ in their bits", text, prec, l.layout, bad);
                su3_program_destroy(p);
                su3_field_free(a); su3_field_free(z);
            }
    std::printf("traces done\n");
}

// The hopping term: one wave per hop bit for bit as one lane per site, and
// rows too long for their tiles (the schedule's fallbacks).
static void hopping()
{
    struct Case { int d[4]; Lay l; };
    static const Case cases[] = {
        {{3, 5, 7, 2}, {SU3_LAYOUT_SOA, 0}}, {{4, 4, 2, 3}, {SU3_LAYOUT_AOS, 0}}, {{5, 3, 2, 6}, {SU3_LAYOUT_AOSOA, 8}},
        {{4, 2, 6, 4}, {SU3_LAYOUT_VNODE, 2}}, {{130, 1, 2, 2}, {SU3_LAYOUT_SOA, 0}}, {{300, 1, 1, 2}, {SU3_LAYOUT_SOA, 0}}};
    for (const Case &c : cases)
        for (int lp : {(int)SU3_F64, (int)SU3_F32, (int)SU3_C12_F32}) {
            const int64_t V = volume(c.d);
            const int sp = lp == SU3_F64 ? (int)SU3_F64 : (int)SU3_F32;
            std::vector<std::vector<double>> q;
            const double *up[4];
            su3_field *u[4];
            for (int mu = 0; mu < 4; ++mu) {
                const std::vector<double> h = host_values(V, M, mu);
                u[mu] = make(c.d, lp, M, c.l, h.data());
                q.push_back(stored(h, V, M, lp));
            }
            for (int mu = 0; mu < 4; ++mu) up[mu] = q[mu].data();
            std::vector<double> in(24 * V), qin(24 * V), want(24 * V), plain(24 * V), got(24 * V);
            su3gen_spinor(21, 77, 0, V, in.data());
            for (int64_t i = 0; i < 24 * V; ++i) qin[i] = sp == SU3_F64 ? in[i] : (double)(float)in[i];
            oracle_dslash(up, qin.data(), want.data(), c.d);
            su3_field *fin = make(c.d, sp, SU3_KIND_SPINOR, c.l, in.data());
            su3_field *out = make(c.d, sp, SU3_KIND_SPINOR, c.l, nullptr);
            // block, persistent, nontemporal, xcd_remap, lds_stage, tile_sites,
            // occupancy, schedule, sites_per_lane
            static const su3_launch ls[] = {
                {64, 0, 0, 0, 0, 1, 0, 0, 0}, {64, 0, 0, 0, 0, 1, 0, 0, 8}, {64, 0, 3, 1, 0, 1, 0, 0, 8},
                {256, 0, 2, 0, 0, 2, 0, 16, 0}, {256, 0, 2, 1, 0, 3, 0, 17, 0}, {256, 0, 2, 2, 0, 1, 0, 12, 0},
                {256, 0, 2, 0, 0, 2, 0, 28, 0}};
            const int lanes = c.l.layout == SU3_LAYOUT_AOSOA || c.l.layout == SU3_LAYOUT_VNODE ? c.l.lanes : 0;
            for (const su3_launch &s : ls) {
                CHECK(su3_launch_set(SU3_EXPR_DSLASH, (su3_precision)lp, (su3_layout)c.l.layout, lanes, c.d, &s) == SU3_OK, "launch: %s", su3_last_error());
                CHECK(su3_dslash(out, u, fin, nullptr) == SU3_OK, "dslash: %s", su3_last_error());
                CHECK(s.sites_per_lane != 8 || blockDim.x == 512, "not one wave per hop");
                su3_field_download(out, &s == ls ? plain.data() : got.data(), nullptr);
                CHECK(&s == ls || std::memcmp(plain.data(), got.data(), sizeof(double) * 24 * V) == 0, "dslash %dx%dx%dx%d layout %d prec %d: launch %d differs", c.d[0], c.d[1], c.d[2], c.d[3], c.l.layout, lp, (int)(&s - ls));
            }
            su3_launch_reset();
            double err = 0;
            for (int64_t i = 0; i < 24 * V; ++i) err = std::max(err, std::fabs(plain[i] - want[i]));
            CHECK(err <= (sp == SU3_F64 ? 1e-13 : 2e-5), "dslash err %.3e", err);
            su3_field_free(fin); su3_field_free(out);
            for (int mu = 0; mu < 4; ++mu) su3_field_free(u[mu]);
        }
    std::printf("hopping term done\n");
}

// The walks' t-links bypass the caches where a lane-block's entry fills whole
// lines (a bypassed line comes once per piece of it) and the call does not fit
// the Infinity Cache, and nowhere else.
static void t_links()
{
    struct Case { int prec; Lay l; int t; bool bypass; };
    static const Case cases[] = {
        {SU3_F64, {SU3_LAYOUT_SOA, 0}, 1, false}, {SU3_F64, {SU3_LAYOUT_SOA, 0}, 4, true},
        {SU3_F64, {SU3_LAYOUT_AOSOA, 8}, 4, true}, {SU3_F64, {SU3_LAYOUT_VNODE, 4}, 4, false}};
    for (const Case &c : cases) {
        const int d[4] = {48, 48, 48, c.t};  // 106 MB, 425 MB
        su3_field *u = make(d, c.prec, M, c.l, nullptr);
        su3_field *in = make(d, c.prec, SU3_KIND_SPINOR, c.l, nullptr), *out = make(d, c.prec, SU3_KIND_SPINOR, c.l, nullptr);
        su3_field *links[4] = {u, u, u, u};
        const int lanes = c.l.layout == SU3_LAYOUT_SOA ? 0 : c.l.lanes;
        const su3_launch s = {256, 0, 2, 0, 0, 1, 0, 9, 0};
        CHECK(su3_launch_set(SU3_EXPR_DSLASH, (su3_precision)c.prec, (su3_layout)c.l.layout, lanes, d, &s) == SU3_OK, "launch: %s", su3_last_error());
        void *p;
        size_t n;
        su3_field_data(u, &p, &n);
        emu_watch_lo = (const char *)p;
        emu_watch_hi = emu_watch_lo + n;
        emu_watched = 0;
        CHECK(su3_dslash(out, links, in, nullptr) == SU3_OK, "dslash: %s", su3_last_error());
        CHECK((emu_watched > 0) == c.bypass, "prec %d layout %d/%d t %d: %ld link loads bypass the caches", c.prec, c.l.layout, c.l.lanes, c.t, emu_watched);
        emu_watch_lo = emu_watch_hi = nullptr;
        su3_launch_reset();
        for (su3_field *f : {u, in, out}) su3_field_free(f);
    }
    std::printf("t-links done\n");
}

// Launches of one batch with a persistent grid share its ticket counter: on
// any streams each waits for the event recorded behind the one before it, and
// captured ones, which nothing orders, draw no tickets.
static void batches()
{
    const int d[4] = {5, 6, 7, 8};
    const Lay l = {SU3_LAYOUT_SOA, 0};
    const int64_t V = volume(d);
    const std::vector<double> hx = host_values(V, M, 0), hy = host_values(V, M, 1);
    su3_field *x = make(d, SU3_F64, M, l, hx.data()), *y = make(d, SU3_F64, M, l, hy.data());
    su3_field *z = make(d, SU3_F64, M, l, nullptr), *ref = make(d, SU3_F64, M, l, nullptr);
    su3_mult(ref, x, y, nullptr);
    std::vector<double> want(18 * V), got(18 * V);
    su3_field_download(ref, want.data(), nullptr);
    const su3_launch s = {64, 2, 3, 0, 0, 64, 0, 0, 0};
    su3_launch_set((su3_expr)(SU3_EXPR_BATCH + SU3_EXPR_MUL), SU3_F64, SU3_LAYOUT_SOA, 0, d, &s);
    const su3_expr ex = SU3_EXPR_MUL;
    const su3_field *ops[4] = {x, y, nullptr, nullptr};
    su3_batch *b = nullptr;
    CHECK(su3_batch_create(&b, &ex, &z, ops, 1, nullptr) == SU3_OK, "batch: %s", su3_last_error());
    const std::vector<double> zero(18 * V, 0.0);
    const auto same = [&](const char *what) {
        su3_field_download(z, got.data(), nullptr);
        CHECK(std::memcmp(got.data(), want.data(), sizeof(double) * 18 * V) == 0, "batch %s: wrong result", what);
        su3_field_upload(z, zero.data(), nullptr);
    };
    hipEvent_t last = nullptr;
    for (uintptr_t stream : {1, 2, 2, 1, 3}) {
        emu_calls.clear();
        CHECK(su3_batch_launch(b, (void *)stream) == SU3_OK, "batch launch: %s", su3_last_error());
        size_t launch = 0;
        while (launch < emu_calls.size() && emu_calls[launch].what != 'L') ++launch;
        bool waits = last == nullptr;
        for (size_t i = 0; i < launch; ++i)
            waits |= emu_calls[i].what == 'W' && emu_calls[i].event == last && emu_calls[i].stream == (void *)stream;
        CHECK(waits, "batch on stream %d does not wait for the launch before it", (int)stream);
        last = nullptr;
        for (size_t i = launch; i < emu_calls.size(); ++i)
            if (emu_calls[i].what == 'R' && emu_calls[i].stream == (void *)stream)
                last = emu_calls[i].event;
        CHECK(last != nullptr, "no event behind the batch");
        same("launch");
    }
    hipGraph_t graph;
    hipStreamBeginCapture((hipStream_t)4, hipStreamCaptureModeThreadLocal);
    CHECK(su3_batch_launch(b, (void *)4) == SU3_OK, "batch capture: %s", su3_last_error());
    hipStreamEndCapture((hipStream_t)4, &graph);
    for (int rep = 0; rep < 3; ++rep) {
        const int tickets = emu_atomics;
        hipGraphLaunch((hipGraphExec_t)graph, nullptr);
        CHECK(emu_atomics == tickets, "a captured batch draws tickets");
        same("replay");
        su3_batch_launch(b, nullptr);
        same("between replays");
    }
    hipGraphDestroy(graph);
    su3_batch_destroy(b);
    su3_launch_reset();
    for (su3_field *f : {x, y, z, ref}) su3_field_free(f);
    std::printf("batches done\n");
}

// The transfers' staging buffers: a handle on borrowed memory ends without a
// HIP call, the last owning one gives them back, and so does an allocation
// that would fail.
static void staging()
{
    const int d[4] = {8, 8, 8, 4};
    const int64_t V = volume(d);
    const Lay l = {SU3_LAYOUT_SOA, 0};
    const std::vector<double> h = host_values(V, M, 0);
    size_t bytes = 0;
    su3_field_bytes(d, SU3_F64, SU3_LAYOUT_SOA, 0, &bytes);
    void *mem = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
    const auto borrowed = [&]() {
        su3_field *f = nullptr;
        CHECK(su3_field_wrap(&f, mem, bytes, d, SU3_F64, SU3_LAYOUT_SOA, 0) == SU3_OK, "wrap: %s", su3_last_error());
        CHECK(su3_field_upload(f, h.data(), nullptr) == SU3_OK, "upload: %s", su3_last_error());
        const int frees = emu_frees;
        su3_field_free(f);
        CHECK(emu_frees == frees, "the end of a borrowed field frees device memory");
    };
    borrowed();
    int frees = emu_frees;
    su3_field *f = make(d, SU3_F64, M, l, h.data());
    su3_field_free(f);
    CHECK(emu_frees == frees + 2, "the last owning field keeps the staging buffer");
    borrowed();
    frees = emu_frees;
    emu_failing_mallocs = 1;
    CHECK(su3_field_alloc(&f, d, SU3_F64, SU3_LAYOUT_SOA, 0) == SU3_OK, "an allocation fails beside kept buffers: %s", su3_last_error());
    CHECK(emu_frees == frees + 1, "no staging buffer given back");
    emu_failing_mallocs = 2;
    su3_field *g = nullptr;
    CHECK(su3_field_alloc(&g, d, SU3_F64, SU3_LAYOUT_SOA, 0) == SU3_ERR_OUT_OF_MEMORY, "no memory, but a field");
    emu_failing_mallocs = 0;
    su3_field_free(f);
    std::free(mem);
    std::printf("staging done\n");
}

// Calls that hold no host memory of their own end well where there is none.
static void no_host_memory()
{
    const int d[4] = {8, 8, 8, 4}, other[4] = {8, 8, 8, 6};
    const std::vector<double> h = host_values(volume(d), M, 0);
    std::vector<double> got(h.size());
    su3_field *f = make(d, SU3_F64, M, {SU3_LAYOUT_SOA, 0}, nullptr);
    emu_calls.reserve(emu_calls.size() + 100);
    try {
        su3_launch c;
        emu_failing_new = true;
        const su3_status planned = su3_launch_get(SU3_EXPR_DSLASH, SU3_F64, SU3_LAYOUT_SOA, 0, other, &c);
        const su3_status up = su3_field_upload(f, h.data(), nullptr), down = su3_field_download(f, got.data(), nullptr);
        emu_failing_new = false;
        CHECK(planned == SU3_OK && up == SU3_OK && down == SU3_OK, "plan %d, upload %d, download %d", planned, up, down);
        CHECK(std::memcmp(got.data(), h.data(), sizeof(double) * h.size()) == 0, "another field than was stored");
    } catch (const std::bad_alloc &) {
        emu_failing_new = false;
        CHECK(false, "an exception crosses the entry point");
    }
    su3_field_free(f);
    std::printf("no host memory done\n");
}

int main()
{
    program_settings();
    programs();
    program_launches();
    tuners();
    traces();
    hopping();
    t_links();
    batches();
    staging();
    no_host_memory();
    std::printf("fails %d\n", fails);
    return fails != 0;
}
