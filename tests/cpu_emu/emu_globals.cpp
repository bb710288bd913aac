// Storage of the emulated launch state and of the kernels' LDS arrays; the
// lanes of a workgroup as contexts that take turns at its barriers.
#include <hip/hip_runtime.h>
#include <csetjmp>
#include <memory>
#include <sanitizer/asan_interface.h>
#include <sanitizer/common_interface_defs.h>
#include <ucontext.h>
thread_local emu_idx blockIdx, threadIdx;
emu_idx blockDim, gridDim;
bool emu_capturing = false;
std::vector<std::function<void()>> emu_graph;
unsigned char emu_lds[1 << 18];
int emu_launches = 0;
bool emu_threaded = false;
bool emu_failing_new = false;
int emu_atomics = 0, emu_failing_mallocs = 0, emu_frees = 0;
std::vector<emu_call> emu_calls;
const char *emu_watch_lo = nullptr, *emu_watch_hi = nullptr;
long emu_watched = 0;
float (*emu_launch_ms)() = nullptr;
namespace su3k { namespace p0 { alignas(16) unsigned char lds[1 << 18]; } namespace p1 { alignas(16) unsigned char lds[1 << 18]; } namespace p2 { alignas(16) unsigned char lds[1 << 18]; } namespace p3 { alignas(16) unsigned char lds[1 << 18]; } }
namespace su3k { char occupancy_reserve[1 << 16]; namespace p0 { char occupancy_reserve[1 << 16]; } namespace p1 { char occupancy_reserve[1 << 16]; } namespace p2 { char occupancy_reserve[1 << 16]; } namespace p3 { char occupancy_reserve[1 << 16]; } namespace dslash { alignas(16) char occupancy_reserve[160 << 10]; } namespace prog { alignas(16) char occupancy_reserve[160 << 10]; } }

void emu_lds_limit(size_t bytes)
{
    const auto limit = [&](void *p, size_t n) {
        ASAN_UNPOISON_MEMORY_REGION(p, n);
        if (bytes < n)
            ASAN_POISON_MEMORY_REGION((char *)p + bytes, n - bytes);
    };
    using namespace su3k;
    limit(occupancy_reserve, sizeof occupancy_reserve);
    limit(p0::lds, sizeof p0::lds);
    limit(p1::lds, sizeof p1::lds);
    limit(p2::lds, sizeof p2::lds);
    limit(p3::lds, sizeof p3::lds);
    limit(dslash::occupancy_reserve, sizeof dslash::occupancy_reserve);
    limit(prog::occupancy_reserve, sizeof prog::occupancy_reserve);
}

namespace {
struct Fiber {
    ucontext_t start;
    bool started = false;
    jmp_buf at;  // (no system call between lanes, as swapcontext makes)
    std::unique_ptr<char[]> stack;
    void *fake = nullptr;
    unsigned lane = 0;
};
constexpr size_t kStack = 512 << 10;
ucontext_t g_unused;
jmp_buf g_main;
void *g_main_fake;
const void *g_main_bottom;
size_t g_main_size;
Fiber *g_fiber;  // the one that runs, or null
unsigned g_next, g_lanes;
bool g_ended;
const std::function<void(unsigned)> *g_body;

void to_main()
{
    Fiber *f = g_fiber;
    __sanitizer_start_switch_fiber(&f->fake, g_main_bottom, g_main_size);
    if (!_setjmp(f->at))
        _longjmp(g_main, 1);
    __sanitizer_finish_switch_fiber(f->fake, &g_main_bottom, &g_main_size);
}

// Lane after lane as long as they run to their end.
void fiber_main()
{
    __sanitizer_finish_switch_fiber(nullptr, &g_main_bottom, &g_main_size);
    for (;;) {
        while (g_next < g_lanes) {
            Fiber *f = g_fiber;
            f->lane = g_next++;
            threadIdx = {f->lane, 0, 0};
            (*g_body)(f->lane);
        }
        g_ended = true;
        to_main();
    }
}

bool run(Fiber *f)  // false: it waits at a barrier
{
    g_fiber = f;
    g_ended = false;
    threadIdx = {f->lane, 0, 0};
    __sanitizer_start_switch_fiber(&g_main_fake, f->stack.get(), kStack);
    if (!_setjmp(g_main)) {
        if (f->started)
            _longjmp(f->at, 1);
        f->started = true;
        swapcontext(&g_unused, &f->start);
    }
    __sanitizer_finish_switch_fiber(g_main_fake, nullptr, nullptr);
    g_fiber = nullptr;
    return g_ended;
}
}  // namespace

void emu_wait()
{
    if (!g_fiber)
        return;
    to_main();
}

void emu_workgroup(unsigned lanes, const std::function<void(unsigned)> &body)
{
    static std::vector<std::unique_ptr<Fiber>> fibers;
    static std::vector<Fiber *> idle;
    g_next = 0;
    g_lanes = lanes;
    g_body = &body;
    std::vector<Fiber *> waiting;
    const auto turn = [&](Fiber *f) { (run(f) ? idle : waiting).push_back(f); };
    while (g_next < lanes) {
        if (idle.empty()) {
            fibers.emplace_back(new Fiber);
            Fiber *f = fibers.back().get();
            f->stack.reset(new char[kStack]);
            getcontext(&f->start);
            f->start.uc_stack.ss_sp = f->stack.get();
            f->start.uc_stack.ss_size = kStack;
            f->start.uc_link = nullptr;
            makecontext(&f->start, fiber_main, 0);
            idle.push_back(f);
        }
        Fiber *f = idle.back();
        idle.pop_back();
        f->lane = g_next;
        turn(f);
    }
    while (!waiting.empty()) {
        std::vector<Fiber *> now;
        now.swap(waiting);
        for (Fiber *f : now)
            turn(f);
    }
}
