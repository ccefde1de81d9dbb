// The native tier, its launches and the finish kernel on the host: what fake_device.cpp does not
// stand in for.  Test infrastructure only.
//
// It is linked with fake_device.cpp's object after objcopy has made that object's symbols weak, so
// that what is defined here takes their place, and has given four of them a second name
// (tests/standin.py), so that they can be called from here.
//
//   * Kernel launches run on one other thread, in order, as a device does; copies, events and
//     hipStreamSynchronize wait for it.  A caller that reads a result without waiting for the finish
//     kernel's store is thus a data race that the thread sanitizer sees.
//   * A native launch executes the generated machine code out of the module's .fescode section
//     (native_emulator.cpp), with the work items, the bound and the report routine of
//     native/es_native.hip.
//   * A launch without workgroups is refused, as by HIP.
//
// Switches for tests: FASTLEC_STANDIN_FAIL_LAUNCH=k fails the k-th kernel launch of the process (from 1),
// FASTLEC_STANDIN_LAUNCH_US=t makes every launch, and the call of one that fails, take t microseconds more,
// FASTLEC_STANDIN_SLOW_CLOCK=k makes launches seem k times as fast, FASTLEC_STANDIN_TRACE=1 prints launches
// and waits.
#include <elf.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <mutex>
#include <thread>

#include "kernels.hpp"
#include "native_emulator.hpp"
#include "runtime.hpp"

namespace {

long env_long(const char* name) {
    const char* v = std::getenv(name);
    return v && *v ? std::atol(v) : 0;
}

void note(const char* what) {
    static const bool on = env_long("FASTLEC_STANDIN_TRACE") != 0;
    if (on) std::fprintf(stderr, "standin: %s\n", what);
}

// One queue for all streams, on a thread that lives as long as the process.
class Queue {
public:
    void add(std::function<void()> f) {
        std::lock_guard<std::mutex> g(mu_);
        work_.push_back(std::move(f));
        cv_.notify_all();
    }
    void drain() {
        std::unique_lock<std::mutex> g(mu_);
        cv_.wait(g, [&] { return work_.empty(); });
    }
    static Queue& get() {
        static Queue* q = [] {
            auto* x = new Queue;
            std::thread([x] { x->loop(); }).detach();
            return x;
        }();
        return *q;
    }

private:
    void loop() {
        const long us = env_long("FASTLEC_STANDIN_LAUNCH_US");
        for (;;) {
            std::function<void()> f;
            {
                std::unique_lock<std::mutex> g(mu_);
                cv_.wait(g, [&] { return !work_.empty(); });
                f = work_.front();
            }
            if (us) std::this_thread::sleep_for(std::chrono::microseconds(us));
            f();
            std::lock_guard<std::mutex> g(mu_);
            work_.pop_front();  // what drain() waits for
            cv_.notify_all();
        }
    }
    std::mutex mu_;
    std::condition_variable cv_;
    std::deque<std::function<void()>> work_;
};

std::atomic<long> g_launches{0};

// Whether this launch may run (see FASTLEC_STANDIN_FAIL_LAUNCH).
hipError_t admit(uint64_t grid) {
    static const long fail = env_long("FASTLEC_STANDIN_FAIL_LAUNCH");
    if (grid == 0) return hipErrorInvalidConfiguration;
    if (g_launches.fetch_add(1) + 1 == fail) {
        std::this_thread::sleep_for(std::chrono::microseconds(env_long("FASTLEC_STANDIN_LAUNCH_US")));
        note("launch refused");
        return hipErrorLaunchFailure;
    }
    note("launch");
    return hipSuccess;
}

// The device's clock, in ticks of 10 ns.
uint64_t ticks() {
    using namespace std::chrono;
    static const long slow = std::max(1l, env_long("FASTLEC_STANDIN_SLOW_CLOCK"));
    return (uint64_t)duration_cast<nanoseconds>(steady_clock::now().time_since_epoch()).count() / 10 / (uint64_t)slow;
}

// A launch finds its claim counters at zero and leaves them used.
void claim(unsigned long long* counters) {
    using namespace fes;
    for (uint32_t i = 0; i < kClaimCounters; ++i)
        if (counters[i * kClaimStride]) std::fprintf(stderr, "standin: claim counter %u is not zero\n", i);
    counters[0] = 64;
    counters[kStartWord] = ticks();
}

struct Function {
    const char* module;
    std::string name;
};

const uint32_t* generated_code(const char* module) {
    Elf64_Ehdr eh;
    std::memcpy(&eh, module, sizeof eh);
    std::vector<Elf64_Shdr> sh(eh.e_shnum);
    std::memcpy(sh.data(), module + eh.e_shoff, sizeof(Elf64_Shdr) * sh.size());
    const char* names = module + sh[eh.e_shstrndx].sh_offset;
    for (const Elf64_Shdr& s : sh)
        if (!std::strcmp(names + s.sh_name, ".fescode")) return (const uint32_t*)(module + s.sh_offset);
    std::abort();
}

void run_native(const char* module, const fes::NativeLaunch& L) {
    const char* code = (const char*)generated_code(module);
    claim(L.counters);
    const fes::NativeDesc* cones = L.cones ? L.cones : &L.one;
    for (uint32_t k = 0; k < L.num_cones; ++k) {
        const fes::NativeDesc& c = cones[k];
        unsigned long long& best = L.best[c.best_index];
        for (uint64_t base = c.u_first; base < c.u_end; base += 64) {
            uint64_t real = base;
            for (uint32_t j = 0; j < c.inner; ++j) {
                const uint64_t low = (1ull << c.inner_bit[j]) - 1u;
                real = ((real & ~low) << 1) | (real & low);
            }
            if (32u * real >= best) break;
            best = std::min<unsigned long long>(
                best, emulate_pass((const uint32_t*)(code + c.code_offset), base, real, c.hw_begin, c.hw_end));
        }
    }
}

}  // namespace

extern "C" {

hipError_t hipStreamSynchronize(hipStream_t stream) {
    Queue::get().drain();
    char what[64];
    std::snprintf(what, sizeof what, "synchronize %p", (void*)stream);
    note(what);
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    Queue::get().drain();
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    Queue::get().drain();
    if (n) std::memmove(d, s, n);
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }

hipError_t hipModuleGetFunction(hipFunction_t* f, hipModule_t module, const char* name) {
    static std::mutex mu;
    static auto* all = new std::map<std::pair<const void*, std::string>, Function>;
    std::lock_guard<std::mutex> g(mu);
    auto it = all->emplace(std::make_pair((const void*)module, std::string(name)),
                           Function{(const char*)module, name}).first;
    *f = (hipFunction_t)&it->second;
    return hipSuccess;
}
hipError_t hipModuleLaunchKernel(hipFunction_t f, unsigned gx, unsigned, unsigned, unsigned, unsigned, unsigned,
                                 unsigned, hipStream_t, void** args, void**) {
    const Function fn = *(const Function*)f;
    if (fn.name.compare(0, 11, "fes_native_")) return hipErrorNotSupported;
    if (const hipError_t e = admit(gx)) return e;
    const fes::NativeLaunch L = *(const fes::NativeLaunch*)args[0];
    Queue::get().add([fn, L] { run_native(fn.module, L); });
    return hipSuccess;
}

}  // extern "C"

namespace fes {

hipError_t standin_interp(const InterpLaunch& L, int K, int B, bool lds, int grid, int block, hipStream_t s) asm("standin_interp");
hipError_t standin_regs(const InterpLaunch& L, int regs, int grid, hipStream_t s) asm("standin_regs");
JitLaunchPlan standin_prepare(Device& dev, JitKernel& k, const HwRange& r, uint64_t tile) asm("standin_prepare");
void standin_enqueue(const JitLaunchPlan& lp, uint64_t* next, uint64_t* best, const int* cancel, hipStream_t s) asm("standin_enqueue");

namespace {

template <class Launch>
hipError_t queue_interp(const InterpLaunch& L, int grid, Launch launch) {
    if (const hipError_t e = admit(grid > 0 ? grid : 0)) return e;
    Queue::get().add([L, launch] {
        InterpLaunch x = L;
        if (!x.cones) x.cones = &x.one;
        claim(x.ctl->next_item);
        (void)launch(x);
    });
    return hipSuccess;
}

}  // namespace

hipError_t launch_interp(const InterpLaunch& L, int K, int B, bool lds, int grid, int block, hipStream_t s) {
    return queue_interp(L, grid, [=](const InterpLaunch& x) { return standin_interp(x, K, B, lds, grid, block, s); });
}
hipError_t launch_interp_regs(const InterpLaunch& L, int regs, int grid, hipStream_t s) {
    if (L.rows_max > (uint32_t)regs) return hipErrorInvalidValue;
    return queue_interp(L, grid, [=](const InterpLaunch& x) { return standin_regs(x, regs, grid, s); });
}

hipError_t launch_finish(unsigned long long* claims, uint32_t words, unsigned long long* best, uint32_t n,
                         unsigned long long* host_best, hipStream_t) {
    if (const hipError_t e = admit(1)) return e;
    Queue::get().add([=] {
        const uint64_t now = ticks();
        uint64_t start = now;
        for (uint32_t i = kStartWord; i < words; i += kClaimCounters * kClaimStride)
            if (claims[i] && claims[i] < start) start = claims[i];
        for (uint32_t i = 0; i < n; ++i) {
            host_best[i] = best[i];
            best[i] = ~0ull;
        }
        std::memset(claims, 0, 8ull * words);
        __atomic_store_n(host_best + n, now - start, __ATOMIC_RELEASE);
    });
    return hipSuccess;
}

JitLaunchPlan jit_prepare(Device& dev, JitKernel& k, const HwRange& r, uint64_t tile) {
    return k.native ? native_prepare(dev, k, r, tile) : standin_prepare(dev, k, r, tile);
}
void jit_enqueue(const JitLaunchPlan& lp, uint64_t* next, uint64_t* best, const int* cancel, hipStream_t s) {
    if (lp.native) return native_enqueue(lp, next, best, s);
    Queue::get().drain();
    standin_enqueue(lp, next, best, cancel, s);
}
void run_jit(Device& dev, Circuit&, JitKernel& k, const HwRange& r, uint64_t tile, hipStream_t s, const int* cancel,
             uint64_t* best, double* kernel_ms, DevMem) {
    const JitLaunchPlan lp = jit_prepare(dev, k, r, tile);
    *best = run_on_slot(dev, s, kernel_ms, [&](const ControlSlot& slot) {
        jit_enqueue(lp, (uint64_t*)slot.claims(), (uint64_t*)slot.best(), cancel, s);
    });
}
hipModule_t CodeObject::module(int) { return (hipModule_t)bytes->data(); }

namespace {
const bool g_registered = (register_finish(&launch_finish), Queue::get().drain(), true);
}

}  // namespace fes
