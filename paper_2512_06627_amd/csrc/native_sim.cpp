// Native simulation passes on the device: when one pays, its module and its launch.
#include <algorithm>
#include <cmath>

#include "native.hpp"
#include "runtime.hpp"

namespace fes {

struct NativeSim {
    CodeObject code;
    int waves = 0;  // per SIMD; 0: the circuit's values do not fit
    uint32_t gates = 0;
    std::mutex mu;
    std::map<int, hipFunction_t> per_device;
};

namespace {

// Longer code than this is left to the interpreter (43k gates).
constexpr uint32_t kMaxCodeBytes = 1u << 20;
// Per gate of a wave alone: the interpreter's pass and the native one; bytes per ms that stores reach
// either way; building a pass per gate, and a module load.
constexpr double kInterpMs = 36e-6, kNativeMs = 13e-6, kBytesPerMs = 5.4e9, kBuildMs = 0.1e-3, kLoadMs = 1.0;

std::shared_ptr<NativeSim> build(const Aig& g) {
    auto k = std::make_shared<NativeSim>();
    k->gates = g.num_ands();
    NativeCode code;
    for (int waves : {4, 3, 2}) {
        if (24ull * g.num_ands() > kMaxCodeBytes) break;
        if (!emit_sim(g, waves == 4 ? 112 : waves == 3 ? 152 : 240, code)) continue;
        std::vector<uint64_t> at;
        k->code.bytes = std::make_shared<const std::vector<char>>(native_code_object({&code}, &at));
        k->waves = waves;
        break;
    }
    return k;
}

bool run(Device& dev, Circuit& c, const uint32_t* pi, uint64_t words, uint32_t* sig, hipStream_t stream,
         double* kernel_ms) {
    const uint32_t gates = c.aig.num_ands();
    if (words >= (1ull << 30) || !gates) return false;
    const uint64_t passes = (words + 63) / 64, cus = dev.prop.multiProcessorCount;
    std::shared_ptr<NativeSim> k;
    {
        std::lock_guard<std::mutex> g(c.mu);
        k = c.native_sim;
    }
    if (!k) {
        // Like a native kernel of a check (native_pays): built once the interpreter has taken as long as
        // building, where the chain of gates and not memory bounds it.  16x16 miter, 2^18 words: 1.05 ms
        // on the interpreter, 5.5 TB/s; 4.3k gates, 1,003 words: 179 us there, 71 native.
        const double rounds = std::ceil((double)passes / (double)(cus * 12));
        const double memory = 4.0 * (double)words * (c.aig.max_var() + 1.0) / kBytesPerMs;
        const double interp = std::max(kInterpMs * gates * rounds, memory);
        if (std::max(kNativeMs * gates * rounds, memory) > 0.8 * interp) return false;
        const double spent = c.sim_ms_spent.load(std::memory_order_relaxed) + interp;
        c.sim_ms_spent.store(spent, std::memory_order_relaxed);
        if (spent < 1.5 * (kBuildMs * gates + kLoadMs)) return false;
        std::lock_guard<std::mutex> one(c.native_sim_mu);
        {
            std::lock_guard<std::mutex> g(c.mu);
            k = c.native_sim;
        }
        if (!k) {
            k = build(c.aig);
            trace("native simulation: %u gates, %d waves per SIMD", k->gates, k->waves);
            std::lock_guard<std::mutex> g(c.mu);
            c.native_sim = k;
        }
    }
    if (!k->waves) return false;
    hipFunction_t fn;
    {
        std::lock_guard<std::mutex> g(k->mu);
        auto it = k->per_device.find(dev.ordinal);
        if (it == k->per_device.end()) {
            const char* name = k->waves == 4 ? "fes_sim_128" : k->waves == 3 ? "fes_sim_168" : "fes_sim_256";
            FES_HIP(hipModuleGetFunction(&fn, k->code.module(dev.ordinal), name));
            it = k->per_device.emplace(dev.ordinal, fn).first;
        }
        fn = it->second;
    }
    // One workgroup per CU and round, of as many waves as share the words out evenly.
    const uint64_t most = cus * 4 * k->waves, rounds = (passes + most - 1) / most;
    const uint64_t waves = (passes + cus * rounds - 1) / (cus * rounds);
    SimLaunch L{};
    L.pi = pi;
    L.sig = sig;
    L.words = words;
    L.items = (passes + waves - 1) / waves;
    const uint64_t grid = (L.items + rounds - 1) / rounds;
    trace("native simulation: %llu words, grid=%llu of %llu waves, %llu rounds", (unsigned long long)words,
          (unsigned long long)grid, (unsigned long long)waves, (unsigned long long)rounds);
    run_on_slot(dev, stream, kernel_ms, [&](const ControlSlot& s) {
        L.counters = s.claims();
        void* args[] = {&L};
        FES_HIP(hipModuleLaunchKernel(fn, (unsigned)grid, 1, 1, (unsigned)(64 * waves), 1, 1, 0, stream, args, nullptr));
    });
    return true;
}

const bool g_registered = (register_sim_runner(&run), true);

}  // namespace
}  // namespace fes
