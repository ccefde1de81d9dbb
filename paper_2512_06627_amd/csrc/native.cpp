// Native tier on the device: kernels per circuit, modules and launches.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <numeric>
#include <thread>

#include "native.hpp"
#include "runtime.hpp"

namespace fes {
namespace {

// Test hook: FASTLEC_ES_NATIVE_INNER fixes the number of inner inputs (where the circuit has them).
int forced_inner() {
    const char* v = std::getenv("FASTLEC_ES_NATIVE_INNER");
    return v && *v ? std::atoi(v) : -1;
}

// Inner inputs of checks that cover `span` half-words at a time: any input for the whole space,
// else inputs whose block of patterns is at most a sixteenth of the span (a range is covered in
// whole blocks, so its ragged ends cost at most an eighth more).  Steps of three inputs keep the
// number of kernels per circuit small.
uint32_t inner_limit(const Circuit& c, uint64_t span) {
    const uint32_t n = c.plan1.num_inputs;
    if (n <= 11 || span >= 1ull << (n - 5)) return std::max<uint32_t>(n, 11);
    uint32_t q = 0;
    while (q < 58 && (span >> (q + 1))) ++q;
    const int top = (int)q + 5 - 4;
    return top <= 11 ? 11 : 11 + (uint32_t)(top - 11) / 3 * 3;
}

double passes_of(double patterns) { return std::max(1.0, patterns / 2048.0); }

std::shared_ptr<JitKernel> ready(Circuit& c, uint64_t span) {
    std::lock_guard<std::mutex> g(c.mu);
    auto it = c.native.find(inner_limit(c, span));
    return it == c.native.end() ? nullptr : it->second;
}

// A build that found no choice of inner inputs to fit is not repeated: native_refused holds its limit, with
// true when every choice was tried (weight 0; a build that weighs its own time tries a few).  Such a
// build is as long as one that succeeds: 27,000 gates 28 ms, for a check of 0.3 ms on the interpreter.
bool refused(const Circuit& c, uint64_t span, double weight) {
    std::lock_guard<std::mutex> g(c.mu);
    auto it = c.native_refused.find(inner_limit(c, span));
    return it != c.native_refused.end() && (weight > 0 || it->second);
}

std::shared_ptr<JitKernel> get(Circuit& c, uint64_t span, double weight, const std::atomic<bool>* stop) {
    if (auto k = ready(c, span)) return k;
    if (refused(c, span, weight)) return nullptr;
    std::unique_lock<std::mutex> build(c.native_mu, std::defer_lock);
    while (stop && !build.try_lock()) {  // another thread's build of this circuit
        if (stop->load(std::memory_order_relaxed)) return nullptr;
        std::this_thread::sleep_for(std::chrono::microseconds(50));
    }
    if (!stop) build.lock();
    if (auto k = ready(c, span)) return k;
    if (refused(c, span, weight)) return nullptr;
    const uint32_t limit = inner_limit(c, span);
    const double patterns = 32.0 * (double)span;
    std::shared_ptr<NativeKernel> n;
    const int inner = forced_inner();
    if (inner >= 0) n = build_native(c.aig, c.plan1.order, limit, passes_of(patterns), 0, inner);
    if (!n) n = build_native(c.aig, c.plan1.order, limit, passes_of(patterns), weight, -1, stop);
    if (!n) {
        if (stop && stop->load(std::memory_order_relaxed)) return nullptr;
        trace("native: no kernel with inner inputs below %u fits", limit);
        std::lock_guard<std::mutex> g(c.mu);
        bool& all = c.native_refused[limit];
        all = all || weight <= 0;
        c.interp_ms_spent.store(0, std::memory_order_relaxed);  // it has bought this
        c.serve_ms_waited.store(0, std::memory_order_relaxed);
        return nullptr;
    }
    auto k = std::make_shared<JitKernel>();
    k->native = n;
    k->name = n->waves == 4 ? "fes_native_128" : n->waves == 3 ? "fes_native_168" : "fes_native_256";
    k->waves_per_eu = k->waves_used = n->waves;
    k->block = 64;
    std::vector<uint64_t> at;
    k->code = std::make_shared<CodeObject>();
    k->code->bytes = std::make_shared<const std::vector<char>>(native_code_object({&n->code}, &at));
    trace("native: %zu inner inputs, %u VALU and %u LDS instructions, %d waves per SIMD, built in %.2f ms",
          n->bits.size(), n->code.valu, n->code.lds, n->waves, n->build_ms);
    std::lock_guard<std::mutex> g(c.mu);
    c.native[limit] = k;
    c.interp_ms_spent.store(0, std::memory_order_relaxed);
    c.serve_ms_waited.store(0, std::memory_order_relaxed);
    return k;
}

double run_ms(const JitKernel& k, double patterns) {
    const NativeKernel& n = *k.native;
    return 0.003 + native_run_ms(n.code.valu + n.code.lds, (uint32_t)n.bits.size(), passes_of(patterns));
}

std::shared_ptr<JitKernel> best(Circuit& c, const HwRange& r, uint64_t span, double* ms, double* aim) {
    const uint32_t limit = inner_limit(c, span);
    const uint64_t size = r.end - r.begin, pieces = span < size ? (size + span - 1) / span : 1;
    std::shared_ptr<JitKernel> pick;
    std::lock_guard<std::mutex> g(c.mu);
    for (auto& kv : c.native) {
        // A range is covered in whole blocks of patterns up to the highest inner input, a piece of it with
        // about one block too many.
        const uint32_t block = kv.second->native->bits.empty() ? 0 : kv.second->native->bits.back() + 1;
        const uint64_t covered = pieces > 1 ? size + (block ? pieces << block : 0)
                                            : (((r.end + ((1ull << block) - 1)) >> block) - (r.begin >> block)) << block;
        const double t = run_ms(*kv.second, 32.0 * (double)covered);
        if (pick && t >= *ms) continue;
        pick = kv.second;
        *ms = t;
        *aim = kv.first == limit ? t : kv.first > limit ? run_ms(*kv.second, 32.0 * (double)size) : 0.0;
    }
    return pick;
}

double share_ms(const JitKernel& k, double patterns) {
    const NativeKernel& n = *k.native;
    return std::ceil(passes_of(patterns) / (double)(1u << n.bits.size())) * (n.code.valu + n.code.lds + 200) * 1.0e-9;
}

double guess_run_ms(const Circuit& c, double patterns) {
    return 0.003 + native_run_ms(0.26 * c.plan1.num_ands_tfi + 10, 0, passes_of(patterns));
}

double guess_build_ms(const Circuit& c) { return native_build_ms(c.plan1.num_ands_tfi); }

void counts(const JitKernel& k, uint32_t* inner, uint32_t* valu, uint32_t* waves) {
    if (inner) *inner = (uint32_t)k.native->bits.size();
    if (valu) *valu = k.native->code.valu;
    if (waves) *waves = (uint32_t)k.native->waves;
}

// Descriptor of kernel k over range r, its work items numbered from item_begin; returns the next
// free item number.
uint64_t fill(const NativeKernel& k, uint64_t code_offset, const HwRange& r, uint64_t tile_hw, uint64_t waves,
              uint64_t item_begin, uint32_t best_index, NativeDesc& d) {
    d = NativeDesc{};
    d.code_offset = code_offset;
    d.hw_begin = r.begin;
    d.hw_end = r.end;
    d.inner = (uint32_t)k.bits.size();
    for (uint32_t j = 0; j < d.inner; ++j) d.inner_bit[j] = k.bits[j];
    if (d.inner == 0) {
        d.u_first = r.begin / 64 * 64;
        d.u_end = r.end;
    } else {  // whole blocks of patterns up to the highest inner input
        const uint32_t block = k.bits.back() + 1, packed = block - d.inner;
        d.u_first = (r.begin >> block) << packed;
        d.u_end = ((r.end + ((1ull << block) - 1)) >> block) << packed;
    }
    const uint64_t span = d.u_end - d.u_first;
    // About 16 work items per wave, of one to 64 passes.
    uint64_t tile = tile_hw >> d.inner;
    if (!tile_hw) {
        const uint64_t target = span / std::max<uint64_t>(1, waves * 16);
        tile = 64;
        while (tile < target && tile < 64ull * 64) tile *= 2;
    }
    d.tile_hw = std::max<uint64_t>(64, (tile + 63) / 64 * 64);
    d.item_begin = item_begin;
    d.best_index = best_index;
    return item_begin + (span + d.tile_hw - 1) / d.tile_hw;
}

hipFunction_t function_of(Device& dev, JitKernel& k) {
    std::lock_guard<std::mutex> g(k.mu);
    auto it = k.per_device.find(dev.ordinal);
    if (it != k.per_device.end()) return it->second;
    hipFunction_t fn;
    FES_HIP(hipModuleGetFunction(&fn, k.code->module(dev.ordinal), k.name.c_str()));
    k.per_device[dev.ordinal] = fn;
    return fn;
}

uint64_t resident_waves(const Device& dev, int waves_per_simd) {
    return (uint64_t)dev.prop.multiProcessorCount * 4 * waves_per_simd;
}

void launch(hipFunction_t fn, const NativeLaunch& L, uint64_t grid, uint32_t lds, hipStream_t stream) {
    void* args[] = {const_cast<NativeLaunch*>(&L)};
    trace("native launch: %u cones, %llu items, grid=%llu", L.num_cones, (unsigned long long)L.total_items,
          (unsigned long long)grid);
    FES_HIP(hipModuleLaunchKernel(fn, (unsigned)grid, 1, 1, 64, 1, 1, lds, stream, args, nullptr));
}

const NativeTier kTier = {ready, get, refused, best, run_ms, share_ms, guess_run_ms, guess_build_ms, counts};
const bool g_registered = (register_native_tier(&kTier), true);

}  // namespace

JitLaunchPlan native_prepare(Device& dev, JitKernel& k, const HwRange& r, uint64_t tile_hw) {
    const NativeKernel& n = *k.native;
    JitLaunchPlan lp;
    lp.native = true;
    lp.fn = function_of(dev, k);
    const uint64_t resident = resident_waves(dev, n.waves);
    lp.total_items = fill(n, 0, r, tile_hw, resident, 0, 0, lp.one);
    lp.grid = (int)std::min(lp.total_items, resident);
    lp.block = 64;
    lp.lds_bytes = n.code.lds_slots * 256;
    lp.hw_begin = r.begin;
    lp.hw_end = r.end;
    return lp;
}

void native_enqueue(const JitLaunchPlan& lp, uint64_t* next_item, uint64_t* best, hipStream_t stream) {
    NativeLaunch L{};
    L.cones = nullptr;
    L.num_cones = 1;
    L.total_items = lp.total_items;
    L.counters = (unsigned long long*)next_item;
    L.best = (unsigned long long*)best;
    L.one = lp.one;
    launch(lp.fn, L, (uint64_t)lp.grid, lp.lds_bytes, stream);
}

NativeMany native_many_fill(Device& dev, const std::vector<std::shared_ptr<JitKernel>>& ks,
                            const std::vector<HwRange>& ranges, const std::vector<uint32_t>& best_index,
                            NativeDesc* host_descs, const NativeDesc* dev_descs, uint8_t* claims,
                            unsigned long long* best) {
    NativeMany m;
    std::vector<const NativeCode*> codes;
    for (auto& k : ks) codes.push_back(&k->native->code);
    std::vector<uint64_t> at;
    m.code = std::make_shared<CodeObject>();
    m.code->bytes = std::make_shared<const std::vector<char>>(native_code_object(codes, &at));
    // Longest first within a register tier, so that the short ones fill the end of the launch.
    std::vector<size_t> order(ks.size());
    std::iota(order.begin(), order.end(), 0);
    std::vector<double> cost(ks.size());
    for (size_t i = 0; i < ks.size(); ++i) cost[i] = share_ms(*ks[i], 32.0 * (double)(ranges[i].end - ranges[i].begin));
    std::stable_sort(order.begin(), order.end(), [&](size_t a, size_t b) { return cost[a] > cost[b]; });
    size_t next = 0;
    for (int t = 0; t < kNativeTiers; ++t) {
        NativeManyLaunch& g = m.tier[t];
        const int waves = 4 - t;
        const uint64_t resident = resident_waves(dev, waves);
        const size_t from = next;
        uint64_t items = 0;
        const char* name = nullptr;
        for (size_t i : order) {
            const NativeKernel& k = *ks[i]->native;
            if (k.waves != waves) continue;
            items = fill(k, at[i], ranges[i], 0, resident, items, best_index[i], host_descs[next++]);
            g.lds = std::max(g.lds, k.code.lds_slots * 256);
            name = ks[i]->name.c_str();
        }
        g.L.cones = dev_descs + from;
        g.L.num_cones = (uint32_t)(next - from);
        if (!g.L.num_cones) continue;
        g.L.total_items = items;
        g.L.counters = (unsigned long long*)(claims + (size_t)t * kClaimBytes);
        g.L.best = best;
        g.grid = std::min(items, resident);
        FES_HIP(hipModuleGetFunction(&g.fn, m.code->module(dev.ordinal), name));
    }
    return m;
}

void native_many_enqueue(const NativeMany& m, hipStream_t stream) {
    for (const NativeManyLaunch& g : m.tier)
        if (g.L.num_cones) launch(g.fn, g.L, g.grid, g.lds, stream);
}

}  // namespace fes
