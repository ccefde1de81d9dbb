// Batched launches: every launch of a call on one stream, results in one go.
//
// A prepared batch holds what its launches read on the device: claim counters, best[] and the
// descriptors of all its cones.  The descriptors are uploaded once; after each call the finish
// kernel copies best[] to pinned host memory and returns the control block to its state before
// a launch, so a call with the same circuits and kernels uploads and reads back nothing.
#include <algorithm>
#include <cstring>

#include "runtime.hpp"

namespace fes {
namespace {

struct Prepared {
    std::mutex mu;  // one call at a time
    bool spoilt = false;  // a call failed: its control block is no longer known to be clean
    int device = 0;
    std::vector<uint64_t> key;
    std::vector<std::shared_ptr<JitKernel>> kernels;  // kept while their code may run
    Buffer buf;
    size_t best_off = 0, claim_words = 0, n = 0;
    struct Launch {
        InterpLaunch L{};
        Schedule sch;
        bool native = false;
        NativeMany many;
    };
    std::vector<Launch> launches;
    uint64_t last_use = 0;
    Device* dev = nullptr;
    ~Prepared() {
        if (dev && buf.dev) dev->release(buf);
    }
};

// At most this many are kept per process (least recently used dropped).
constexpr size_t kMaxPrepared = 16;
std::mutex g_mu;
std::vector<std::shared_ptr<Prepared>>& kept() {
    static auto* v = new std::vector<std::shared_ptr<Prepared>>;  // outlives the HIP runtime's own statics
    return *v;
}
uint64_t g_clock = 0;

std::vector<uint64_t> key_of(const std::vector<BatchPart>& parts, size_t n) {
    std::vector<uint64_t> k{n};
    for (const BatchPart& p : parts) {
        k.push_back(p.native.empty() ? 1 : 2);
        k.push_back(p.entries.size());
        for (size_t i = 0; i < p.entries.size(); ++i) {
            k.push_back(p.entries[i]);
            k.push_back(p.ranges[i].begin);
            k.push_back(p.ranges[i].end);
            k.push_back(p.native.empty() ? p.cs[i]->uid : (uint64_t)(uintptr_t)p.native[i].get());
        }
        if (p.native.empty())
            for (uint64_t x : {(uint64_t)p.sch.K, (uint64_t)p.sch.B, (uint64_t)p.sch.block, (uint64_t)p.sch.grid,
                               (uint64_t)p.sch.lds, (uint64_t)p.sch.regs, p.sch.tile_hw})
                k.push_back(x);
    }
    return k;
}

std::shared_ptr<Prepared> prepare(Device& dev, const std::vector<BatchPart>& parts, size_t n, hipStream_t stream,
                                  std::vector<uint64_t> key) {
    auto b = std::make_shared<Prepared>();
    b->device = dev.ordinal;
    b->dev = &dev;
    b->key = std::move(key);
    b->n = n;
    // Claim counters: one set per interpreter launch, one per native register tier.
    size_t sets = 0, interp_cones = 0, native_cones = 0, file_bytes = 0;
    for (const BatchPart& p : parts) {
        if (!p.native.empty()) {
            sets += kNativeTiers;
            native_cones += p.native.size();
            continue;
        }
        ++sets;
        interp_cones += p.cs.size();
        if (!p.sch.lds && !p.sch.regs)  // the launches run one after the other: one set of value files
            file_bytes = std::max<size_t>(file_bytes, (size_t)p.sch.grid * (p.sch.block / 64) * rows_for(p.cs, p.sch.B) *
                                                          64ull * p.sch.K * 4ull);
    }
    b->claim_words = sets * (kClaimBytes / 8);
    b->best_off = sets * kClaimBytes;
    const size_t interp_off = (b->best_off + 8 * (n + 1) + 63) & ~size_t(63);
    const size_t native_off = (interp_off + sizeof(ConeDesc) * interp_cones + 63) & ~size_t(63);
    const size_t files_off = (native_off + sizeof(NativeDesc) * native_cones + 255) & ~size_t(255);
    b->buf = dev.acquire(files_off + file_bytes, files_off);
    uint8_t *host = (uint8_t*)b->buf.host, *devp = (uint8_t*)b->buf.dev;
    std::memset(host, 0, b->best_off);
    std::memset(host + b->best_off, 0xFF, 8 * n);
    size_t set = 0, cone = 0, kernel = 0;
    for (const BatchPart& p : parts) {
        Prepared::Launch l;
        std::vector<uint32_t> at(p.entries.begin(), p.entries.end());
        if (!p.native.empty()) {
            l.native = true;
            const size_t off = native_off + sizeof(NativeDesc) * kernel;
            l.many = native_many_fill(dev, p.native, p.ranges, at, (NativeDesc*)(host + off),
                                      (const NativeDesc*)(devp + off), devp + set * kClaimBytes,
                                      (unsigned long long*)(devp + b->best_off));
            b->kernels.insert(b->kernels.end(), p.native.begin(), p.native.end());
            set += kNativeTiers;
            kernel += p.native.size();
        } else {
            const size_t off = interp_off + sizeof(ConeDesc) * cone;
            l.sch = p.sch;
            l.L.total_items = build_descs(dev, p.cs, p.ranges, at, p.sch, stream, (ConeDesc*)(host + off));
            l.L.cones = (const ConeDesc*)(devp + off);
            l.L.num_cones = (uint32_t)p.cs.size();
            l.L.rows_max = rows_for(p.cs, p.sch.B);
            l.L.ctl = (LaunchCtl*)(devp + set * kClaimBytes);
            l.L.best = (unsigned long long*)(devp + b->best_off);
            l.L.hbm_rows = (p.sch.lds || p.sch.regs) ? nullptr : (uint32_t*)(devp + files_off);
            l.L.cancel = nullptr;
            const uint64_t per_block = (uint64_t)(p.sch.block / 64);
            l.sch.grid = (int)std::min<uint64_t>((uint64_t)p.sch.grid, (l.L.total_items + per_block - 1) / per_block);
            ++set;
            cone += p.cs.size();
        }
        b->launches.push_back(std::move(l));
    }
    FES_HIP(hipMemcpyAsync(devp, host, files_off, hipMemcpyHostToDevice, stream));
    FES_HIP(hipStreamSynchronize(stream));  // other calls may use it on other streams
    return b;
}

// After a failed call: launches of it may still run, on memory and code that b holds.
void give_up(const std::shared_ptr<Prepared>& b, hipStream_t stream) {
    b->spoilt = true;
    {
        std::lock_guard<std::mutex> g(g_mu);
        auto& v = kept();
        v.erase(std::remove(v.begin(), v.end(), b), v.end());
    }
    if (hipStreamSynchronize(stream) != hipSuccess) new std::shared_ptr<Prepared>(b);  // kept for good
}

void run_batch(Device& dev, const std::vector<BatchPart>& parts, size_t n, hipStream_t stream,
               std::vector<uint64_t>& best, double* ms) {
    const std::vector<uint64_t> key = key_of(parts, n);
    std::shared_ptr<Prepared> b;
    std::unique_lock<std::mutex> one;
    for (;;) {
        b = nullptr;
        {
            std::lock_guard<std::mutex> g(g_mu);
            for (auto& x : kept())
                if (x->device == dev.ordinal && x->key == key) b = x;
            if (b) b->last_use = ++g_clock;
        }
        if (!b) {
            b = prepare(dev, parts, n, stream, key);
            std::lock_guard<std::mutex> g(g_mu);
            auto& v = kept();
            if (v.size() >= kMaxPrepared)
                v.erase(std::min_element(v.begin(), v.end(),
                                         [](const auto& x, const auto& y) { return x->last_use < y->last_use; }));
            b->last_use = ++g_clock;
            v.push_back(b);
        }
        one = std::unique_lock<std::mutex>(b->mu);
        if (!b->spoilt) break;  // another thread's call failed meanwhile
        one.unlock();
    }
    uint8_t *host = (uint8_t*)b->buf.host, *devp = (uint8_t*)b->buf.dev;
    unsigned long long* const found = (unsigned long long*)(host + b->best_off);
    double t = 0;
    try {
        __atomic_store_n(found + n, kPending, __ATOMIC_RELEASE);
        for (const Prepared::Launch& l : b->launches) {
            if (l.native) native_many_enqueue(l.many, stream);
            else if (l.L.num_cones) FES_HIP(launch_schedule(l.L, l.sch, stream));
        }
        FES_HIP(launch_finish((unsigned long long*)devp, (uint32_t)b->claim_words,
                              (unsigned long long*)(devp + b->best_off), (uint32_t)n, found, stream));
        t = wait_finished(found + n, stream);
    } catch (...) {
        give_up(b, stream);
        throw;
    }
    if (ms) *ms = t;
    best.assign((uint64_t*)found, (uint64_t*)found + n);
}

const bool g_registered = (register_batch_runner(&run_batch), true);

}  // namespace

// A batch of one interpreter launch.
void run_batch_graph(Device& dev, const std::vector<Circuit*>& cs, const std::vector<HwRange>& ranges,
                     const Schedule& sch, hipStream_t stream, std::vector<uint64_t>& best, double* ms) {
    BatchPart p;
    p.cs = cs;
    p.ranges = ranges;
    p.sch = sch;
    for (size_t i = 0; i < cs.size(); ++i) p.entries.push_back(i);
    run_batch(dev, {p}, cs.size(), stream, best, ms);
}

}  // namespace fes
