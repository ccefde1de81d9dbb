// Interpreter schedule autotuner.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <numeric>

#include "runtime.hpp"

namespace fes {
namespace {

struct TuneKey {
    int device;
    uint32_t rows_log2, cones_log2, work_log2;
    bool hbm;
    bool operator<(const TuneKey& o) const {
        return std::tie(device, rows_log2, cones_log2, work_log2, hbm) <
               std::tie(o.device, o.rows_log2, o.cones_log2, o.work_log2, o.hbm);
    }
};

uint32_t log2_bucket(double x) {
    uint32_t b = 0;
    while (x >= 2.0) {
        x /= 2.0;
        ++b;
    }
    return b;
}

std::mutex g_tune_mu;
std::map<TuneKey, Schedule>& tune_cache() {
    static std::map<TuneKey, Schedule> m;
    return m;
}

}  // namespace

Schedule autotune(Device& dev, const std::vector<Circuit*>& cs, const std::vector<HwRange>& ranges, hipStream_t stream,
                  bool hbm) {
    // FASTLEC_ES_TUNE_FORCE="K,B,block" takes that candidate, when it fits, without timing
    // (a test hook for schedule-dependent paths).
    const char* force = std::getenv("FASTLEC_ES_TUNE_FORCE");
    // Value files that fit the register tier run there: five times the rate of LDS files, so no
    // other candidate is worth its timing (and the streams of two more bundle sizes).
    Schedule regs;
    if (!hbm && !force && make_schedule_regs(dev, rows_for(cs, 4), regs)) return regs;
    double work = 0;
    for (size_t i = 0; i < cs.size(); ++i)
        work += (double)cs[i]->plan1.num_gate_instrs * 32.0 * (double)(ranges[i].end - ranges[i].begin);
    TuneKey key{dev.ordinal, log2_bucket(rows_for(cs, 8)), log2_bucket((double)cs.size()), log2_bucket(work), hbm};
    {
        // A cached choice is re-fitted to this batch: the key buckets the value-file rows, and
        // within a bucket a larger cone may no longer fit the chosen workgroup in LDS.
        std::lock_guard<std::mutex> g(g_tune_mu);
        auto it = tune_cache().find(key);
        if (it != tune_cache().end()) {
            Schedule s;
            if (make_schedule(dev, cs, it->second.K, it->second.B, it->second.block, it->second.lds, s)) return s;
            trace("autotune: cached K=%d B=%d block=%d does not fit this batch; re-tuning", it->second.K,
                  it->second.B, it->second.block);
        }
    }
    // Bounded sample: a prefix of every cone, about 2e11 gate evaluations in total.
    const double budget = 2e11;
    std::vector<HwRange> sample(ranges.size());
    double sample_work = 0;
    for (size_t i = 0; i < cs.size(); ++i) {
        const double per_hw = 32.0 * std::max<uint32_t>(1, cs[i]->plan1.num_gate_instrs);
        uint64_t hw = (uint64_t)std::max(512.0, budget / (double)cs.size() / per_hw);
        hw = std::min<uint64_t>(hw, ranges[i].end - ranges[i].begin);
        sample[i] = HwRange{ranges[i].begin, ranges[i].begin + hw};
        sample_work += per_hw * (double)hw;
    }
    std::vector<Schedule> cands;
    for (int K : {1, 2, 4})
        for (int B : {4, 8, 16})
            for (int block : {64, 128, 256}) {
                if (B == 16 && K > 2) continue;  // 16 bundles of 4 words per lane spill registers
                Schedule s;
                if (make_schedule(dev, cs, K, B, block, !hbm, s)) cands.push_back(s);
            }
    // Device-memory files with one or two words per lane compete with the LDS candidates (files too
    // large for registers leave at most two waves per CU in LDS).
    if (!hbm)
        for (int K : {1, 2})
            for (int B : {8, 16})
                for (int block : {64, 128}) {
                    Schedule s;
                    if (make_schedule(dev, cs, K, B, block, false, s)) cands.push_back(s);
                }
    if (cands.empty()) {
        fastlec_es_options o{};
        o.kernel = hbm ? FASTLEC_KERNEL_INTERP_HBM : FASTLEC_KERNEL_INTERP;
        cands.push_back(default_schedule(dev, cs, &o));
    }
    Schedule best = cands[0];
    double best_rate = -1;
    std::vector<uint64_t> b;
    double ms = 0;
    if (const char* f = force) {
        int fk = 0, fb = 0, fw = 0;
        if (std::sscanf(f, "%d,%d,%d", &fk, &fb, &fw) == 3)
            for (const Schedule& s : cands)
                if (s.K == fk && s.B == fb && s.block == fw) {
                    std::lock_guard<std::mutex> g(g_tune_mu);
                    tune_cache()[key] = s;
                    return s;
                }
    }
    run_interp(dev, cs, sample, cands[0], stream, nullptr, b, &ms);  // uploads programs, warms caches
    for (const Schedule& s : cands) {
        run_interp(dev, cs, sample, s, stream, nullptr, b, &ms);
        const double rate = sample_work / std::max(1e-3, (double)ms);
        trace("autotune: K=%d B=%d block=%d grid=%d %s -> %.3f ms", s.K, s.B, s.block, s.grid,
              s.lds ? "lds" : "hbm", ms);
        if (rate > best_rate) {
            best_rate = rate;
            best = s;
        }
    }
    std::lock_guard<std::mutex> g(g_tune_mu);
    tune_cache()[key] = best;
    return best;
}

}  // namespace fes
