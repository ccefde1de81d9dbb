// Host threads around native kernels under ThreadSanitizer: plain checks that build a kernel beside the
// interpreter, checks in pieces, and batches whose descriptors are kept, all on shared handles.
//
// Several threads check the same circuits until the library has built their kernels (AUTO counts what
// the interpreter takes), with deadlines, cancel flags and ranges in between; then threads run the same
// batches at once, so that they meet on one prepared batch.  Every answer must be the one that a single
// thread got first.  Control slots, the polling wait and the finish kernel's store take part
// in each call (native_device.cpp runs launches on a thread of its own).
//
// Usage: native_race_driver file.aig...   Prints "ok" on success.
#include <atomic>
#include <cstdio>
#include <fstream>
#include <iterator>
#include <string>
#include <thread>
#include <vector>

#include "fastlec_es.h"

namespace {

fastlec_es_circuit* load(const char* path) {
    std::ifstream f(path, std::ios::binary);
    const std::string s((std::istreambuf_iterator<char>(f)), std::istreambuf_iterator<char>());
    fastlec_es_circuit* c = nullptr;
    return fastlec_es_load_aig(s.data(), s.size(), &c) ? nullptr : c;
}

uint64_t answer(const fastlec_es_result& r) { return r.verdict == FASTLEC_NONEQUIVALENT ? r.cex : ~0ull; }

std::atomic<int> g_wrong{0};

void expect(bool ok, const char* what, size_t i) {
    if (ok) return;
    if (g_wrong.fetch_add(1) < 10) std::fprintf(stderr, "wrong: %s, circuit %zu: %s\n", what, i, fastlec_es_last_error());
}

template <class F>
void on_threads(int n, F f) {
    std::vector<std::thread> th;
    for (int t = 0; t < n; ++t) th.emplace_back(f, t);
    for (auto& t : th) t.join();
}

}  // namespace

int main(int argc, char** argv) {
    std::vector<fastlec_es_circuit*> cs;
    std::vector<uint64_t> want;
    fastlec_es_options o;
    fastlec_es_options_init(&o);
    for (int i = 1; i < argc; ++i) {
        cs.push_back(load(argv[i]));
        if (!cs.back()) return 1;
        fastlec_es_options po = o;
        po.kernel = FASTLEC_KERNEL_INTERP;
        fastlec_es_result r;
        if (fastlec_es_check(cs.back(), &po, &r)) return 2;
        want.push_back(answer(r));
    }
    on_threads(4, [&](int t) {
        volatile int never = 0;
        for (int round = 0; round < 40; ++round)
            for (size_t k = 0; k < cs.size(); ++k) {
                const size_t i = (k + (size_t)t) % cs.size();
                fastlec_es_options po = o;
                const int kind = (round + t) % 5;
                if (kind == 3) po.deadline_s = 3600;
                if (kind == 4) po.cancel_flag = &never;
                fastlec_es_result r;
                expect(!fastlec_es_check(cs[i], &po, &r) && answer(r) == want[i], "check", i);
                if (kind == 0) {  // the words below the counterexample are clean
                    po.end_word = want[i] == ~0ull ? 2 : want[i] / 64;
                    if (po.end_word)
                        expect(!fastlec_es_check(cs[i], &po, &r) && r.verdict == FASTLEC_EQUIVALENT, "range", i);
                }
            }
    });
    std::printf("checks: %d wrong\n", g_wrong.load());
    std::vector<fastlec_es_circuit*> fresh;
    for (int i = 1; i < argc; ++i) fresh.push_back(load(argv[i]));
    on_threads(3, [&](int t) {
        for (int round = 0; round < 12; ++round) {
            // The same handles in the same order meet on one prepared batch; the third thread's do not.
            std::vector<fastlec_es_circuit*> mix = t < 2 ? fresh : cs;
            if (round % 2) mix.insert(mix.end(), cs.begin(), cs.end());
            fastlec_es_options bo = o;
            bo.kernel = round % 3 == 2 ? FASTLEC_KERNEL_SPECIALIZED : FASTLEC_KERNEL_AUTO;
            std::vector<fastlec_es_result> r(mix.size());
            const bool ok = !fastlec_es_check_batch(mix.data(), mix.size(), &bo, r.data());
            for (size_t i = 0; i < mix.size(); ++i) expect(ok && answer(r[i]) == want[i % cs.size()], "batch", i);
        }
    });
    std::printf("batches: %d wrong\n", g_wrong.load());
    uint32_t native = 0;
    for (auto* c : cs) native += fastlec_es_native_info(c, nullptr, nullptr, nullptr) == 0;
    for (auto* c : cs) fastlec_es_free(c);
    for (auto* c : fresh) fastlec_es_free(c);
    if (g_wrong.load()) return 3;
    std::printf("%u native kernels\nok\n", native);
    return 0;
}
