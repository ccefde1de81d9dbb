// Data layouts shared by the native tier's host code and its kernel (native/es_native.hip).
#pragma once
#include <cstdint>

namespace fes {

// Work claims are spread over C = min(kClaimCounters, waves in the grid) counters, each on
// its own 128-byte line: the wave with global index w claims from counter s = w % C and gets
// the items s, s + C, s + 2C, ... in that order.  One shared counter
// serialises every claim of the launch at the atomic unit (about 30 ns each), which bounds
// launches of many short work items; spread over separate lines the claims proceed in
// parallel, and the items still start in roughly ascending order.
constexpr uint32_t kClaimCounters = 16;
constexpr uint32_t kClaimStride = 16;  // 64-bit words from one counter to the next (128 bytes)
// Word of the claim block where a launch's first workgroup notes when it starts (realtime counter,
// 100 MHz); the finish kernel makes the launch's time of it.
constexpr uint32_t kStartWord = 1;

constexpr uint32_t kMaxInner = 5;  // inner inputs of a native pass: up to 2^5 assignments

// One circuit of a native launch.  Half-word h holds patterns 32h .. 32h+31.
struct NativeDesc {
    uint64_t code_offset;  // of its pass in the generated section
    uint64_t hw_begin;     // checked range, real half-words
    uint64_t hw_end;
    uint64_t u_first;      // packed half-words covered (inner positions removed)
    uint64_t u_end;
    uint64_t tile_hw;      // packed half-words per work item (multiple of 64)
    uint64_t item_begin;   // first work item of this cone in the launch
    uint32_t best_index;
    uint32_t inner;                 // inner inputs
    uint32_t inner_bit[kMaxInner];  // their bits of the real half-word index, ascending
    uint32_t pad;
};
static_assert(sizeof(NativeDesc) == 88, "descriptor layout");

struct NativeLaunch {
    const NativeDesc* cones;  // device array, or null for a launch of the single cone `one`
    uint32_t num_cones;
    uint64_t total_items;
    unsigned long long* counters;  // claim counters, zero before the launch
    unsigned long long* best;      // per cone: lowest failing pattern, ~0 = none yet
    NativeDesc one;
};

// A native simulation pass (native_sim.cpp): columns [0, words) of the caller's input words, in items of
// one column per thread of a workgroup.
struct SimLaunch {
    uint64_t code_offset;
    const uint32_t* pi;
    uint32_t* sig;
    uint64_t words;  // below 2^30
    uint64_t items;
    unsigned long long* counters;  // claim block, for kStartWord only
};

}  // namespace fes
