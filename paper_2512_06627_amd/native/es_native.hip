// Host kernel of generated machine code (gfx950).
//
// A circuit's pass is straight-line machine code that the library writes itself
// (csrc/native_emit.cpp); this file is everything around it.  It is compiled once, when the
// library is built, into a code object whose last executable section, .fescode, is a place
// holder: at run time the library makes a copy of the code object with the generated passes of
// one or many circuits in that section and loads it as a module.  No compiler runs after the
// build, so a circuit's kernel costs milliseconds of planning and one module load instead of
// about 0.1 s of hipRTC.
//
// Work decomposition.  The circuit has k "inner" inputs; one call of its pass evaluates all 2^k
// assignments of them on the 2,048 patterns of a wave (64 lanes x 32 bits), sharing every value
// that does not depend on an inner input.  The remaining inputs form a packed space of
// 2^(n-k) patterns that is tiled like the interpreter's: waves claim work items in ascending
// order from the launch's claim counters.  A packed half-word index becomes the real one by a zero
// bit at each inner position; that is monotone, so an item whose first pattern is at or above the
// lowest failure found so far cannot lower it and is dropped.  A launch may hold many cones (each
// with its own code address).
//
// The pass is bound by VALU issue (one v_bitop3_b32 per three-input LUT; a wave issues at most one
// every five clocks, a SIMD one every two): one wave per workgroup, and as many of two to four waves
// per SIMD as the pass's registers allow.  16x16 miter without inner inputs, 2^32 patterns: 2.96 ms
// at four waves (1.10e12 instructions a second), 3.05 at three, 3.48 at two; with the four inner inputs
// that the library takes 0.77 ms at three (0.68 in calls one after the other), with five 0.71 at two.
//
// Contract with the generated code.  Inputs: v2..v7 lane words of inputs 5..10, v8 byte address
// of the lane's first LDS spill slot, s[38:39] packed half-word index, s[48:49] fes_native_report,
// s[42:43] real half-word index, s[44:47] the checked half-word range, s[50:51] its own address.
// Output: s[40:41], the lowest failing pattern seen (all ones before the first).  It may use v15 up
// to the kernel's register count, s36, s37, s52..s99, VCC and SCC, and returns to s[36:37].  Where a
// miter word is not zero it calls fes_native_report (return address in s[52:53]) with the word in
// v15, its nonzero lanes in VCC and the half-word offset of the inner assignment in s[54:55].
#include <hip/hip_runtime.h>

#include "../csrc/native_launch.hpp"

namespace {

using fes::kClaimCounters;
using fes::kClaimStride;
using fes::kStartWord;
using fes::NativeDesc;
using fes::NativeLaunch;
using fes::SimLaunch;

constexpr uint32_t kXcds = 8;  // workgroup b runs on XCD b % 8

#define FES_CONST __attribute__((address_space(4)))

__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Addresses of the generated section and of the report routine, relative to the kernel's own code.
__device__ __forceinline__ uint64_t code_base() {
    uint64_t a;
    asm volatile(
        "s_getpc_b64 s[36:37]\n"
        "s_add_u32 s36, s36, fes_native_code@rel32@lo+4\n"
        "s_addc_u32 s37, s37, fes_native_code@rel32@hi+12\n"
        "s_mov_b64 %0, s[36:37]\n"
        : "=s"(a)
        :
        : "s36", "s37", "scc");
    return a;
}
__device__ __forceinline__ uint64_t report_address() {
    uint64_t a;
    asm volatile(
        "s_getpc_b64 s[36:37]\n"
        "s_add_u32 s36, s36, fes_native_report@rel32@lo+4\n"
        "s_addc_u32 s37, s37, fes_native_report@rel32@hi+12\n"
        "s_mov_b64 %0, s[36:37]\n"
        : "=s"(a)
        :
        : "s36", "s37", "scc");
    return a;
}

#define V10(d) "v" #d "0", "v" #d "1", "v" #d "2", "v" #d "3", "v" #d "4", "v" #d "5", "v" #d "6", "v" #d "7", \
               "v" #d "8", "v" #d "9"
#define S10(d) "s" #d "0", "s" #d "1", "s" #d "2", "s" #d "3", "s" #d "4", "s" #d "5", "s" #d "6", "s" #d "7", \
               "s" #d "8", "s" #d "9"
#define SCLOB "s36", "s37", "s52", "s53", "s54", "s55", "s56", "s57", "s58", "s59", S10(6), S10(7), S10(8), S10(9)
#define VCLOB_128                                                                                            \
    "v15", "v16", "v17", "v18", "v19", V10(2), V10(3), V10(4), V10(5), V10(6), V10(7), V10(8), V10(9), V10(10), \
        V10(11), "v120", "v121", "v122", "v123", "v124", "v125", "v126", "v127"
#define VCLOB_168                                                                                            \
    "v15", "v16", "v17", "v18", "v19", V10(2), V10(3), V10(4), V10(5), V10(6), V10(7), V10(8), V10(9), V10(10), \
        V10(11), V10(12), V10(13), V10(14), V10(15), "v160", "v161", "v162", "v163", "v164", "v165", "v166", "v167"
#define VCLOB_256                                                                                          \
    VCLOB_168, "v168", "v169", V10(17), V10(18), V10(19), V10(20), V10(21), V10(22), V10(23), V10(24), "v250", \
        "v251", "v252", "v253", "v254", "v255"
#define PASS_OPERANDS                                                                                       \
    : "+{s[40:41]}"(found)                                                                                 \
    : "{s[38:39]}"(base), "{s[42:43]}"(real), "{s[44:45]}"(hw_begin), "{s[46:47]}"(hw_end),                  \
      "{s[48:49]}"(report), "{s[50:51]}"(code), "{v2}"(x5), "{v3}"(x6), "{v4}"(x7), "{v5}"(x8), "{v6}"(x9),     \
      "{v7}"(x10), "{v8}"(spill)

template <int R>
__device__ __forceinline__ void native_body(const NativeLaunch& L) {
    extern __shared__ uint32_t spill_area[];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t x5 = 0u - (lane & 1u), x6 = 0u - ((lane >> 1) & 1u), x7 = 0u - ((lane >> 2) & 1u);
    const uint32_t x8 = 0u - ((lane >> 3) & 1u), x9 = 0u - ((lane >> 4) & 1u), x10 = 0u - ((lane >> 5) & 1u);
    const uint32_t spill = (uint32_t)(unsigned long)(__attribute__((address_space(3))) uint32_t*)(spill_area + lane);
    const uint64_t base_code = uniform64(code_base()), report = uniform64(report_address());
    const uint32_t waves = gridDim.x;
    const uint32_t nclaim = waves < kClaimCounters ? waves : kClaimCounters;
    const uint32_t claim = __builtin_amdgcn_readfirstlane(blockIdx.x % nclaim);
    unsigned long long* const counter = L.counters + claim * kClaimStride;
    // Control flow stays wave-uniform: every lane takes part in the claim and in the atomicMin.
    // A claim adds 1 from each of the 64 lanes, which the compiler turns into one atomic of 64; a
    // value that differs by lane (1 from lane 0 only) becomes a 64-step scalar prefix loop.
    // A launch with a wave for every item claims nothing: wave w takes item w.
    if (blockIdx.x == 0 && lane == 0) L.counters[kStartWord] = __builtin_amdgcn_s_memrealtime();
    const bool one_each = L.total_items <= waves;
    for (bool more = true; more;) {
        uint64_t item = blockIdx.x;
        if (one_each) {
            more = false;
        } else {
            const uint64_t k = uniform64(atomicAdd(counter, 1ull)) >> 6;
            item = claim + k * nclaim;
        }
        if (item >= L.total_items) break;
        // A single cone's descriptor comes with the kernel's arguments: nothing to upload.
        const FES_CONST NativeDesc* cones = (const FES_CONST NativeDesc*)L.cones;
        if (!cones) cones = &((const FES_CONST NativeLaunch*)__builtin_amdgcn_kernarg_segment_ptr())->one;
        uint32_t lo = 0, hi = L.num_cones - 1;  // cone holding this item (uniform search)
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1) >> 1;
            if (cones[mid].item_begin <= item) lo = mid; else hi = mid - 1;
        }
        const FES_CONST NativeDesc* c = cones + lo;
        unsigned long long* const best = L.best + c->best_index;
        const uint64_t hw_begin = c->hw_begin, hw_end = c->hw_end, code = base_code + c->code_offset;
        const uint64_t u0 = c->u_first + (item - c->item_begin) * c->tile_hw;
        const uint64_t u_stop = min(u0 + c->tile_hw, c->u_end);
        const uint32_t inner = c->inner;
        // The bound found by other waves is read once per work item.
        uint64_t limit = uniform64(__hip_atomic_load(best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        for (uint64_t base = u0; base < u_stop; base += 64u) {
            uint64_t real = base;
            for (uint32_t j = 0; j < inner; ++j) {  // a zero bit at each inner position, lowest first
                const uint32_t at = c->inner_bit[j];
                const uint64_t low = (1ull << at) - 1u;
                real = ((real & ~low) << 1) | (real & low);
            }
            if (32u * real >= limit) {  // nothing at or above here can lower best
                more = more && (L.num_cones > 1 || base > u0);
                break;
            }
            uint64_t found = ~0ull;
            if constexpr (R == 128)
                asm volatile("s_swappc_b64 s[36:37], s[50:51]" PASS_OPERANDS
                             : SCLOB, "vcc", "scc", "memory", VCLOB_128);
            else if constexpr (R == 168)
                asm volatile("s_swappc_b64 s[36:37], s[50:51]" PASS_OPERANDS
                             : SCLOB, "vcc", "scc", "memory", VCLOB_168);
            else
                asm volatile("s_swappc_b64 s[36:37], s[50:51]" PASS_OPERANDS
                             : SCLOB, "vcc", "scc", "memory", VCLOB_256);
            if (found != ~0ull) {
                // Later passes of the item may still hold a lower failing pattern (another inner
                // assignment): they stop at the bound above.
                if (found < limit) limit = found;
                // Where most patterns fail every wave comes here in its first pass, and an atomic
                // on one address takes 25 ns: those that come after a lower pattern leave it out.
                const uint64_t now = uniform64(__hip_atomic_load(best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                if (found < now) atomicMin(best, (unsigned long long)found);
            }
        }
    }
}

// Simulation: the generated code loads the input words of the wave's 64 columns, stores row 0 and the
// input rows, then evaluates and stores gate by gate, rows ascending.  It has the registers from v15 up,
// the lane's byte offset in a row in v2, the addresses of the first input row and of row 0 in s[38:39]
// and s[40:41] (which it moves), the bytes of a row in s42 and the lanes that have a column in s[44:45].
// Adjacent workgroups share an XCD, and the code holds barriers that every wave of a workgroup reaches,
// so that the parts of cache lines at the ends of a ragged row's stores meet in L2.
template <int R>
__device__ __forceinline__ void sim_body(const SimLaunch& L) {
    const uint64_t code = uniform64(code_base()) + L.code_offset;
    if (blockIdx.x == 0 && threadIdx.x == 0) L.counters[kStartWord] = __builtin_amdgcn_s_memrealtime();
    const uint32_t xcds = min(gridDim.x, kXcds), xcd = blockIdx.x % xcds;
    const uint64_t share = L.items / xcds, odd = L.items % xcds;
    const uint64_t first = xcd * share + min((uint64_t)xcd, odd), stop = first + share + (xcd < odd ? 1u : 0u);
    const uint32_t step = (gridDim.x - xcd + xcds - 1u) / xcds;
    for (uint64_t item = first + blockIdx.x / xcds; item < stop; item += step) {
        const uint64_t w = item * blockDim.x + threadIdx.x;
        const uint64_t lanes = __ballot(w < L.words);
        const uint32_t off = (uint32_t)(w * 4u), row_bytes = (uint32_t)(L.words * 4u);
        uint64_t in = (uint64_t)L.pi, out = (uint64_t)L.sig;
#define SIM_OPERANDS                                                                              \
    : "+{s[38:39]}"(in), "+{s[40:41]}"(out)                                                       \
    : "{s42}"(row_bytes), "{s[44:45]}"(lanes), "{s[50:51]}"(code), "{v2}"(off)
        if constexpr (R == 128)
            asm volatile("s_swappc_b64 s[36:37], s[50:51]" SIM_OPERANDS : SCLOB, "vcc", "scc", "memory", VCLOB_128);
        else if constexpr (R == 168)
            asm volatile("s_swappc_b64 s[36:37], s[50:51]" SIM_OPERANDS : SCLOB, "vcc", "scc", "memory", VCLOB_168);
        else
            asm volatile("s_swappc_b64 s[36:37], s[50:51]" SIM_OPERANDS : SCLOB, "vcc", "scc", "memory", VCLOB_256);
#undef SIM_OPERANDS
    }
}

}  // namespace

// 128 registers per lane: four waves per SIMD; 168: three; 256: two.  The pass has those from v16 up.
extern "C" __global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4, 4)))
fes_native_128(NativeLaunch L) {
    native_body<128>(L);
}
extern "C" __global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3, 3)))
fes_native_168(NativeLaunch L) {
    native_body<168>(L);
}
extern "C" __global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2)))
fes_native_256(NativeLaunch L) {
    native_body<256>(L);
}

extern "C" __global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4, 4)))
fes_sim_128(SimLaunch L) {
    sim_body<128>(L);
}
extern "C" __global__ void __launch_bounds__(768) __attribute__((amdgpu_waves_per_eu(3, 3)))
fes_sim_168(SimLaunch L) {
    sim_body<168>(L);
}
extern "C" __global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
fes_sim_256(SimLaunch L) {
    sim_body<256>(L);
}

// Never launched: it holds the report routine and the place holder of the generated code.
//
// fes_native_report: VCC = lanes whose miter word (v15) is not zero, s[54:55] = half-word offset of
// the inner assignment.  Lanes outside the checked range [s[44:45], s[46:47]) are dropped; the
// lowest lane left and its lowest bit give the failing pattern, and s[40:41] keeps the lowest.
// Scalar code only, off the path of passes that find nothing.
extern "C" __global__ void fes_native_space() {
    asm volatile(
        ".pushsection .text\n"
        ".p2align 8\n"
        ".globl fes_native_report\n"
        ".hidden fes_native_report\n"
        "fes_native_report:\n"
        "s_add_u32 s56, s42, s54\n"  // half-word of lane 0
        "s_addc_u32 s57, s43, s55\n"
        "s_sub_u32 s58, s44, s56\n"  // lanes below the range
        "s_subb_u32 s59, s45, s57\n"
        "s_cbranch_scc1 fes_report_low_done\n"
        "s_cmp_lg_u32 s59, 0\n"
        "s_cbranch_scc1 fes_report_none\n"
        "s_cmp_gt_u32 s58, 63\n"
        "s_cbranch_scc1 fes_report_none\n"
        "s_lshl_b64 s[60:61], -1, s58\n"
        "s_and_b64 vcc, vcc, s[60:61]\n"
        "fes_report_low_done:\n"
        "s_sub_u32 s58, s46, s56\n"  // lanes inside the range's end
        "s_subb_u32 s59, s47, s57\n"
        "s_cbranch_scc1 fes_report_none\n"
        "s_cmp_lg_u32 s59, 0\n"
        "s_cbranch_scc1 fes_report_high_done\n"
        "s_cmp_gt_u32 s58, 63\n"
        "s_cbranch_scc1 fes_report_high_done\n"
        "s_lshl_b64 s[60:61], -1, s58\n"
        "s_andn2_b64 vcc, vcc, s[60:61]\n"
        "fes_report_high_done:\n"
        "s_cmp_eq_u64 vcc, 0\n"
        "s_cbranch_scc1 fes_report_none\n"
        "s_ff1_i32_b64 s58, vcc\n"
        "s_nop 4\n"
        "v_readlane_b32 s59, v15, s58\n"
        "s_add_u32 s56, s56, s58\n"
        "s_addc_u32 s57, s57, 0\n"
        "s_lshl_b64 s[56:57], s[56:57], 5\n"
        "s_ff1_i32_b32 s59, s59\n"
        "s_or_b32 s56, s56, s59\n"
        "s_sub_u32 s58, s56, s40\n"
        "s_subb_u32 s59, s57, s41\n"
        "s_cselect_b32 s40, s56, s40\n"
        "s_cselect_b32 s41, s57, s41\n"
        "fes_report_none:\n"
        "s_setpc_b64 s[52:53]\n"
        ".popsection\n"
        ".pushsection .fescode,\"ax\",@progbits\n"
        ".p2align 8\n"
        ".globl fes_native_code\n"
        ".hidden fes_native_code\n"
        "fes_native_code:\n"
        ".fill 1024,4,0xbf800000\n"
        ".popsection\n");
}
