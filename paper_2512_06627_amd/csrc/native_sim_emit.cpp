// Machine code of a simulation pass: the whole circuit as straight-line code, gates in file order.
//
// A gate is one v_bitop3, its store, and two scalar adds that move the row address on, 24 bytes in all,
// against 14 instructions of the interpreter's pass: a wave alone takes 13 ns a gate instead of 36, which
// is what a simulation of few words waits for (27-input cone of 4.3k gates, 1,003 words: 179 -> 71 us;
// 12x12 multiplier miter, 2,928 words: 129 -> 53).  Gates go in file order, so that the address steps by
// a row; a circuit that needs more registers in that order than there are stays with the interpreter.
#include <algorithm>
#include <set>

#include "native.hpp"

namespace fes {
namespace {

constexpr int kOff = 2, kFirst = 16, kZero = 15, kIn = 38, kOut = 40, kRowBytes = 42, kLanes = 44, kReturn = 36;
constexpr uint32_t kExec = 126, kConst0 = 128, kMinus1 = 193;
constexpr uint32_t kGatesPerBarrier = 8;

struct Code {
    std::vector<uint32_t>& w;
    void mov64(uint32_t dst, uint32_t src) { w.push_back(0xBE800100u | dst << 16 | src); }
    void nop() { w.push_back(0xBF800000u); }
    void barrier() { w.push_back(0xBF8A0000u); }
    void wait_memory() { w.push_back(0xBF8C0F70u); }  // s_waitcnt vmcnt(0)
    void setpc(uint32_t s) { w.push_back(0xBE801D00u | s); }
    void zero(int v) {
        w.push_back(0xD1410000u | (uint32_t)v);
        w.push_back(kConst0);
    }
    void load(int v) {  // global_load_dword v, v2, s[38:39]
        w.push_back(0xDC508000u);
        w.push_back((uint32_t)kOff | (uint32_t)kIn << 16 | (uint32_t)v << 24);
        next_row(kIn);
    }
    void store(int v) {  // global_store_dword v2, v, s[40:41]
        w.push_back(0xDC708000u);
        w.push_back((uint32_t)kOff | (uint32_t)v << 8 | (uint32_t)kOut << 16);
        next_row(kOut);
    }
    void next_row(int s) {
        w.push_back(0x80000000u | (uint32_t)s << 16 | (uint32_t)kRowBytes << 8 | (uint32_t)s);
        w.push_back(0x82000000u | (uint32_t)(s + 1) << 16 | kConst0 << 8 | (uint32_t)(s + 1));
    }
    // v_bitop3 of two operands, each complemented or not: the third source does not matter.
    void land(int dst, uint32_t a, bool na, uint32_t b, bool nb) {
        const uint32_t t = (na ? 0x0Fu : 0xF0u) & (nb ? 0x33u : 0xCCu);
        w.push_back(0xD2340000u | (uint32_t)dst | ((t >> 3) & 7u) << 8);
        w.push_back(a | b << 9 | kConst0 << 18 | ((t >> 6) & 3u) << 27 | (t & 7u) << 29);
    }
};

}  // namespace

bool emit_sim(const Aig& g, int vgprs, NativeCode& out) {
    const uint32_t n = g.num_inputs, A = g.num_ands();
    out = NativeCode{};
    std::vector<uint32_t> left(g.max_var() + 1, 0);  // reads still to come
    for (uint32_t k = 0; k < A; ++k) {
        ++left[g.and_r0[k] >> 1];
        ++left[g.and_r1[k] >> 1];
    }
    std::set<int> free_regs;
    for (int r = kFirst; r < kFirst + vgprs; ++r) free_regs.insert(r);
    std::vector<int> reg(g.max_var() + 1, -1);
    auto take = [&](uint32_t v) {
        if (free_regs.empty()) return false;
        reg[v] = *free_regs.begin();
        free_regs.erase(free_regs.begin());
        return true;
    };
    Code c{out.words};
    c.mov64(kExec, kLanes);
    c.nop();
    for (uint32_t i = 1; i <= n; ++i) {
        if (!take(i)) return false;
        c.load(reg[i]);
    }
    c.zero(kZero);
    c.store(kZero);
    c.wait_memory();
    c.nop();
    for (uint32_t i = 1; i <= n; ++i) c.store(reg[i]);
    for (uint32_t i = 1; i <= n; ++i)
        if (!left[i]) free_regs.insert(reg[i]);
    for (uint32_t k = 0; k < A; ++k) {
        const uint32_t a = g.and_r0[k], b = g.and_r1[k], v = n + 1 + k;
        auto src = [&](uint32_t lit) { return lit >> 1 ? 256u + (uint32_t)reg[lit >> 1] : kConst0; };
        const uint32_t sa = src(a), sb = src(b);
        for (uint32_t x : {a >> 1, b >> 1})
            if (--left[x] == 0 && x) free_regs.insert(reg[x]);
        if (!take(v)) return false;
        c.land(reg[v], sa, a & 1, sb, b & 1);
        c.store(reg[v]);
        if (!left[v]) free_regs.insert(reg[v]);
        if (k % kGatesPerBarrier == kGatesPerBarrier - 1) {
            c.barrier();
            c.nop();
        }
    }
    c.mov64(kExec, kMinus1);
    c.setpc(kReturn);
    out.valu = A;
    return true;
}

}  // namespace fes
