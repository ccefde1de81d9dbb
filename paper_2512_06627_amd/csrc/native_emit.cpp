// Machine code of a native pass (gfx950), from the mapped LUT program.
//
// The pass is straight-line code, so a value's life is an interval of steps and one scan assigns
// registers: VGPRs v16.. to LUT results, plan-time words and copies of wave-uniform inputs, SGPRs
// s62.. to wave-uniform inputs.  When the VGPRs run out, the value read farthest ahead leaves: a
// word or a copy is simply made again, a LUT result goes to an LDS slot of the wave and is read
// back a few steps before its next reader.
//
// Instructions: v_bitop3_b32 (a three-input LUT; its table is split over the abs, omod and neg
// fields), v_mov_b32, s_bfe_i32 (one bit of the half-word index as a mask), and per assignment
// v_cmp_ne_u32 with a branch to code behind the pass that reports its lowest failing lane.  A VALU
// instruction reads at most one SGPR; a second one goes through a VGPR copy.
#include <algorithm>
#include <climits>
#include <set>

#include "native.hpp"

namespace fes {
namespace {

constexpr int kFirstVgpr = 16, kReportVgpr = 15, kSpillVgpr = 8, kLaneVgpr = 2;
constexpr int kFirstSgpr = 62, kSgprs = 38;
constexpr int kIndexSgpr = 38;    // s[38:39] packed half-word index
constexpr int kReportSgpr = 48;   // s[48:49] the report routine
constexpr int kReturnSgpr = 36;   // s[36:37]
constexpr int kCallSgpr = 52;     // s[52:53] return address of the report
constexpr int kOffsetSgpr = 54;   // s[54:55] half-word offset of the assignment
constexpr uint32_t kAhead = 8;    // steps between an LDS read-back and its reader

// Every instruction of the straight path takes 8 bytes at a multiple of 8 (the compare and its
// branch together): 8-byte instructions that cross such a boundary issue slower.  With 4-byte
// forms for the two-input LUTs the 16x16 pass took 4.06 ms instead of 2.99 (four waves per SIMD),
// though it was a fifth shorter.
struct Encoder {
    std::vector<uint32_t>& w;
    static uint32_t vsrc(int v) { return 256u + (uint32_t)v; }
    static bool inline_const(uint32_t x, uint32_t* src) {
        const int32_t s = (int32_t)x;
        if (s >= 0 && s <= 64) {
            *src = 128u + (uint32_t)s;
            return true;
        }
        if (s >= -16 && s < 0) {
            *src = 192u + (uint32_t)(-s);
            return true;
        }
        return false;
    }
    // Source codes: 0..101 SGPR, 128..208 constants, 256.. VGPR.
    void bitop3(int vdst, uint32_t s0, uint32_t s1, uint32_t s2, uint32_t t) {
        w.push_back(0xD2340000u | (uint32_t)vdst | ((t >> 3) & 7u) << 8);
        w.push_back(s0 | s1 << 9 | s2 << 18 | ((t >> 6) & 3u) << 27 | (t & 7u) << 29);
    }
    void mov_v(int vdst, uint32_t src) {  // the 8-byte form
        w.push_back(0xD1410000u | (uint32_t)vdst);
        w.push_back(src);
    }
    void mov_v_literal(int vdst, uint32_t x) {
        w.push_back(0x7E0002FFu | (uint32_t)vdst << 17);
        w.push_back(x);
    }
    void not_v(int vdst, uint32_t src) { w.push_back(0x7E005600u | (uint32_t)vdst << 17 | src); }
    void bit_mask(int sdst, uint32_t bit) {  // s_bfe_i32 of one index bit
        w.push_back(0x93000000u | (uint32_t)sdst << 16 | 255u << 8 | (uint32_t)(kIndexSgpr + (bit >= 32 ? 1 : 0)));
        w.push_back(0x00010000u | (bit & 31u));
    }
    void mov_s(int sdst, uint32_t x) {
        uint32_t c = 255;
        inline_const(x, &c);
        w.push_back(0xBE800000u | (uint32_t)sdst << 16 | c);
        if (c == 255) w.push_back(x);
    }
    void cmp_ne(uint32_t src0, int v) { w.push_back(0x7D9A0000u | src0 | (uint32_t)v << 9); }
    void ds_write(int vdata, int slot) {
        w.push_back(0xD81A0000u | 256u * (uint32_t)slot);
        w.push_back((uint32_t)kSpillVgpr | (uint32_t)vdata << 8);
    }
    void ds_read(int vdst, int slot) {
        w.push_back(0xD86C0000u | 256u * (uint32_t)slot);
        w.push_back((uint32_t)kSpillVgpr | (uint32_t)vdst << 24);
    }
    void wait_lds() {
        w.push_back(0xBF8CC07Fu);
        w.push_back(0xBF800000u);  // s_nop: see above
    }
    void setpc(int s) { w.push_back(0xBE801D00u | (uint32_t)s); }
    void swappc(int sdst, int s) { w.push_back(0xBE801E00u | (uint32_t)sdst << 16 | (uint32_t)s); }
    // s_branch / s_cbranch_vccnz at word `at` to word `to`
    static uint32_t rel(size_t at, size_t to) { return (uint32_t)((int64_t)to - (int64_t)at - 1) & 0xFFFFu; }
    void branch(size_t to) { w.push_back(0xBF820000u | rel(w.size(), to)); }
};

// Free VGPRs by bank (number mod 4).
struct Vgprs {
    uint64_t free[4] = {0, 0, 0, 0};
    explicit Vgprs(int count) {
        for (int r = kFirstVgpr; r < kFirstVgpr + count; ++r) give(r);
    }
    void give(int r) { free[r & 3] |= 1ull << (r >> 2); }
    // The lowest free register outside the banks of `avoid`, else the lowest free one, else -1.
    int take(unsigned avoid) {
        for (unsigned skip : {avoid & 15u, 0u}) {
            int best = INT_MAX;
            for (int b = 0; b < 4; ++b)
                if (free[b] && !((skip >> b) & 1u)) best = std::min(best, __builtin_ctzll(free[b]) * 4 + b);
            if (best != INT_MAX) {
                free[best & 3] &= ~(1ull << (best >> 2));
                return best;
            }
        }
        return -1;
    }
};

}  // namespace

void order_for_registers(LutProgram& lp) {
    // Of the steps whose operands are there, the one that ends the most lives (its own result counts
    // against it) goes next; of equals the first in the program's order, but not one that reads the
    // result just computed if another will do: a wave waits out the VALU latency on those.
    const uint32_t N = lp.num_values;
    std::vector<uint32_t> step_of(N, UINT32_MAX), luts;
    for (uint32_t s = 0; s < lp.steps.size(); ++s)
        if (lp.steps[s].op == LutStep::Lut) {
            step_of[lp.steps[s].dst] = (uint32_t)luts.size();
            luts.push_back(s);
        }
    const uint32_t T = (uint32_t)luts.size();
    std::vector<std::vector<uint32_t>> readers(T);
    std::vector<uint32_t> left(T, 0), waiting(T, 0);
    auto operands = [&](uint32_t t, auto&& f) {
        const LutStep& st = lp.steps[luts[t]];
        for (uint32_t j = 0; j < st.nleaves; ++j)
            if (st.leaf[j].kind == LutRef::Varying) f(step_of[st.leaf[j].index]);
    };
    for (uint32_t t = 0; t < T; ++t)
        operands(t, [&](uint32_t q) {
            readers[q].push_back(t);
            ++left[q];
            ++waiting[t];
        });
    // Ready steps by what they do to the number of live values: -3 .. 1.
    std::set<uint32_t> ready[5];
    std::vector<int8_t> gain(T, 0);
    std::vector<uint8_t> state(T, 0);  // 0 waiting, 1 ready, 2 done
    auto change_of = [&](uint32_t t) {
        int d = left[t] ? 1 : 0;
        operands(t, [&](uint32_t q) { d -= left[q] == 1 ? 1 : 0; });
        return (int8_t)d;
    };
    auto make_ready = [&](uint32_t t) {
        state[t] = 1;
        gain[t] = change_of(t);
        ready[gain[t] + 3].insert(t);
    };
    for (uint32_t t = 0; t < T; ++t)
        if (!waiting[t]) make_ready(t);
    std::vector<uint32_t> order;
    order.reserve(T);
    uint32_t last = UINT32_MAX;
    while (order.size() < T) {
        uint32_t pick = UINT32_MAX;
        for (int b = 0; b < 5 && pick == UINT32_MAX; ++b) {
            if (ready[b].empty()) continue;
            pick = *ready[b].begin();
            int looked = 0;
            for (uint32_t t : ready[b]) {
                bool reads_last = false;
                operands(t, [&](uint32_t q) { reads_last |= q == last; });
                if (!reads_last) {
                    pick = t;
                    break;
                }
                if (++looked == 8) break;
            }
        }
        ready[gain[pick] + 3].erase(pick);
        state[pick] = 2;
        order.push_back(pick);
        last = pick;
        operands(pick, [&](uint32_t q) {
            if (--left[q] != 1) return;
            for (uint32_t r : readers[q])  // its last reader ends its life now
                if (state[r] == 1) {
                    ready[gain[r] + 3].erase(r);
                    gain[r] = change_of(r);
                    ready[gain[r] + 3].insert(r);
                }
        });
        for (uint32_t r : readers[pick])
            if (--waiting[r] == 0) make_ready(r);
    }
    std::vector<LutStep> out;
    out.reserve(lp.steps.size());
    for (uint32_t t : order) out.push_back(lp.steps[luts[t]]);
    for (const LutStep& st : lp.steps)
        if (st.op != LutStep::Lut) out.push_back(st);
    lp.steps.swap(out);
}

bool emit_native(const LutProgram& lp, const std::vector<uint64_t>& offset, int vgprs, int lds_slots, NativeCode& out) {
    out = NativeCode{};
    Encoder e{out.words};
    const uint32_t n = lp.num_inputs;
    // Items: LUT results, then plan-time words, then inputs.
    const uint32_t W0 = lp.num_values, I0 = W0 + (uint32_t)lp.words.size(), items = I0 + n;
    auto item_of = [&](const LutRef& r) {
        return r.kind == LutRef::Word ? W0 + r.index : r.kind == LutRef::Input ? I0 + r.index : r.index;
    };
    std::vector<const LutStep*> luts;
    struct Out {
        LutRef ref;
        bool neg;
        uint32_t which;
    };
    std::vector<Out> fixed_outs;                       // outputs that are an input or a word
    std::vector<std::vector<std::pair<uint32_t, bool>>> outs_of;  // LUT result -> assignments it answers
    outs_of.resize(lp.num_values);
    uint32_t which = 0;
    for (const LutStep& st : lp.steps) {
        if (st.op == LutStep::Lut) luts.push_back(&st);
        else if (st.op == LutStep::Output) {
            if (st.leaf[0].kind == LutRef::Varying) outs_of[st.leaf[0].index].push_back({which, st.out_neg});
            else fixed_outs.push_back({st.leaf[0], st.out_neg, which});
            ++which;
        } else return false;  // scalar-unit steps do not occur in all-VALU programs
    }
    if (which != offset.size()) return false;
    const uint32_t T = (uint32_t)luts.size();
    // Readers of every item, in order.
    std::vector<uint32_t> first(items + 1, 0), uses, cursor;
    for (const LutStep* st : luts)
        for (uint32_t j = 0; j < st->nleaves; ++j) ++first[item_of(st->leaf[j]) + 1];
    for (uint32_t i = 0; i < items; ++i) first[i + 1] += first[i];
    uses.resize(first[items]);
    cursor.assign(first.begin(), first.end() - 1);
    for (uint32_t t = 0; t < T; ++t)
        for (uint32_t j = 0; j < luts[t]->nleaves; ++j) uses[cursor[item_of(luts[t]->leaf[j])]++] = t;
    cursor.assign(first.begin(), first.end() - 1);
    constexpr uint32_t kNever = UINT32_MAX;
    auto next_use = [&](uint32_t i) { return cursor[i] < first[i + 1] ? uses[cursor[i]] : kNever; };

    Vgprs vp(vgprs);
    std::vector<int> vreg(items, -1), sreg(items, -1), slot(items, -1);
    std::vector<uint8_t> pending(items, 0);  // LDS read-back issued, not waited for
    std::vector<uint32_t> in_flight;         // the items with that mark
    bool failed = false;
    std::vector<uint32_t> owner(256, kNever);
    std::vector<uint32_t> sowner(kSgprs, kNever);
    std::vector<int> free_slots;
    uint32_t now = 0;
    auto take_v = [&](unsigned avoid) {
        int r = vp.take(avoid);
        if (r >= 0) return r;
        // Leaves: the item read farthest ahead; a word or a copy (made again for one instruction)
        // before a LUT result (an LDS write and read) unless it is read within 16 steps.
        uint32_t cheap = kNever, cheap_at = 0, dear = kNever, dear_at = 0;
        for (int q = kFirstVgpr; q < kFirstVgpr + vgprs; ++q) {
            const uint32_t i = owner[q];
            if (i == kNever || pending[i]) continue;
            const uint32_t at = next_use(i);
            if (at == now) continue;
            if (i >= W0) {
                if (cheap == kNever || at > cheap_at) cheap = i, cheap_at = at;
            } else if (dear == kNever || at > dear_at) {
                dear = i;
                dear_at = at;
            }
        }
        uint32_t victim = cheap != kNever && (cheap_at > now + 16 || dear == kNever) ? cheap : dear;
        if (victim == kNever) {
            failed = true;
            return kFirstVgpr;
        }
        r = vreg[victim];
        if (victim < W0 && slot[victim] < 0) {  // an earlier copy in LDS is still good
            if (free_slots.empty()) {
                if ((int)out.lds_slots >= lds_slots) {
                    failed = true;
                    return r;
                }
                free_slots.push_back((int)out.lds_slots++);
            }
            slot[victim] = free_slots.back();
            free_slots.pop_back();
            e.ds_write(r, slot[victim]);
            ++out.lds;
        }
        vreg[victim] = -1;
        owner[r] = kNever;
        return r;
    };
    auto bind = [&](uint32_t i, int r) {
        vreg[i] = r;
        owner[r] = i;
    };
    auto read_back = [&](uint32_t i) {
        const int r = take_v(0);
        if (failed) return;
        e.ds_read(r, slot[i]);
        ++out.lds;
        bind(i, r);
        pending[i] = 1;
        in_flight.push_back(i);
    };
    auto wait = [&] {
        e.wait_lds();
        for (uint32_t i : in_flight) pending[i] = 0;
        in_flight.clear();
    };
    auto take_s = [&] {
        int pick = 0;
        uint32_t far = 0;
        for (int q = 0; q < kSgprs; ++q) {
            if (sowner[q] == kNever) {
                pick = q;
                break;
            }
            const uint32_t at = next_use(sowner[q]);
            if (at != now && at >= far) {
                far = at;
                pick = q;
            }
        }
        if (sowner[pick] != kNever) sreg[sowner[pick]] = -1;
        return pick;
    };
    // An item's source code for a VALU reader (wave-uniform inputs: their SGPR unless a copy exists).
    auto locate = [&](const LutRef& r) -> uint32_t {
        const uint32_t i = item_of(r);
        uint32_t c;
        if (r.kind == LutRef::Word && Encoder::inline_const(lp.words[r.index], &c)) return c;
        if (r.kind == LutRef::Input && r.index < 11) return Encoder::vsrc(kLaneVgpr + (int)r.index - 5);
        if (vreg[i] >= 0) {
            if (pending[i]) wait();
            return Encoder::vsrc(vreg[i]);
        }
        if (r.kind == LutRef::Input) {
            if (sreg[i] < 0) {
                const int q = take_s();
                e.bit_mask(kFirstSgpr + q, r.index - 5);
                ++out.salu;
                sreg[i] = q;
                sowner[q] = i;
            }
            return (uint32_t)(kFirstSgpr + sreg[i]);
        }
        if (r.kind == LutRef::Word) {
            const int q = take_v(0);
            if (failed) return 0;
            e.mov_v_literal(q, lp.words[r.index]);
            ++out.valu;
            bind(i, q);
            return Encoder::vsrc(q);
        }
        if (slot[i] < 0) {
            failed = true;
            return 0;
        }
        read_back(i);
        if (failed) return 0;
        wait();
        return Encoder::vsrc(vreg[i]);
    };
    auto release = [&](uint32_t i) {
        if (vreg[i] >= 0) {
            owner[vreg[i]] = kNever;
            vp.give(vreg[i]);
            vreg[i] = -1;
        }
        if (sreg[i] >= 0) {
            sowner[sreg[i]] = kNever;
            sreg[i] = -1;
        }
        if (slot[i] >= 0) {
            free_slots.push_back(slot[i]);
            slot[i] = -1;
        }
    };
    // Where an assignment's miter word is not zero, code behind the pass reports it.
    struct Report {
        size_t branch_at;  // word of the s_cbranch_vccnz
        uint32_t which;
        int reg;
        bool neg;
    };
    std::vector<Report> reports;
    auto answer = [&](int reg, bool neg, uint32_t w) {
        e.cmp_ne(neg ? 193u : 128u, reg);  // a word of all ones is zero after its complement
        reports.push_back({out.words.size(), w, reg, neg});
        out.words.push_back(0);
        ++out.valu;
        ++out.salu;
    };
    for (const Out& o : fixed_outs) {
        const uint32_t src = locate(o.ref);
        if (failed) return false;
        int reg = (int)src - 256;
        const int own = src >= 256 ? -1 : kReportVgpr;
        if (own >= 0) {
            e.mov_v(own, src);
            ++out.valu;
            reg = own;
        }
        answer(reg, o.neg, o.which);
    }
    for (uint32_t t = 0; t < T; ++t) {
        now = t;
        const LutStep& st = *luts[t];
        if (out.lds && t + kAhead < T) {  // spilled operands of a step soon to come
            const LutStep& soon = *luts[t + kAhead];
            for (uint32_t j = 0; j < soon.nleaves && in_flight.size() < (size_t)vgprs / 8; ++j) {
                const uint32_t i = item_of(soon.leaf[j]);
                if (i < W0 && vreg[i] < 0 && slot[i] >= 0) read_back(i);
            }
        }
        uint32_t src[3] = {0, 0, 0};
        int used = -1;  // the one SGPR this instruction reads
        for (uint32_t j = 0; j < st.nleaves && !failed; ++j) {
            src[j] = locate(st.leaf[j]);
            if (src[j] >= 102 || failed) continue;
            if (used < 0 || used == (int)src[j]) {
                used = (int)src[j];
                continue;
            }
            const uint32_t i = item_of(st.leaf[j]);
            const int q = take_v(0);
            if (failed) break;
            e.mov_v(q, src[j]);
            ++out.valu;
            bind(i, q);
            src[j] = Encoder::vsrc(q);
        }
        if (failed) return false;
        for (uint32_t j = 0; j < st.nleaves; ++j) {
            const uint32_t i = item_of(st.leaf[j]);
            while (cursor[i] < first[i + 1] && uses[cursor[i]] <= t) ++cursor[i];
            if (next_use(i) == kNever) release(i);
        }
        // Bank choice: not the banks of the operands that this result's first reader already has in
        // VGPRs (three operands in one bank are read one after the other).
        unsigned avoid = 0;
        if (first[st.dst] < first[st.dst + 1]) {
            const LutStep& rd = *luts[uses[first[st.dst]]];
            for (uint32_t j = 0; j < rd.nleaves; ++j) {
                const uint32_t i = item_of(rd.leaf[j]);
                if (i != st.dst && vreg[i] >= 0) avoid |= 1u << (vreg[i] & 3);
            }
        }
        const int d = take_v(avoid);
        if (failed) return false;
        const uint32_t s1 = st.nleaves >= 2 ? src[1] : src[0];
        e.bitop3(d, src[0], s1, st.nleaves >= 3 ? src[2] : s1, st.table);
        ++out.valu;
        bind(st.dst, d);
        for (auto& o : outs_of[st.dst]) answer(d, o.second, o.first);
        if (next_use(st.dst) == kNever) release(st.dst);
    }
    if (out.lds) e.wait_lds();  // no spill write outlives the pass
    e.setpc(kReturnSgpr);
    for (const Report& r : reports) {
        if (out.words.size() - r.branch_at > 32000) return false;  // 16-bit branch distance
        out.words[r.branch_at] = 0xBF870000u | Encoder::rel(r.branch_at, out.words.size());
        if (r.neg) e.not_v(kReportVgpr, Encoder::vsrc(r.reg));
        else if (r.reg != kReportVgpr) e.mov_v(kReportVgpr, Encoder::vsrc(r.reg));
        e.mov_s(kOffsetSgpr, (uint32_t)offset[r.which]);
        e.mov_s(kOffsetSgpr + 1, (uint32_t)(offset[r.which] >> 32));
        e.swappc(kCallSgpr, kReportSgpr);
        e.branch(r.branch_at + 1);
    }
    return true;
}

}  // namespace fes
