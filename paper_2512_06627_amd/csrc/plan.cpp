#include "plan.hpp"

#include <algorithm>
#include <string>

namespace fes {
namespace {

struct Cone {
    std::vector<uint8_t> in;      // per AND index
    std::vector<uint32_t> level;  // per var
    std::vector<uint32_t> label;  // per var: slots needed to evaluate a var's cone as a tree
};

inline bool is_and(const Aig& g, uint32_t var) { return var > g.num_inputs; }
inline uint32_t and_index(const Aig& g, uint32_t var) { return var - g.num_inputs - 1; }

Cone cone_of(const Aig& g) {
    Cone c;
    const uint32_t A = g.num_ands();
    c.in.assign(A, 0);
    std::vector<uint32_t> stack;
    for (uint32_t o : g.outputs)
        if (is_and(g, o >> 1)) stack.push_back(o >> 1);
    while (!stack.empty()) {
        uint32_t v = stack.back();
        stack.pop_back();
        uint32_t k = and_index(g, v);
        if (c.in[k]) continue;
        c.in[k] = 1;
        for (uint32_t f : {g.and_r0[k] >> 1, g.and_r1[k] >> 1})
            if (is_and(g, f)) stack.push_back(f);
    }
    c.level.assign(g.max_var() + 1, 0);
    c.label.assign(g.max_var() + 1, 0);
    for (uint32_t k = 0; k < A; ++k) {  // topological index order
        uint32_t v = g.num_inputs + 1 + k, a = g.and_r0[k] >> 1, b = g.and_r1[k] >> 1;
        c.level[v] = 1 + std::max(c.level[a], c.level[b]);
        uint32_t la = c.label[a], lb = c.label[b];
        c.label[v] = la == lb ? la + 1 : std::max(la, lb);
    }
    return c;
}

// Post-order DFS from the outputs; `first_child` picks which fanin to descend into first.
std::vector<uint32_t> dfs_order(const Aig& g, const Cone& c, bool by_label) {
    std::vector<uint32_t> order;
    std::vector<uint8_t> done(g.num_ands(), 0);
    std::vector<std::pair<uint32_t, uint8_t>> stack;  // (var, children pushed)
    for (uint32_t o : g.outputs) {
        uint32_t root = o >> 1;
        if (!is_and(g, root) || done[and_index(g, root)]) continue;
        stack.push_back({root, 0});
        while (!stack.empty()) {
            auto& top = stack.back();
            uint32_t v = top.first, k = and_index(g, v);
            if (done[k]) {
                stack.pop_back();
                continue;
            }
            if (top.second == 0) {
                top.second = 1;
                uint32_t a = g.and_r0[k] >> 1, b = g.and_r1[k] >> 1;
                uint32_t first = a, second = b;
                if (by_label && c.label[b] > c.label[a]) std::swap(first, second);
                // Push the second child below the first so the first is evaluated first.
                if (is_and(g, second) && !done[and_index(g, second)]) stack.push_back({second, 0});
                if (is_and(g, first) && !done[and_index(g, first)]) stack.push_back({first, 0});
                continue;
            }
            done[k] = 1;
            order.push_back(k);
            stack.pop_back();
        }
    }
    return order;
}

// Set of numbers below a bound with its smallest member at hand: one bit each, and one bit per word
// of the level below.
class MinSet {
public:
    explicit MinSet(uint32_t bound) {
        do {
            bound = (bound + 63) / 64;
            levels_.emplace_back(bound, 0);
        } while (bound > 1);
    }
    void insert(uint32_t x) {
        for (auto& l : levels_) {
            const uint64_t was = l[x >> 6];
            l[x >> 6] |= 1ull << (x & 63);
            if (was) return;
            x >>= 6;
        }
    }
    bool empty() const { return levels_.back()[0] == 0; }
    uint32_t take_min() {
        uint32_t x = 0;
        for (size_t i = levels_.size(); i-- > 0;) x = x * 64 + (uint32_t)__builtin_ctzll(levels_[i][x]);
        uint32_t at = x;
        for (auto& l : levels_) {
            l[at >> 6] &= ~(1ull << (at & 63));
            if (l[at >> 6]) break;
            at >>= 6;
        }
        return x;
    }

private:
    std::vector<std::vector<uint64_t>> levels_;
};

// An order cut into bundles: bundle i holds gates[ends[i - 1] .. ends[i]).
struct Bundles {
    std::vector<uint32_t> gates, ends;
};

// Readers of each gate among the gates of the cone, in the order `order`.
struct Readers {
    std::vector<uint32_t> first, gate, missing;  // gate[first[k] .. first[k + 1]): readers of k
};

Readers readers_of(const Aig& g, const std::vector<uint32_t>& order) {
    Readers r;
    const uint32_t A = g.num_ands();
    r.first.assign(A + 1, 0);
    r.missing.assign(A, 0);
    for (uint32_t k : order)
        for (uint32_t f : {g.and_r0[k] >> 1, g.and_r1[k] >> 1})
            if (is_and(g, f)) {
                ++r.missing[k];
                ++r.first[and_index(g, f) + 1];
            }
    for (uint32_t k = 0; k < A; ++k) r.first[k + 1] += r.first[k];
    r.gate.resize(r.first[A]);
    std::vector<uint32_t> at(r.first.begin(), r.first.end() - 1);
    for (uint32_t k : order)
        for (uint32_t f : {g.and_r0[k] >> 1, g.and_r1[k] >> 1})
            if (is_and(g, f)) r.gate[at[and_index(g, f)]++] = k;
    return r;
}

// Group an order into bundles of independent gates by list scheduling: a gate is ready when
// its AND fanins were computed in an earlier bundle; each bundle takes up to `B` ready gates
// in order of their position in `order`.
Bundles bundle_order(const Aig& g, std::vector<uint32_t> order, const Readers& readers, uint32_t B) {
    Bundles out;
    if (B <= 1) {
        out.ends.resize(order.size());
        for (uint32_t i = 0; i < order.size(); ++i) out.ends[i] = i + 1;
        out.gates = std::move(order);
        return out;
    }
    std::vector<uint32_t> pos(g.num_ands(), UINT32_MAX), missing = readers.missing;
    for (uint32_t i = 0; i < order.size(); ++i) pos[order[i]] = i;
    MinSet ready((uint32_t)order.size());  // by position
    for (uint32_t k : order)
        if (missing[k] == 0) ready.insert(pos[k]);
    out.gates.reserve(order.size());
    while (out.gates.size() < order.size()) {
        const size_t first = out.gates.size();
        while (out.gates.size() < first + B && !ready.empty()) out.gates.push_back(order[ready.take_min()]);
        for (size_t i = first; i < out.gates.size(); ++i) {
            const uint32_t k = out.gates[i];
            for (uint32_t j = readers.first[k]; j < readers.first[k + 1]; ++j)
                if (--missing[readers.gate[j]] == 0) ready.insert(pos[readers.gate[j]]);
        }
        out.ends.push_back((uint32_t)out.gates.size());
    }
    return out;
}

// Reads of every variable by the cone's gates, and by outputs plain and complemented.
struct Refs {
    std::vector<uint32_t> reads, pos, neg;
};

Refs refs_of(const Aig& g, const std::vector<uint32_t>& cone) {
    Refs r;
    const uint32_t V = g.max_var();
    r.reads.assign(V + 1, 0);
    r.pos.assign(V + 1, 0);
    r.neg.assign(V + 1, 0);
    for (uint32_t k : cone) {
        ++r.reads[g.and_r0[k] >> 1];
        ++r.reads[g.and_r1[k] >> 1];
    }
    for (uint32_t o : g.outputs) (o & 1 ? r.neg : r.pos)[o >> 1]++;
    return r;
}

// Slots an order needs: values alive at once, a bundle's operands given up before its results.
uint32_t count_slots(const Aig& g, const Bundles& b, const Refs& refs) {
    std::vector<uint32_t> rc = refs.reads;
    uint32_t slots = 0, live = 0, at = 0;
    for (uint32_t end : b.ends) {
        const uint32_t first = at;
        for (; at < end; ++at)
            for (uint32_t f : {g.and_r0[b.gates[at]] >> 1, g.and_r1[b.gates[at]] >> 1})
                if (is_and(g, f) && --rc[f] == 0) --live;
        live += end - first;
        slots = std::max(slots, live);
        for (uint32_t i = first; i < end; ++i)
            if (rc[g.num_inputs + 1 + b.gates[i]] == 0) --live;
    }
    return slots;
}

// The stream: every result in the lowest free slot.
std::vector<Instr> allocate(const Aig& g, const Bundles& bundles, const Refs& refs, uint32_t slots, uint32_t B,
                            uint32_t* gates) {
    const uint32_t n = g.num_inputs, V = g.max_var(), sink = n + 1 + slots;
    std::vector<uint32_t> rc = refs.reads, slot(V + 1, UINT32_MAX);
    MinSet free_slots(std::max(slots, 1u));
    for (uint32_t i = 0; i < slots; ++i) free_slots.insert(i);
    std::vector<Instr> prog;
    prog.reserve(bundles.ends.size() * B + g.outputs.size() + B);
    auto row_of = [&](uint32_t var) { return is_and(g, var) ? n + 1 + slot[var] : var; };
    auto release = [&](uint32_t var) {
        if (is_and(g, var) && --rc[var] == 0) free_slots.insert(slot[var]);
    };
    const Instr nop = {0u, 0u, sink, 0u};
    uint32_t at = 0;
    for (uint32_t end : bundles.ends) {
        const size_t first = prog.size();
        const uint32_t* b = bundles.gates.data() + at;
        const uint32_t count = end - at;
        at = end;
        // Operands are read before any result of the bundle is written, so the slots whose
        // last reader is in this bundle are free for the bundle's own results.
        for (uint32_t t = 0; t < count; ++t) {
            const uint32_t a = g.and_r0[b[t]], c = g.and_r1[b[t]];
            prog.push_back({row_of(a >> 1) | ((a & 1) ? kCompl : 0u), row_of(c >> 1) | ((c & 1) ? kCompl : 0u), 0u, 0u});
        }
        for (uint32_t t = 0; t < count; ++t) {
            release(g.and_r0[b[t]] >> 1);
            release(g.and_r1[b[t]] >> 1);
        }
        for (uint32_t t = 0; t < count; ++t) {
            const uint32_t v = n + 1 + b[t];
            slot[v] = free_slots.take_min();
            Instr& ins = prog[first + t];
            ins.d = n + 1 + slot[v];
            ins.flags = (refs.pos[v] ? kOutPos : 0u) | (refs.neg[v] ? kOutNeg : 0u) | (g.is_xor(b[t]) ? kXor : 0u);
        }
        for (uint32_t t = 0; t < count; ++t)
            if (rc[n + 1 + b[t]] == 0) free_slots.insert(slot[n + 1 + b[t]]);
        while ((prog.size() - first) % B) prog.push_back(nop);
    }
    *gates = (uint32_t)bundles.gates.size();
    // Outputs driven by a constant or a primary input: value AND true, into the sink row.
    const size_t first = prog.size();
    for (uint32_t o : g.outputs) {
        if (is_and(g, o >> 1)) continue;
        prog.push_back({(o >> 1) | ((o & 1) ? kCompl : 0u), 0u | kCompl, sink, kOutPos});
        ++*gates;
    }
    while ((prog.size() - first) % B) prog.push_back(nop);
    return prog;
}

}  // namespace

Aig fuse_xors(const Aig& g) {
    const uint32_t A = g.num_ands();
    std::vector<uint32_t> readers(g.max_var() + 1, 0);
    for (uint32_t k = 0; k < A; ++k) {
        ++readers[g.and_r0[k] >> 1];
        ++readers[g.and_r1[k] >> 1];
    }
    for (uint32_t o : g.outputs) ++readers[o >> 1];
    Aig f = g;
    f.xor_gate.assign(A, 0);
    std::vector<uint8_t> absorbed(A, 0);
    for (uint32_t k = 0; k < A; ++k) {
        const uint32_t l1 = g.and_r0[k], l2 = g.and_r1[k];
        if (!(l1 & 1) || !(l2 & 1)) continue;  // both fanins complemented
        const uint32_t t1 = l1 >> 1, t2 = l2 >> 1;
        if (t1 == t2 || !is_and(g, t1) || !is_and(g, t2) || readers[t1] != 1 || readers[t2] != 1) continue;
        const uint32_t k1 = and_index(g, t1), k2 = and_index(g, t2);
        if (f.xor_gate[k1] || f.xor_gate[k2] || absorbed[k1] || absorbed[k2]) continue;
        const uint32_t x = g.and_r0[k1], y = g.and_r1[k1];
        const uint32_t p = g.and_r0[k2], q = g.and_r1[k2];
        if (!((p == (x ^ 1u) && q == (y ^ 1u)) || (p == (y ^ 1u) && q == (x ^ 1u)))) continue;
        if ((x >> 1) == (y >> 1)) continue;  // x & ~x: leave constant gates to the AND path
        f.and_r0[k] = x;
        f.and_r1[k] = y;
        f.xor_gate[k] = 1;
        absorbed[k1] = absorbed[k2] = 1;
    }
    return f;
}

Plan make_plan(const Aig& g, Order order, uint32_t bundle) {
    if (bundle == 0) bundle = 1;
    Cone c = cone_of(g);
    Plan p;
    p.num_inputs = g.num_inputs;
    p.num_ands_file = g.num_ands();
    p.num_outputs = (uint32_t)g.outputs.size();
    for (uint32_t k = 0; k < g.num_ands(); ++k) p.num_ands_tfi += c.in[k];
    for (uint32_t o : g.outputs) p.levels = std::max(p.levels, c.level[o >> 1]);

    std::vector<std::pair<Order, std::vector<uint32_t>>> cands;
    if (order == Order::Auto || order == Order::DfsLabel) cands.push_back({Order::DfsLabel, dfs_order(g, c, true)});
    if (order == Order::Auto || order == Order::DfsFanin0) cands.push_back({Order::DfsFanin0, dfs_order(g, c, false)});
    if (order == Order::Auto || order == Order::File) {
        std::vector<uint32_t> file;
        for (uint32_t k = 0; k < g.num_ands(); ++k)
            if (c.in[k]) file.push_back(k);
        cands.push_back({Order::File, std::move(file)});
    }
    // The first of the candidates that need the fewest slots; only its stream is made.
    const Refs refs = refs_of(g, cands.front().second);
    Readers readers;
    if (bundle > 1) readers = readers_of(g, cands.front().second);
    Bundles best;
    bool have = false;
    for (auto& cand : cands) {
        Bundles b = bundle_order(g, std::move(cand.second), readers, bundle);
        const uint32_t slots = count_slots(g, b, refs);
        if (have && slots >= p.peak_slots) continue;
        have = true;
        p.peak_slots = slots;
        p.order_used = cand.first;
        best = std::move(b);
    }
    p.prog = allocate(g, best, refs, p.peak_slots, bundle, &p.num_gate_instrs);
    p.order = std::move(best.gates);
    p.bundle = bundle;
    p.rows = g.num_inputs + p.peak_slots + 2;
    // Gate instructions write a slot row and appear in the stream in evaluation order;
    // padding and output-only steps write the sink row.
    const uint32_t sink = g.num_inputs + 1 + p.peak_slots;
    p.instr_gate.assign(p.prog.size(), UINT32_MAX);
    size_t next = 0;
    for (size_t t = 0; t < p.prog.size(); ++t)
        if (p.prog[t].d != sink) p.instr_gate[t] = p.order[next++];
    if (next != p.order.size()) throw Error{kErrInvalid, "planner: gate instructions do not match the order"};
    return p;
}

std::string validate_plan(const Aig& g, const Plan& p) {
    // Symbolic replay of the stream.  holds[row] is the variable a row holds.  Within a
    // bundle all operands are resolved first, then all results are written; a result may
    // only overwrite a row whose value has no reads left once the bundle's reads are done.
    const uint32_t n = g.num_inputs, V = g.max_var(), sink = n + 1 + p.peak_slots;
    if (p.bundle == 0 || p.prog.size() % p.bundle) return "stream is not a whole number of bundles";
    std::vector<int64_t> holds(p.rows, -1);
    holds[0] = 0;
    for (uint32_t i = 1; i <= n; ++i) holds[i] = i;
    std::vector<std::vector<uint32_t>> by_fanin0(V + 1);
    for (uint32_t k = 0; k < g.num_ands(); ++k) by_fanin0[g.and_r0[k] >> 1].push_back(k);
    std::vector<uint32_t> reads(V + 1, 0);
    std::vector<uint8_t> in_cone(g.num_ands(), 0);
    {  // cone of the outputs and its read counts
        std::vector<uint32_t> st;
        for (uint32_t o : g.outputs) {
            ++reads[o >> 1];
            if (is_and(g, o >> 1)) st.push_back(o >> 1);
        }
        while (!st.empty()) {
            uint32_t k = and_index(g, st.back());
            st.pop_back();
            if (in_cone[k]) continue;
            in_cone[k] = 1;
            for (uint32_t f : {g.and_r0[k] >> 1, g.and_r1[k] >> 1}) {
                ++reads[f];
                if (is_and(g, f)) st.push_back(f);
            }
        }
    }
    std::vector<uint8_t> done(g.num_ands(), 0);
    std::vector<uint8_t> out_only_done(g.outputs.size(), 0);
    for (size_t b0 = 0; b0 < p.prog.size(); b0 += p.bundle) {
        struct Step { uint32_t la, lb, d, flags; int64_t gate; };
        std::vector<Step> steps;
        for (size_t t = b0; t < b0 + p.bundle; ++t) {
            const Instr& ins = p.prog[t];
            uint32_t ra = ins.a & kRowMask, rb = ins.b & kRowMask;
            if (ra >= p.rows || rb >= p.rows || ins.d >= p.rows) return "row out of range at " + std::to_string(t);
            if (holds[ra] < 0 || holds[rb] < 0) return "read of an empty row at " + std::to_string(t);
            Step s{2 * (uint32_t)holds[ra] + ((ins.a & kCompl) ? 1u : 0u),
                   2 * (uint32_t)holds[rb] + ((ins.b & kCompl) ? 1u : 0u), ins.d, ins.flags, -1};
            if (ins.d == sink) {
                if (ins.flags == 0) continue;  // padding
                bool found = false;
                for (size_t j = 0; j < g.outputs.size(); ++j)
                    if (g.outputs[j] == s.la && !is_and(g, s.la >> 1) && !out_only_done[j]) {
                        out_only_done[j] = 1;
                        found = true;
                        break;
                    }
                if (!found || s.lb != 1 || ins.flags != kOutPos) return "bad output-only step at " + std::to_string(t);
                --reads[s.la >> 1];
                continue;
            }
            for (uint32_t k : by_fanin0[s.la >> 1])
                if (!done[k] && in_cone[k] && g.and_r0[k] == s.la && g.and_r1[k] == s.lb &&
                    ((ins.flags & kXor) != 0) == g.is_xor(k)) {
                    bool taken = false;
                    for (auto& o : steps) taken |= o.gate == (int64_t)k;
                    if (!taken) { s.gate = k; break; }
                }
            if (s.gate < 0) return "instruction " + std::to_string(t) + " computes no pending cone gate";
            steps.push_back(s);
        }
        for (auto& s : steps) {
            --reads[s.la >> 1];
            --reads[s.lb >> 1];
        }
        for (size_t i = 0; i < steps.size(); ++i) {
            auto& s = steps[i];
            if (s.d <= n) return "write into a constant or input row";
            for (size_t j = 0; j < i; ++j)
                if (steps[j].d == s.d) return "two results of one bundle share a row";
            int64_t prev = holds[s.d];
            if (prev > (int64_t)n && reads[prev] != 0) return "live value overwritten";
        }
        for (auto& s : steps) {
            uint32_t v = n + 1 + (uint32_t)s.gate;
            holds[s.d] = v;
            done[s.gate] = 1;
            uint32_t want = 0;
            for (uint32_t o : g.outputs)
                if ((o >> 1) == v) {
                    want |= (o & 1) ? kOutNeg : kOutPos;
                    --reads[v];
                }
            if ((s.flags & ~kXor) != want) return "output flags wrong";
        }
    }
    for (uint32_t k = 0; k < g.num_ands(); ++k)
        if (in_cone[k] && !done[k]) return "cone gate never computed";
    for (size_t j = 0; j < g.outputs.size(); ++j)
        if (!is_and(g, g.outputs[j] >> 1) && !out_only_done[j]) return "output-only step missing";
    for (uint32_t v = 0; v <= V; ++v)
        if (reads[v] != 0) return "unbalanced reads of variable " + std::to_string(v);
    return "";
}

}  // namespace fes
