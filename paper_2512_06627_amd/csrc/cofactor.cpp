// Inner inputs of a native pass and the graph that shares work between their assignments.
//
// Exact simulation evaluates the circuit at every input assignment (paper, Section 2.2).  Two
// assignments that differ in one input agree on every gate that input does not reach, so a pass
// that covers all 2^k assignments of k inner inputs evaluates such a gate once instead of 2^k times.
// With structural hashing and constant folding over the assignments, the 16x16 multiplier miter
// needs 1,554 VALU instructions per 2,048 patterns with no inner input and 316 with four (its last operand bits,
// which reach only the last rows of either multiplier).
#include <algorithm>
#include <utility>

#include "native.hpp"

namespace fes {

std::vector<InnerChoice> plan_inner(const Aig& g, const std::vector<uint32_t>& cone, uint32_t limit) {
    const uint32_t n = g.num_inputs, top = std::min(n, limit);
    std::vector<uint64_t> support(g.max_var() + 1, 0);
    for (uint32_t i = 11; i < top; ++i) support[i + 1] = 1ull << i;
    std::vector<uint64_t> masks;
    masks.reserve(cone.size());
    for (uint32_t k : cone) {
        const uint64_t m = support[g.and_r0[k] >> 1] | support[g.and_r1[k] >> 1];
        support[n + 1 + k] = m;
        masks.push_back(m);
    }
    std::sort(masks.begin(), masks.end());
    std::vector<std::pair<uint64_t, uint64_t>> kinds;  // support -> gates with it
    for (uint64_t m : masks) {
        if (kinds.empty() || kinds.back().first != m) kinds.push_back({m, 0});
        ++kinds.back().second;
    }
    auto gates_with = [&](uint64_t set) {
        uint64_t total = 0;
        for (auto& k : kinds) total += k.second << __builtin_popcountll(k.first & set);
        return total;
    };
    std::vector<InnerChoice> choices{{{}, cone.size()}};
    // By the gates' supports: each input that leaves the fewest evaluations beside those before it.
    std::vector<uint32_t> in;
    uint64_t chosen = 0;
    while (in.size() < kMaxInner) {
        uint64_t best = ~0ull;
        uint32_t pick = n;
        for (uint32_t i = 11; i < top; ++i) {
            if ((chosen >> i) & 1u) continue;
            const uint64_t total = gates_with(chosen | 1ull << i);
            if (total < best) {
                best = total;
                pick = i;
            }
        }
        if (pick == n) break;
        chosen |= 1ull << pick;
        in.push_back(pick);
        choices.push_back({in, best});
    }
    // The last inputs, from the last one down: in arithmetic they are the operand bits whose
    // products come last, so the assignments differ in one end of the circuit and fewer values stay
    // alive between them (16x16 miter, four inner inputs: 215 registers against more than 400).
    in.clear();
    chosen = 0;
    for (uint32_t i = top; i > 11 && in.size() < kMaxInner; --i) {
        in.push_back(i - 1);
        chosen |= 1ull << (i - 1);
        if (choices[in.size()].inputs != in) choices.push_back({in, gates_with(chosen)});
    }
    return choices;
}

namespace {

// Structural hashing of two-input gates (open addressing).
class Strash {
public:
    Strash(Aig& g, size_t expect) : g_(g) {
        size_t cap = 1024;
        while (cap < 2 * expect) cap *= 2;
        slots_.assign(cap, 0);
    }
    uint32_t land(uint32_t a, uint32_t b) {
        if (a > b) std::swap(a, b);
        if (a == 0) return 0;
        if (a == 1) return b;
        if (a == b) return a;
        if ((a ^ 1u) == b) return 0;
        if (2 * (size_t)g_.num_ands() + 2 > slots_.size()) grow();
        size_t h = hash(a, b);
        while (slots_[h]) {
            const uint32_t k = slots_[h] - 1;
            if (g_.and_r0[k] == b && g_.and_r1[k] == a) return 2 * (g_.num_inputs + 1 + k);
            h = (h + 1) & (slots_.size() - 1);
        }
        const uint32_t k = g_.num_ands();
        g_.and_r0.push_back(b);
        g_.and_r1.push_back(a);
        slots_[h] = k + 1;
        return 2 * (g_.num_inputs + 1 + k);
    }

private:
    size_t hash(uint32_t a, uint32_t b) const {
        const uint64_t x = (((uint64_t)a << 32) | b) * 0x9E3779B97F4A7C15ull;
        return (size_t)(x >> 20) & (slots_.size() - 1);
    }
    void grow() {
        std::vector<uint32_t> old(slots_.size() * 2, 0);
        slots_.swap(old);
        for (uint32_t k = 0; k < g_.num_ands(); ++k) {
            size_t h = hash(g_.and_r1[k], g_.and_r0[k]);
            while (slots_[h]) h = (h + 1) & (slots_.size() - 1);
            slots_[h] = k + 1;
        }
    }
    Aig& g_;
    std::vector<uint32_t> slots_;  // gate index + 1, 0 = empty
};

// Depth-first orders from the outputs, one assignment after the other: the fanin that needs more
// values first (Sethi-Ullman), fanin 0 first, fanin 1 first, and the graph's own order; the one with
// the fewest values alive at once is kept.
void order_gates(SharedCone& s) {
    const Aig& g = s.aig;
    const uint32_t n = g.num_inputs, A = g.num_ands();
    std::vector<uint32_t> label(g.max_var() + 1, 0);
    for (uint32_t k = 0; k < A; ++k) {
        const uint32_t a = label[g.and_r0[k] >> 1], b = label[g.and_r1[k] >> 1];
        label[n + 1 + k] = a == b ? a + 1 : std::max(a, b);
    }
    std::vector<uint8_t> state(A), needed(A, 0);  // state: 0 new, 1 fanins pushed, 2 ordered
    std::vector<uint32_t> stack, left(A), order;
    for (int kind = 0; kind < 4; ++kind) {
        order.clear();
        if (kind < 3) {
            std::fill(state.begin(), state.end(), 0);
            for (uint32_t o : g.outputs) {
                if ((o >> 1) <= n) continue;
                stack.push_back((o >> 1) - n - 1);
                while (!stack.empty()) {
                    const uint32_t k = stack.back();
                    if (state[k]) {
                        stack.pop_back();
                        if (state[k] == 1) order.push_back(k);
                        state[k] = 2;
                        continue;
                    }
                    state[k] = 1;
                    uint32_t first = g.and_r0[k] >> 1, second = g.and_r1[k] >> 1;
                    if (kind == 0 ? label[second] > label[first] : kind == 2) std::swap(first, second);
                    if (second > n && state[second - n - 1] == 0) stack.push_back(second - n - 1);
                    if (first > n && state[first - n - 1] == 0) stack.push_back(first - n - 1);
                }
            }
            if (kind == 0)
                for (uint32_t k : order) needed[k] = 1;
        } else {
            for (uint32_t k = 0; k < A; ++k)
                if (needed[k]) order.push_back(k);
        }
        std::fill(left.begin(), left.end(), 0);
        for (uint32_t k : order)
            for (uint32_t f : {g.and_r0[k] >> 1, g.and_r1[k] >> 1})
                if (f > n) ++left[f - n - 1];
        uint32_t live = 0, peak = 0;
        for (uint32_t k : order) {
            for (uint32_t f : {g.and_r0[k] >> 1, g.and_r1[k] >> 1})
                if (f > n && --left[f - n - 1] == 0) --live;
            if (left[k]) ++live;
            peak = std::max(peak, live);
        }
        if (kind == 0 || peak < s.peak_live) {
            s.peak_live = peak;
            s.order = order;
        }
    }
}

}  // namespace

SharedCone share_cofactors(const Aig& g, const std::vector<uint32_t>& cone, const std::vector<uint32_t>& inner) {
    const uint32_t n = g.num_inputs, k = (uint32_t)inner.size(), C = 1u << k;
    SharedCone s;
    s.aig.num_inputs = n - k;
    std::vector<int> place(n, -1);
    for (uint32_t j = 0; j < k; ++j) place[inner[j]] = (int)j;
    // lit[v] (or lit[at[v] + c] for a variable that depends on inner inputs, c restricted to those)
    std::vector<uint32_t> lit(g.max_var() + 1, 0), dep(g.max_var() + 1, 0);
    std::vector<uint32_t> many;
    uint32_t next = 0;
    for (uint32_t i = 0; i < n; ++i) {
        if (place[i] < 0) {
            lit[i + 1] = 2 * (++next);
            continue;
        }
        dep[i + 1] = 1u << place[i];
        lit[i + 1] = (uint32_t)many.size();
        for (uint32_t c = 0; c < C; ++c) many.push_back((c >> place[i]) & 1u);
    }
    auto get = [&](uint32_t l, uint32_t c) {
        const uint32_t v = l >> 1;
        return (dep[v] ? many[lit[v] + (c & dep[v])] : lit[v]) ^ (l & 1u);
    };
    Strash st(s.aig, 2 * cone.size());
    for (uint32_t q : cone) {
        const uint32_t v = n + 1 + q, a = g.and_r0[q], b = g.and_r1[q];
        dep[v] = dep[a >> 1] | dep[b >> 1];
        if (!dep[v]) {
            lit[v] = st.land(get(a, 0), get(b, 0));
            continue;
        }
        const uint32_t at = (uint32_t)many.size();
        many.resize(at + C);
        for (uint32_t c = 0; c < C; ++c)
            if ((c & ~dep[v]) == 0) many[at + c] = st.land(get(a, c), get(b, c));
        lit[v] = at;
    }
    for (uint32_t c = 0; c < C; ++c) {
        // The circuit's miter value is the OR of its outputs (paper, Section 2.1).
        std::vector<uint32_t> outs;
        for (uint32_t o : g.outputs) outs.push_back(get(o, c));
        while (outs.size() > 1) {
            std::vector<uint32_t> up;
            for (size_t i = 0; i + 1 < outs.size(); i += 2) up.push_back(st.land(outs[i] ^ 1u, outs[i + 1] ^ 1u) ^ 1u);
            if (outs.size() & 1u) up.push_back(outs.back());
            outs.swap(up);
        }
        s.aig.outputs.push_back(outs.empty() ? 0u : outs[0]);
        uint64_t off = 0;
        for (uint32_t j = 0; j < k; ++j)
            if ((c >> j) & 1u) off |= 1ull << (inner[j] - 5);
        s.offset.push_back(off);
    }
    for (uint32_t i : inner) s.bits.push_back(i - 5);
    std::sort(s.bits.begin(), s.bits.end());
    order_gates(s);
    return s;
}

}  // namespace fes
