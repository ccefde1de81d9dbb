// Runs the machine code of native passes on the host, word by word (CPU test of the planner,
// the mapper and the encoder).  No GPU and no HIP.
//
//   native_driver FILE.aig K VGPRS LDS_SLOTS BASE...
//
// plans the file's circuit with the first K inner inputs that plan_inner picks, encodes its pass into
// VGPRS registers and LDS_SLOTS spill slots, and for every packed half-word BASE prints
//   pass BASE
//   word OFFSET LANE0 .. LANE63     one line per assignment: the miter words the pass compares
// first "inner BITS..." and "size WORDS VALU SALU LDS SLOTS", last the pass as assembly text, one
// "asm" line per instruction with its words in hex.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <iterator>
#include <map>
#include <string>

#include "native.hpp"

using namespace fes;

namespace {

struct Machine {
    uint32_t v[256][64] = {};
    uint32_t s[106] = {};
    std::map<uint32_t, uint32_t> lds;
    uint64_t vcc = 0;
};

struct Text {
    std::string line;
    int words;
};

std::string src_text(uint32_t c, uint32_t literal) {
    char b[32];
    if (c >= 256) std::snprintf(b, sizeof b, "v%u", c - 256);
    else if (c <= 101) std::snprintf(b, sizeof b, "s%u", c);
    else if (c >= 128 && c <= 192) std::snprintf(b, sizeof b, "%u", c - 128);
    else if (c >= 193 && c <= 208) std::snprintf(b, sizeof b, "-%u", c - 192);
    else if (c == 255) std::snprintf(b, sizeof b, "0x%x", literal);
    else std::snprintf(b, sizeof b, "?%u", c);
    return b;
}

uint32_t src_value(const Machine& m, uint32_t c, uint32_t literal, int lane) {
    if (c >= 256) return m.v[c - 256][lane];
    if (c <= 101) return m.s[c];
    if (c >= 128 && c <= 192) return c - 128;
    if (c >= 193 && c <= 208) return 0u - (c - 192);
    return literal;
}

// Executes (run) and describes the instruction at w[pc].
Text step(const std::vector<uint32_t>& w, size_t pc, Machine& m, bool run) {
    char b[160];
    const uint32_t x = w[pc], y = pc + 1 < w.size() ? w[pc + 1] : 0;
    if ((x >> 16) == 0xD234) {
        const uint32_t s0 = y & 511, s1 = (y >> 9) & 511, s2 = (y >> 18) & 511;
        const uint32_t t = ((y >> 29) & 7) | ((x >> 8) & 7) << 3 | ((y >> 27) & 3) << 6, d = x & 255;
        std::snprintf(b, sizeof b, "v_bitop3_b32 v%u, %s, %s, %s bitop3:0x%x", d, src_text(s0, 0).c_str(),
                      src_text(s1, 0).c_str(), src_text(s2, 0).c_str(), t);
        int sg = -1;
        for (uint32_t c : {s0, s1, s2})
            if (c <= 101) {
                if (sg >= 0 && sg != (int)c) std::exit(3);  // two different SGPRs in one VALU instruction
                sg = (int)c;
            }
        if (run)
            for (int l = 0; l < 64; ++l) {
                const uint32_t p = src_value(m, s0, 0, l), q = src_value(m, s1, 0, l), r = src_value(m, s2, 0, l);
                uint32_t o = 0;
                for (uint32_t i = 0; i < 8; ++i)
                    if ((t >> i) & 1) o |= ((i & 4) ? p : ~p) & ((i & 2) ? q : ~q) & ((i & 1) ? r : ~r);
                m.v[d][l] = o;
            }
        return {b, 2};
    }
    if ((x & 0xFE01FE00u) == 0x7E000200u || (x & 0xFE01FE00u) == 0x7E005600u) {
        const bool inv = (x & 0x1FE00u) == 0x5600u;
        const uint32_t d = (x >> 17) & 255, c = x & 511;
        std::snprintf(b, sizeof b, "%s v%u, %s", inv ? "v_not_b32" : "v_mov_b32", d, src_text(c, y).c_str());
        if (run)
            for (int l = 0; l < 64; ++l) m.v[d][l] = src_value(m, c, y, l) ^ (inv ? ~0u : 0u);
        return {b, c == 255 ? 2 : 1};
    }
    if ((x & 0xFFFFFF00u) == 0xD1410000u) {
        const uint32_t d = x & 255, c = y & 511;
        std::snprintf(b, sizeof b, "v_mov_b32_e64 v%u, %s", d, src_text(c, 0).c_str());
        if (run)
            for (int l = 0; l < 64; ++l) m.v[d][l] = src_value(m, c, 0, l);
        return {b, 2};
    }
    if (x == 0xBF800000u) return {"s_nop 0", 1};
    if ((x >> 23) == 0x126) {  // s_bfe_i32
        const uint32_t d = (x >> 16) & 127, c = x & 255;
        if (((x >> 8) & 255) != 255) std::exit(4);
        std::snprintf(b, sizeof b, "s_bfe_i32 s%u, %s, 0x%x", d, src_text(c, 0).c_str(), y);
        if (run) m.s[d] = (m.s[c] >> (y & 31)) & 1 ? ~0u : 0u;
        if ((y >> 16) != 1) std::exit(5);
        return {b, 2};
    }
    if ((x & 0xFFFE0000u) == 0x7D9A0000u) {
        const uint32_t v = (x >> 9) & 255, c = x & 511;
        std::snprintf(b, sizeof b, "v_cmp_ne_u32 vcc, %s, v%u", src_text(c, 0).c_str(), v);
        if (run) {
            m.vcc = 0;
            for (int l = 0; l < 64; ++l) m.vcc |= (uint64_t)(src_value(m, c, 0, l) != m.v[v][l]) << l;
        }
        return {b, 1};
    }
    if ((x >> 16) == 0xBF87 || (x >> 16) == 0xBF82) {
        std::snprintf(b, sizeof b, "%s %d", (x >> 16) == 0xBF87 ? "s_cbranch_vccnz" : "s_branch", (int)(int16_t)x);
        return {b, 1};
    }
    if (x == 0xBF8CC07Fu) return {"s_waitcnt lgkmcnt(0)", 1};
    if ((x & 0xFFFF0000u) == 0xD81A0000u || (x & 0xFFFF0000u) == 0xD86C0000u) {
        const bool wr = (x >> 16) == 0xD81A;
        const uint32_t off = x & 0xFFFF, a = y & 255, r = wr ? (y >> 8) & 255 : y >> 24;
        if (wr) std::snprintf(b, sizeof b, "ds_write_b32 v%u, v%u offset:%u", a, r, off);
        else std::snprintf(b, sizeof b, "ds_read_b32 v%u, v%u offset:%u", r, a, off);
        if (run)
            for (int l = 0; l < 64; ++l) {
                if (wr) m.lds[m.v[a][l] + off] = m.v[r][l];
                else m.v[r][l] = m.lds.at(m.v[a][l] + off);
            }
        return {b, 2};
    }
    if ((x & 0xFF80FF00u) == 0xBE800000u) {
        const uint32_t c = x & 255;
        std::snprintf(b, sizeof b, "s_mov_b32 s%u, %s", (x >> 16) & 127, src_text(c, y).c_str());
        if (run) m.s[(x >> 16) & 127] = src_value(m, c, y, 0);
        return {b, c == 255 ? 2 : 1};
    }
    if ((x & 0xFFFFFF00u) == 0xBE801D00u) {
        std::snprintf(b, sizeof b, "s_setpc_b64 s[%u:%u]", x & 255, (x & 255) + 1);
        return {b, 1};
    }
    if ((x & 0xFF80FF00u) == 0xBE801E00u) {
        const uint32_t d = (x >> 16) & 127;
        std::snprintf(b, sizeof b, "s_swappc_b64 s[%u:%u], s[%u:%u]", d, d + 1, x & 255, (x & 255) + 1);
        return {b, 1};
    }
    std::fprintf(stderr, "unknown instruction %08x at %zu\n", x, pc);
    std::exit(2);
}

}  // namespace

int main(int argc, char** argv) {
    if (argc < 5) return 1;
    std::ifstream f(argv[1], std::ios::binary);
    const std::string bytes((std::istreambuf_iterator<char>(f)), std::istreambuf_iterator<char>());
    const Aig g = parse_aiger((const uint8_t*)bytes.data(), bytes.size());
    const Plan p1 = make_plan(g);
    const uint32_t k = (uint32_t)std::atoi(argv[2]);
    const std::vector<InnerChoice> choices = plan_inner(g, p1.order, g.num_inputs);
    if (choices.size() <= k || choices[k].inputs.size() != k) return 6;
    const SharedCone s = share_cofactors(g, p1.order, choices[k].inputs);
    Plan p;
    p.order = s.order;
    const LutProgram lp = make_lut_program(s.aig, p, 2);
    NativeCode c;
    if (!emit_native(lp, s.offset, std::atoi(argv[3]), std::atoi(argv[4]), c)) {
        std::printf("does not fit\n");
        return 0;
    }
    std::printf("inner");
    for (uint32_t b : s.bits) std::printf(" %u", b);
    std::printf("\nsize %zu %u %u %u %u\n", c.words.size(), c.valu, c.salu, c.lds, c.lds_slots);
    for (int a = 5; a < argc; ++a) {
        const uint64_t base = std::strtoull(argv[a], nullptr, 0);
        std::printf("pass %llu\n", (unsigned long long)base);
        static Machine m;
        m = Machine();
        for (auto& r : m.v)
            for (uint32_t& x : r) x = 0xDEADBEEFu;  // nothing is left over from before a pass
        for (int l = 0; l < 64; ++l) {
            for (int i = 0; i < 6; ++i) m.v[2 + i][l] = 0u - ((uint32_t)(l >> i) & 1u);
            m.v[8][l] = 4u * (uint32_t)l;
        }
        m.s[38] = (uint32_t)base;
        m.s[39] = (uint32_t)(base >> 32);
        for (size_t pc = 0;;) {
            const uint32_t x = c.words[pc];
            if ((x & 0xFFFFFF00u) == 0xBE801D00u) break;  // back to the kernel
            if ((x >> 16) == 0xBF87) {  // always take the report, then go on behind the branch
                size_t q = pc + 1 + (size_t)(int64_t)(int16_t)x;
                while ((c.words[q] & 0xFF80FF00u) != 0xBE801E00u) q += (size_t)step(c.words, q, m, true).words;
                if (c.words[q] != 0xBEB41E30u) return 7;  // the report routine, return address in s[52:53]
                std::printf("word %llu", (unsigned long long)m.s[54] | (unsigned long long)m.s[55] << 32);
                for (int l = 0; l < 64; ++l) {
                    if (((m.vcc >> l) & 1) != (m.v[15][l] != 0)) return 8;
                    std::printf(" %x", m.v[15][l]);
                }
                std::printf("\n");
                ++q;
                if ((c.words[q] >> 16) != 0xBF82 || q + 1 + (size_t)(int64_t)(int16_t)c.words[q] != pc + 1) return 9;
            }
            pc += (size_t)step(c.words, pc, m, true).words;
        }
    }
    Machine none;
    for (size_t pc = 0; pc < c.words.size();) {
        const Text t = step(c.words, pc, none, false);
        std::printf("asm %s |", t.line.c_str());
        for (int i = 0; i < t.words; ++i) std::printf(" %08x", c.words[pc + i]);
        std::printf("\n");
        pc += (size_t)t.words;
    }
    return 0;
}
