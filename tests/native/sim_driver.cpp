// Runs the machine code of a native simulation pass on the host, word by word (CPU test of emit_sim).
//
//   sim_driver FILE.aig VGPRS WORDS
//
// encodes the file's circuit into VGPRS registers and runs one wave over WORDS columns (at most 64) of
// random input words, every register filled with rubbish first.  Compares every row with a plain
// evaluation, and prints the code as assembly text, one "asm" line per instruction with its words
// in hex; "does not fit" when the registers are too few.  Exit status 1 on a difference.
#include <cstdio>
#include <cstdlib>
#include <fstream>
#include <iterator>
#include <random>
#include <string>

#include "native.hpp"

using namespace fes;

int main(int argc, char** argv) {
    if (argc != 4) return 2;
    std::ifstream f(argv[1], std::ios::binary);
    const std::string bytes((std::istreambuf_iterator<char>(f)), {});
    const Aig g = parse_aiger((const uint8_t*)bytes.data(), bytes.size());
    const int vgprs = std::atoi(argv[2]);
    const uint32_t W = (uint32_t)std::atoi(argv[3]), n = g.num_inputs, rows = g.max_var() + 1;
    NativeCode code;
    if (!emit_sim(g, vgprs, code)) {
        std::printf("does not fit\n");
        return 0;
    }
    std::mt19937 rng(7);
    std::vector<uint32_t> pi((size_t)n * W), sig((size_t)rows * W + 64, 0xA5A5A5A5u), want((size_t)rows * W, 0);
    for (uint32_t& x : pi) x = rng();
    for (uint32_t i = 0; i < n; ++i)
        for (uint32_t c = 0; c < W; ++c) want[(size_t)(i + 1) * W + c] = pi[(size_t)i * W + c];
    for (uint32_t k = 0; k < g.num_ands(); ++k)
        for (uint32_t c = 0; c < W; ++c) {
            auto lit = [&](uint32_t l) { return want[(size_t)(l >> 1) * W + c] ^ (l & 1 ? ~0u : 0u); };
            want[(size_t)(n + 1 + k) * W + c] = lit(g.and_r0[k]) & lit(g.and_r1[k]);
        }
    // Addresses: input words at 1 << 40, the signature at 1 << 41.
    const uint64_t in = 1ull << 40, out = 1ull << 41;
    uint32_t v[256][64], s[106];
    for (auto& r : v)
        for (uint32_t& x : r) x = rng();
    for (uint32_t& x : s) x = rng();
    for (uint32_t l = 0; l < 64; ++l) v[2][l] = 4 * l;
    s[38] = (uint32_t)in, s[39] = (uint32_t)(in >> 32), s[40] = (uint32_t)out, s[41] = (uint32_t)(out >> 32);
    s[42] = 4 * W;
    uint64_t exec = ~0ull;
    const uint64_t lanes = W == 64 ? ~0ull : (1ull << W) - 1;
    s[44] = (uint32_t)lanes, s[45] = (uint32_t)(lanes >> 32);
    bool scc = false, waited = false, done = false;
    auto fail = [](const char* what, size_t pc) {
        std::printf("%s at word %zu\n", what, pc);
        std::exit(1);
    };
    const std::vector<uint32_t>& w = code.words;
    for (size_t pc = 0; pc < w.size() && !done;) {
        const uint32_t x = w[pc], y = pc + 1 < w.size() ? w[pc + 1] : 0;
        char t[96];
        int len = 1;
        if (x == 0xBF800000u) std::snprintf(t, sizeof t, "s_nop 0");
        else if (x == 0xBF8A0000u) std::snprintf(t, sizeof t, "s_barrier");
        else if (x == 0xBF8C0F70u) waited = true, std::snprintf(t, sizeof t, "s_waitcnt vmcnt(0)");
        else if (x == (0xBE800100u | 126u << 16 | 44u)) exec = s[44] | (uint64_t)s[45] << 32, std::snprintf(t, sizeof t, "s_mov_b64 exec, s[44:45]");
        else if (x == (0xBE800100u | 126u << 16 | 193u)) exec = ~0ull, std::snprintf(t, sizeof t, "s_mov_b64 exec, -1");
        else if (x == (0xBE801D00u | 36u)) done = true, std::snprintf(t, sizeof t, "s_setpc_b64 s[36:37]");
        else if (x >> 23 == 0x80000000u >> 23 || x >> 23 == 0x82000000u >> 23) {
            const uint32_t d = (x >> 16) & 127, b = (x >> 8) & 255, a = x & 255;
            const bool carry = x >> 23 == 0x82000000u >> 23;
            const uint64_t sum = (uint64_t)s[a] + (b == 128 ? 0u : s[b]) + (carry && scc ? 1 : 0);
            s[d] = (uint32_t)sum;
            scc = sum >> 32;
            if (b == 128) std::snprintf(t, sizeof t, "%s s%u, s%u, 0", carry ? "s_addc_u32" : "s_add_u32", d, a);
            else std::snprintf(t, sizeof t, "%s s%u, s%u, s%u", carry ? "s_addc_u32" : "s_add_u32", d, a, b);
        } else if ((x & 0xFFFFFF00u) == 0xD1410000u) {
            len = 2;
            if (y != 128) fail("move of something else", pc);
            for (int l = 0; l < 64; ++l)
                if (exec >> l & 1) v[x & 255][l] = 0;
            std::snprintf(t, sizeof t, "v_mov_b32_e64 v%u, 0", x & 255);
        } else if ((x & 0xFFFFF800u) == 0xD2340000u) {
            len = 2;
            const uint32_t tab = ((x >> 8) & 7) << 3 | ((y >> 27) & 3) << 6 | y >> 29;
            const uint32_t src[3] = {y & 511, (y >> 9) & 511, (y >> 18) & 511};
            uint32_t res[64];
            for (int l = 0; l < 64; ++l) {
                uint32_t val[3], r = 0;
                for (int i = 0; i < 3; ++i) val[i] = src[i] >= 256 ? v[src[i] - 256][l] : 0;
                for (int bit = 0; bit < 32; ++bit)
                    r |= ((tab >> ((val[0] >> bit & 1) * 4 + (val[1] >> bit & 1) * 2 + (val[2] >> bit & 1))) & 1u) << bit;
                res[l] = r;
            }
            for (int l = 0; l < 64; ++l)
                if (exec >> l & 1) v[x & 255][l] = res[l];
            char a[3][16];
            for (int i = 0; i < 3; ++i) src[i] >= 256 ? std::snprintf(a[i], 16, "v%u", src[i] - 256) : std::snprintf(a[i], 16, "0");
            std::snprintf(t, sizeof t, "v_bitop3_b32 v%u, %s, %s, %s bitop3:0x%x", x & 255, a[0], a[1], a[2], tab);
        } else if (x == 0xDC508000u || x == 0xDC708000u) {
            len = 2;
            const bool load = x == 0xDC508000u;
            const uint32_t base = (y >> 16) & 127, data = load ? y >> 24 : (y >> 8) & 255;
            for (int l = 0; l < 64; ++l) {
                if (!(exec >> l & 1)) continue;
                const uint64_t at = (s[base] | (uint64_t)s[base + 1] << 32) + v[y & 255][l];
                if (load ? at < in || at >= in + 4 * pi.size() || waited : at < out || at >= out + 4ull * rows * W) fail("address", pc);
                if (load) v[data][l] = pi[(at - in) / 4];
                else sig[(at - out) / 4] = v[data][l];
            }
            if (load) std::snprintf(t, sizeof t, "global_load_dword v%u, v%u, s[%u:%u]", data, y & 255, base, base + 1);
            else std::snprintf(t, sizeof t, "global_store_dword v%u, v%u, s[%u:%u]", y & 255, data, base, base + 1);
        } else fail("unknown word", pc);
        std::printf("asm %08x", x);
        if (len == 2) std::printf(" %08x", y);
        std::printf(" %s\n", t);
        pc += len;
    }
    if (!done || exec != ~0ull) fail("no return with all lanes on", w.size());
    for (size_t i = 0; i < (size_t)rows * W; ++i)
        if (sig[i] != want[i]) {
            std::printf("row %zu column %zu differs\n", i / W, i % W);
            return 1;
        }
    for (size_t i = 0; i < 64; ++i)
        if (sig[(size_t)rows * W + i] != 0xA5A5A5A5u) return 1;
    return 0;
}
