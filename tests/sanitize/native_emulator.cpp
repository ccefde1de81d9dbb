// Executes the machine code of a native pass, with the report routine of native/es_native.hip.  The
// instructions are those of tests/native/native_driver.cpp.  A file of its own, compiled without a
// sanitizer: it shares nothing with other threads.
#include <vector>

#include "native_emulator.hpp"

#define main native_driver_main
#include "../native/native_driver.cpp"
#undef main

uint64_t emulate_pass(const uint32_t* code, uint64_t base, uint64_t real, uint64_t hw_begin, uint64_t hw_end) {
    static thread_local Machine m;
    m.lds.clear();
    for (int l = 0; l < 64; ++l) {
        for (int i = 0; i < 6; ++i) m.v[2 + i][l] = 0u - ((uint32_t)(l >> i) & 1u);
        m.v[8][l] = 4u * (uint32_t)l;
    }
    m.s[38] = (uint32_t)base;
    m.s[39] = (uint32_t)(base >> 32);
    uint64_t found = ~0ull;
    std::vector<uint32_t> w(2);
    auto run = [&](const uint32_t* at) {
        w[0] = at[0];
        w[1] = at[1];
        return step(w, 0, m, true).words;
    };
    for (const uint32_t* pc = code;;) {
        const uint32_t x = *pc;
        if ((x & 0xFFFFFF00u) == 0xBE801D00u) return found;  // back to the kernel
        if ((x >> 16) == 0xBF87 && m.vcc) {                  // the report
            const uint32_t* q = pc + 1 + (int64_t)(int16_t)x;
            while ((*q & 0xFF80FF00u) != 0xBE801E00u) q += run(q);
            const uint64_t hw0 = real + ((uint64_t)m.s[54] | (uint64_t)m.s[55] << 32);
            for (int l = 0; l < 64; ++l) {
                const uint64_t hw = hw0 + (uint64_t)l;
                if (!((m.vcc >> l) & 1) || hw < hw_begin || hw >= hw_end) continue;
                const uint64_t p = 32 * hw + (uint64_t)__builtin_ctz(m.v[15][l]);
                if (p < found) found = p;
                break;
            }
            ++pc;
            continue;
        }
        pc += run(pc);
    }
}
