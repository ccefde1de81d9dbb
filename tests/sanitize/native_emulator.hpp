// One pass of a native kernel on the host (native_emulator.cpp).
#pragma once
#include <cstdint>

// The lowest failing pattern of the pass at `code` (all ones when there is none): packed half-word `base`,
// real half-word `real`, patterns of half-words [hw_begin, hw_end) only.
uint64_t emulate_pass(const uint32_t* code, uint64_t base, uint64_t real, uint64_t hw_begin, uint64_t hw_end);
