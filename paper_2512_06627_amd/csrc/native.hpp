// Native tier: a circuit's pass as gfx950 machine code written by the library itself.
//
// plan      cofactor.cpp     inner inputs and one shared graph of all their assignments
// map       lut.cpp          three-input LUTs
// encode    native_emit.cpp  registers and machine words
// run       native.cpp       code object, module, launches
#pragma once
#include <atomic>
#include <cstdint>
#include <memory>
#include <vector>

#include "aig.hpp"
#include "native_launch.hpp"
#include "plan.hpp"

namespace fes {

// The circuit evaluated under every assignment of some inner inputs, as one graph: gates that do
// not depend on an inner input are computed once and read by every assignment; the others once
// per distinct assignment of the inner inputs they depend on, with the constants folded in.
struct SharedCone {
    Aig aig;                      // over the remaining inputs (in their order), one output per assignment
    std::vector<uint32_t> order;  // gates of `aig` in evaluation order
    std::vector<uint64_t> offset; // per output: half-word offset of its assignment
    std::vector<uint32_t> bits;   // inner inputs' bits of the half-word index, ascending
    uint32_t peak_live = 0;       // values alive at once in that order
};

// Sets of inner inputs worth a try, the empty set first, each with its input of fewest dependent
// gates first, and the gate evaluations that the gates' supports predict for all of its assignments
// together.  Inputs 0..10 (bits of a word and of the lane) and inputs at or above `limit` are
// never inner.
struct InnerChoice {
    std::vector<uint32_t> inputs;
    uint64_t gates;
};
std::vector<InnerChoice> plan_inner(const Aig& g, const std::vector<uint32_t>& cone, uint32_t limit);
SharedCone share_cofactors(const Aig& g, const std::vector<uint32_t>& cone, const std::vector<uint32_t>& inner);

// The program's LUT steps in an order that keeps few values alive (outputs stay last): list
// scheduling by how many operands a step is the last to read.
void order_for_registers(LutProgram& lp);

// Machine code of one pass.
struct NativeCode {
    std::vector<uint32_t> words;
    uint32_t valu = 0, salu = 0, lds = 0;  // instructions on the straight path
    uint32_t lds_slots = 0;
};
// Encodes the mapped program; `offset` as in SharedCone (output t of the program belongs to
// assignment t).  vgprs: registers from v16 up.  lds_slots: spill slots of 256 bytes it may use.
// False when the pass needs more than that.
bool emit_native(const LutProgram& lp, const std::vector<uint64_t>& offset, int vgprs, int lds_slots, NativeCode& out);

// A simulation pass (native_sim.cpp, sim_body in native/es_native.hip): every variable's word, in order,
// to its row of the signature matrix.  vgprs: registers from v16 up.  False when the values alive at
// once need more.
bool emit_sim(const Aig& g, int vgprs, NativeCode& out);

// A circuit's pass, ready to run.  Immutable once built.
struct NativeKernel {
    NativeCode code;
    std::vector<uint32_t> bits;  // inner inputs' bits of the half-word index, ascending
    int waves = 3;               // per SIMD: 4, 3 or 2 (112, 152 or 240 registers)
    uint32_t limit = 0;          // inner inputs are below this input
    double build_ms = 0;
};

// The code object with the passes `codes` in its generated section; at[i] = offset of pass i.
std::vector<char> native_code_object(const std::vector<const NativeCode*>& codes, std::vector<uint64_t>* at);

// `limit`: as plan_inner.  `passes`: passes of 2,048 patterns that the kernel is built for.
// `weight`: what a millisecond of building costs against one of kernel time (0: nothing).
// `inner`: the number of inner inputs, or -1 for the one expected to be fastest.  Null when no
// choice fits the registers and LDS, or when *stop is set meanwhile.
std::shared_ptr<NativeKernel> build_native(const Aig& g, const std::vector<uint32_t>& cone, uint32_t limit,
                                           double passes, double weight, int inner = -1,
                                           const std::atomic<bool>* stop = nullptr);

// Expected kernel time of a pass of `valu` instructions with j inner inputs over `passes` passes.
double native_run_ms(double valu, uint32_t j, double passes);
// Expected time of build_native, for a cone of `gates` gates.
double native_build_ms(double gates);

}  // namespace fes
