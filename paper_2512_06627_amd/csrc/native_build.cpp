// From a circuit to the machine code of its pass, and from passes to a loadable code object.
// Host only: nothing here needs a device.
#include <elf.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>

#include "native.hpp"

// The code object of native/es_native.hip, embedded by the build.
extern "C" const char fes_native_template[];
extern "C" const char fes_native_template_end[];

namespace fes {
namespace {

double clock_ms() {
    using namespace std::chrono;
    return duration<double, std::milli>(steady_clock::now().time_since_epoch()).count();
}

// Milliseconds of a wave64 VALU instruction over the whole chip (1.0e12 a second) and in one wave
// alone (about five clocks); of building, per gate of the shared graph.
constexpr double kMsPerWaveInstr = 1.0e-9, kMsPerLoneInstr = 2.1e-6, kBuildMsPerGate = 0.8e-3;
constexpr double kLutsPerSharedGate = 0.26;
constexpr double kChipWaves = 256 * 4 * 2;
// A pass that shares work is not made longer than this: beyond 64 KB it streams through the instruction
// cache.  16x16 miter, 2^32 patterns: 8,519 instructions with five inner inputs, two waves per SIMD, 0.71 ms;
// 5,055 with four, three waves, 0.77.  MAC8: 5,368 with five 0.48 ms, 2,468 with four 0.43.  The estimate
// below takes four for both.
constexpr double kMaxSharedValu = 9000;
// Registers of the mapped and reordered program against values alive at once in the graph (0.5 to
// 0.75 on multipliers, up to 0.97 on layered cones).
constexpr double kVgprsPerLive = 0.58;

// Registers from v16 up and LDS spill slots by waves per SIMD (512 registers per SIMD lane, 160 KB
// of LDS per CU).
struct Tier {
    int waves, vgprs, slots;
};
constexpr Tier kTiers[] = {{4, 112, 0}, {3, 152, 0}, {3, 152, 53}, {2, 240, 0}, {2, 240, 80}};

// Time of an instruction against one at full rate, by the registers a pass is expected to take and
// its length.  16x16 and MAC8 miters: four waves per SIMD 1.04 to 1.10e12 instructions a second,
// three 1.00 to 1.07e12, two 0.88 to 0.94e12 (a wave issues at most every fifth clock); passes of
// 40 KB and more 0.78 to 0.86e12 against 12 KB, through the instruction cache.
double slowdown(double vgprs, double valu) {
    const double waves = vgprs <= 112 ? 1.0 : vgprs <= 152 ? 1.03 : vgprs <= 205 ? 1.1 : vgprs <= 240 ? 1.2 : vgprs / 200;
    return waves * (1.0 + 0.25 * std::min(1.0, std::max(0.0, (8 * valu - 12e3) / 28e3)));
}

}  // namespace

double native_run_ms(double valu, uint32_t j, double passes) {
    const double calls = std::max(1.0, std::ceil(passes / (double)(1u << j)));
    const double rounds = std::ceil(calls / kChipWaves);  // calls of the wave that has the most
    return std::max(calls * valu * kMsPerWaveInstr, std::min(calls, rounds) * valu * kMsPerLoneInstr);
}

double native_build_ms(double gates) { return 0.05 + kBuildMsPerGate * gates; }

std::shared_ptr<NativeKernel> build_native(const Aig& g, const std::vector<uint32_t>& cone, uint32_t limit,
                                           double passes, double weight, int inner, const std::atomic<bool>* stop) {
    auto stopped = [&] { return stop && stop->load(std::memory_order_relaxed); };
    const double t0 = clock_ms();
    struct Option {
        double ms;
        InnerChoice c;
        SharedCone s;
    };
    auto estimate = [&](double gates, uint32_t j) {
        return native_run_ms(kLutsPerSharedGate * gates, j, passes) + weight * kBuildMsPerGate * gates;
    };
    std::vector<Option> options;
    for (InnerChoice& c : plan_inner(g, cone, limit)) {
        const uint32_t j = (uint32_t)c.inputs.size();
        if (inner >= 0 ? j != (uint32_t)inner : j && kLutsPerSharedGate * (double)c.gates > 1.5 * kMaxSharedValu) continue;
        options.push_back({estimate((double)c.gates, j), std::move(c), {}});
    }
    auto by_time = [](const Option& a, const Option& b) { return a.ms < b.ms; };
    std::stable_sort(options.begin(), options.end(), by_time);
    // The shared graph of the best ones tells their true size and how many values they keep alive.
    std::vector<Option> tried;
    const size_t most = weight > 0 ? 2 : 6;
    for (Option& o : options) {
        const uint32_t j = (uint32_t)o.c.inputs.size();
        if (tried.size() >= most && j) continue;
        if (stopped()) return nullptr;
        o.s = share_cofactors(g, cone, o.c.inputs);
        const double vgprs = kVgprsPerLive * o.s.peak_live;
        const double luts = kLutsPerSharedGate * (double)o.s.order.size();
        if (inner < 0 && j && (vgprs > 320 || luts > kMaxSharedValu)) continue;
        o.ms = estimate((double)o.s.order.size(), j) * slowdown(vgprs, luts);
        tried.push_back(std::move(o));
    }
    std::stable_sort(tried.begin(), tried.end(), by_time);
    for (Option& o : tried) {
        Plan p;
        p.order = std::move(o.s.order);
        if (stopped()) return nullptr;
        LutProgram lp = make_lut_program(o.s.aig, p, 2);
        if (stopped()) return nullptr;
        order_for_registers(lp);
        auto k = std::make_shared<NativeKernel>();
        k->bits = o.s.bits;
        k->limit = limit;
        bool ok = false;
        for (const Tier& t : kTiers) {
            if (stopped()) return nullptr;
            k->waves = t.waves;
            ok = emit_native(lp, o.s.offset, t.vgprs, t.slots, k->code);
            // The third wave pays for a few LDS operations (one in twenty instructions), shared work
            // for one in eight; beyond that the wave, or the sharing, costs more than it saves.
            if (ok && k->code.lds > k->code.valu / (t.waves == 3 ? 20 : inner < 0 && !o.c.inputs.empty() ? 8 : 1)) ok = false;
            if (ok) break;
        }
        if (!ok) continue;
        k->build_ms = clock_ms() - t0;
        return k;
    }
    return nullptr;
}

std::vector<char> native_code_object(const std::vector<const NativeCode*>& codes, std::vector<uint64_t>* at) {
    const char* t = fes_native_template;
    const size_t size = (size_t)(fes_native_template_end - fes_native_template);
    Elf64_Ehdr eh;
    if (size < sizeof eh) throw Error{kErrDevice, "native template is not a code object"};
    std::memcpy(&eh, t, sizeof eh);
    std::vector<Elf64_Shdr> sh(eh.e_shnum);
    std::memcpy(sh.data(), t + eh.e_shoff, sizeof(Elf64_Shdr) * sh.size());
    std::vector<Elf64_Phdr> ph(eh.e_phnum);
    std::memcpy(ph.data(), t + eh.e_phoff, sizeof(Elf64_Phdr) * ph.size());
    const char* names = t + sh[eh.e_shstrndx].sh_offset;
    size_t sec = 0;
    for (size_t i = 0; i < sh.size(); ++i)
        if (!std::strcmp(names + sh[i].sh_name, ".fescode")) sec = i;
    if (!sec) throw Error{kErrDevice, "native template has no generated section"};
    // Passes on 64-byte lines (instruction cache), then a line of s_nop past the last one for the
    // instruction prefetcher.
    uint64_t need = 0;
    at->clear();
    for (const NativeCode* c : codes) {
        at->push_back(need);
        need += (4 * (uint64_t)c->words.size() + 63) & ~63ull;
    }
    need += 256;
    const uint64_t have = sh[sec].sh_size, off = sh[sec].sh_offset, addr = sh[sec].sh_addr;
    // The section grows by whole pages; everything behind it in the file or in memory moves by as much.
    const uint64_t grow = need > have ? (need - have + 4095) & ~4095ull : 0;
    std::vector<char> out(size + grow);
    std::memcpy(out.data(), t, off + have);
    std::memcpy(out.data() + off + have + grow, t + off + have, size - off - have);
    const uint32_t nop = 0xBF800000u;
    for (uint64_t b = 0; b < have + grow; b += 4) std::memcpy(out.data() + off + b, &nop, 4);
    for (size_t i = 0; i < codes.size(); ++i)
        std::memcpy(out.data() + off + (*at)[i], codes[i]->words.data(), 4 * codes[i]->words.size());
    if (!grow) return out;
    const uint64_t end_off = off + have, end_addr = addr + have;
    auto moved_off = [&](uint64_t o) { return o >= end_off ? o + grow : o; };
    auto moved_addr = [&](uint64_t a) { return a >= end_addr ? a + grow : a; };
    for (size_t i = 0; i < sh.size(); ++i) {
        Elf64_Shdr& s = sh[i];
        if (i == sec) {
            s.sh_size += grow;
            continue;
        }
        s.sh_offset = moved_off(s.sh_offset);
        if (s.sh_flags & SHF_ALLOC) s.sh_addr = moved_addr(s.sh_addr);
    }
    for (Elf64_Phdr& p : ph) {
        if (p.p_type == PT_LOAD && p.p_offset <= off && off < p.p_offset + p.p_filesz) {
            p.p_filesz += grow;
            p.p_memsz += grow;
        } else if (p.p_filesz || p.p_memsz) {
            p.p_offset = moved_off(p.p_offset);
            p.p_vaddr = moved_addr(p.p_vaddr);
            p.p_paddr = moved_addr(p.p_paddr);
        }
    }
    eh.e_shoff = moved_off(eh.e_shoff);
    std::memcpy(out.data(), &eh, sizeof eh);
    std::memcpy(out.data() + eh.e_phoff, ph.data(), sizeof(Elf64_Phdr) * ph.size());
    std::memcpy(out.data() + eh.e_shoff, sh.data(), sizeof(Elf64_Shdr) * sh.size());
    for (const Elf64_Shdr& s : sh) {
        if (s.sh_type != SHT_SYMTAB && s.sh_type != SHT_DYNSYM) continue;
        for (uint64_t o = 0; o + sizeof(Elf64_Sym) <= s.sh_size; o += sizeof(Elf64_Sym)) {
            Elf64_Sym sym;
            std::memcpy(&sym, out.data() + s.sh_offset + o, sizeof sym);
            if (sym.st_shndx == SHN_UNDEF || sym.st_shndx >= SHN_LORESERVE) continue;
            sym.st_value = moved_addr(sym.st_value);
            std::memcpy(out.data() + s.sh_offset + o, &sym, sizeof sym);
        }
    }
    return out;
}

}  // namespace fes
