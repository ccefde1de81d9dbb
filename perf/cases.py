"""The work that users of this framework have it do, as cases that can be timed.

A verification flow calls the library in six ways, and each listed case stands for one of them at
a size that such a flow meets:

* ``check``     one miter, every input pattern: the smallest (latency), ordinary datapath miters,
                cones too wide for the register file, the headline multiplier, a resumed word range;
* ``batch``     many cones in one call: the cones a partitioner hands over, and very small ones;
* ``simulate``  random-pattern simulation of every variable: a large signature matrix, a ragged one;
* ``hash``      signature hashes of a matrix whose rows are an odd number of words long;
* ``sweep``     a whole sweeping pass: simulate, hash, classes, sub-miters, one batched check;
* ``serve``     jobs submitted together to a server and polled until done.

The miters are the seeded ones of ``miters/``.  A checked miter is equivalent except at one input
pattern near the end of its space, drawn from the seed (a difference that only exhaustive
simulation shows), so an answer depends on the inputs and nearly the whole space is evaluated.
"""
import functools

import numpy as np
import torch

import miters
import paper_2512_06627_amd as es

_M64 = (1 << 64) - 1


def listed():
    return [
        # The smallest call: a 12-input miter, 4,096 patterns; launch and host latency.
        {"name": "check_mult6", "kind": "check", "circuit": "mult", "width": 6, "impl": "wallace", "kernel": "auto"},
        # An ordinary datapath miter (24 inputs) that a flow checks without asking for a compile.
        {"name": "check_mult12", "kind": "check", "circuit": "mult", "width": 12, "impl": "booth", "kernel": "auto"},
        # A wide cone (about 19,000 gates): its value file is larger than a wave's registers.
        {"name": "check_wide", "kind": "check", "circuit": "layered", "inputs": 23, "gates": 14000, "kernel": "auto"},
        # The headline: 16x16 multipliers, 2^32 patterns, on the kernel compiled for the circuit.
        {"name": "check_mult16", "kind": "check", "circuit": "mult", "width": 16, "impl": "booth",
         "kernel": "specialized"},
        # A multiply-accumulate datapath over an odd part of its words (a resumed or split check).
        {"name": "check_mac8_range", "kind": "check", "circuit": "mac", "width": 8, "kernel": "specialized",
         "begin_word": 12345677, "end_word": 54321011},
        # Cones of a partitioned design, a tenth of them faulty.
        {"name": "batch_cones", "kind": "batch", "count": 96, "faulty": 9, "n_lo": 18, "n_hi": 28, "gates_lo": 200,
         "gates_hi": 5000},
        # Many very small cones: launches and descriptors rather than patterns.
        {"name": "batch_small", "kind": "batch", "count": 512, "faulty": 51, "n_lo": 8, "n_hi": 16, "gates_lo": 50,
         "gates_hi": 2000},
        # Signatures of every node of the headline miter, 2^23 random patterns.
        {"name": "simulate_mult16", "kind": "simulate", "circuit": "mult", "width": 16, "impl": "booth",
         "words": 1 << 18},
        # A short ragged simulation (the first look at a cone).
        {"name": "simulate_ragged", "kind": "simulate", "circuit": "layered", "inputs": 27, "gates": 3000,
         "words": 1003},
        # Hashes of a signature matrix with odd row length, so most rows are not 8-byte aligned.
        {"name": "hash_ragged", "kind": "hash", "rows": 3111, "words": 100003},
        # One sweeping pass over the 12x12 miter, sub-miters loaded and checked as one batch.
        {"name": "sweep_mult12", "kind": "sweep", "circuit": "mult", "width": 12, "impl": "booth", "words": 1 << 12},
        # A burst of jobs served by continuous batching.
        {"name": "serve_burst", "kind": "serve", "count": 24, "n_lo": 16, "n_hi": 26, "gates_lo": 500,
         "gates_hi": 8000},
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["check", "check", "check", "check", "batch", "batch", "simulate", "simulate", "hash", "sweep",
                       "serve"])
    if kind == "check":
        form = rng.choice(["mult", "mac", "layered", "layered", "specialized", "range"])
        if form == "mult":
            return {"kind": kind, "circuit": "mult", "width": rng.randint(3, 13),
                    "impl": rng.choice(["booth", "wallace"]), "kernel": rng.choice(["auto", "interp"])}
        if form == "mac":
            return {"kind": kind, "circuit": "mac", "width": rng.randint(2, 6), "kernel": "auto"}
        if form == "layered":
            n = rng.randint(8, 25)
            return {"kind": kind, "circuit": "layered", "inputs": n, "gates": _log_int(rng, 150, 14000),
                    "kernel": rng.choice(["auto", "auto", "interp"])}
        if form == "specialized":
            return {"kind": kind, "circuit": "mult", "width": rng.randint(11, 15),
                    "impl": rng.choice(["booth", "wallace"]), "kernel": "specialized"}
        w = rng.randint(12, 14)
        words = 1 << (2 * w - 6)
        begin = rng.randrange(words // 2)
        return {"kind": kind, "circuit": "mult", "width": w, "impl": rng.choice(["booth", "wallace"]),
                "kernel": rng.choice(["auto", "specialized"]), "begin_word": begin,
                "end_word": begin + _log_int(rng, 1000, words // 2)}
    if kind == "batch":
        if rng.random() < 0.5:
            lo = rng.randint(6, 12)
            count = _log_int(rng, 16, 512)
            return {"kind": kind, "count": count, "faulty": rng.randint(0, count // 8), "n_lo": lo,
                    "n_hi": lo + rng.randint(0, 5), "gates_lo": 50, "gates_hi": _log_int(rng, 200, 2000)}
        lo = rng.randint(14, 20)
        count = _log_int(rng, 8, 80)
        return {"kind": kind, "count": count, "faulty": rng.randint(0, count // 8), "n_lo": lo,
                "n_hi": lo + rng.randint(2, 7), "gates_lo": 200, "gates_hi": _log_int(rng, 600, 6000)}
    if kind == "simulate":
        if rng.random() < 0.5:
            return {"kind": kind, "circuit": "mult", "width": rng.randint(6, 16),
                    "impl": rng.choice(["booth", "wallace"]), "words": _log_int(rng, 200, 250000)}
        return {"kind": kind, "circuit": "layered", "inputs": rng.randint(10, 40), "gates": _log_int(rng, 300, 16000),
                "words": _log_int(rng, 60, 70000)}
    if kind == "hash":
        rows = _log_int(rng, 300, 6000)
        return {"kind": kind, "rows": rows, "words": _log_int(rng, 100, min(250000, 600000000 // rows))}
    if kind == "sweep":
        return {"kind": kind, "circuit": "mult", "width": rng.randint(6, 12), "impl": rng.choice(["booth", "wallace"]),
                "words": _log_int(rng, 256, 8192)}
    lo = rng.randint(12, 18)
    return {"kind": kind, "count": rng.randint(8, 32), "n_lo": lo, "n_hi": lo + rng.randint(3, 8), "gates_lo": 300,
            "gates_hi": _log_int(rng, 800, 8000)}


# ---- circuits -----------------------------------------------------------------------------

@functools.lru_cache(maxsize=8)
def _base(circuit, width, impl, inputs, gates):
    if circuit == "mult":
        return miters.mult_miter(width, impl)
    if circuit == "mac":
        return miters.mac_miter(width)
    return miters.layered_cone_miter(1000 * inputs + gates, inputs, gates)


def _miter(case):
    return _base(case["circuit"], case.get("width"), case.get("impl"), case.get("inputs"), case.get("gates"))


def _words(case, n):
    whole = max(1, 1 << n >> 6)
    return case.get("begin_word", 0), case.get("end_word", whole)


def _rare_pattern(case, n, seed):
    """A pattern in the last 16th of the checked range (the upper half of a tiny one)."""
    begin, end = _words(case, n)
    lo, hi = 64 * begin, min(64 * end, 1 << n)
    return hi - 1 - miters.SplitMix64(seed).below((hi - lo) // (16 if hi - lo >= 4096 else 2))


def _with_difference(g, p):
    """Copy of a miter that is 1 at input pattern p too."""
    h = miters.Aig(g.num_inputs)
    out = miters.import_into(h, g)
    term = 1
    for i in range(g.num_inputs):
        term = h.AND(term, h.input(i) ^ (0 if (p >> i) & 1 else 1))
    acc = term
    for o in out:
        acc = h.OR(o, acc)
    h.add_output(acc)
    return h


@functools.lru_cache(maxsize=4)
def _cones(kind, seed, count, faulty, n_lo, n_hi, gates_lo, gates_hi):
    if kind == "serve":
        return miters.serve_pool(miters.SplitMix64(seed), seed, count, (n_lo, n_hi), (gates_lo, gates_hi))
    return miters.cone_batch(seed, count, faulty, (n_lo, n_hi), (gates_lo, gates_hi))


def _cones_of(case, seed):
    return _cones(case["kind"], seed, case["count"], case.get("faulty", 0), case["n_lo"], case["n_hi"],
                  case["gates_lo"], case["gates_hi"])


# ---- a case's inputs and one pass ----------------------------------------------------------

def _random_words(rows, words, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return torch.randint(-(1 << 31), 1 << 31, (rows, words), dtype=torch.int32, device="cuda", generator=gen)


def prepare(case, seed):
    kind = case["kind"]
    torch.cuda.init()
    s = {"kind": kind, "stream": torch.cuda.current_stream()}
    if kind == "check":
        g = _miter(case)
        c = es.fastlec_es_load_aig(_with_difference(g, _rare_pattern(case, g.num_inputs, seed)).to_aig())
        if case["kernel"] == "specialized":
            es.fastlec_es_compile_specialized(c, 3)
        s.update(circuit=c, kernel=case["kernel"])
        if "begin_word" in case:
            s["range"] = {"begin_word": case["begin_word"], "end_word": case["end_word"]}
    elif kind == "batch":
        s["circuits"] = [es.fastlec_es_load_aig(g.to_aig()) for g, _ in _cones_of(case, seed)]
    elif kind == "serve":
        s["circuits"] = [es.fastlec_es_load_aig(g.to_aig()) for g, _ in _cones_of(case, seed)]
        s["server"] = es.Server(8 << 30)
    elif kind == "hash":
        s["sig"] = _random_words(case["rows"], case["words"], seed)
        s["rows"], s["words"] = case["rows"], case["words"]
        s["hash"] = torch.empty(case["rows"], dtype=torch.int64, device="cuda")
        s["ones"] = torch.empty(case["rows"], dtype=torch.int64, device="cuda")
    else:  # simulate, sweep
        g = _miter(case)
        rows = g.max_var + 1
        s["circuit"] = es.fastlec_es_load_aig(g.to_aig())
        s["n"], s["rows"], s["words"] = g.num_inputs, rows, case["words"]
        s["pi"] = _random_words(g.num_inputs, case["words"], seed)
        s["sig"] = torch.empty((rows, case["words"]), dtype=torch.int32, device="cuda")
        s["hash"] = torch.empty(rows, dtype=torch.int64, device="cuda")
        s["ones"] = torch.empty(rows, dtype=torch.int64, device="cuda")
    return s


def _answers(results):
    return {f: np.array([r[f] for r in results], dtype=np.uint64).view(np.int64)
            for f in ("verdict", "cex", "patterns_evaluated", "next_word")}


def run(s):
    kind, stream = s["kind"], s["stream"]
    if kind == "check":
        return _answers([es.fastlec_es_check(s["circuit"], stream=stream, kernel=s["kernel"], **s.get("range", {}))])
    if kind == "batch":
        return _answers(es.fastlec_es_check_batch(s["circuits"], stream=stream))
    if kind == "serve":
        tickets = [s["server"].submit(c) for c in s["circuits"]]
        return _answers([s["server"].poll(t, wait=True) for t in tickets])
    if kind == "hash":
        es.fastlec_es_signature_hash(s["sig"], s["rows"], s["words"], s["hash"], s["ones"], stream=stream)
        return {"hash": s["hash"], "ones": s["ones"]}
    es.fastlec_es_simulate(s["circuit"], s["pi"], s["words"], s["sig"], stream=stream)
    if kind == "simulate":
        return {"sig": s["sig"]}
    es.fastlec_es_signature_hash(s["sig"], s["rows"], s["words"], s["hash"], s["ones"], stream=stream)
    classes = es.fastlec_es_classes(s["hash"].cpu().numpy().view(np.uint64))
    polarity = (s["sig"][:, 0] & 1).to(torch.uint8).cpu().numpy()
    targets = [v for v in range(s["n"] + 1, s["rows"]) if classes[v] != v]
    subs = [es.fastlec_es_load_aig(es.fastlec_es_submiter_aag(s["circuit"], classes, polarity, v)[0])
            for v in targets]
    found = _answers(es.fastlec_es_check_batch(subs, stream=stream)) if subs else _answers([])
    out = {"hash": s["hash"], "ones": s["ones"], "classes": classes.astype(np.int64)}
    for f, v in found.items():  # one entry per variable, -1 where it is its class's representative
        out[f] = np.full(s["rows"], -1, dtype=np.int64)
        out[f][targets] = v
    return out


# ---- what a pass cannot do without ------------------------------------------------------------

def _check_work(gates, patterns):
    """Circuit in, answer out; one 32-bit operation per AND gate and 32 patterns."""
    return 8.0 * gates + 32.0, gates * max(1.0, patterns / 32.0)


def work(case):
    kind = case["kind"]
    if kind == "hash":
        n = case["rows"] * case["words"]
        return {"bytes": 4.0 * n + 16.0 * case["rows"], "flops": 2.0 * n}
    if kind in ("batch", "serve"):
        every = [_check_work(g.num_ands(), 1 if fault is not None else 1 << g.num_inputs)
                 for g, fault in _cones_of(case, 1)]
        return {"bytes": sum(b for b, _ in every), "flops": sum(f for _, f in every)}
    g = _miter(case)
    if kind == "check":
        begin, end = _words(case, g.num_inputs)
        b, f = _check_work(g.num_ands(), min(64 * (end - begin), 1 << g.num_inputs))
        return {"bytes": b, "flops": f}
    rows = g.max_var + 1
    b = 4.0 * case["words"] * (rows + g.num_inputs) + 8.0 * g.num_ands()
    f = float(g.num_ands() * case["words"])
    if kind == "sweep":  # the matrix is read once more for its hashes
        b += 4.0 * case["words"] * rows + 16.0 * rows
        f += 2.0 * case["words"] * rows
    return {"bytes": b, "flops": f}


# ---- the same outputs in plain torch ------------------------------------------------------------

def _plain_rows(g, pi):
    """Every variable's words, one gate at a time."""
    sig = torch.empty((g.max_var + 1, pi.shape[1]), dtype=torch.int32, device=pi.device)
    sig[0] = 0
    sig[1:1 + g.num_inputs] = pi
    for k, (a, b) in enumerate(g.ands):
        x, y = sig[a >> 1], sig[b >> 1]
        sig[1 + g.num_inputs + k] = (~x if a & 1 else x) & (~y if b & 1 else y)
    return sig


def _plain_hash(sig):
    rows, words = sig.shape
    h = torch.arange(words, dtype=torch.int64, device=sig.device)
    h = h ^ (h >> 16)
    h = (h * 0x85EBCA6B) & 0xFFFFFFFF
    h = h ^ (h >> 13)
    h = (h * 0xC2B2AE35) & 0xFFFFFFFF
    key = (h ^ (h >> 16)) | 1
    hashes, ones = [], []
    for r in range(rows):
        w = sig[r].to(torch.int64) & 0xFFFFFFFF
        flip = 0xFFFFFFFF if int(w[0]) & 1 else 0
        hashes.append(((w ^ flip) * key).sum())
        c = w - ((w >> 1) & 0x55555555)
        c = (c & 0x33333333) + ((c >> 2) & 0x33333333)
        c = (c + (c >> 4)) & 0x0F0F0F0F
        ones.append((((c * 0x01010101) >> 24) & 0xFF).sum())
    return torch.stack(hashes), torch.stack(ones)


def exact(case, seed):
    """Signatures and hashes by plain torch; a check's answer where its space is small.  Larger
    spaces, batches and whole flows have no such value here (every pattern would be simulated one
    gate at a time)."""
    kind = case["kind"]
    if kind == "simulate":
        g = _miter(case)
        return {"sig": _plain_rows(g, _random_words(g.num_inputs, case["words"], seed))}
    if kind == "hash":
        h, ones = _plain_hash(_random_words(case["rows"], case["words"], seed))
        return {"hash": h, "ones": ones}
    if kind == "check":
        g = _miter(case)
        n = g.num_inputs
        if n <= 16 and "begin_word" not in case:
            g = _with_difference(g, _rare_pattern(case, n, seed))
            p = np.arange(1 << n, dtype=np.uint32)
            bits = np.stack([(p >> i) & 1 for i in range(n)]).astype(np.int32)
            out = g.outputs[0]
            v = _plain_rows(g, torch.from_numpy(-bits))[out >> 1]
            bad = torch.nonzero(~v if out & 1 else v)
            if len(bad):
                cex = int(bad[0])
                return _answers([{"verdict": 1, "cex": cex, "patterns_evaluated": cex + 1, "next_word": cex // 64}])
    return None
