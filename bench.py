"""Benchmark: exact simulation of the 16x16 multiplier miter on one MI355X.

One step = one complete exact simulation of the miter of a 16x16 array
multiplier against a radix-4 Booth/Wallace multiplier (32 inputs, 2^32
patterns, every pattern simulated because the miter is equivalent), through
the C ABI (fastlec_es_check), on PyTorch's current stream.  The metric is AND
node * pattern evaluations per second: N (AND gates in the output cone) times
2^32 per step.

Prints one JSON line.  Besides the headline it reports the roofline of the
simulation kernel (integer VALU bound; achieved from the kernel's own HIP
event time) and the plain CPU oracle timed on a bounded sample on the host.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

# Integer-VALU roofline of MI355X.  The published fp32 vector rate, 157.3 TFLOP/s = 256 CUs x
# 2.4 GHz x 128 lanes x 2 flops per FMA, gives 128 32-bit lanes per CU per cycle, and a 32-bit
# bitwise op issues at that lane rate (two wave64 VALU instructions per CU per cycle).  The
# roofline's peak is the larger of that figure and the issue rate the library's probe measures
# for the specialized kernel's instruction (fastlec_es_valu_probe: independent v_bitop3_b32
# chains).  One lane-op of the algorithmic view evaluates one AND gate on 32 patterns.
CUS, LANES_PER_CYCLE, CLOCK_HZ = 256, 128, 2.4e9
PEAK_LANE_OPS = CUS * LANES_PER_CYCLE * CLOCK_HZ        # 7.86e13 int32 lane-ops/s
PEAK_WAVE_INSTR = PEAK_LANE_OPS / 64                     # 1.23e12 wave64 VALU instructions/s
PEAK_NODE_PATTERNS = PEAK_LANE_OPS * 32                   # 2.52e15 AND-node*patterns/s
PEAK_HBM = 8.0e12                                        # bytes/s, MI355X HBM3E
PROBE_WAVES = (1, 2, 3, 4, 6, 7)                         # waves per SIMD swept by the probe leg
PROBE_ITERS = 20000                                      # 256 instructions per iteration


PROBE_VARIANTS = {0: "v_bitop3_b32, three VGPR sources in three banks", 1: "v_bitop3_b32, two VGPRs and an SGPR",
                  2: "v_xor_b32, two VGPRs"}


def valu_peak(es, waves=PROBE_WAVES, variants=(0, 1, 2), iters=PROBE_ITERS):
    """The library's issue-rate probe for each operand form and occupancy; returns the rates and
    the best (16 independent chains per wave, 256 instructions per loop iteration)."""
    rows = []
    for v in variants:
        for w in waves:
            es.fastlec_es_valu_probe(v, w, 100)  # first launch loads the code object
            r = es.fastlec_es_valu_probe(v, w, iters)
            rows.append({"variant": v, "waves_per_simd": w, "instr_per_s": r["instr_per_s"],
                         "kernel_ms": r["kernel_ms"], "per_cu_per_clock_at_2_4_GHz": r["instr_per_s"] / CUS / CLOCK_HZ})
    best = max(rows, key=lambda x: x["instr_per_s"])
    return {"variants": {str(k): v for k, v in PROBE_VARIANTS.items() if k in variants}, "iters": iters,
            "sweep": rows, "best_instr_per_s": best["instr_per_s"], "best_variant": best["variant"],
            "best_waves_per_simd": best["waves_per_simd"], "spec_instr_per_s": PEAK_WAVE_INSTR}


def cpu_model() -> str:
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def cpu_baseline(aag: bytes, num_ands: int, n: int, target_s: float = 12.0):
    """The oracle (one pattern at a time, all host cores) on an ascending prefix of the space;
    also its estimated time for the whole space at the measured rate."""
    import oracle
    c = oracle.Circuit(aag)
    threads = len(os.sched_getaffinity(0)) if hasattr(os, "sched_getaffinity") else os.cpu_count()
    threads = max(1, min(threads, int(os.environ.get("OMP_NUM_THREADS", threads))))
    patterns = 1 << 14
    while True:
        t0 = time.perf_counter()
        p, ev = c.lowest_failure(0, patterns, threads=threads)
        dt = time.perf_counter() - t0
        if p is not None:
            raise RuntimeError("oracle found a failure in an equivalent miter")
        if dt >= target_s / 4 or patterns >= 1 << 30:
            break
        patterns = min(1 << 30, int(patterns * max(2.0, min(16.0, target_s / max(dt, 1e-3)))))
        patterns = 1 << (patterns.bit_length() - 1)
    rate = num_ands * ev / dt
    return {"value": rate, "unit": "node*patterns/s", "cores": threads, "kind": "oracle",
            "cpu_model": cpu_model(),
            "sample": f"patterns [0, {patterns}) of the same miter, {dt:.1f} s on {threads} threads",
            "full_space_eta_s": num_ands * float(1 << n) / rate}


def batch_leg(es, stream, seed: int = 4, count: int = 256, faulty: int = 26, n_range=(18, 30),
              size_range=(200, 5000)):
    """`count` XOR-dense layered cones (n ~ U{n_range}, ~U[size_range] AND gates, `faulty` of them
    with an injected fault), checked four ways with identical answers: one plain check per cone on
    the interpreter; one batched call on the interpreter (persistent grouped launches, autotuned);
    one batched call with the runtime model's routing (native kernels where they pay, the other
    cones on the interpreter); one plain check per cone with the model's kernel choice once those
    kernels exist."""
    import miters
    t0 = time.perf_counter()
    cones, work = [], 0
    for g, _ in miters.cone_batch(seed, count, faulty, n_range, size_range):
        c = es.fastlec_es_load_aig(g.to_aig())
        cones.append(c)
        info = c.info()
        work += info["num_ands_tfi"] * (1 << info["num_pis"])
    gen_s = time.perf_counter() - t0

    def answers(rs):
        return [r["cex"] if r["verdict"] == es.FASTLEC_NONEQUIVALENT else None for r in rs]

    def timed(f, reps):
        ts, out = [], None
        for _ in range(reps):
            t0 = time.perf_counter()
            out = f()
            ts.append(time.perf_counter() - t0)
        return sorted(ts)[len(ts) // 2], out

    plain = answers([es.fastlec_es_check(c, stream=stream, kernel="interp") for c in cones])  # warm: uploads
    t_plain, plain2 = timed(lambda: answers([es.fastlec_es_check(c, stream=stream, kernel="interp") for c in cones]), 1)
    interp_first = answers(es.fastlec_es_check_batch(cones, stream=stream, kernel="interp"))  # autotune + capture
    t_batch_interp, got_interp = timed(lambda: answers(es.fastlec_es_check_batch(cones, stream=stream, kernel="interp")), 3)
    t0 = time.perf_counter()
    first = answers(es.fastlec_es_check_batch(cones, stream=stream))  # compiles + autotune + capture
    t_first = time.perf_counter() - t0
    t_batch, got = timed(lambda: answers(es.fastlec_es_check_batch(cones, stream=stream)), 3)
    t_plain_auto, plain_auto = timed(lambda: answers([es.fastlec_es_check(c, stream=stream) for c in cones]), 1)
    return {"cones": count, "n_range": list(n_range), "gates_range": list(size_range), "faulty_injected": faulty,
            "found_nonequivalent": sum(a is not None for a in got), "node_patterns_upper_bound": work,
            "plain_cones_per_s": count / t_plain, "batched_interp_cones_per_s": count / t_batch_interp,
            "batched_interp_vs_plain_speedup": t_plain / t_batch_interp,
            "batched_cones_per_s": count / t_batch, "batched_vs_plain_speedup": t_plain / t_batch,
            "plain_auto_cones_per_s": count / t_plain_auto, "batched_vs_plain_auto_speedup": t_plain_auto / t_batch,
            "identical_verdicts": plain == plain2 == interp_first == got_interp == first == got == plain_auto,
            "first_batch_call_s": t_first, "first_batch_call_cones_per_s": count / t_first, "generate_s": gen_s}


def interp_leg(es, stream, seed: int = 4, count: int = 256, faulty: int = 26, n_range=(18, 30),
               size_range=(200, 5000), reps: int = 3):
    """The interpreter alone on the batched workload's equivalent cones (every pattern simulated):
    one plain check per cone, so each cone is its own launch.  Rate in stream instructions x
    patterns per second (a fused three-AND XOR is one instruction) and in AND gates x patterns,
    over the summed kernel times."""
    import miters
    cones = []
    for g, fault in miters.cone_batch(seed, count, faulty, n_range, size_range):
        if fault is None:
            cones.append(es.fastlec_es_load_aig(g.to_aig()))
    instr_work = and_work = 0
    for c in cones:
        i = c.info()
        instr_work += (i["num_instrs"] - 2 * i["num_xors"]) * (1 << i["num_pis"])
        and_work += i["num_ands_tfi"] * (1 << i["num_pis"])
    for c in cones:  # uploads and schedules
        es.fastlec_es_check(c, stream=stream, kernel="interp")
    best = None
    for _ in range(reps):
        ms = 0.0
        for c in cones:
            r = es.fastlec_es_check(c, stream=stream, kernel="interp")
            assert r["verdict"] == es.FASTLEC_EQUIVALENT
            ms += r["kernel_ms"]
        best = ms if best is None else min(best, ms)
    return {"cones": len(cones), "kernel_ms_sum": best, "instr_patterns_per_s": instr_work / (best / 1e3),
            "and_patterns_per_s": and_work / (best / 1e3)}


def rsim_leg(es, stream, workload: str = "mult16_array_booth", words: int = 1 << 18, reps: int = 5):
    """Random-pattern simulation (sweeping step 1) on the headline miter: every variable's
    signature row over `words` 32-bit columns of seeded random input words, then the
    signature hashes and the candidate classes.  Both kernels are bound by HBM: the
    simulation writes (max_var + 1) x words x 4 bytes and reads n x words x 4; the hash
    kernel reads the signature matrix once."""
    import numpy as np
    import torch
    import miters
    g = miters.workload(workload)
    c = es.fastlec_es_load_aig(g.to_aig())
    info = c.info()
    n, V = info["num_pis"], info["num_pis"] + info["num_ands"]
    rng = np.random.default_rng(8)
    pi = torch.from_numpy(rng.integers(0, 1 << 32, size=(n, words), dtype=np.uint64).astype(np.uint32)
                          .view(np.int32)).cuda()
    sig = torch.empty((V + 1, words), dtype=torch.int32, device="cuda")
    h = torch.empty(V + 1, dtype=torch.int64, device="cuda")
    ones = torch.empty(V + 1, dtype=torch.int64, device="cuda")
    es.fastlec_es_simulate(c, pi, words, sig, stream=stream)
    es.fastlec_es_signature_hash(sig, V + 1, words, h, ones, stream=stream)
    sim_ms = sorted(es.fastlec_es_simulate(c, pi, words, sig, stream=stream) for _ in range(reps))[reps // 2]
    hash_ms = sorted(es.fastlec_es_signature_hash(sig, V + 1, words, h, ones, stream=stream)
                     for _ in range(reps))[reps // 2]
    t0 = time.perf_counter()
    cls = es.fastlec_es_classes(h.cpu().numpy().view(np.uint64))
    classes_ms = (time.perf_counter() - t0) * 1e3
    sizes = np.bincount(cls)
    sim_bytes = (V + 1) * words * 4 + n * words * 4
    hash_bytes = (V + 1) * words * 4
    del sig
    torch.cuda.empty_cache()
    return {"workload": workload, "words": words, "patterns": 32 * words, "rows": V + 1,
            "simulate_ms": sim_ms, "simulate_GBps": sim_bytes / (sim_ms / 1e3) / 1e9,
            "simulate_hbm_frac": sim_bytes / (sim_ms / 1e3) / PEAK_HBM,
            "simulate_node_patterns_per_s": info["num_ands"] * 32 * words / (sim_ms / 1e3),
            "hash_ms": hash_ms, "hash_GBps": hash_bytes / (hash_ms / 1e3) / 1e9,
            "hash_hbm_frac": hash_bytes / (hash_ms / 1e3) / PEAK_HBM,
            "classes_host_ms": classes_ms, "classes_with_2_or_more": int((sizes >= 2).sum()),
            "rows_in_such_classes": int(sizes[sizes >= 2].sum())}


def sweep_leg(es, stream, workload: str = "mult12_array_booth", words: int = 1 << 12):
    """One virtual sweeping pass (paper, Sections 2.3 and 3.2): simulate seeded random words,
    hash, group candidate classes, cut out every candidate pair's sub-miter and check them all
    with one batched exact-simulation call.  Times each stage; returns verdict counts."""
    import numpy as np
    import torch
    import miters
    g = miters.workload(workload)
    c = es.fastlec_es_load_aig(g.to_aig())
    info = c.info()
    n, V = info["num_pis"], info["num_pis"] + info["num_ands"]
    rng = np.random.default_rng(9)
    pi = torch.from_numpy(rng.integers(0, 1 << 32, size=(n, words), dtype=np.uint64).astype(np.uint32)
                          .view(np.int32)).cuda()
    sig = torch.empty((V + 1, words), dtype=torch.int32, device="cuda")
    h = torch.empty(V + 1, dtype=torch.int64, device="cuda")
    ones = torch.empty(V + 1, dtype=torch.int64, device="cuda")
    t = {}
    t0 = time.perf_counter()
    es.fastlec_es_simulate(c, pi, words, sig, stream=stream)
    es.fastlec_es_signature_hash(sig, V + 1, words, h, ones, stream=stream)
    hh = h.cpu().numpy().view(np.uint64)
    pol = (sig[:, 0] & 1).to(torch.uint8).cpu().numpy()
    t["simulate_hash_s"] = time.perf_counter() - t0
    t0 = time.perf_counter()
    cls = es.fastlec_es_classes(hh)
    targets = [v for v in range(n + 1, V + 1) if cls[v] != v]
    subs = [es.fastlec_es_submiter_aag(c, cls, pol, v)[0] for v in targets]
    circuits = [es.fastlec_es_load_aig(text) for text in subs]
    t["classes_extract_load_s"] = time.perf_counter() - t0
    work = sum(x.info()["num_ands_tfi"] * (1 << x.info()["num_pis"]) for x in circuits)
    t0 = time.perf_counter()
    res = es.fastlec_es_check_batch(circuits, stream=stream)
    t["batch_check_s"] = time.perf_counter() - t0
    eq = sum(r["verdict"] == es.FASTLEC_EQUIVALENT for r in res)
    return {"workload": workload, "words": words, "patterns": 32 * words, "targets": len(targets),
            "equivalent": eq, "nonequivalent": len(targets) - eq, "submiter_node_patterns": work,
            "batch_node_patterns_per_s": work / t["batch_check_s"], **t,
            "total_s": sum(t.values())}


def serve_leg(es, stream, seed: int = 5, seconds: float = 30.0, max_requests: int = 400,
              pool: int = 40, budget_gib: int = 64, load: float = 0.7):
    """Poisson stream of cones (n ~ U{16..34}, ~U[500, 20000] AND gates, 10% faulty) served by
    continuous batching with an HBM budget; large jobs move to their specialized kernel once it is
    compiled.  Capacity is measured on the same server first (every pool cone submitted at once;
    work = gates x patterns each job actually evaluated), and the arrival rate is set to `load` of
    it.  Reports p50/p90/p99 latency and checks every answer against the same cone checked
    alone."""
    import miters
    rng = miters.SplitMix64(seed)
    t0 = time.perf_counter()
    circs, gates = [], []
    for g, _ in miters.serve_pool(rng, seed, pool):
        c = es.fastlec_es_load_aig(g.to_aig())
        circs.append(c)
        gates.append(c.info()["num_ands_tfi"])
    gen_s = time.perf_counter() - t0
    srv = es.Server(budget_gib << 30, stream=None)
    t0 = time.perf_counter()
    cal = [srv.poll(t, wait=True) for t in [srv.submit(c) for c in circs]]
    cal_s = time.perf_counter() - t0
    works = [g * r["patterns_evaluated"] for g, r in zip(gates, cal)]
    capacity = sum(works) / cal_s
    lam = load / (cal_s / pool)
    print(json.dumps({"progress": "serve calibration", "seconds": cal_s, "capacity_node_patterns_per_s": capacity,
                      "arrival_rate_per_s": lam}), file=sys.stderr, flush=True)
    steps0 = srv.stats()["steps"]
    tickets, which = [], []
    start = time.perf_counter()
    t_next = 0.0
    while len(tickets) < max_requests and t_next < seconds:
        now = time.perf_counter() - start
        if now < t_next:
            time.sleep(min(0.05, t_next - now))
            continue
        k = rng.below(pool)
        tickets.append(srv.submit(circs[k]))
        which.append(k)
        t_next += rng.exponential(lam)
    results = [srv.poll(t, wait=True) for t in tickets]
    wall = time.perf_counter() - start
    st = srv.stats()
    srv.close()
    alone = {}
    for k in sorted(set(which)):  # the library's own choice of kernel (compiled ones are reused)
        r = es.fastlec_es_check(circs[k], stream=stream)
        alone[k] = r["cex"] if r["verdict"] == es.FASTLEC_NONEQUIVALENT else None
    served = [r["cex"] if r["verdict"] == es.FASTLEC_NONEQUIVALENT else None for r in results]
    lat = sorted(r["latency_ms"] for r in results)
    slow = sorted(range(len(results)), key=lambda i: -results[i]["latency_ms"])[:3]
    slowest = [{"n": circs[which[i]].info()["num_pis"], "gates": gates[which[i]],
                "latency_ms": round(results[i]["latency_ms"], 1), "queued_ms": round(results[i]["queued_ms"], 1),
                "device_ms": round(results[i]["kernel_ms"], 1), "work": works[which[i]]} for i in slow]
    q = lambda f: lat[min(len(lat) - 1, int(f * len(lat)))]
    done_work = sum(works[k] for k in which)
    return {"requests": len(tickets), "arrival_rate_per_s": lam, "offered_load": load,
            "capacity_node_patterns_per_s": capacity, "calibration_s": cal_s, "wall_s": wall,
            "latency_ms_p50": q(0.50), "latency_ms_p99": q(0.99), "requests_per_s": len(tickets) / wall,
            "node_patterns_per_s": done_work / wall, "max_jobs_in_flight": st["max_active"],
            "peak_charge_bytes": st["peak_charge_bytes"], "budget_bytes": st["budget_bytes"],
            "server_device_bytes": st["device_bytes"], "steps": st["steps"] - steps0,
            "specialized_slices": st["specialized_slices"], "latency_ms_p90": q(0.90), "latency_ms_max": lat[-1],
            "slowest": slowest,
            "each_equal_alone": served == [alone[k] for k in which], "pool": pool, "generate_s": gen_s}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=10)  # the first includes the compile; then clocks settle
    ap.add_argument("--kernel", default="specialized")
    ap.add_argument("--workload", default="mult16_array_booth")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-secondary", action="store_true", help="skip the MAC, batch and serving legs")
    ap.add_argument("--serve-seconds", type=float, default=30.0)
    ap.add_argument("--copy-calibration-mib", type=int, default=0,
                    help="also run one device-to-device copy of this many MiB (HBM counter calibration)")
    ap.add_argument("--leg", choices=["rsim", "sweep", "valu_peak", "interp", "batch", "serve"], default=None,
                    help="run only this leg (random simulation, a sweeping pass, the VALU issue-rate "
                         "probe, the interpreter, batch or serving workload) and print its JSON")
    a = ap.parse_args()
    if a.gpus != 1:
        print(f"bench.py runs on one GPU only: exact simulation here is a single-GPU build "
              f"(--gpus {a.gpus} requested)", file=sys.stderr)
        sys.exit(2)

    import torch
    import miters
    import paper_2512_06627_amd as es

    torch.cuda.init()
    stream = torch.cuda.current_stream()
    if a.copy_calibration_mib:
        src = torch.empty(a.copy_calibration_mib << 20, dtype=torch.uint8, device="cuda")
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    if a.leg:
        if a.leg == "valu_peak":
            print(json.dumps({"leg": a.leg, **valu_peak(es)}), flush=True)
            return
        leg = {"rsim": rsim_leg, "sweep": sweep_leg, "interp": interp_leg, "batch": batch_leg,
               "serve": lambda e, s: serve_leg(e, s, seconds=a.serve_seconds)}[a.leg]
        print(json.dumps({"leg": a.leg, **leg(es, stream)}), flush=True)
        return
    g = miters.workload(a.workload)
    aig = g.to_aig()
    t0 = time.perf_counter()
    c = es.fastlec_es_load_aig(aig)
    load_ms = (time.perf_counter() - t0) * 1e3
    info = c.info()
    n, N = info["num_pis"], info["num_ands_tfi"]
    node_patterns = N * (1 << n)

    compile_ms = 0.0
    for _ in range(a.warmup):
        r = es.fastlec_es_check(c, stream=stream, kernel=a.kernel)
        compile_ms += r["compile_ms"]
        if r["verdict"] != es.FASTLEC_EQUIVALENT:
            raise RuntimeError(f"expected an equivalent miter, got {r}")

    kernel_ms = []
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(a.steps):
        r = es.fastlec_es_check(c, stream=stream, kernel=a.kernel)
        kernel_ms.append(r["kernel_ms"])
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    for_each_ok = r["verdict"] == es.FASTLEC_EQUIVALENT and r["patterns_evaluated"] == 1 << n

    ms_per_step = elapsed * 1e3 / a.steps
    value = node_patterns * a.steps / elapsed
    k_ms = sorted(kernel_ms)[len(kernel_ms) // 2]
    k_mean_s = sum(kernel_ms) / len(kernel_ms) / 1e3
    achieved_np = node_patterns / k_mean_s
    # Roofline of the specialized kernel: executed wave64 VALU instructions per second (the
    # generated pass's count per call times the calls that cover the space; a call evaluates 2^inner
    # times 2,048 patterns) against the issue peak, the larger of the published figure and the
    # probe's measurement.
    probe = valu_peak(es, waves=(3, 7), variants=(1, 2))
    peak = max(PEAK_WAVE_INSTR, probe["best_instr_per_s"])
    counts = es.fastlec_es_native_info(c) if a.kernel == "specialized" else None
    if counts:
        valu, passes = counts["valu"], 1 << max(0, n - 11 - counts["inner"])
        roofline = {"bound": "alu", "achieved": valu * passes / k_mean_s, "peak": peak, "unit": "wave64 VALU instr/s",
                    "frac": valu * passes / k_mean_s / peak,
                    "traffic": None,
                    "kernel_ms_mean": k_mean_s * 1e3, "kernel_ms_median": k_ms,
                    "valu_per_call": valu, "inner_inputs": counts["inner"], "calls": passes,
                    "waves_per_simd": counts["waves_per_simd"],
                    "peak_spec": PEAK_WAVE_INSTR, "peak_probe": probe["best_instr_per_s"],
                    "note": "achieved = VALU instructions of the generated pass x its 2^(n-11-inner) calls / mean "
                            "kernel time (from its first workgroup's start); peak = max(256 CU x 2 wave64 instr/clk x 2.4 GHz, v_bitop3 probe)"}
    else:
        roofline = {"bound": "alu", "achieved": achieved_np, "peak": PEAK_NODE_PATTERNS, "unit": "node*patterns/s",
                    "frac": achieved_np / PEAK_NODE_PATTERNS, "traffic": None, "kernel_ms_mean": k_mean_s * 1e3,
                    "kernel_ms_median": k_ms, "note": "interpreter: algorithmic node*patterns against one lane-op per AND"}
    out = {
        "metric": "ES node*patterns/s (16x16 mult miter)",
        "value": value,
        "unit": "node*patterns/s",
        "n_gpus": 1,
        "steps": a.steps,
        "warmup": a.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "u32",
        "data": "synthetic",
        "config": {"workload": f"{a.workload}: {n} inputs, 2^{n} patterns, {N} AND gates in cone, "
                               f"equivalent (all patterns simulated)",
                   "kernel": a.kernel, "peak_live_slots": info["peak_live_slots"]},
        "roofline": roofline,
        "roofline_algorithmic": {"achieved": achieved_np, "one_op_per_and_peak": PEAK_NODE_PATTERNS,
                                 "unit": "node*patterns/s", "ratio": achieved_np / PEAK_NODE_PATTERNS,
                                 "and_gates_per_valu_instr": N * (1 << counts["inner"]) / counts["valu"] if counts else None,
                                 "note": "N*2^n per launch over a peak of one int32 lane-op per AND gate per 32 "
                                         "patterns; above 1 because one LUT instruction evaluates several AND gates "
                                         "and one call shares what its 2^inner input assignments have in common"},
        "load_ms": load_ms,
        "compile_ms": compile_ms,
        "all_steps_equivalent": bool(for_each_ok),
    }
    if not a.no_cpu:
        out["cpu_baseline"] = cpu_baseline(g.to_aag(), N, n)
    if not a.no_secondary:
        sec = {}
        mac = es.fastlec_es_load_aig(miters.workload("mac8_fused_separate").to_aig())
        for _ in range(3):  # compile, then let the clocks settle after the host-side compile
            es.fastlec_es_check(mac, stream=stream, kernel=a.kernel)
        rs = [es.fastlec_es_check(mac, stream=stream, kernel=a.kernel) for _ in range(5)]
        mac_ms = sorted(r["kernel_ms"] for r in rs)[2]
        mi = mac.info()
        sec["mac8"] = {"kernel_ms": mac_ms, "equivalent": all(r["verdict"] == es.FASTLEC_EQUIVALENT for r in rs),
                       "node_patterns_per_s": mi["num_ands_tfi"] * (1 << mi["num_pis"]) / (mac_ms / 1e3)}
        print(json.dumps({"progress": "mac8", **sec["mac8"]}), file=sys.stderr, flush=True)
        sec["batch"] = batch_leg(es, stream)
        print(json.dumps({"progress": "batch", **sec["batch"]}), file=sys.stderr, flush=True)
        sec["batch_small"] = batch_leg(es, stream, seed=6, count=2048, faulty=205, n_range=(8, 16),
                                       size_range=(50, 2000))
        print(json.dumps({"progress": "batch_small", **sec["batch_small"]}), file=sys.stderr, flush=True)
        sec["rsim"] = rsim_leg(es, stream)
        print(json.dumps({"progress": "rsim", **sec["rsim"]}), file=sys.stderr, flush=True)
        sec["sweep"] = sweep_leg(es, stream)
        print(json.dumps({"progress": "sweep", **sec["sweep"]}), file=sys.stderr, flush=True)
        sec["serve"] = serve_leg(es, stream, seconds=a.serve_seconds)
        out["secondary"] = sec
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
