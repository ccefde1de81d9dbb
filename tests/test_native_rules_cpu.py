"""When native kernels are built, waited for and used: checks, batches and the server on the host
stand-in of a GPU (tests/standin.py), driven through the package.

Each test runs a script in a process of its own, with the library's trace switched on.
"""
import os
import subprocess
import sys

import pytest

import standin

HEAD = """
import sys, time
sys.path.insert(0, {root!r})
import miters, paper_2512_06627_amd as es
es.LIB_PATH = {lib!r}

def load(g):
    return es.fastlec_es_load_aig(g.to_aig())

def chain(steps, n=12):
    "Rounds of s[i] ^= s[i+1] & s[i+5]: four gates a step, few values alive."
    g = miters.Aig(n)
    s = [g.input(i) for i in range(n)]
    for k in range(steps):
        i = k % n
        s[i] = g.XOR(s[i], g.AND(s[(i + 1) % n] ^ (k // n & 1), s[(i + 5) % n] ^ (k // (2 * n) & 1)))
    g.add_output(g.AND(s[0], s[1]))
    return g

def chain_value(steps, pattern, n=12):
    s = [(pattern >> i) & 1 for i in range(n)]
    for k in range(steps):
        i = k % n
        s[i] ^= (s[(i + 1) % n] ^ (k // n & 1)) & (s[(i + 5) % n] ^ (k // (2 * n) & 1))
    return s[0] & s[1]
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not os.path.exists(standin.CLANG):
        pytest.skip("clang++ not found")
    return standin.build(tmp_path_factory.mktemp("native_rules"))


def run(lib, script, **env):
    env = dict(os.environ, FASTLEC_ES_TRACE="1", **env)
    r = subprocess.run([sys.executable, "-c", HEAD.format(root=standin.ROOT, lib=lib) + script], capture_output=True,
                       text=True, timeout=300, env=env)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-4000:])
    return r


def test_one_word_of_a_long_circuit(lib):
    """A word that takes the interpreter more than a millisecond is still one piece of a check while the
    kernel is being built."""
    r = run(lib, """
steps, want = 32000, [p for p in range(64) if chain_value(32000, p)]
c = load(chain(steps))
for i in range(160):
    r = es.fastlec_es_check(c, begin_word=0, end_word=1)
    assert (r["verdict"], r["cex"]) == ((1, want[0]) if want else (0, 0)), r
""")
    assert "native: 0 inner inputs" in r.stderr, r.stderr[-2000:]


def test_a_circuit_without_kernel_is_tried_once(lib):
    """A cone too wide for registers and LDS: AUTO checks, batches and explicit builds all end in no kernel, and
    only the first of each weight goes through the planning, mapping and encoding (some 20 ms)."""
    r = run(lib, """
c = load(miters.layered_cone_miter(1, 14, 27000))
def spent(f, times):
    t = time.perf_counter()
    for _ in range(times):
        f()
    return time.perf_counter() - t
def auto():
    assert es.fastlec_es_check(c, begin_word=0, end_word=1)["verdict"] == 0
def batch():
    assert [x["verdict"] for x in es.fastlec_es_check_batch([c, c])] == [0, 0]
def info():
    try:
        es.fastlec_es_native_info(c)
        assert False
    except es.EsError:
        pass
spent(auto, 200)   # more than a build's time on the interpreter
late = min(spent(auto, 20) / 20 for _ in range(3))
whole = min(spent(info, 1) for _ in range(3))
print("late", late, "info", whole)
assert late < 5e-3 and whole < 1e-3
for _ in range(3):
    batch()
for _ in range(3):
    assert es.fastlec_es_check(c, kernel="specialized", begin_word=0, end_word=1)["verdict"] == 0
""")
    # one word, under AUTO and SPECIALIZED; the whole space for info, which tries every choice
    assert r.stderr.count("native: no kernel") == 3, r.stdout + r.stderr[-3000:]


def test_a_deadline_holds_while_a_kernel_is_built(lib):
    """Checks of a word, a fraction of a millisecond on the interpreter, with deadlines that are shorter than
    building the kernel (about 0.25 s): none runs into its deadline.  With time enough the kernel is built."""
    r = run(lib, """
word = 64 * 7
want = next((p for p in range(word, word + 64) if chain_value(64000, p)), None)
c = load(chain(64000))
def check(**kw):
    t = time.perf_counter()
    r = es.fastlec_es_check(c, begin_word=7, end_word=8, **kw)
    assert (r["verdict"], r["cex"]) == ((0, 0) if want is None else (1, want)), r
    return time.perf_counter() - t
for i in range(200):
    check(deadline_s=0.1)
print("no kernel yet", flush=True)
print("no kernel yet", file=sys.stderr, flush=True)
for i in range(3):
    check(deadline_s=60.0)
""")
    before, after = r.stderr.split("no kernel yet")
    assert "inner inputs" not in before and "native: 0 inner inputs" in after, r.stderr[-2000:]


@pytest.mark.parametrize("how", ["cancel", "deadline"])
def test_a_check_is_stopped_while_its_kernel_is_built(lib, how):
    """In the caller's device memory nothing is interpreted meanwhile: cancelled, or at its deadline, in the middle
    of the building, a check ends without the kernel and says that it has covered nothing."""
    r = run(lib, """
import ctypes, threading
g = miters.Aig(32)
for o in miters.import_into(g, chain(40000, 32)):
    g.add_output(o)
g.add_output(g.input(0) ^ 1)  # a check that is not stopped ends at once
c = load(g)
how, flag = %r, ctypes.c_int(0)
class Scratch:
    mem = ctypes.create_string_buffer(1 << 16)
    def data_ptr(self): return (ctypes.addressof(self.mem) + 255) // 256 * 256
    def numel(self): return 4096
    def element_size(self): return 1
kw = {"cancel_flag": flag} if how == "cancel" else {"deadline_s": 0.03}
if how == "cancel":
    threading.Timer(0.02, lambda: setattr(flag, "value", 1)).start()
try:
    es.fastlec_es_check(c, scratch=Scratch(), **kw)
    assert False
except es.EsError as e:
    assert e.code == (es.FASTLEC_CANCELLED if how == "cancel" else es.FASTLEC_TIMEOUT), e
    assert e.result["patterns_evaluated"] == 0 and e.result["next_word"] == 0, e.result
""" % how)
    assert "inner inputs" not in r.stderr, r.stderr[-2000:]


def test_no_thread_to_be_had(lib, tmp_path):
    """A process at its limit of threads: checks go on without a kernel built beside them, batches plan and
    build on the calling thread."""
    pre = tmp_path / "no_threads.so"
    subprocess.run(["g++", "-shared", "-fPIC", os.path.join(standin.SAN, "no_threads.cpp"), "-o", str(pre), "-ldl"],
                   check=True)
    run(lib, """
import ctypes
es.lib()
cs = [load(miters.layered_cone_miter(40 + i, 12, 1500, fault_seed=i or None)) for i in range(3)]
want = [es.fastlec_es_check(c, kernel="interp") for c in cs]
fresh = [load(miters.layered_cone_miter(40 + i, 12, 1500, fault_seed=i or None)) for i in range(3)]
ctypes.CDLL(None).refuse_threads(1)
same = lambda r, w: (r["verdict"], r["cex"]) == (w["verdict"], w["cex"])
for i in range(150):  # more than a kernel's building on the interpreter
    assert same(es.fastlec_es_check(cs[0]), want[0])
for kernel in ("auto", "interp", "specialized"):
    assert all(map(same, es.fastlec_es_check_batch(fresh, kernel=kernel), want)), kernel
""", LD_PRELOAD=str(pre))


@pytest.mark.parametrize("call", ["auto", "specialized", "batch", "batch_specialized"])
def test_a_kernel_made_for_a_few_words_does_not_stay(lib, call):
    """A 14x14 multiplier miter (with the first pattern failing, so that a check is quick) checked over two words
    first, on a kernel without inner inputs; checks of its whole space have their own kernel built, once, when by
    the model they have paid for it."""
    r = run(lib, """
call = %r
g = miters.Aig(28)
for o in miters.import_into(g, miters.mult_miter(14, "booth")):
    g.add_output(o)
g.add_output(g.input(0) ^ 1)
c = load(g)
kernel = "specialized" if "specialized" in call else "auto"
for _ in range(3):
    es.fastlec_es_check(c, kernel="specialized", end_word=2)
print("whole", file=sys.stderr, flush=True)
for _ in range(300):
    if "batch" in call:
        r = es.fastlec_es_check_batch([c], kernel=kernel)[0]
    else:
        r = es.fastlec_es_check(c, kernel=kernel)
    assert r["verdict"] == 1 and r["cex"] == 0, r
""" % call)
    before, after = r.stderr.split("whole")
    made = [ln.split("native: ")[1] for ln in after.splitlines() if "inner inputs" in ln]
    assert "native: 0 inner inputs" in before, before[-2000:]
    assert len(made) == 1, (made, after[-2000:])


def test_simulations_do_not_wait_for_a_check_s_kernel(lib):
    """A thread simulates a circuit while another one builds its native kernel (0.2 s and more); the stand-in
    has no simulation, so that every call ends at its launch, but none comes late."""
    run(lib, """
import ctypes, threading
c = load(chain(60000, 32))
sig = ctypes.addressof(ctypes.create_string_buffer(64))
def simulate():
    t = time.perf_counter()
    try:
        es.fastlec_es_simulate(c, sig, 64, sig)
        assert False
    except es.EsError:
        return time.perf_counter() - t
simulate()  # plans
t = threading.Thread(target=lambda: es.fastlec_es_native_info(c))
start = time.perf_counter()
t.start()
late = []
while t.is_alive():
    late.append(simulate())
    time.sleep(0.001)
build = time.perf_counter() - start
assert len(late) > 20 and max(late) < 0.4 * build, (build, len(late), max(late))
""")


def test_server_jobs_without_native_kernel_are_interpreted(lib):
    """Jobs of a cone for which no native kernel fits: eight at a time are by the model worth a native kernel (its
    first pattern fails, which the model does not know) and not a hipRTC compile, so none is compiled and all
    run on the interpreter."""
    r = run(lib, """
g = miters.Aig(24)
for o in miters.import_into(g, miters.layered_cone_miter(3, 24, 60000)):
    g.add_output(o)
g.add_output(g.input(0) ^ 1)
cs = [load(g) for _ in range(8)]
srv = es.Server(1 << 36)
res = [srv.poll(t, wait=True) for t in [srv.submit(c) for c in cs]]
assert all((x["verdict"], x["cex"]) == (1, 0) for x in res), res
st = srv.stats()
print(st)
assert st["specialized_slices"] == 0 and st["completed"] == 8, st
srv.close()
""")
    assert "native: no kernel" in r.stderr, r.stderr[-2000:]


def test_server_waits_for_a_kernel_without_spinning(lib):
    """One job waits for its kernel (0.2 s of building) while another finds no room in the budget: the server's
    loop sleeps, and the process takes the time of one thread that builds."""
    run(lib, """
def first_fails(seed):
    g = miters.Aig(32)
    for o in miters.import_into(g, chain(60000 + seed, 32)):
        g.add_output(o)
    g.add_output(g.input(0) ^ 1)
    return load(g)
a, b = first_fails(0), first_fails(1)
charge = first_fails(0).info()["peak_live_slots"] * (1 << 22) * 8  # info() plans the interpreter's stream
srv = es.Server(charge + charge // 2)
cpu, wall = time.process_time(), time.perf_counter()
t = [srv.submit(a), srv.submit(b)]
assert srv.poll(t[0], wait=True)["cex"] == 0
cpu, wall = time.process_time() - cpu, time.perf_counter() - wall
print(cpu, wall)
assert srv.poll(t[1], wait=True)["cex"] == 0
assert srv.stats()["max_active"] == 1
assert cpu < 1.4 * wall + 0.02, (cpu, wall)
srv.close()
""")


def test_server_counts_what_a_job_took(lib):
    """Jobs of many small steps: what counts towards a native kernel is what the steps took, not all that is left
    at each of them.  A job that is by the model some ten times too short for a kernel gets none, however
    many steps it is cut into."""
    r = run(lib, """
c = load(miters.layered_cone_miter(7, 24, 300))
p = es.fastlec_es_predict(c)
srv = es.Server(1 << 34)
for _ in range(2):
    x = srv.poll(srv.submit(c), wait=True)
    assert x["verdict"] == 0 and x["patterns_evaluated"] == 1 << 24, x
print(p, srv.stats())
assert srv.stats()["steps"] >= 500, srv.stats()
srv.close()
""", FASTLEC_ES_SERVER_RATE="1000000000", FASTLEC_ES_SERVER_STEP_MS="1", FASTLEC_STANDIN_SLOW_CLOCK="10000")
    assert "native: " not in r.stderr, r.stdout + r.stderr[-2000:]


def test_a_failing_batch_waits_for_its_launches(lib):
    """A batch's second launch (its finish kernel) is refused while the first one runs: what they read on the device goes back to
    the pool only when nothing runs any more, and the same batch works again."""
    r = run(lib, """
cs = [load(miters.layered_cone_miter(50 + i, 12, 300, fault_seed=2)) for i in range(2)]
cs += [load(miters.layered_cone_miter(60 + i, 12, 12000, fault_seed=2)) for i in range(2)]
try:
    es.fastlec_es_check_batch(cs, kernel="interp")
    assert False
except es.EsError as e:
    print("failed", file=sys.stderr, flush=True)
want = [es.fastlec_es_check(c, kernel="interp") for c in cs]
got = es.fastlec_es_check_batch(cs, kernel="interp")
assert [(x["verdict"], x["cex"]) for x in got] == [(x["verdict"], x["cex"]) for x in want]
""", FASTLEC_STANDIN_FAIL_LAUNCH="2", FASTLEC_STANDIN_LAUNCH_US="50000", FASTLEC_STANDIN_TRACE="1")
    during = r.stderr.split("failed")[0]
    assert "launch refused" in during and "synchronize" in during.split("launch refused")[1], during[-1500:]


def test_threads_with_one_batch_when_a_call_fails(lib):
    """Two threads run the same batch and meet on what is kept for it; the first one's finish kernel is refused.  The
    other one does not use the claim counters that it left."""
    r = run(lib, """
import threading
cs = [load(miters.layered_cone_miter(50 + i, 12, 300, fault_seed=2)) for i in range(2)]
cs += [load(miters.layered_cone_miter(60 + i, 12, 12000, fault_seed=2)) for i in range(2)]
want = [(x["verdict"], x["cex"]) for x in es.fastlec_es_check_batch(cs, kernel="interp")]  # launches 1 and 2
errors, good = [], []
def call():
    try:
        good.append([(x["verdict"], x["cex"]) for x in es.fastlec_es_check_batch(cs, kernel="interp")])
    except es.EsError as e:
        errors.append(e)
threads = [threading.Thread(target=call) for _ in range(2)]
[t.start() for t in threads]
[t.join() for t in threads]
assert len(errors) == 1 and good == [want], (errors, good)
""", FASTLEC_STANDIN_FAIL_LAUNCH="4", FASTLEC_STANDIN_LAUNCH_US="50000", FASTLEC_STANDIN_TRACE="1")
    assert "launch refused" in r.stderr and "not zero" not in r.stderr, r.stderr[-2000:]


def test_server_budget_just_above_the_job_table(lib):
    """The table is 551 pages of device memory; every budget above that is accepted, and jobs run in it."""
    run(lib, """
table = 551 * 4096
try:
    es.Server(table)
    assert False
except es.EsError as e:
    assert e.code == es.FASTLEC_ERR_INVALID
srv = es.Server(table + 1)
cs = [load(miters.layered_cone_miter(70 + i, 12, 300, fault_seed=i or None)) for i in range(4)]
want = [es.fastlec_es_check(c, kernel="interp") for c in cs]
got = [srv.poll(t, wait=True) for t in [srv.submit(c) for c in cs]]
assert [(x["verdict"], x["cex"]) for x in got] == [(x["verdict"], x["cex"]) for x in want]
assert srv.stats()["device_bytes"] == table
srv.close()
""")


def test_calls_wait_on_their_own_stream(lib):
    """Checks, batches and explicit kernels on a stream of the caller wait for no other one (the library's may be
    busy with another thread's check), from the first call on."""
    r = run(lib, """
c = load(miters.layered_cone_miter(80, 12, 300, fault_seed=1))
want = None
for kernel in ("interp", "specialized", "auto"):
    x = es.fastlec_es_check(c, kernel=kernel, stream=0x7000)
    y = es.fastlec_es_check_batch([c, c], kernel=kernel, stream=0x7000)
    want = want or (x["verdict"], x["cex"])
    assert all((z["verdict"], z["cex"]) == want for z in [x] + y)
""", FASTLEC_STANDIN_TRACE="1")
    waits = [ln.split()[-1] for ln in r.stderr.splitlines() if ln.startswith("standin: synchronize")]
    assert waits and set(waits) == {"0x7000"}, waits
