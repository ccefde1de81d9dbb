"""The host threads of what the library ships under ThreadSanitizer, on the CPU: native kernels and the
threads that build them, kept batches, control slots, the polling wait and the finish kernel.

tests/test_server_race_cpu.py builds the host sources without the native tier; these programs hold it
(tests/standin.py).  A native launch executes the generated machine code, launches run on a thread of
their own, and every answer must be the one a circuit gave alone.  Any sanitizer report fails the test.
"""
import os
import subprocess

import pytest

import miters

import standin


@pytest.fixture(scope="module")
def drivers(tmp_path_factory):
    if not os.path.exists(standin.CLANG):
        pytest.skip("clang++ not found")
    return standin.build(tmp_path_factory.mktemp("native_race"), "thread",
                         ("native_race_driver.cpp", "server_race_driver.cpp"), "-O1")


def write(d, specs):
    files = []
    for k, (seed, n, gates, fault) in enumerate(specs):
        p = d / f"c{k}.aig"
        p.write_bytes(miters.layered_cone_miter(seed, n, gates, fault_seed=fault).to_aig())
        files.append(str(p))
    return files


def run(exe, files, **env):
    env = dict(os.environ, FASTLEC_ES_TRACE="1", TSAN_OPTIONS="halt_on_error=1 exitcode=66", **env)
    r = subprocess.run([exe] + files, capture_output=True, text=True, timeout=600, env=env)
    assert "ThreadSanitizer" not in r.stderr, r.stderr[-8000:]
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-8000:])
    return r


def test_checks_and_batches_have_no_data_races(drivers, tmp_path):
    files = write(tmp_path, [(8101, 12, 1500, None), (8102, 13, 800, 2), (8103, 14, 600, None), (8104, 12, 2500, 4)])
    r = run(drivers[0], files)
    assert r.stdout.strip().endswith("4 native kernels\nok"), r.stdout
    assert "native: " in r.stderr, r.stderr[-3000:]  # kernels were built while checks ran


@pytest.mark.parametrize("jit", ["1", "2"])
def test_server_has_no_data_races(drivers, tmp_path, jit):
    files = write(tmp_path, [(8001, 12, 400, 1), (8002, 14, 600, None), (8003, 13, 500, 2), (8004, 14, 400, None),
                             (8005, 18, 300, 3), (8006, 18, 350, None), (8007, 20, 300, None), (8008, 20, 250, 4)])
    r = run(drivers[1], files, FASTLEC_ES_SERVER_JIT=jit, FASTLEC_ES_SERVER_RATE="1000000000",
            FASTLEC_ES_SERVER_STEP_MS="1")
    assert r.stdout.strip().endswith("ok 96"), r.stdout
    line = [ln for ln in r.stdout.splitlines() if ln.startswith("server:")][0]
    assert " 0 mismatches, 0 errors" in line, line
    assert " 0 specialized slices" not in line, line
