"""The runtime calls that the host side makes, without a GPU: libexageo.so on a
stand-in for the HIP runtime (fakehip.c) that runs no kernel and writes every
call to a file.  In a process of its own, so that nothing else binds to it."""
import os
import re
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_1908_06936_amd", "libexageo.so")

CHILD = """
import ctypes, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
i64, d = ctypes.c_int64, ctypes.c_double
mark = lambda s: fake.fakehip_mark(s.encode())
theta = (d * 3)(1.0, 0.1, 0.5)
ll, grad, info, ctx = d(), (d * 3)(), i64(), ctypes.c_void_p()

def create(ts):
    mark("create")
    assert lib.exageo_create(ctypes.byref(ctx), 0, i64(ts), None) == 0

def field(n):
    return [i64(n)] + [(d * n)() for _ in range(3)]
"""


@pytest.fixture(scope="module")
def calls(tmp_path_factory):
    if not os.path.exists(LIB):
        pytest.skip("libexageo.so not built")
    tmp = tmp_path_factory.mktemp("fakehip")
    so = str(tmp / "fakehip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-Wall", os.path.join(HERE, "fakehip.c"), "-o", so], check=True)

    def run(script):
        log = str(tmp / "log.txt")
        r = subprocess.run([sys.executable, "-c", CHILD + script, so, LIB], capture_output=True, text=True, timeout=120,
                           env=dict(os.environ, FAKEHIP_LOG=log))
        assert r.returncode == 0, r.stderr
        return open(log).read().splitlines()

    return run


# the allocation-free entry point, one tile and several, on a context that has
# made no other call: no memory, stream or event is made or freed inside it
@pytest.mark.parametrize("n", [200, 1100])
@pytest.mark.parametrize("grad", ["grad", "None"])
def test_noalloc_call_makes_nothing(calls, n, grad):
    log = calls(f"""
create(256)
mark("call")
assert lib.exageo_loglik_grad_noalloc(ctx, *field({n}), theta, ctypes.byref(ll), {grad}, ctypes.byref(info)) == 0
""")
    inside = log[log.index("call"):]
    assert any("k_potrf_blk" in c for c in inside) and inside[-1] == "hipStreamSynchronize"
    made = [c for c in inside if c.startswith("hip") and any(w in c for w in ("Malloc", "Free", "Create", "Destroy"))]
    assert made == []


# the phases of exageo_get_timings: five tiles, so four are solved before the
# event that ends the Cholesky phase and one after it; bench.py takes no rate
# from the phase of the last one
def test_forward_solve_in_the_phases(calls):
    log = calls("""
create(256)
assert lib.exageo_set_profiling(ctx, 1) == 0
mark("call")
assert lib.exageo_loglik_grad(ctx, *field(1100), theta, 0, ctypes.byref(ll), grad, ctypes.byref(info)) == 0
""")
    ev = [c.split()[1] for c in log if c.startswith("hipEventCreate ")]
    rec = [next(i for i, c in enumerate(log) if c.startswith(f"hipEventRecord {e} ")) for e in ev[:6]]
    assert rec == sorted(rec) and rec[0] > log.index("call")

    def launched(name, phase):  # between the events that bound it
        return sum(name in c for c in log[rec[phase - 1]:rec[phase]])

    assert [launched("k_potrf_blk", p) for p in range(1, 6)] == [0, 0, 9, 0, 0]
    assert [launched("k_tile_fwd", p) for p in range(1, 6)] == [0, 0, 4, 1, 0]
    assert launched("k_copy_diag_lower", 5) == 1  # FP64: the diagonal tiles' inverses
    root = os.path.dirname(HERE)
    header = " ".join(open(os.path.join(root, "include", "exageo.h")).read().replace("*", " ").split())
    assert "forward solve of every tile but the last" in header and "forward solve of the last tile" in header
    rates = re.findall(r'/ *\(avg\("(\w+)"\)', open(os.path.join(root, "bench.py")).read())
    assert "gen_ms" in rates and "solve_ms" not in rates
