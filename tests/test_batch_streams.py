"""How a batch's chains of launches are ordered, on the CPU against a HIP runtime that logs the calls: no run waits
for another caller's, and no chain that was launched is left behind when a later call of the same run fails."""
import ctypes
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)   # before the library, so that it binds to these
stub.stub_log.restype = ctypes.c_char_p
import paper_2103_11847_amd as dk
L = dk.lib()
P = ctypes.c_void_p

def ok(r):
    assert r == 0, r

def log():
    out = [l.split() for l in stub.stub_log().decode().splitlines()]
    stub.stub_clear()
    return [(n, int(a, 16), int(b, 16), bad == "1") for n, a, b, bad in out]

def context(stream):
    c = P()
    ok(L.dctk_create(ctypes.byref(c), 0, stream))
    return c

class Plan:
    def __init__(self, ctx, ps=(3, 8, 31), n=4):
        self.ctx, self.h, self.ops, self.ws = ctx, P(), [], []
        self.bufs = [(ctypes.c_double * (p * n * n))(*([1.0] * (p * n * n))) for p in ps]
        for p, A in zip(ps, self.bufs):
            op, ws = P(), P()
            ok(L.dctk_op_create(ctx, 0, dk.DCTK_F32, p, n, n, ctypes.cast(A, P), n, None, ctypes.byref(op)))
            ok(L.dctk_krylov_create(ctx, op, 0, 4, 0, ctypes.byref(ws)))
            self.ops.append(op)
            self.ws.append(ws)
        arr = lambda v: (P * len(v))(*v)
        data = [ctypes.cast(b, P) for b in self.bufs]
        self.opts = dk.make_opts(4)
        ok(L.dctk_batch_create(ctx, len(ps), arr(self.ws), arr(data), arr(data), ctypes.byref(self.opts), None, 1.0, 1,
                               ctypes.byref(self.h)))

    def run(self):
        log()
        r = L.dctk_batch_run(self.ctx, self.h)
        return r, log()

    def close(self):
        ok(L.dctk_batch_destroy(self.h))
        for w in self.ws:
            ok(L.dctk_krylov_destroy(w))
        for o in self.ops:
            ok(L.dctk_op_destroy(o))

def launched(calls):
    return [s for n, s, _, bad in calls if n == "launch" and not bad]
"""

STREAMS = CHILD + r"""
a, b = context(0x100), context(0x200)
plans = [Plan(a), Plan(b), Plan(a)]

def run(i):
    r, calls = plans[i].run()
    ok(r)
    s = launched(calls)
    assert len(s) == 3
    # only streams and events of this run are waited for
    recorded = {e for n, _, e, _ in calls if n == "record"}
    assert all(e in recorded for n, _, e, _ in calls if n == "wait")
    return s, (0x100, 0x200, 0x100)[i]

def apart(i):
    s, own = run(i)
    assert len(set(s)) == 3 and s.count(own) == 1, s
    return set(s) - {own}

def alone(i):
    s, own = run(i)
    assert set(s) == {own}, s

first = apart(0)
stub.stub_ready(0)
assert apart(2) == first == apart(0)   # the same stream orders its runs itself
alone(1)                               # another one waits for none of them
stub.stub_ready(1)
assert apart(1) == first
stub.stub_ready(0)
alone(0)
L.dctk_set_stream(a, 0x200)
plans[0].run()
assert launched(plans[0].run()[1]).count(0x200) == 1
log()
for p in plans:
    p.close()
gone = [s for n, s, _, _ in log() if n == "destroy"]
assert all(gone.count(s) == 1 for s in first), gone
p = Plan(b)                            # a plan after the last one has streams again
plans[1] = p
apart(1)
p.close()
print("done")
"""

JOIN = CHILD + r"""
name, nth = sys.argv[2], int(sys.argv[3])
c = context(0x100)
p = Plan(c)
stub.stub_fail(name.encode(), nth)
r, calls = p.run()
assert r == dk.DCTK_EHIP, r
assert sum(bad for _, _, _, bad in calls) == 1
for i, (n, s, _, bad) in enumerate(calls):
    if n != "launch" or bad or s == 0x100:
        continue
    rest = calls[i + 1:]
    synced = any(m == "sync" and t == s for m, t, _, _ in rest)
    joined = any(m == "record" and t == s and not b2 and
                 any(m2 == "wait" and t2 == 0x100 and e2 == e and not b3 for m2, t2, e2, b3 in rest[k + 1:])
                 for k, (m, t, e, b2) in enumerate(rest))
    assert synced or joined, (hex(s), calls)
stub.stub_fail(b"", 0)
r, calls = p.run()          # the plan is whole
ok(r)
assert len(launched(calls)) == 3
p.close()
print("done")
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    out = str(tmp_path_factory.mktemp("stub") / "libstubhip.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", out, os.path.join(ROOT, "tests", "stub_hip.cpp")], check=True)
    return out


def child(code, *args):
    r = subprocess.run([sys.executable, "-c", code, *args], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("done"), r.stdout + r.stderr


def test_no_run_waits_for_another_stream(stub):
    child(STREAMS, stub)


@pytest.mark.parametrize("name,nth", [("launch", i) for i in (1, 2, 3)] + [("record", i) for i in (1, 2, 3)] +
                         [("wait", i) for i in (1, 2, 3, 4)])
def test_failed_run_joins_its_chains(stub, name, nth):
    child(JOIN, stub, name, str(nth))
