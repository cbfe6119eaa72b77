"""What the library's host code asks of the HIP runtime, recorded by a stand-in for the
runtime (hip_stub.c): no GPU, nothing is computed.  Each case runs in a process of its
own, where the stand-in's symbols come before the runtime's."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(ROOT, "paper_2409_07222_amd", "liblabs.so")

pytestmark = [pytest.mark.skipif(not os.path.exists(LIB), reason="library not built"),
              pytest.mark.skipif(shutil.which("gcc") is None, reason="no C compiler")]

PRELUDE = """
import ctypes, os, sys
sys.path.insert(0, %(root)r)
S = ctypes.CDLL(%(stub)r, mode=ctypes.RTLD_GLOBAL)
from paper_2409_07222_amd import labs
H = labs.lib()
class Launch(ctypes.Structure):
    _fields_ = [("name", ctypes.c_char_p), ("grid", ctypes.c_uint32), ("block", ctypes.c_uint32),
                ("shmem", ctypes.c_size_t)]
class Attr(ctypes.Structure):
    _fields_ = [("name", ctypes.c_char_p), ("attr", ctypes.c_int), ("value", ctypes.c_int)]
def launches():
    n = ctypes.c_int.in_dll(S, "stub_n_launches").value
    return list((Launch * 65536).in_dll(S, "stub_launches"))[:n]
def attrs():
    n = ctypes.c_int.in_dll(S, "stub_n_attrs").value
    return list((Attr * 65536).in_dll(S, "stub_attrs"))[:n]
P = 1 << 20       # an aligned address that nothing reads
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    stub = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", stub, os.path.join(HERE, "hip_stub.c")], check=True)

    def go(body):
        r = subprocess.run([sys.executable, "-c", PRELUDE % {"root": ROOT, "stub": stub} + body],
                           capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr
    return go


def test_lds_limits_do_not_depend_on_the_call(run):
    """A kernel's limit of dynamic LDS belongs to the process: if every call set it to its
    own network's need, a thread with a small network could lower it between another
    thread's call and launch.  Every call sets the same value, which no launch exceeds."""
    run("""
for L, hidden in ((1023, 256), (21, 64), (501, 256)):
    lay = labs.mlp_layout(L, hidden)
    r = ctypes.byref(lay)
    assert H.labs_mlp_train_step(r, P, P, P, P, P, 1, 1e-3, .9, .999, 1e-8, 100, P, P, P, P, P, 1 << 40, None) == 0
    assert H.labs_mlp_grads(r, P, P, 100, P, P, P, P, P, P, 1 << 40, None) == 0
    for n in (1, 5000, 20000):
        assert H.labs_mlp_forward(r, P, P, n, P, P, P, 1 << 40, None) == 0
limit = {}
for a in attrs():
    limit.setdefault(a.name, set()).add(a.value)
assert len(limit) >= 4, limit       # two training kernels, the forward's row tiles
assert all(len(v) == 1 for v in limit.values()), limit
for l in launches():
    if l.shmem > 64 * 1024:
        assert l.shmem <= min(limit[l.name])
""")


@pytest.mark.parametrize("L", [101, 301, 501, 639])
def test_autotuner_times_the_untuned_residency(run, L):
    """The tuner replaces the residency that an untuned launch asks for, so it has to have
    timed it: where that one is the fastest, tuning keeps it."""
    run("""
L, p, walkers = %d, 16, 20000
untuned = labs.autotune_get(L, p)
F = ctypes.CFUNCTYPE(ctypes.c_float, ctypes.c_uint32)
elapsed = F(lambda grid: 1.0 + abs(int(grid) - 4 * 256 * untuned[1]))     # 256 CUs, 4 SIMDs each
ctypes.c_void_p.in_dll(S, "elapsed_of_grid").value = ctypes.cast(elapsed, ctypes.c_void_p).value
ctypes.c_char_p.in_dll(S, "timed_kernel").value = b"k_walk_persistent"
assert H.labs_autotune_step1((ctypes.c_int32 * 1)(L), 1, p, walkers, 10, None) == 0
assert sum(b"k_walk_persistent" in l.name for l in launches()) >= 10
assert labs.autotune_get(L, p) == untuned
""" % L)


def test_network_workspaces_are_16_byte_aligned(run):
    """The network's kernels read and write their workspace 16 bytes at a time: one that
    is not aligned for that is refused before any launch, at every width.  Calls that run
    no network take any."""
    run("""
for hidden in (64, 256, 320):
    lay = labs.mlp_layout(101, hidden)
    r = ctypes.byref(lay)
    for off in (1, 4, 8):
        W = P + off
        assert H.labs_mlp_forward(r, P, P, 100, P, P, W, 1 << 40, None) == -1
        assert b"16-byte" in H.labs_last_error()
        assert H.labs_mlp_grads(r, P, P, 100, P, P, P, P, P, W, 1 << 40, None) == -1
        assert H.labs_mlp_train_step(r, P, P, P, P, P, 1, 1e-3, .9, .999, 1e-8, 100, P, P, P, P, W, 1 << 40, None) == -1
    assert not launches()

def walk(mode, every, steps, ws, hidden):
    cfg = labs.Step1Cfg(101, 8, steps, 10, 20, -1, 0, 100, 1, 0, 0)
    pr = labs.Proposer(mode, 8, every, hidden, P, P, 0, 0, 0)
    out = labs.LearnedOut()
    out.flip_evals = P
    return H.labs_learned_walk(ctypes.byref(cfg), ctypes.byref(pr), ctypes.byref(out), ws, 1 << 40, None)

for hidden in (64, 320):
    assert walk(labs.PROPOSE_MLP, 4, 10, P + 8, hidden) == -1 and b"16-byte" in H.labs_last_error()
    assert not launches()
    assert walk(labs.PROPOSE_MLP, 4, 10, P + 16, hidden) == 0
    assert walk(labs.PROPOSE_MLP, 1, 10, P + 8, hidden) == 0
    assert walk(labs.PROPOSE_MLP, 4, 1, P + 8, hidden) == 0
    assert walk(labs.PROPOSE_RANDOM, 4, 10, P + 8, hidden) == 0
    ctypes.c_int.in_dll(S, "stub_n_launches").value = 0
lay = labs.mlp_layout(101, 64)
assert H.labs_mlp_grads(ctypes.byref(lay), P, P, 0, None, None, None, P, P, P + 4, 1 << 40, None) == 0
assert H.labs_mlp_forward(ctypes.byref(lay), P, P, 0, P, P, P + 4, 1 << 40, None) == 0
""")
