"""What libnf's host code asks of the HIP runtime, call by call, against a stub
runtime on the CPU (tests/hip_stub.cpp) in a child process: no GPU is used."""

import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1307_7820_amd", "libnf.so")

HEAD = """
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # found before the real runtime
L = ctypes.CDLL(sys.argv[2])
vp, c_int, c_sz = ctypes.c_void_p, ctypes.c_int, ctypes.c_size_t
stub.stub_log.restype = stub.stub_grids.restype = ctypes.c_char_p
stub.stub_capture.argtypes = [vp]
L.nf_last_error.restype = ctypes.c_char_p
L.nf_fold_dev.argtypes = [vp, c_int, c_int, vp, vp, vp]
L.nf_submit.argtypes = [ctypes.c_char_p, c_int, c_int, c_int]
L.nf_submit.restype = ctypes.c_int64
L.nf_wait.argtypes = [ctypes.c_int64, c_int, vp, vp]
L.nf_batch_create.argtypes = [vp, vp, c_int, c_int, vp]
L.nf_batch_run.argtypes = [vp, vp]
L.nf_batch_scores.argtypes = [vp, vp]
L.nf_batch_destroy.argtypes = [vp]
L.nf_batch_destroy.restype = None
L.nf_fold_batch.argtypes = [vp, vp, c_int, c_int, vp, vp]
mem = ctypes.create_string_buffer(1 << 16)
score = c_int(0)
STREAM = 0x1230

def log():
    out = stub.stub_log().decode().split("\\n")[:-1]
    stub.stub_clear()
    return out

def fold(n, stream=STREAM):
    return L.nf_fold_dev(mem, n, 8, ctypes.byref(score), None, stream)

def batch(ns, q=8):
    seqs = (ctypes.c_char_p * len(ns))(*[b"ACGU" * (n // 4) + b"A" * (n % 4) for n in ns])
    h = vp()
    assert L.nf_batch_create(seqs, (c_int * len(ns))(*ns), len(ns), q, ctypes.byref(h)) == 0, L.nf_last_error()
    return h
"""


@pytest.fixture(scope="module")
def child(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "libhipstub.so")
    subprocess.check_call(["g++", "-O1", "-shared", "-fPIC", "-std=c++17", "-D__HIP_PLATFORM_AMD__",
                           "-I/opt/rocm/include", os.path.join(ROOT, "tests", "hip_stub.cpp"), "-o", so])

    def run(body, **env):
        keep = {k: v for k, v in os.environ.items() if not k.startswith("NF_")}
        subprocess.run([sys.executable, "-c", HEAD + textwrap.dedent(body), so, LIB], check=True, timeout=120,
                       env=dict(keep, **env))
    return run


def test_a_stream_under_capture_is_refused_at_every_length(child):
    """Before anything is enqueued or allocated, with a workspace at hand or
    without; the streams beside it and the calls after it are served."""
    child("""
    for warm in (0, 1):
        for n in (60, 500, 2000):
            stub.stub_capture(STREAM)
            log()
            assert fold(n) == -1, (n, warm)
            assert b"nf_fold_dev_noalloc" in L.nf_last_error()
            work = [x for x in log() if x != "stream synchronize"]
            assert work == [], (n, warm, work)
            assert fold(n, STREAM + 16) == 0
            stub.stub_capture(None)
            log()
            assert fold(n) == 0 and ("kernel" in log())
    b = batch([60, 500])
    stub.stub_capture(STREAM)
    log()
    assert L.nf_batch_run(b, STREAM) == -1 and log() == []
    stub.stub_capture(None)
    assert L.nf_batch_run(b, STREAM) == 0
    L.nf_batch_destroy(b)
    """)


def test_a_graph_is_destroyed_only_when_the_device_is_idle(child):
    """Between the last launch and the end of a graph lies a wait for the device:
    a workspace dropped from the cache behind a fold that nothing waited for, a
    batch destroyed after its run, the one-shot batch call."""
    child("""
    def ordered(calls):
        busy, destroyed = False, 0
        for c in calls:
            if c in ("graph launch", "kernel"):
                busy = True
            elif c == "device synchronize":
                busy = False
            elif c in ("exec destroy", "graph destroy"):
                destroyed += 1
                assert not busy, calls
        return destroyed
    for n in (2000, 1900, 2100):
        assert fold(n) == 0
    assert ordered(log()) >= 4
    for ns in ([60], [500, 700], [900] * 40, [1500] * 40):
        b = batch(ns)
        assert L.nf_batch_run(b, STREAM) == 0
        L.nf_batch_destroy(b)
        assert ordered(log()) == 2
        seqs = (ctypes.c_char_p * len(ns))(*[b"A" * n for n in ns])
        assert L.nf_fold_batch(seqs, (c_int * len(ns))(*ns), len(ns), 8, (c_int * len(ns))(), None) == 0
        assert ordered(log()) == 2
    """, NF_PLAN_CACHE_BYTES="1")


@pytest.mark.parametrize("q,least", [(8, 6), (4, 4)])
def test_served_steps_are_cut_like_batches(child, q, least):
    """A chunk of a served step spans at least as many group tiles as one of a
    batch's step: the workgroups of every step of one served fold."""
    child("""
    n, q, least = 2000, %d, %d
    L.nf_serve_config.argtypes = [c_sz, c_int, c_int]
    assert L.nf_serve_config(1 << 28, 0, 0) == 0
    t = L.nf_submit(b"ACGU" * 500, n, q, 0)
    assert t > 0, L.nf_last_error()
    assert L.nf_wait(t, 20000, None, None) == 1
    L.nf_shutdown()
    grids = [int(x) for x in stub.stub_grids().split()]
    NT = (n + 64) // 64
    want = []
    for s in range(1, NT):
        dd, chunks = s + 1, 0
        if 4 <= dd < NT:
            chunk = max(least, -(-(NT - dd) * (dd - 3) // 1024))
            chunks = (NT - dd) * -(-(dd - 3) // chunk)
        want.append(NT - s + chunks)
    assert grids[-NT - 1:] == [NT] + want + [1], (grids, want)
    """ % (q, least))
