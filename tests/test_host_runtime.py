"""The library's host code over a HIP runtime whose kernels do nothing and whose streams the test stops (fake_hip.c), each
case in a process of its own: what the server does between submit and completion."""
import ctypes
import os
import subprocess
import sys
import tempfile
import threading
import time
import traceback

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "fake_hip.c"), "-lpthread"], check=True)
    return so


def _run(fake, name):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), fake, name], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


# ------------------------------------------------------------------------ in the child process


def _plan(B, n_cheb=32, precisions=("fp32",), n_chi=6, n_R=5, n_ell=4):
    chi, w = B.grid_chi_simpson(n_chi, 100.0, 2000.0)
    R, wR = B.grid_R_fejer(n_R, 0.3)
    return B.Plan(np.arange(2, 2 + n_ell), chi, w, R, wR, 1e-4, 1.0, n_cheb, precisions=precisions)


class _Server:
    """A server whose first request runs for as long as time stands still, and more requests of its shape."""

    def __init__(self, B, F, max_wait_ms=1e6):
        self.B, self.F, self.plan = B, F, _plan(B)
        self.srv = B.Server(self.plan, batch=64, n_sets=2, max_g=2, max_s=1, max_wait_ms=max_wait_ms)
        F.fake_hold(1)
        self.submit(False)
        self.until(lambda: self.srv.stats()["in_flight"] == 1)

    def submit(self, pin):
        P, K, K2 = np.ones((6, 5, 32), np.float32), np.ones((3, 6)), np.ones((3, 6, 5))
        if pin:
            self.F.fake_pin(P.ctypes.data, P.nbytes)
        return self.srv.submit(P, K, K2, 2, 1, [0, 1, 2, 3]), P

    def pending(self, P):
        return self.F.fake_pending(P.ctypes.data, P.nbytes)

    def until(self, f):
        t = time.time()
        while not f():
            assert time.time() - t < 10
            time.sleep(1e-3)

    def done(self):
        self.F.fake_hold(0)
        self.srv.close()
        self.plan.close()


def pageable_requests_are_asked_once(B, F):
    s = _Server(B, F)
    n0 = F.fake_attr_calls()
    for _ in range(20):
        s.submit(False)
    time.sleep(0.3)  # the scheduler takes a turn every 50 us
    assert s.srv.stats()["queued"] == 0
    assert F.fake_attr_calls() - n0 <= 20, F.fake_attr_calls() - n0
    s.done()


def _in_thread(f):
    t = threading.Thread(target=f, daemon=True)
    t.start()
    return t


def cancelling_waits_for_its_own_copy_only(B, F):
    s = _Server(B, F)
    (ta, a), (tb, _), (tc, c), (td, d) = s.submit(True), s.submit(False), s.submit(True), s.submit(True)
    s.until(lambda: s.pending(a) and s.pending(c) and s.pending(d))
    t = _in_thread(lambda: s.srv.cancel(tb))  # nothing of it is on the way
    t.join(5)
    assert not t.is_alive()
    s.until(lambda: s.pending(c) == 2 and s.pending(d) == 2)  # moved up and sent again
    left = []

    def cancel(ticket, P):
        s.srv.cancel(ticket)
        left.append(s.pending(P))

    ts = [_in_thread(lambda: cancel(ta, a)), _in_thread(lambda: cancel(tc, c))]
    time.sleep(0.1)
    assert all(t.is_alive() for t in ts)
    t = _in_thread(s.srv.stats)  # others are not kept waiting
    t.join(5)
    assert not t.is_alive()
    F.fake_hold(0)
    for t in ts:
        t.join(5)
    assert left == [0, 0]
    for ticket in (ta, tb, tc):
        try:
            s.srv.wait(ticket, 5000)
            assert False
        except B.BlastError as e:
            assert e.status == B.E_CANCELLED
    s.srv.wait(td, 5000)
    assert s.srv.stats()["cancelled"] == 3
    s.done()


def a_failed_launch_ends_after_its_copies(B, F):
    s = _Server(B, F, max_wait_ms=300.0)
    F.fake_fail_graph(1)
    (ta, a), (tb, b) = s.submit(True), s.submit(False)
    st = []

    def wait(t):
        try:
            s.srv.wait(t)
        except B.BlastError as e:
            st.append((e.status, s.pending(a), s.pending(b)))

    ts = [_in_thread(lambda: wait(ta)), _in_thread(lambda: wait(tb))]
    s.until(lambda: s.pending(a) and s.pending(b))  # b with the launch, after 300 ms
    time.sleep(0.2)
    F.fake_hold(0)
    for t in ts:
        t.join(5)
    assert st == [(B.E_HIP, 0, 0)] * 2, st
    s.done()


def the_optional_nodal_copy_comes_last(B, F):
    """The FP64 nodal basis of an even n_cheb that is no multiple of 32: only for plans asked for FP64, and only out
    of memory that nothing else of the plan needs and that leaves as much again."""
    size = dict(n_chi=256, n_R=96, n_ell=60, n_cheb=34)
    n = 256 * 96 * 192 * 64 * 8  # rows of 3 types x 60 multipoles and columns padded: bytes of one FP64 copy

    def make(budget, precisions):
        F.fake_budget(budget)
        p = _plan(B, precisions=precisions, **size)
        got = p.basis_bytes[0], F.fake_used()
        p.close()
        assert F.fake_used() == 0
        return got

    room = 1 << 40
    every = ("fp64", "fp32", "bf16x3")
    assert make(room, ())[0] == make(room, ("fp32",))[0] == make(room, ("bf16x3", "fp16x3"))[0] == n
    has, full = make(room, every)
    assert has == 2 * n
    assert make(full + n, every) == (2 * n, full)
    for budget in (full + n - 1, full, full - 1, full - n):  # the last: just what the plan has to have
        assert make(budget, every) == (n, full - n), budget
    try:
        make(full - n - 1, every)
        assert False
    except B.BlastError as e:
        assert e.status == B.E_OOM
    F.hipGetLastError()
    F.fake_budget(room)
    with tempfile.TemporaryDirectory() as d:  # a saved plan comes back with what it was asked for
        for precisions in (("bf16x3",), ("fp64", "fp32")):
            p = _plan(B, n_cheb=34, precisions=precisions)
            p.save(d + "/p")
            q = B.Plan.load(d + "/p")
            assert p.basis_bytes == q.basis_bytes
            p.close(), q.close()


CASES = [pageable_requests_are_asked_once, cancelling_waits_for_its_own_copy_only, a_failed_launch_ends_after_its_copies,
         the_optional_nodal_copy_comes_last]


@pytest.mark.parametrize("case", [c.__name__ for c in CASES])
def test_host(fake, case):
    _run(fake, case)


if __name__ == "__main__":
    sys.path.insert(0, os.path.dirname(HERE))
    F = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
    F.fake_pin.argtypes = F.fake_pending.argtypes = [ctypes.c_void_p, ctypes.c_size_t]
    F.fake_budget.argtypes, F.fake_used.restype = [ctypes.c_size_t], ctypes.c_size_t
    for f in (F.fake_attr_calls, F.fake_waits, F.fake_copies):
        f.restype = ctypes.c_long
    from paper_2410_03632_amd import blast

    try:
        {c.__name__: c for c in CASES}[sys.argv[2]](blast, F)
    except BaseException:  # (not through the interpreter's end, which would wait for a server whose time stands still)
        traceback.print_exc()
        sys.stderr.flush()
        os._exit(1)
