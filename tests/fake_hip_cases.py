"""Host-logic cases that test_host_logic.py runs in a process of its own, with
fake_hip.c in place of the HIP runtime (argv: its library, the case)."""
import ctypes
import os
import sys
import threading

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)

from mess_inputs import generators as G  # noqa: E402
from paper_2406_03121_amd import mess  # noqa: E402

assert "torch" not in sys.modules
CREATES = [b"hipMalloc", b"hipFree", b"hipStreamCreateWithFlags", b"hipEventCreate", b"hipEventCreateWithFlags"]
STREAM = b"hipStreamCreateWithFlags"


def system():
    """A basis with d shells (all 21 classes), and its density and outputs."""
    B = mess.basis_from_molecule(G.water_cluster(0, n_waters=2, box=6.0))
    D = np.eye(B.nbf)
    return B, D, np.zeros_like(D), np.zeros_like(D)


def p(a):
    return None if a is None else a.ctypes.data_as(ctypes.c_void_p)


def jk(s, stream=0):
    B, D, J, K = s
    rc = mess.lib().mess_jk(B.handle, p(D), p(J), p(K), 0, 0, 0.0, ctypes.c_void_p(stream))
    assert rc == 0, mess.mess_last_error()


def noalloc(s, stream=0):
    B, D, J, K = s
    rc = mess.lib().mess_jk_noalloc(B.handle, p(D), p(J), p(K), 0, 0.0, ctypes.c_void_p(stream))
    assert rc == 0, mess.mess_last_error()


def noalloc_creates_nothing():
    s = system()
    # lists and tables made by a build that forks no streams
    mess.mess_prof_enable(True)
    jk(s)
    mess.mess_prof_enable(False)
    before = [fake.fake_count(n) for n in CREATES]
    noalloc(s)
    assert [fake.fake_count(n) for n in CREATES] == before
    # once another build has made them, it runs on the class streams too
    jk(s)
    waits = fake.fake_count(b"hipStreamWaitEvent")
    before = [fake.fake_count(n) for n in CREATES]
    noalloc(s)
    assert [fake.fake_count(n) for n in CREATES] == before
    assert fake.fake_count(b"hipStreamWaitEvent") > waits


def streams_per_caller():
    s = system()
    jk(s, 0x10)
    assert fake.fake_count(STREAM) == 3
    jk(s, 0x10)
    assert fake.fake_count(STREAM) == 3      # the same caller again
    jk(s, 0x20)
    assert fake.fake_count(STREAM) == 6      # another caller's work queues behind neither
    jk(s, 0x10)
    jk(s, 0x20)
    assert fake.fake_count(STREAM) == 6
    for k in range(3, 40):                   # bounded
        jk(s, 0x10 * k)
    assert fake.fake_count(STREAM) == 24


def streams_per_device():
    n = 8
    sets = [system() for _ in range(n)]
    for s in sets:
        mess.mess_work_stats(s[0], 0.0, 0)
    fake.fake_gate(n)
    th = [threading.Thread(target=jk, args=(s, 0x10 * (i + 1))) for i, s in enumerate(sets)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    fake.fake_gate(0)
    assert fake.fake_count(STREAM) == 3 * n  # the first device has its eight
    fake.fake_device(1)
    jk(system())
    assert fake.fake_count(STREAM) == 3 * n + 3


def gradient_waits_for_its_copy():
    B, D, _, _ = system()
    g = np.zeros(3 * B.n_atoms)
    f = mess.lib().mess_hf_gradient

    def run():
        return f(B.handle, p(D), p(D), ctypes.c_double(0.0), p(g), None)

    assert run() == 0, mess.mess_last_error()
    assert fake.fake_pending_copies() == 0
    # every launch of the call failing in turn
    n0 = fake.fake_count(b"hipGetLastError")
    assert run() == 0
    checks = fake.fake_count(b"hipGetLastError") - n0
    failed = 0
    for k in range(1, checks + 1):
        fake.fake_fail(b"hipGetLastError", k)
        rc = run()
        fake.fake_fail(None, 0)
        failed += rc != 0
        assert fake.fake_pending_copies() == 0, f"returned {rc} with its host table still being copied (launch {k})"
    assert failed > 5


def xc(s, pbe, V, E):
    B, D, J, _ = s
    v, e = p(J) if V else None, ctypes.byref(ctypes.c_double()) if E else None
    if pbe:
        rc = mess.lib().mess_pbe_xc(B.handle, p(D), v, e, None, None, None)
    else:
        rc = mess.lib().mess_lda_x(B.handle, p(D), v, e, None, None)
    assert rc == 0, mess.mess_last_error()


def xc_buffers_stay():
    # what a captured call could hold is neither made by a later call of the
    # same functional nor freed by any
    for first in (0, 1):
        s = system()
        xc(s, first, False, True)
        n = fake.fake_count(b"hipMalloc")
        xc(s, first, True, False)
        assert fake.fake_count(b"hipMalloc") == n
        fake.fake_watch()
        xc(s, 1 - first, True, True)
        xc(s, first, True, True)
        assert fake.fake_freed_watched() == 0
        s[0].close()


def tensor_workspace():
    B, D, J, K = system()
    jk((B, D, J, K))
    out = np.zeros(B.nbf ** 4)

    def eri(stream):
        rc = mess.lib().mess_eri(B.handle, 0, 0, 0.0, p(out), out.nbytes, ctypes.c_void_p(stream))
        assert rc == 0, mess.mess_last_error()
        return fake.fake_count(b"hipLaunchKernel"), fake.fake_count(b"hipMalloc")

    l0, _ = eri(0x10)
    l1, m1 = eri(0x10)
    assert eri(0x20) == (l1 + (l1 - l0), m1)  # kept, whatever the stream
    B.close()
    # without the workspace the tensor is built without it: one launch fewer
    B, D, J, K = system()
    jk((B, D, J, K))
    k0 = fake.fake_count(b"hipLaunchKernel")
    fake.fake_fail(b"hipMalloc", 1)
    k1, _ = eri(0x10)
    assert k1 - k0 == (l1 - l0) - 1


globals()[sys.argv[2]]()
print("ok")
