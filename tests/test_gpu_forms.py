"""Every kernel form of every class (the choices the autotuner makes) meets
the same parity bar: with the form of one class forced, dense ERIs within
1e-12 * max(1, |x|) of the extended-precision oracle and direct J/K within
1e-11 * max(1, |x|) of the oracle's defining sums, for a molecule holding
every angular class.  FP32 table: with one class's FP32 form forced, FP32
J/K within 2e-5 of max|J|, max|K| (the FP32 bar of the mixed-precision
tests)."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(__file__))
from gpu_common import announce, dev, host, need_gpu, random_density, zeros  # noqa: E402

from mess_inputs import generators as G  # noqa: E402
from oracle import core  # noqa: E402

pytestmark = pytest.mark.gpu

PC = ["ss", "ps", "pp", "ds", "dp", "dd"]
FORMS = {1: "lane", 2: "rows", 3: "plane", 4: "coop", 5: "wave", 6: "fp64"}


def _cases(forms, prec):
    """The (class, form) pairs the library has kernels for (the form table's
    validity check is host logic: no device needed to ask)."""
    out = [(cb, ck, f) for cb in range(6) for ck in range(cb + 1) for f in forms]
    try:
        from paper_2406_03121_amd import mess
        lib = mess.lib()
        p = mess.MESS_FP64 if prec == 64 else mess.MESS_FP32
    except Exception:  # library not built: every pair, each skipped at run time
        return out
    built = []
    for cb, ck, f in out:
        cls = cb * (cb + 1) // 2 + ck
        if lib.mess_kernel_form(p, cls, f, None) == mess.MESS_OK:
            built.append((cb, ck, f))
        lib.mess_kernel_form(p, cls, mess.MESS_FORM_AUTO, None)
    return built


@pytest.fixture(scope="module")
def ref():
    mol = G.water_cluster(0, n_waters=2, box=7.0)
    with core.extended_precision():
        eri = core.eri_dense(mol)
    D = random_density(mol.n_bf, seed=51)
    J, K = core.jk_from_dense(core.eri_dense(mol), D)
    return mol, eri, D, J, K


@pytest.mark.parametrize("cb,ck,form", _cases([1, 2, 3, 4, 5], 64))
def test_form_parity(ref, cb, ck, form):
    mess = need_gpu()
    cls = mess.class_index(cb, ck)
    if mess.lib().mess_kernel_form(mess.MESS_FP64, cls, form, None) != mess.MESS_OK:
        pytest.skip(f"form {FORMS[form]} not built for ({PC[cb]}|{PC[ck]})")
    try:
        mol, eri, D, Jo, Ko = ref
        announce(f"form {FORMS[form]} for ({PC[cb]}|{PC[ck]})")
        B = mess.basis_from_molecule(mol)
        N = B.nbf
        out = zeros(N, N, N, N)
        mess.mess_eri(B, out, schwarz_tol=0.0)
        got = host(out)
        err = np.abs(got - eri) / np.maximum(1.0, np.abs(eri))
        assert err.max() < 1e-12, err.max()
        for tau in (0.0, 1e-10):
            J, K = zeros(N, N), zeros(N, N)
            mess.mess_jk(B, dev(D), J, K, schwarz_tol=tau)
            if tau == 0.0:
                rel = lambda a, b: np.max(np.abs(a - b) / np.maximum(1.0, np.abs(b)))  # noqa: E731
                assert rel(host(J), Jo) < 1e-11 and rel(host(K), Ko) < 1e-11
            else:
                Jt, Kt, _ = core.jk_unique(mol, D, tau)
                rel = lambda a, b: np.max(np.abs(a - b) / np.maximum(1.0, np.abs(b)))  # noqa: E731
                assert rel(host(J), Jt) < 1e-11 and rel(host(K), Kt) < 1e-11
        B.close()
    finally:
        mess.mess_kernel_form(cls, mess.MESS_FORM_AUTO)


@pytest.mark.parametrize("cb,ck,form", _cases([1, 2, 3, 4, 5, 6], 32))
def test_fp32_form_parity(ref, cb, ck, form):
    mess = need_gpu()
    cls = mess.class_index(cb, ck)
    if mess.lib().mess_kernel_form(mess.MESS_FP32, cls, form, None) != mess.MESS_OK:
        pytest.skip(f"FP32 form {FORMS[form]} not built for ({PC[cb]}|{PC[ck]})")
    try:
        mol, eri, D, Jo, Ko = ref
        announce(f"fp32 form {FORMS[form]} for ({PC[cb]}|{PC[ck]})")
        B = mess.basis_from_molecule(mol)
        N = B.nbf
        J, K = zeros(N, N), zeros(N, N)
        mess.mess_jk(B, dev(D), J, K, prec=mess.MESS_FP32, schwarz_tol=0.0)
        dJ = np.max(np.abs(host(J) - Jo)) / np.max(np.abs(Jo))
        dK = np.max(np.abs(host(K) - Ko)) / np.max(np.abs(Ko))
        assert dJ < 2e-5 and dK < 2e-5, (dJ, dK)
        B.close()
    finally:
        mess.mess_kernel_form(cls, mess.MESS_FORM_AUTO, prec=mess.MESS_FP32)


@pytest.mark.parametrize("waters", [1, 3, 7, 13])
def test_shared_quartets_match_single_lanes(waters):
    """Direct J/K with the built-in forms, which on lists of these lengths put
    64, 16, 4 or 1 lanes on a quartet by class, against every unrolled class
    forced to one lane per quartet: sums of the same terms in another order,
    1e-12 * max(1, |x|) apart at the most (the bar of one form against the
    oracle is 1e-11)."""
    mess = need_gpu()
    mol = G.water_cluster(3, n_waters=waters, box=18.0 * (waters / 20) ** (1 / 3) + 3.0)
    announce(f"shared quartets, {waters} waters, {mol.n_bf} functions")
    B = mess.basis_from_molecule(mol)
    N = mol.n_bf
    D = dev(random_density(N, seed=7))
    got, ref = [zeros(N, N), zeros(N, N)], [zeros(N, N), zeros(N, N)]
    mess.mess_jk(B, D, *got, schwarz_tol=1e-10)
    forced = [c for c in range(21)
              if mess.lib().mess_kernel_form(mess.MESS_FP64, c, mess.MESS_FORM_LANE, None) == mess.MESS_OK]
    try:
        assert len(forced) == 14
        mess.mess_jk(B, D, *ref, schwarz_tol=1e-10)
    finally:
        for c in forced:
            mess.mess_kernel_form(c, mess.MESS_FORM_AUTO)
    for a, b in zip(got, ref):
        a, b = host(a), host(b)
        assert np.all(np.abs(a - b) <= 1e-12 * np.maximum(1.0, np.abs(b)).max())
    B.close()


@pytest.mark.parametrize("atoms,half", [(2, None), (4, None), (6, None), (6, "J"), (6, "K"), (9, None), (15, None)])
def test_small_molecules_in_one_launch(atoms, half):
    """s and p molecules whose lists take 64 (2 and 4 atoms) or 16 lanes a
    quartet (6, 9) run their classes in one launch, longer ones (15) in one each:
    J, K (or one of them) and the dense tensor against the same builds with a
    form asked for, which keeps the separate launches.  Sums of the same terms
    in another order: 1e-12 * max(1, |x|)."""
    mess = need_gpu()
    mol = G.random_small_molecule(3, n_atoms=atoms, box=6.0 * (atoms / 6) ** (1 / 3) + 1.0)
    announce(f"one launch, {atoms} atoms, {mol.n_bf} functions, {half}")
    B = mess.basis_from_molecule(mol)
    N = mol.n_bf
    D = dev(random_density(N, seed=9))

    def builds():
        J, K = (None if half == "K" else zeros(N, N)), (None if half == "J" else zeros(N, N))
        mess.mess_jk(B, D, J, K, schwarz_tol=0.0)
        out = [x for x in (J, K) if x is not None]
        if half is None and N <= 50:
            out.append(zeros(N, N, N, N))
            mess.mess_eri(B, out[-1], schwarz_tol=0.0)
        return [host(x) for x in out]

    got = builds()
    try:
        assert mess.lib().mess_kernel_form(mess.MESS_FP64, 0, mess.MESS_FORM_LANE, None) == mess.MESS_OK
        ref = builds()
    finally:
        mess.mess_kernel_form(0, mess.MESS_FORM_AUTO)
    for a, b in zip(got, ref):
        assert np.all(np.abs(a - b) <= 1e-12 * np.maximum(1.0, np.abs(b)).max())
    B.close()


@pytest.mark.parametrize("mode", ["direct", "stored"])
def test_class_streams_order_and_capture(mode):
    """The classes of a build run on several streams between a fork and a
    join: calls on two streams at once, buffers overwritten right after a call
    on its stream, and a captured call (one stream) all give the eager result
    (same terms, order of the atomics aside: 1e-12 * max(1, |x|))."""
    import torch
    mess = need_gpu()
    mode = mess.MESS_JK_STORED if mode == "stored" else mess.MESS_JK_DIRECT
    mols = [G.water_cluster(k, n_waters=2, box=8.0) for k in (1, 2)]
    Bs = [mess.basis_from_molecule(m) for m in mols]
    N = mols[0].n_bf
    Ds = [dev(random_density(N, seed=k)) for k in (1, 2)]
    ref = []
    for B, D in zip(Bs, Ds):
        J, K = zeros(N, N), zeros(N, N)
        mess.mess_jk(B, D, J, K, schwarz_tol=1e-10, mode=mode)
        ref.append((host(J), host(K)))
    bar = [tuple(1e-12 * max(1.0, np.abs(x).max()) for x in r) for r in ref]
    streams = [torch.cuda.Stream() for _ in Bs]
    out = [(zeros(N, N), zeros(N, N)) for _ in Bs]
    torch.cuda.synchronize()
    for _ in range(3):
        for k, st in enumerate(streams):
            with torch.cuda.stream(st):
                D = Ds[k].clone()
                mess.mess_jk(Bs[k], D, *out[k], schwarz_tol=1e-10, mode=mode)
                D.fill_(float("nan"))  # ordered after the call on its stream
        torch.cuda.synchronize()
        for k in range(2):
            for a, b, t in zip(out[k], ref[k], bar[k]):
                assert np.abs(host(a) - b).max() <= t
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        mess.mess_jk(Bs[0], Ds[0], *out[0], schwarz_tol=1e-10, mode=mode)
    for _ in range(3):
        for x in out[0]:
            x.zero_()
        g.replay()
        mess.mess_jk(Bs[1], Ds[1], *out[1], schwarz_tol=1e-10, mode=mode)  # eager work between the replays
        torch.cuda.synchronize()
        for k in range(2):
            for a, b, t in zip(out[k], ref[k], bar[k]):
                assert np.abs(host(a) - b).max() <= t
    for B in Bs:
        B.close()


def test_wide_exchange_rows():
    """480 functions: the exchange rows of a dd bra take 46 KB of LDS beside
    the Boys rows of the segment kernels, together beyond 64 KB.  Eager and
    captured builds against the d-bra classes forced to one lane per quartet:
    sums of the same terms in another order, 1e-12 * max(1, |x|)."""
    import torch
    mess = need_gpu()
    mol = G.water_cluster(5, n_waters=32, box=26.0)
    assert mol.n_bf == 480
    announce("wide exchange rows, 480 functions")
    B = mess.basis_from_molecule(mol)
    N = mol.n_bf
    D = dev(random_density(N, seed=11))
    J, K, Jc, Kc = (zeros(N, N) for _ in range(4))
    tau = 1e-7
    g = torch.cuda.CUDAGraph()
    mess.mess_jk(B, D, J, K, schwarz_tol=tau)
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        mess.mess_jk(B, D, Jc, Kc, schwarz_tol=tau)
    forced = [mess.class_index(5, 0), mess.class_index(3, 0)]
    Jr, Kr = zeros(N, N), zeros(N, N)
    try:
        for c in forced:
            assert mess.lib().mess_kernel_form(mess.MESS_FP64, c, mess.MESS_FORM_LANE, None) == mess.MESS_OK
        mess.mess_jk(B, D, Jr, Kr, schwarz_tol=tau)
    finally:
        for c in forced:
            mess.mess_kernel_form(c, mess.MESS_FORM_AUTO)
    for _ in range(2):
        Jc.zero_()
        Kc.zero_()
        g.replay()
        torch.cuda.synchronize()
        for a, b in ((J, Jr), (K, Kr), (Jc, Jr), (Kc, Kr)):
            a, b = host(a), host(b)
            assert np.abs(a - b).max() <= 1e-12 * max(1.0, np.abs(b).max())
    B.close()
