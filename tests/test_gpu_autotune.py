"""mess_autotune keeps the fastest: the built-in choice of every class is one
of its candidates, in the form that later builds run it (several lanes per
quartet on short FP64 lists, small s and p molecules in one launch), and a
class is taken off it only for a form that measured faster."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(__file__))
from gpu_common import announce, dev, need_gpu, random_density, torch, zeros  # noqa: E402

from mess_inputs import generators as G  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _default_forms():
    yield
    if torch.cuda.is_available():
        from paper_2406_03121_amd import mess
        for prec in (mess.MESS_FP64, mess.MESS_FP32):
            for c in range(21):
                mess.mess_kernel_form(c, mess.MESS_FORM_AUTO, prec)


def _build_us(mess, B, D, J, K, reps=30):
    """Best time of one direct J/K build, us (events)."""
    best = 1e30
    for _ in range(reps):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        mess.mess_jk(B, D, J, K, schwarz_tol=0.0)
        e1.record()
        e1.synchronize()
        best = min(best, e0.elapsed_time(e1) * 1e3)
    return best


@pytest.mark.parametrize("name,mol", [("hco6_sp/5", lambda: G.random_small_molecule(5)),
                                      ("water3_spd/0", lambda: G.water_cluster(0, n_waters=3, box=8.0))])
@pytest.mark.parametrize("prec", [0, 1])
def test_autotune_keeps_what_is_fastest(name, mol, prec):
    mess = need_gpu()
    announce(f"autotune {name} prec={prec}")
    B = mess.basis_from_molecule(mol())
    D = dev(random_density(B.nbf, seed=4))
    J, K = zeros(B.nbf, B.nbf), zeros(B.nbf, B.nbf)
    builtin = [mess.mess_kernel_form(c, prec=prec) for c in range(21)]
    before = _build_us(mess, B, D, J, K)
    forms, ms = mess.mess_autotune(B, D, schwarz_tol=0.0, reps=5, prec=prec)
    for c in range(21):
        active = mess.mess_kernel_form(c, prec=prec)
        assert forms[c] == active
        if mess.mess_work_stats(B, 0.0, c)[0] == 0:
            assert np.all(ms[c] == -1.0) and active == builtin[c]
            continue
        assert ms[c, 0] > 0.0, f"class {c}: the built-in choice was not timed"
        if active != builtin[c]:
            assert ms[c, active] < ms[c, 0], f"class {c}: form {active} at {ms[c, active]} ms, built-in {ms[c, 0]}"
    # a tuned FP64 build is no slower than an untuned one, within the scatter
    # of the best of 30 runs of some 0.1 to 1 ms
    if prec == 0:
        after = _build_us(mess, B, D, J, K)
        print(f"[gpu-case] {name}: {before:.1f} us untuned, {after:.1f} us tuned", flush=True)
        assert after < 1.25 * before
    B.close()
