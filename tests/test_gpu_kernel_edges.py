"""Sizes and branches at the edge of what a kernel's tables and LDS hold."""
import math
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(__file__))
from gpu_common import announce, dev, host, need_gpu, random_density, torch  # noqa: E402
from test_gpu_pbe import test_xc_at_tile_edges as _xc_at  # noqa: E402

from mess_inputs import generators as G  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nbf", [160, 640, 1280])
def test_xc_at_full_panels(nbf):
    """The last sizes of a point tile: 160 functions with 64 points (80 KB, two
    blocks a CU), 640 with 32 and 1280 with 16, whose basis values take all
    160 KB of LDS."""
    _xc_at(nbf)


def test_gradient_beyond_512_atoms():
    """Above 512 atoms the gradient kernels add to the gradient in memory
    instead of LDS.  The gradient at a given density and Fock matrix is a sum
    over nuclei, so that of two waters among 520 protons without functions
    follows from three calls with 6, 266 and 266 atoms and the repulsion
    between the two halves of the protons: sums of some 1e4 terms in FP64,
    1e-12 of the largest component."""
    mess = need_gpu()
    w = G.water_cluster(1, n_waters=2, box=8.0)
    rng = np.random.Generator(np.random.PCG64(3))
    half = 260
    # protons on shells 15 to 40 bohr from the waters, no two within 1 bohr
    pts = []
    while len(pts) < 2 * half:
        d = rng.normal(size=3)
        x = np.asarray(w.xyz).reshape(-1, 3).mean(axis=0) + d / np.linalg.norm(d) * rng.uniform(15.0, 40.0)
        if all(np.linalg.norm(x - y) > 1.0 for y in pts):
            pts.append(x)
    pts = np.array(pts)
    D = random_density(w.n_bf, seed=5) / w.n_bf
    F = random_density(w.n_bf, seed=6)
    n = len(w.Z)

    def gradient(extra):
        Z = np.concatenate([w.Z, np.ones(len(extra), np.int32)]).astype(np.int32)
        xyz = np.concatenate([np.asarray(w.xyz).reshape(-1, 3), extra]) if len(extra) else np.asarray(w.xyz)
        B = mess.mess_basis_create(Z, xyz, w.shell_atom, w.shell_l, w.shell_nprim, w.exps, w.coefs, len(extra))
        g = np.asarray(mess.mess_hf_gradient(B, dev(D), dev(F), schwarz_tol=1e-12)).reshape(-1, 3)
        B.close()
        return g

    announce("gradient of 526 atoms")
    g0, g1, g2, g = (gradient(e) for e in (pts[:0], pts[:half], pts[half:], pts))
    ref = np.empty_like(g)
    ref[:n] = g1[:n] + g2[:n] - g0
    d = pts[:half, None] - pts[None, half:]
    rep = d / np.linalg.norm(d, axis=-1, keepdims=True) ** 3
    ref[n:n + half] = g1[n:] - rep.sum(axis=1)
    ref[n + half:] = g2[n:] + rep.sum(axis=0)
    assert np.abs(g - ref).max() <= 1e-12 * np.abs(ref).max()


def test_boys_rows_of_the_segment_kernels():
    """The segment kernels take the Boys function's row number from the low
    word of a sum and the inverse root in one step of third order, which
    mess_boys does not run.  Pairs of s, p and d functions on one centre
    against an s pair on another: with the density on the s pair alone, each J
    element is one integral (ab|ss), of order 0 (ss) to 4 (dd).  Every row of
    the table at its middle and both ends, and the large-argument form, against
    the oracle in extended precision: a few tens of FP64 operations, 1e-13 of
    the shell pair's largest element."""
    mess = need_gpu()
    from oracle import core
    a, b = 0.8, 1.3
    rho = (2 * a) * (2 * b) / (2 * a + 2 * b)
    T = [k / 4 + e for k in range(241) for e in (-0.125 + 1e-9, 0.0, 0.125 - 1e-9)]
    T = [t for t in T if t > 1e-3] + [1e-3, 60.0 - 1e-9, 60.0, 75.0, 400.0]
    mols = [G.Molecule(np.array([1, 1], np.int32), np.array([[0, 0, 0], [R / 3, 2 * R / 3, -2 * R / 3]]),
                       np.array([0, 0, 0, 1], np.int32), np.array([0, 1, 2, 0], np.int32), np.ones(4, np.int32),
                       np.array([a, a, a, b]), np.ones(4), 0, f"boys/{t}")
            for t in T for R in [math.sqrt(t / rho)]]
    n = mols[0].n_bf
    D = np.zeros((n, n))
    D[n - 1, n - 1] = 1.0
    announce(f"Boys rows of the segment kernels, {len(mols)} pairs of centres")
    B = mess.mess_batch_create(mols)
    Dp = torch.as_tensor(np.tile(D.ravel(), len(mols)), device="cuda")
    J, K = torch.zeros_like(Dp), torch.zeros_like(Dp)
    classes = [mess.class_index(cb, 0) for cb in range(6)]  # (ss|ss) .. (dd|ss)
    try:
        for c in classes:
            assert mess.mess_kernel_form(c, mess.MESS_FORM_ROWS) == mess.MESS_FORM_ROWS
        mess.mess_jk(B, Dp, J, K, schwarz_tol=0.0)
        torch.cuda.synchronize()
    finally:
        for c in classes:
            mess.mess_kernel_form(c, mess.MESS_FORM_AUTO)
    got = host(J).reshape(len(mols), n, n)
    B.close()
    first = [0, 1, 4, 10]
    worst = 0.0
    for m, t, g in zip(mols, T, got):
        with core.extended_precision():
            ref = core.jk_unique(m, D, 0.0)[0]
        for i in range(3):
            for j in range(3):
                s = np.s_[first[i]:first[i + 1], first[j]:first[j + 1]]
                err = np.abs(g[s] - ref[s]).max() / np.abs(ref[s]).max()
                worst = max(worst, err)
                assert err <= 1e-13, (t, i, j, err)
    print(f"[gpu-case] largest error {worst:.1e}", flush=True)
