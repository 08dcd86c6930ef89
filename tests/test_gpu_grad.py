"""GPU parity of the analytic Hartree-Fock nuclear gradient (mess_hf_gradient)
against the oracle's central differences of its converged energy, given the
oracle's converged density and Fock matrix:

* minimal-basis H2: the force along the bond against the derivative of the
  textbook closed-form energy (within 1e-9 Ha/bohr);
* an s/p molecule (6 atoms) and a water molecule with d functions: every
  component within 1e-6 Ha/bohr of the differences (their own accuracy is
  about 1e-8);
* invariants of the analytic forces: they sum to zero and exert no torque
  (to rounding, far tighter than the differences);
* the SCF handle's gradient (its own converged D and F) agrees with the one
  at the oracle's D and F.
"""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(__file__))
from closed_forms import h2_minimal_energy  # noqa: E402
from gpu_common import announce, dev, need_gpu  # noqa: E402

from mess_inputs import generators as G  # noqa: E402
from oracle import grad as ograd  # noqa: E402

pytestmark = pytest.mark.gpu

CASES = {
    "hco6_sp/1": lambda: G.random_small_molecule(1),
    "water1_spd/0": lambda: G.water_cluster(0, n_waters=1),
}


def test_h2_force_closed_form():
    mess = need_gpu()
    alpha, R = 0.42, 1.3
    mol = G.single_gaussian_system("H2", alpha, bond=R)
    D, F, E = ograd.converged(mol)
    B = mess.basis_from_molecule(mol)
    g = mess.mess_hf_gradient(B, dev(D), dev(F))
    h = 1e-3
    dE = (8 * (h2_minimal_energy(alpha, R + h) - h2_minimal_energy(alpha, R - h))
          - (h2_minimal_energy(alpha, R + 2 * h) - h2_minimal_energy(alpha, R - 2 * h))) / (12 * h)
    announce(f"H2 force {g[1, 2]!r} vs closed-form dE/dR {dE!r}")
    assert abs(g[1, 2] - dE) < 1e-9 and abs(g[0, 2] + dE) < 1e-9
    assert np.abs(g[:, :2]).max() < 1e-12


@pytest.mark.parametrize("case", list(CASES))
def test_gradient_matches_oracle_differences(case):
    mess = need_gpu()
    mol = CASES[case]()
    D, F, E = ograd.converged(mol)
    B = mess.basis_from_molecule(mol)
    g = mess.mess_hf_gradient(B, dev(D), dev(F))
    fd = ograd.fd_gradient(mol)
    err = np.abs(g - fd).max()
    xyz = np.asarray(mol.xyz).reshape(-1, 3)
    announce(f"gradient {case}: max |g - fd| {err:.2e} (max |g| {np.abs(g).max():.3f}); "
             f"sum {np.abs(g.sum(0)).max():.1e}, torque {np.abs(np.cross(xyz, g).sum(0)).max():.1e}")
    assert err < 1e-6
    assert np.abs(g.sum(axis=0)).max() < 1e-10 * max(1.0, np.abs(g).max())
    assert np.abs(np.cross(xyz, g).sum(axis=0)).max() < 1e-8
    # the SCF handle's own converged state
    st = mess.mess_scf_create(B, schwarz_tol=0.0, conv_tol=1e-12, diis_size=8)
    for _ in range(200):
        e, de, r, c = mess.mess_scf_step(st)
        if c:
            break
    assert c
    g2 = mess.mess_scf_gradient(st)
    assert np.abs(g2 - g).max() < 1e-7
    st.close()
    B.close()


@pytest.mark.parametrize("waters,tau", [(1, 0.0), (2, 1e-10)])
def test_gradient_of_given_density_and_fock(waters, tau):
    """Every angular class on one and on several centres: the gradient of
    Tr[D H] + Tr[D J]/2 - Tr[D K]/4 - Tr[W S] + E_nuc at a fixed density D and
    W = D F D / 2 against fourth-order central differences of the oracle's
    integrals.  The differences (step 5e-3 bohr on exponents up to 50) are off
    by h^4/30 times a fifth derivative, of order (2 alpha)^(5/2) = 1e5 of
    terms of order 1: 2e-6 of the largest component at the most."""
    mess = need_gpu()
    from oracle import core
    mol = G.water_cluster(4, n_waters=waters, box=18.0 * (waters / 20) ** (1 / 3) + 4.0, alpha_range=(0.05, 50.0))
    N = mol.n_bf
    rng = np.random.Generator(np.random.PCG64(8))
    A, Fr = rng.normal(size=(N, N)), rng.normal(size=(N, N))
    D, F = (A + A.T) / N, Fr + Fr.T
    W = D @ F @ D / 2

    def energy(m):
        S, T, V = core.one_electron(m)
        J, K, _ = core.jk_unique(m, D, 0.0)
        return (np.sum(D * (T + V)) + 0.5 * np.sum(D * J) - 0.25 * np.sum(D * K) - np.sum(W * S)
                + core.nuclear_repulsion(m))

    h = 5e-3
    fd = np.zeros((len(mol.Z), 3))
    for a in range(len(mol.Z)):
        for k in range(3):
            e = {s: energy(ograd.displaced(mol, a, k, s * h)) for s in (-2, -1, 1, 2)}
            fd[a, k] = (8.0 * (e[1] - e[-1]) - (e[2] - e[-2])) / (12.0 * h)
    B = mess.basis_from_molecule(mol)
    g = mess.mess_hf_gradient(B, dev(D), dev(F), schwarz_tol=tau)
    B.close()
    err = np.abs(g - fd).max() / np.abs(fd).max()
    announce(f"fixed-density gradient, {waters} waters: max |g - fd| / max |fd| {err:.2e}")
    assert err < 2e-6
    assert np.abs(g.sum(axis=0)).max() < 1e-10 * np.abs(g).max()
