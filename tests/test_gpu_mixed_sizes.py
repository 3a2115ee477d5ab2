"""The matrix-free A f and its Chebyshev recursion at field and orbital
counts around the edges of their kernels (one thread per point up to 12
fields, 16-field and 64-orbital tiles, projections in groups of 48 fields),
and the FP64 A on the same contractions, against the oracle on random
orthonormal orbitals."""
import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu

# FP64: sums of 4096 grid points and up to 4 applications of A, whose kinetic
# part spans about 100 Hartree: eps 4096^(1/2) 4 ~ 6e-14 of the largest term
TOL = 1e-11


@pytest.mark.parametrize("n_o,n_occ,n_c", [(1, 1, 1), (2, 17, 3), (5, 16, 2), (11, 65, 1), (12, 33, 2), (13, 64, 2),
                                           (16, 31, 1), (17, 40, 2)])
def test_mixed_recursion_sizes(n_o, n_occ, n_c):
    from oracle import bse as obse
    from oracle.grid import Grid
    from paper_2205_06690_amd import bse
    n, h, n_mom = 16, 0.6, 8
    rng = np.random.default_rng(n_o + n_occ)
    q, _ = np.linalg.qr(rng.standard_normal((n ** 3, n_occ + n_c)))
    phi = np.ascontiguousarray(q.T) / np.sqrt(h ** 3)
    v = rng.uniform(-2.0, 0.0, n ** 3)
    eps = np.sort(rng.uniform(-1.0, 1.0, n_occ + n_c))
    s = bse.System(n, h, v, n_occ=n_occ, n_stoch=2, n_steps=2, clean_every=0, precision=bse.BSE_FP64, max_batch=200)
    s.set_orbitals(phi, eps)
    A = s.build_a(n_o, n_c)
    w = s.valence_w()
    grid = Grid((n, n, n), h)
    g = phi.reshape(-1, n, n, n)
    pairs = [(a, b) for a in range(n_o) for b in range(a, n_o)]
    full = obse.w_stack(n_o, pairs, w.reshape(-1, n, n, n))
    A_o = obse.build_a(grid, g[n_occ - n_o:n_occ], g[n_occ:], eps[n_occ - n_o:n_occ], eps[n_occ:], full)
    eA = np.abs(A - A_o).max() / np.abs(A_o).max()
    f = rng.standard_normal((n_o, n, n, n))

    def apply(x):
        return obse.apply_a_mixed(grid, v.reshape(n, n, n), g[:n_occ], eps[n_occ - n_o:n_occ], full, x)
    y_o = apply(f)
    e1 = np.abs(s.apply_a_mixed(f.reshape(n_o, -1)).reshape(f.shape) - y_o).max() / np.abs(y_o).max()
    lo, hi = -10.0, 1.5 * (np.pi / h) ** 2 + 10.0
    a, b = obse.chebyshev_scale(lo, hi)
    f0 = obse.mixed_dipole_start(grid, g[:n_occ], n_o)
    R = obse.chebyshev_residues_op(apply, f0, n_mom, a, b, lambda x, z: float(np.sum(x * z)) * grid.dv).T
    _, res = s.chebyshev_mixed(n_mom, (lo, hi))
    e2 = np.abs(res - R).max() / np.abs(R[:, 0]).max()
    F_o = obse.chebyshev_states_op(apply, f0, 4, a, b, np.array([0.5]), 3.0)
    amp, _ = s.exciton_states_mixed(4, (lo, hi), [0.5], 3.0, n_a=n_c)
    am_o = np.stack([obse.mixed_amplitudes(grid, g[n_occ:], F_o[0, p]) for p in range(3)])[None]
    e3 = np.abs(amp - am_o).max() / max(np.abs(am_o).max(), 1e-3)
    say(f"n_o {n_o} n_occ {n_occ}: A {eA:.1e}, A f {e1:.1e}, residues {e2:.1e}, amplitudes {e3:.1e}")
    assert max(eA, e1, e2, e3) < TOL
    s.close()


@pytest.mark.parametrize("n_o,n_occ,n_c", [(1, 16, 16), (3, 17, 17), (15, 32, 33), (16, 33, 48), (16, 48, 49), (17, 49, 64),
                                           (8, 80, 81), (33, 100, 2)])
def test_projection_tiles(n_o, n_occ, n_c):
    """Coefficients of a field set on the occupied and on the virtual orbitals at
    every tile shape of their product (one or two row tiles, one to four column
    tiles, several groups) and few or many outputs of its reduction, through
    amplitudes and densities of exciton states of the mixed form."""
    from oracle import bse as obse
    from oracle.grid import Grid
    from paper_2205_06690_amd import bse
    n, h = 16, 0.6
    rng = np.random.default_rng(100 * n_o + n_occ)
    q, _ = np.linalg.qr(rng.standard_normal((n ** 3, n_occ + n_c)))
    phi = np.ascontiguousarray(q.T) / np.sqrt(h ** 3)
    v = rng.uniform(-2.0, 0.0, n ** 3)
    eps = np.sort(rng.uniform(-1.0, 1.0, n_occ + n_c))
    s = bse.System(n, h, v, n_occ=n_occ, n_stoch=2, n_steps=1, clean_every=0, precision=bse.BSE_FP64, max_batch=600)
    s.set_orbitals(phi, eps)
    s.build_a(n_o, 1)
    pairs = [(a, b) for a in range(n_o) for b in range(a, n_o)]
    full = obse.w_stack(n_o, pairs, s.valence_w().reshape(-1, n, n, n))
    grid = Grid((n, n, n), h)
    g = phi.reshape(-1, n, n, n)

    def apply(x):
        return obse.apply_a_mixed(grid, v.reshape(n, n, n), g[:n_occ], eps[n_occ - n_o:n_occ], full, x)
    lo, hi = -10.0, 1.5 * (np.pi / h) ** 2 + 10.0
    a, b = obse.chebyshev_scale(lo, hi)
    F_o = obse.chebyshev_states_op(apply, obse.mixed_dipole_start(grid, g[:n_occ], n_o), 3, a, b, np.array([0.5]), 3.0)
    amp, dens = s.exciton_states_mixed(3, (lo, hi), [0.5], 3.0, n_a=n_c)
    am_o = np.stack([obse.mixed_amplitudes(grid, g[n_occ:], F_o[0, p]) for p in range(3)])[None]
    de_o = np.stack([2.0 * np.einsum("ixyz,ixyz->xyz", g[n_occ - n_o:n_occ], F_o[0, p]) for p in range(3)])[None]
    ea = np.abs(amp - am_o).max() / np.abs(am_o).max()
    ed = np.abs(dens - de_o).max() / np.abs(de_o).max()
    say(f"n_o {n_o} n_occ {n_occ} n_a {n_c}: amplitudes {ea:.1e}, densities {ed:.1e}")
    assert max(ea, ed) < TOL
    s.close()
