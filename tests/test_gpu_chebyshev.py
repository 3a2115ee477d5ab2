"""The Chebyshev recursion with A on the chip, at sizes around every change
of its layout (one workgroup per polarisation up to 256 rows, groups of
workgroups to 1024, a launch per step beyond and for few moments) and step
counts that end inside, at and past a segment, against the oracle's
recursion on the same A."""
import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


def _system(n_o, n_c, seed):
    """A 16^3 system on random orthonormal orbitals: any A will do."""
    from paper_2205_06690_amd import bse
    n, h = 16, 0.6
    rng = np.random.default_rng(seed)
    q, _ = np.linalg.qr(rng.standard_normal((n ** 3, n_o + n_c)))
    phi = np.ascontiguousarray(q.T) / np.sqrt(h ** 3)
    s = bse.System(n, h, np.zeros(n ** 3), n_occ=n_o, n_stoch=2, n_steps=1, clean_every=0, precision=bse.BSE_FP64,
                   max_batch=600)
    s.set_orbitals(phi, np.sort(rng.uniform(-1.0, 1.0, n_o + n_c)))
    A = s.build_a(n_o, n_c)
    from oracle import bse as obse
    from oracle.grid import Grid
    g = phi.reshape(-1, n, n, n)
    return s, A, obse.dipoles(Grid((n, n, n), h), g[:n_o], g[n_o:]), phi


# a residue sums n products of vectors that carry the rounding of the steps
# before them: eps n_mom^2 / 2 at the worst, 1.3e-10 at 1540 moments; random
# signs leave far less
TOL = 1e-10


@pytest.mark.parametrize("n_o,n_c,n_mom", [(1, 1, 40), (8, 8, 1026), (5, 13, 32), (8, 16, 30), (3, 43, 1024), (16, 13, 60), (11, 19, 60), (16, 16, 64),
                                           (1, 257, 1026), (16, 32, 1540), (19, 27, 64), (32, 32, 130), (25, 41, 40)])
def test_resident_recursion(n_o, n_c, n_mom):
    from oracle import bse as obse
    s, A, f0, phi = _system(n_o, n_c, 7 * n_o + n_c)
    n = n_o * n_c
    lo, hi = obse.spectral_bounds(A) if n > 1 else (A[0, 0] - 1.0, A[0, 0] + 1.0)
    a, b = obse.chebyshev_scale(lo, hi)
    bounds = (lo, hi)
    wg = np.linspace(lo, hi, 9)[1:-1]
    sig = 4.0 * (hi - lo) / n_mom
    R = obse.chebyshev_residues(A, f0, n_mom, a, b).T
    sg, res, _ = s.chebyshev_spectrum(n_mom, wg, sig, bounds=bounds)
    e = np.abs(res - R).max() / np.abs(R[:, 0]).max()
    sg_o = obse.chebyshev_absorption(R.T, wg, a, b, sig)
    es = np.abs(sg - sg_o).max() / np.abs(sg_o).max()
    sg_n, res_n, _ = s.chebyshev_spectrum_noalloc(n_mom, wg, sig, bounds=bounds)
    assert np.array_equal(res_n, res) and np.array_equal(sg_n, sg)
    F, dn, _ = s.exciton_states(n_mom - 1, wg[:3], sig, bounds=bounds)
    F_o = obse.chebyshev_states(A, f0, n_mom - 1, a, b, wg[:3], sig)        # [n_w, n, 3]
    eF = np.abs(F - F_o.transpose(0, 2, 1)).max() / np.abs(F_o).max()
    dn_o = np.stack([[obse.exciton_density(phi[:n_o].reshape(-1, 16, 16, 16), phi[n_o:].reshape(-1, 16, 16, 16), F_o[q, :, p])
                      for p in range(3)] for q in range(3)])
    ed = np.abs(dn - dn_o).max() / np.abs(dn_o).max()
    say(f"n = {n}, {n_mom} moments: residues {e:.1e}, sigma {es:.1e}, states {eF:.1e}, densities {ed:.1e}")
    assert max(e, es, eF, ed) < TOL
    s.close()


@pytest.mark.parametrize("n_o,n_c", [(2, 3), (8, 8), (5, 13), (8, 16), (3, 43), (13, 16), (11, 19)])
def test_resident_lanczos(n_o, n_c):
    """The Lanczos steps with A on the chip (up to 208 rows; the path before
    it takes 209) to the last basis vector, against a dense eigensolve:
    excitons to the convergence test's 1e-10 residual, dipoles to the
    residual over the level spacing."""
    s, A, f0, _ = _system(n_o, n_c, 11 * n_o + n_c)
    n = n_o * n_c
    n_exc = min(n, 6)
    om, d2 = s.spectrum(n_exc)
    ev, X = np.linalg.eigh(A)
    gap = np.diff(ev[:n_exc + 1]).min() if n > n_exc else 1e-2
    e = np.abs(om - ev[:n_exc]).max()
    ed = np.abs(d2 - (X[:, :n_exc].T @ f0) ** 2).max() / np.abs(f0).max() ** 2
    om_all, _ = s.spectrum(n)
    ea = np.abs(om_all - ev).max()
    say(f"n = {n}: {n_exc} excitons {e:.1e}, dipoles {ed:.1e} (spacing {gap:.1e}), all {n} {ea:.1e}")
    assert e < 1e-9 and ea < 1e-9
    assert ed < max(1e-8, 4e-10 / gap)
    s.close()


@pytest.mark.parametrize("n_o,n_c", [(5, 13), (3, 43), (19, 27)])
def test_recursion_whose_workgroups_never_met(n_o, n_c):
    """Below and above 256 rows, a resident recursion that gives up (forced: rows
    empty, its flag raised) ends in the launch per step: the residues and the
    interval of both entry points equal bit for bit those of a short call, which
    always runs so (the residues of fewer moments are a prefix), the states
    agree with the oracle, and the next call is resident again."""
    from oracle import bse as obse
    s, A, f0, phi = _system(n_o, n_c, 5 * n_o + n_c)
    n, n_mom = n_o * n_c, 64
    lo, hi = obse.spectral_bounds(A)
    a, b = obse.chebyshev_scale(lo, hi)
    wg = np.linspace(lo, hi, 9)[1:-1]
    sig = 4.0 * (hi - lo) / n_mom
    _, short, bo_s = s.chebyshev_spectrum(30, None)          # 15 steps: one launch each
    sg_r, res_r, bo_r = s.chebyshev_spectrum(n_mom, wg, sig)
    F_r, dn_r, _ = s.exciton_states(n_mom, wg[:3], sig, bounds=(lo, hi))
    s.inject_resident_miss(2)
    got = [s.chebyshev_spectrum(n_mom, wg, sig), s.chebyshev_spectrum_noalloc(n_mom, wg, sig)]
    for sg, res, bo in got:
        assert np.array_equal(res[:, :30], short) and np.array_equal(bo, bo_s)
        assert np.array_equal(sg, got[0][0]) and np.array_equal(res, got[0][1])
    e = np.abs(got[0][1] - res_r).max() / np.abs(res_r[:, 0]).max()
    es = np.abs(got[0][0] - sg_r).max() / np.abs(sg_r).max()
    s.inject_resident_miss(1)
    F, dn, _ = s.exciton_states(n_mom, wg[:3], sig, bounds=(lo, hi))
    F_o = obse.chebyshev_states(A, f0, n_mom, a, b, wg[:3], sig).transpose(0, 2, 1)
    eF = np.abs(F - F_o).max() / np.abs(F_o).max()
    ed = np.abs(dn - dn_r).max() / np.abs(dn_r).max()
    say(f"n = {n}: against the resident recursion residues {e:.1e}, sigma {es:.1e}, densities {ed:.1e}; states {eF:.1e}")
    assert max(e, es, eF, ed) < TOL
    sg2, res2, bo2 = s.chebyshev_spectrum(n_mom, wg, sig)
    assert np.array_equal(sg2, sg_r) and np.array_equal(res2, res_r) and np.array_equal(bo2, bo_r)
    F2, dn2, _ = s.exciton_states(n_mom, wg[:3], sig, bounds=(lo, hi))
    assert np.array_equal(F2, F_r) and np.array_equal(dn2, dn_r)
    s.close()
