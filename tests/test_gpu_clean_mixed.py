"""Mixed-precision cleaning at orbital counts whose pairs fill the update's half
tiles exactly (1, 4, 16), with a remainder (3, 9, 14), not at all (11, 33: the
density is a pass of its own), one and two row tiles of the unperturbed set's
coefficients (8 and 9 orbitals), and state counts around its 64-state tiles,
against the oracle."""
import numpy as np
import pytest

from gpu_util import gpu_system, oracle_w, rel, small_spec

pytestmark = pytest.mark.gpu

# FP32 rounding of 20 steps, two transforms of 3 x 16 points a step: about
# 6e-8 sqrt(20 * 24) = 1.3e-6 per field, cleaning in three BF16 terms (2^-16 of
# the products) on top; a factor of eight of margin
TOL = 2e-5


@pytest.mark.parametrize("n_occ,n_stoch,n_pairs", [(3, 1, 35), (17, 3, 4), (64, 4, 9), (65, 8, 3), (6, 9, 8), (33, 11, 3),
                                                   (5, 14, 5), (66, 16, 2), (4, 33, 2)])
def test_mixed_cleaning_tile_edges(n_occ, n_stoch, n_pairs):
    from paper_2205_06690_amd import bse, inputs
    spec = small_spec(n_occ=n_occ, n_o=1, n_c=3, n_steps=20, n_stoch=n_stoch)
    sysd = inputs.make_system(spec)
    rng = np.random.default_rng(n_occ)
    pairs = rng.integers(0, n_occ + 3, (n_pairs, 2)).astype(np.int32)
    w_o, _ = oracle_w(spec, sysd, pairs)
    w = gpu_system(spec, sysd, bse.BSE_MIXED, max_batch=n_pairs).apply_w(pairs)
    e = rel(w, w_o.reshape(n_pairs, -1))
    print(f"n_occ {n_occ} L {n_stoch} pairs {n_pairs}: {e.max():.1e}", flush=True)
    assert e.max() < TOL


@pytest.mark.parametrize("n_occ,n_stoch,n_pairs", [(64, 16, 1), (48, 17, 2), (49, 17, 2), (48, 32, 1), (49, 32, 1), (16, 33, 1),
                                                   (130, 66, 1)])
def test_unperturbed_coefficients_of_many_orbitals(n_occ, n_stoch, n_pairs):
    """The same where the unperturbed set's coefficients change kernels (16 and 32
    orbitals, 48 states)."""
    test_mixed_cleaning_tile_edges(n_occ, n_stoch, n_pairs)
