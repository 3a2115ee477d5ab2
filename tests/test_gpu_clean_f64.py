"""FP64 cleaning on the matrix cores (Eq. 15): occupied counts and field
counts at and around the tiles' edges (16 states and 16 fields a tile, up to
four state tiles a wave, 64 fields an update group), against the oracle."""
import numpy as np
import pytest

from gpu_util import gpu_system, oracle_w, rel, small_spec

pytestmark = pytest.mark.gpu


# FP64 rounding of 20 steps, two transforms of 4096 points a step: about
# eps sqrt(20 * 24) = 2.5e-15 per field; three orders of margin
TOL = 3e-12


@pytest.mark.parametrize("n_occ,n_stoch,n_pairs", [(1, 1, 1), (3, 5, 2), (15, 4, 3), (16, 3, 5), (17, 5, 3), (33, 4, 17),
                                                   (64, 16, 1), (65, 13, 5)])
def test_fp64_cleaning_tile_edges(n_occ, n_stoch, n_pairs):
    from paper_2205_06690_amd import bse, inputs
    spec = small_spec(n_occ=n_occ, n_o=1, n_c=3, n_steps=20, n_stoch=n_stoch)
    sysd = inputs.make_system(spec)
    rng = np.random.default_rng(n_occ)
    pairs = rng.integers(0, n_occ + 3, (n_pairs, 2)).astype(np.int32)
    w_o, _ = oracle_w(spec, sysd, pairs)
    w = gpu_system(spec, sysd, bse.BSE_FP64, max_batch=n_pairs).apply_w(pairs)
    e = rel(w, w_o.reshape(n_pairs, -1))
    print(f"n_occ {n_occ} L {n_stoch} pairs {n_pairs}: {e.max():.1e}", flush=True)
    assert e.max() < TOL
