"""The FP64 kinetic step as matrix products, on every grid it takes (blocks of
12 and 16 points, one to four residues) with orbital counts around the five or
two density groups (fewer orbitals than groups included) and pair counts on
both sides of the line from which one workgroup takes all groups, against the
oracle."""
import dataclasses

import numpy as np
import pytest

from gpu_util import gpu_system, oracle_w, rel, small_spec

pytestmark = pytest.mark.gpu

# FP64 rounding of 12 steps, three axes of chains of 2 x 16 products and two
# transforms of the grid a step: about eps sqrt(12 (96 + 36)) = 9e-15 per
# field; more than two orders of margin
TOL = 3e-12


@pytest.mark.timeout(300)
@pytest.mark.parametrize("n,n_stoch,n_pairs", [(16, 1, 1), (16, 5, 3), (16, 7, 129), (24, 2, 3), (24, 11, 2),
                                               (24, 6, 58), (32, 4, 5), (32, 6, 33), (48, 1, 2), (48, 5, 1),
                                               (64, 3, 1)])
def test_fp64_kinetic_step(n, n_stoch, n_pairs):
    from paper_2205_06690_amd import bse, inputs
    spec = dataclasses.replace(small_spec(n=n, h=0.5, n_occ=6, n_o=1, n_c=3, n_steps=12, n_stoch=n_stoch))
    sysd = inputs.make_system(spec)
    rng = np.random.default_rng(n + n_stoch)
    pairs = rng.integers(0, 9, (n_pairs, 2)).astype(np.int32)
    w_o, _ = oracle_w(spec, sysd, pairs[:8])
    w = gpu_system(spec, sysd, bse.BSE_FP64, max_batch=n_pairs).apply_w(pairs)
    # beyond the oracle's pairs, a repeated pair is the same pair
    e = rel(w[:8], w_o.reshape(min(n_pairs, 8), -1)).max()
    for k in range(8, n_pairs):
        same = [j for j in range(8) if sorted(pairs[j]) == sorted(pairs[k])]
        if same:
            e = max(e, rel(w[k:k + 1], w_o.reshape(8, -1)[same[0]][None]).max())
    print(f"{n}^3 L {n_stoch} pairs {n_pairs}: {e:.1e}", flush=True)
    assert e < TOL
