"""Propagation passes whose orbitals run in workgroups of their own on small
batches: W of the same pairs from the largest batch that runs so and from the
next larger one that does not are equal bit for bit (no cleaning step, whose
sums depend on the batch; an even number of pairs, so that the same two share
a transform of the density), with fewer, as many and more orbitals than the
density groups of the FP64 pass."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(300)
@pytest.mark.parametrize("n,fp64,n_stoch,small,large", [(16, 0, 4, 48, 50), (24, 0, 3, 32, 34), (32, 0, 7, 24, 26),
                                                        (48, 0, 2, 12, 14), (64, 0, 3, 4, 6), (112, 0, 2, 2, 4),
                                                        (16, 1, 7, 126, 128), (24, 1, 5, 56, 58), (32, 1, 3, 30, 32),
                                                        (48, 1, 1, 40, 44), (64, 1, 3, 22, 24)])
def test_split_and_unsplit_passes_agree(n, fp64, n_stoch, small, large):
    from paper_2205_06690_amd import bse
    n_occ, h = 5, 0.5
    rng = np.random.default_rng(n + n_stoch)
    x = (np.arange(n) + 0.5) * h
    v = -2.0 * np.exp(-((x[:, None, None] - n * h / 3) ** 2 + (x[None, :, None] - n * h / 2) ** 2 +
                        (x[None, None, :] - n * h / 2) ** 2) / 4)
    phi = rng.standard_normal((n_occ, n, n, n)) / (n * h) ** 1.5
    pairs = rng.integers(0, n_occ, (large, 2)).astype(np.int32)
    res = []
    for B in (small, large):
        s = bse.System(n, h, v, n_occ=n_occ, n_stoch=n_stoch, seed=3, dt=0.05, n_steps=4, gamma=0.5, clean_every=0,
                       precision=bse.BSE_FP64 if fp64 else bse.BSE_MIXED, max_batch=B)
        s.set_signs(np.where(np.random.default_rng(1).random((n_stoch, n_occ)) < 0.5, -1, 1).astype(np.int8))
        s.set_orbitals(phi.reshape(n_occ, -1), np.zeros(n_occ))
        res.append(s.apply_w(pairs[:B])[:small])
        s.close()
    assert np.isfinite(res[0]).all()
    print(f"{n}^3 L {n_stoch}, {small} and {large} pairs: max|dW| {np.abs(res[0] - res[1]).max():.1e}", flush=True)
    assert np.array_equal(res[0], res[1])


def test_parts_of_many_orbitals_are_not_slower():
    """With many orbitals the partial densities outgrow the last-level cache and
    the pairs run whole: 24 pairs of 30 orbitals at 32^3 (768 planes, in parts
    with fewer orbitals) must not take longer than 25, which always run whole
    (5 % for the clock; 13 % slower in parts)."""
    import time
    import torch
    from paper_2205_06690_amd import bse
    n, h, n_occ, L = 32, 0.5, 6, 30
    rng = np.random.default_rng(2)
    s = bse.System(n, h, np.zeros(n ** 3), n_occ=n_occ, n_stoch=L, seed=3, dt=0.05, n_steps=20, gamma=0.5,
                   clean_every=0, precision=bse.BSE_MIXED, max_batch=25)
    s.set_orbitals(rng.standard_normal((n_occ, n ** 3)) / (n * h) ** 1.5, np.zeros(n_occ))
    pq = torch.from_numpy(rng.integers(0, n_occ, (25, 2)).astype(np.int32)).cuda()
    w = torch.empty((25, n ** 3), dtype=torch.float64, device="cuda")
    t = {24: [], 25: []}
    for k in range(8):
        for B in t:
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            s.apply_w_device(pq[:B], w[:B])
            torch.cuda.synchronize()
            t[B].append(time.perf_counter() - t0)
    a, b = min(t[24][1:]), min(t[25][1:])
    print(f"32^3, 30 orbitals: 24 pairs {a * 1e3:.2f} ms, 25 pairs {b * 1e3:.2f} ms", flush=True)
    assert a < 1.05 * b
    s.close()
