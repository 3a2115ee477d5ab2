"""Device memory that a system holds between calls."""
import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


def _free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.timeout(300)
def test_large_recursion_scratch_is_given_back():
    """The vectors of a matrix-free recursion (nine sets, 566 MB for 30 valence
    orbitals at 64^3, and six more of its steps) do not stay with the system;
    one set of 63 MB and small buffers may."""
    from paper_2205_06690_amd import bse
    n, h, n_o = 64, 0.5, 30
    rng = np.random.default_rng(4)
    s = bse.System(n, h, np.zeros(n ** 3), n_occ=n_o, n_stoch=1, n_steps=1, clean_every=0, precision=bse.BSE_MIXED,
                   max_batch=93)
    s.set_orbitals(rng.standard_normal((n_o + 1, n ** 3)) / (n * h) ** 1.5, np.zeros(n_o + 1))
    s.build_a(n_o, 1)
    s.apply_a_mixed(np.ones((n_o, n ** 3)))
    before = _free()
    _, r1 = s.chebyshev_mixed(4, (-50.0, 50.0))
    held = before - _free()
    _, r2 = s.chebyshev_mixed(4, (-50.0, 50.0))
    say(f"64^3, {n_o} valence orbitals: {held / 2 ** 20:.0f} MiB held after the recursion")
    assert held < 128 << 20
    assert np.array_equal(r1, r2)
    s.close()


def test_no_third_unperturbed_buffer_where_it_is_not_used():
    """set_orbitals at 112^3 holds, for each stochastic orbital and point, its
    t = 0 forms (8 + 8 bytes) and two steps of the unperturbed set (8 each in
    mixed precision); the third step's buffer is for grids up to 64^3."""
    from paper_2205_06690_amd import bse
    n, h, n_occ = 112, 0.5, 2
    phi = np.random.default_rng(5).standard_normal((n_occ, n ** 3)) / (n * h) ** 1.5
    used = {}
    for L in (4, 24):
        s = bse.System(n, h, np.zeros(n ** 3), n_occ=n_occ, n_stoch=L, n_steps=1, precision=bse.BSE_MIXED, max_batch=1)
        before = _free()
        s.set_orbitals(phi, np.zeros(n_occ))
        used[L] = before - _free()
        s.close()
    per = (used[24] - used[4]) / 20 / n ** 3
    say(f"112^3 mixed: {per:.1f} bytes a point and stochastic orbital")
    assert per < 36
