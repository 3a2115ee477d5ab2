"""The autotuner keeps the fastest of the shapes that later calls run, the
built-in ones among them."""
import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


def _system(n, L, max_batch, fp64=False, n_occ=6, n_steps=12):
    """Random orbitals in a well: the time of a step does not depend on them."""
    from paper_2205_06690_amd import bse
    h = 0.5
    rng = np.random.default_rng(n)
    x = (np.arange(n) + 0.5 - n / 2) * h
    v = -2.0 * np.exp(-(x[:, None, None] ** 2 + x[None, :, None] ** 2 + x[None, None, :] ** 2) / 4)
    s = bse.System(n, h, v, n_occ=n_occ, n_stoch=L, seed=5, dt=0.05, n_steps=n_steps, gamma=0.5, clean_every=0,
                   precision=bse.BSE_FP64 if fp64 else bse.BSE_MIXED, max_batch=max_batch)
    s.set_orbitals(rng.standard_normal((n_occ, n ** 3)) / (n * h) ** 1.5, np.zeros(n_occ))
    return s


def _pass_times(s, B, n_occ=6, reps=4):
    """The fastest of a few calls' mean times (ms) of the x and plane passes."""
    pairs = np.array([(k % n_occ, (k // n_occ) % n_occ) for k in range(B)], dtype=np.int32)
    s.set_timing(1)
    t = []
    for _ in range(reps):
        s.apply_w(pairs)
        k = s.kernel_times()
        t.append((k["prop_x"][0], k["prop_yz"][0]))
    s.set_timing(0)
    return tuple(min(x) for x in zip(*t))


def test_default_plane_shape_is_kept_at_24():
    """At 24^3 in mixed precision the default plane pass runs on 192 threads, a
    fifth faster than on 256: a tuned run must not be slower than an untuned
    one (10 % for the clock)."""
    s = _system(24, 10, 96)
    before = _pass_times(s, 96)[1]
    tc, nt = s.autotune(96)
    after = _pass_times(s, 96)[1]
    say(f"24^3, 96 pairs: plane pass {before * 1e3:.1f} us untuned, {after * 1e3:.1f} us tuned (x tile {tc}, block {nt})")
    assert nt in (256, 512)
    assert after < 1.1 * before
    s.close()
