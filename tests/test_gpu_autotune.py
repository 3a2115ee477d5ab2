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


@pytest.mark.parametrize("n,L,B,fp64", [(64, 10, 1, False), (32, 6, 2, False), (48, 8, 1, True), (64, 10, 12, False)])
def test_timed_launches_are_those_that_run(n, L, B, fp64, tmp_path):
    """The times behind a choice (written to the cache file) are those of the
    passes of a batch of this size: where a small batch runs its orbitals in
    parts and the unperturbed set beside the pairs, the passes timed do so
    too.  Whole, the plane pass of one 64^3 pair takes three times as long; a
    factor of 1.5 is left for the gaps between launches."""
    s = _system(n, L, B, fp64)
    cache = str(tmp_path / "tune.txt")
    s.autotune(B, cache)
    x, yz = _pass_times(s, B)
    f = open(cache).read().split()
    say(f"{n}^3 {'FP64' if fp64 else 'mixed'} {B} pairs: x pass {x * 1e3:.1f} us, timed {float(f[3]) * 1e3:.1f}; "
        f"plane pass {yz * 1e3:.1f} us, timed {float(f[4]) * 1e3:.1f}")
    for ran, timed in ((x, float(f[3])), (yz, float(f[4]))):
        assert timed < 1.5 * ran + 2e-3 and ran < 1.5 * timed + 2e-3
    s.close()


def test_lines_of_former_kernels_are_not_applied(tmp_path):
    """A cache line written for other kernels (its key without their version)
    is timed anew and stays in the file; the new line is then read."""
    cache = tmp_path / "tune.txt"
    old = "n24_f64_B3_L4 16 512 0.001 0.001 0 -1 0\n"
    cache.write_text(old)
    s = _system(24, 4, 3, fp64=True)
    shape = s.autotune(3, str(cache))
    lines = cache.read_text().splitlines(keepends=True)
    say(f"24^3 FP64: {lines}")
    assert lines[0] == old and len(lines) == 2
    assert s.autotune(3, str(cache)) == shape
    assert cache.read_text() == "".join(lines)
    s.close()
