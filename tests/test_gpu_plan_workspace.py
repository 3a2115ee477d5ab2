"""A captured plan outlives the other calls of its systems: none of the spectrum
calls moves a buffer that the plan's kernels use."""
import numpy as np
import pytest

from gpu_util import say, small_spec, gpu_system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_plan_runs_after_the_spectrum_calls(precision):
    import torch
    from paper_2205_06690_amd import bse, inputs
    spec = small_spec(n=16, n_occ=6, n_o=2, n_c=3, n_steps=20)
    sysd = inputs.make_system(spec)
    s = gpu_system(spec, sysd, bse.BSE_MIXED if precision == "mixed" else bse.BSE_FP64, max_batch=2)
    s.build_a(2, 1)      # few transitions: its own transforms need no more room than a batch of two
    pairs = np.array([[5, 5], [4, 5]], dtype=np.int32)
    out = torch.zeros((2, spec.ng), dtype=torch.float64, device="cuda")
    plan = bse.BatchPlan([s], [pairs], [out.data_ptr()])
    plan.run()
    torch.cuda.synchronize()
    ref = out.clone()
    bounds, wg = (-20.0, 60.0), np.array([0.2, 0.4])
    calls = [("apply_a_mixed", lambda: s.apply_a_mixed(np.ones((2, 2, spec.ng)))),
             ("chebyshev_mixed", lambda: s.chebyshev_mixed(4, bounds, wg, 1.0)),
             ("exciton_states_mixed", lambda: s.exciton_states_mixed(4, bounds, wg, 1.0, n_a=1)),
             ("chebyshev_spectrum", lambda: s.chebyshev_spectrum(64, wg, 0.1)),
             ("exciton_states", lambda: s.exciton_states(64, wg, 0.1)),
             ("spectrum", lambda: s.spectrum(1))]
    for name, call in calls:
        call()
        out.zero_()
        torch.cuda.synchronize()
        plan.run()          # refused (BSE_ERR_STATE) if a buffer has moved
        torch.cuda.synchronize()
        say(f"{precision}: plan after {name}")
        assert torch.equal(out, ref)
    plan.close()
    s.close()
