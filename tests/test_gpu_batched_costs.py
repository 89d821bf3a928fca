"""The autotuner's costs (GPU time per orbit-step) from ensembles that do not fill
the device: they serve calls of their kind only, and a later large
ensemble is timed for itself."""
import pytest

import seeded_inputs as S

pytestmark = pytest.mark.gpu


def test_small_ensembles_leave_no_cost_for_large_ones():
    import torch
    assert torch.cuda.is_available()
    import paper_2507_00622_amd as P
    from oracle import oracle as O
    ind = 9  # SALI, LD: no other batched test's

    def call(n):
        print(f"case: autotuned cost at {n} orbits", flush=True)
        y, py = S.section_points(21, 2 * n + 16)
        x, m = O.hh_points(0.125, y, py)
        _, s = P.integrate_batched([dict(sys=P.henon_heiles(), x0=x[m == 1][:n], dt=0.01, T=2.0)],
                                   indicators=ind, seed=3)
        print("  stats:", s, flush=True)
        return s

    small, again, large = call(100), call(300), call(400000)
    small2 = call(100)
    assert small["from_cache"] == 0 and again["from_cache"] == 1
    assert large["from_cache"] == 0
    # at most three times the full device's rate by the estimate, and the
    # probe's 400 steps carry the launch besides
    assert small["cost_ps"][0] < 8 * large["cost_ps"][0]
    assert small2["from_cache"] == 1 and small2["cost_ps"] == large["cost_ps"]
