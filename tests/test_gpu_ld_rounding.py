"""The LD of the lane kernels is rounded once from one checkpoint to the next.

ld += dt/2 (g_0 + 2 (g_1 + ... ) + g_K) over the K steps of a checkpoint
interval: the integrands g come from the states at every step (the state does
not depend on the checkpoints), summed here in extended precision.  Late in a
run the interval's own error (the roots' 1e-14 of a 2,000th of the LD at
K = 10) is below a tenth of the LD's last place, so the rounding of the
update, half a place, leaves the difference below 0.6 places; a second
rounding reaches 1.
"""
import numpy as np
import pytest

import seeded_inputs as S

pytestmark = pytest.mark.gpu

S0, CHECKED = 20000, 100  # steps before, and steps that are looked at


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available()
    import paper_2507_00622_amd as P
    from oracle import oracle as O
    return torch, P, O


# one lane, two lanes, a row per orbit
@pytest.mark.parametrize("form", ["ld", "sali", "spectrum"])
def test_ld_rounds_once_per_checkpoint(env, form):
    torch, P, O = env
    print(f"case: LD rounding, {form}", flush=True)
    ind = O.IND_LD | {"ld": 0, "sali": O.IND_SALI, "spectrum": O.IND_SALI | O.IND_LYAP}[form]
    y, py = S.section_points(17, 300)
    x, m = O.hh_points(0.05, y, py)
    x = x[m == 1][:64]
    dt = 0.01
    hist = {}
    for K in (1, 10):
        with P.Ensemble(P.henon_heiles(), x, dt=dt, T=dt * (S0 + CHECKED), indicators=ind,
                        renorm_every=K, seed=4) as e:
            out = []
            for s in range(S0, S0 + CHECKED + 1, K):
                e.advance(s)
                r = e.results()
                out.append((r["x_final"], r["ld"]))
            hist[K] = out
    for a, b in zip(hist[1][::10], hist[10]):
        assert np.array_equal(a[0], b[0])
    X = np.array([a for a, _ in hist[1]]).astype(np.longdouble)
    q0, q1, p0, p1 = np.moveaxis(X, 2, 0)
    F0, F1 = q0 + 2 * q0 * q1, q1 + q0 * q0 - q1 * q1
    g = sum(np.sqrt(np.abs(v)) for v in (p0, p1, F0, F1))
    for K in (1, 10):
        ld = np.array([b for _, b in hist[K]])
        worst = 0.0
        for j in range(1, len(ld)):
            i = (j - 1) * K
            inc = (g[i] + g[i + K]) / 2 + g[i + 1:i + K].sum(0)
            err = np.abs(ld[j].astype(np.longdouble) - ld[j - 1] - np.longdouble(dt) * inc)
            worst = max(worst, float((err / np.spacing(ld[j])).max()))
        print(f"  K = {K}: {worst:.3f} places", flush=True)
        assert worst < 0.6
