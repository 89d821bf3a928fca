"""The SALI/GALI set kept as coordinates in the frame of the full Lyapunov
set, against the same set integrated.

A run with all 2N Lyapunov vectors and at most 16 steps per checkpoint keeps
the set in the frame; the same run with 2N - 1 of them integrates it.  The
state, the energy error and the exponents do not depend on the set and
agree bit for bit; the set's growth and GALI differ by rounding only:
each checkpoint adds a few 1e-16 times the stretching of its interval
(below 10 here), so 30 checkpoints stay below 1e-12.
"""
import numpy as np
import pytest

import seeded_inputs as S

pytestmark = pytest.mark.gpu
N_ORB = 70  # eight orbits to a wavefront, the last one not full


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available()
    import paper_2507_00622_amd as P
    from oracle import oracle as O
    return torch, P, O


@pytest.mark.parametrize("K", [1, 10, 16])
def test_frame_against_integrated_set(env, K):
    torch, P, O = env
    print(f"case: frame FPU N=8 K={K}", flush=True)
    N, dt = 8, 0.02
    x0 = O.fput_ic(O.fput(N), S.fput_mode_draws(5, N_ORB))
    for m in (2, 5, 8):
        # SALI needs n_lyap a multiple of 16 here, so GALI alone
        kw = dict(dt=dt, T=dt * (30 * K - (K > 1)),
                  indicators=O.IND_GALI | O.IND_LYAP | O.IND_ENERGY, gali_kmax=m, renorm_every=K)
        w0 = S.deviation_vectors(6, N_ORB, m, 2 * N)
        t = lambda a: torch.as_tensor(a, device="cuda:0")
        a = P.integrate_ensemble(P.fput(N), t(x0), w0=t(w0), n_lyap=2 * N, **kw)
        b = P.integrate_ensemble(P.fput(N), t(x0), w0=t(w0), n_lyap=2 * N - 1, **kw)
        torch.cuda.synchronize()
        a, b = ({k: v.cpu().numpy() for k, v in r.items()} for r in (a, b))
        for k in ("x_final", "t_end", "status", "energy_err"):
            assert np.array_equal(a[k], b[k]), k
        assert np.abs(a["lyap"][:, :-1] - b["lyap"]).max() < 1e-12
        assert np.abs(a["ln_growth"] - b["ln_growth"]).max() < 1e-12
        assert np.abs(a["gali"] - b["gali"]).max() < 1e-12
