"""GALI of more orbits than the rows of one pass: 65,536 blocks of 16 rows (2N of
9..16 and 17..32 components), the rows striding over the rest."""
import numpy as np
import pytest

import seeded_inputs as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,kmax", [(5, 2), (9, 3)])
def test_gali_rows_stride_over_orbits(N, kmax):
    import torch
    assert torch.cuda.is_available()
    import paper_2507_00622_amd as P
    from oracle import oracle as O
    m, n = 37, (1 << 20) + 37
    print(f"case: GALI of {n} orbits, N={N}", flush=True)
    x0 = O.fput_ic(O.fput(N), S.fput_mode_draws(60 + N, m))
    x0[5, 1] = np.nan
    w0 = S.deviation_vectors(61, m, kmax, 2 * N)
    idx = torch.arange(n, device="cuda:0") % m
    t = lambda a: torch.as_tensor(a, device="cuda:0")
    kw = dict(dt=0.05, T=0.1, indicators=O.IND_GALI, gali_kmax=kmax)
    few = P.integrate_ensemble(P.fput(N), t(x0), w0=t(w0), outputs=("gali",), **kw)["gali"]
    many = P.integrate_ensemble(P.fput(N), t(x0)[idx], w0=t(w0)[idx], outputs=("gali",), **kw)["gali"]
    assert torch.isnan(few[5]).all() and not torch.isnan(few[6]).any()
    assert torch.equal(many.nan_to_num(-1.0), few[idx].nan_to_num(-1.0))
