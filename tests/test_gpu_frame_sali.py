"""SALI, GALI, early exit, escape and resume of N = 8 chains whose SALI/GALI set
is kept in the frame of the full Lyapunov set (at most 16 steps per
checkpoint), against the same chains with the set integrated (more steps).

The state does not depend on the checkpoints and has the same bits.  Either form
rounds a unit vector's 16 components once per step, which leaves SALI an absolute
error of a few 1e-16 per step, and what it was once rounded at it carries when
it grows again: relative to SALI, steps * 16 * 2^-52 over its smallest value so
far.
"""
import numpy as np
import pytest

import seeded_inputs as S

pytestmark = pytest.mark.gpu
N, DT = 8, 0.02
EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available()
    import paper_2507_00622_amd as P
    from oracle import oracle as O
    return torch, P, O


def chains(O, n, scale):
    return scale * O.fput_ic(O.fput(N), S.fput_mode_draws(5, n))


def full(O):
    return O.IND_SALI | O.IND_GALI | O.IND_LYAP | O.IND_LD | O.IND_ENERGY


# 93 orbits: the last wavefront holds five of eight; amplitude 4: chaotic, SALI
# crosses 1e-8 and comes back, amplitude 1: mostly regular
@pytest.mark.parametrize("scale,T,coarse", [(4.0, 320.0, 1), (1.0, 64.0, 1), (2.0, 320.0, 10)])
def test_sali_below_1e8_and_back(env, scale, T, coarse):
    torch, P, O = env
    print(f"case: SALI in the frame, amplitude {scale}, dt {DT * coarse}", flush=True)
    n, dt = 93, DT * coarse
    steps = int(round(T / dt))
    x0, w0 = chains(O, n, scale), S.deviation_vectors(6, n, 4, 2 * N)
    kw = dict(dt=dt, T=T, indicators=full(O), gali_kmax=4, n_lyap=2 * N, w0=w0)
    worst, low, back = 0.0, 9.0, 0
    with P.Ensemble(P.fput(N), x0, renorm_every=16, **kw) as a, \
            P.Ensemble(P.fput(N), x0, renorm_every=32, **kw) as b:
        smallest = np.full(n, 2.0)
        for s in range(32, steps + 1, 32):
            a.advance(s)
            b.advance(s)
            ra, rb = a.results(), b.results()
            # (a coarse step makes some chains blow up: the forms stop them at
            # their own checkpoints)
            fin = (ra["status"] == 0) & (rb["status"] == 0)
            assert np.array_equal(ra["status"], rb["status"]) and fin.sum() > n // 2
            assert np.array_equal(ra["x_final"][fin], rb["x_final"][fin])
            sa, sb = ra["sali_final"], rb["sali_final"]
            smallest = np.minimum(smallest, ra["sali_min"])
            tol = s * 16 * EPS / smallest
            ok = fin & (tol < 0.1)
            assert (np.abs(sa / sb - 1)[ok] < tol[ok]).all(), s
            assert (np.abs(ra["gali"] - rb["gali"])[fin] < s * 16 * EPS).all(), s
            worst, low = max(worst, np.abs(sa / sb - 1)[ok].max()), min(low, np.nanmin(smallest))
            back = max(back, int(np.sum(ok & (smallest < 1e-8) & (sa > 1e-7))))
        assert np.abs(ra["lyap"] - rb["lyap"])[fin].max() < 1e-10
        assert np.abs(ra["ln_growth"] - rb["ln_growth"])[fin].max() < 1e-8
    print(f"  largest relative difference {worst:.1e}, smallest SALI {low:.1e}, back {back}",
          flush=True)
    if scale == 4.0:
        assert low < 1e-8


def test_early_exit_and_threshold(env):
    torch, P, O = env
    print("case: early exit in the frame", flush=True)
    n = 93
    x0, w0 = chains(O, n, 4.0), S.deviation_vectors(6, n, 2, 2 * N)
    kw = dict(dt=DT, T=160.0, indicators=full(O), gali_kmax=2, n_lyap=2 * N, renorm_every=10,
              w0=w0, sali_threshold=1e-3)
    run = P.integrate_ensemble(P.fput(N), x0, **kw)
    ee = P.integrate_ensemble(P.fput(N), x0, early_exit=True, **kw)
    hit = np.isfinite(run["t_chaos"])
    assert 10 < hit.sum() < n - 10
    assert np.array_equal(hit, run["sali_min"] < 1e-3)
    assert np.array_equal(ee["t_chaos"], run["t_chaos"], equal_nan=True)
    assert np.array_equal(ee["status"], np.where(hit, O.ST_EXITED, O.ST_OK))
    assert np.array_equal(ee["t_end"], np.where(hit, run["t_chaos"], 160.0))
    # an orbit that exits leaves its row's other orbit alone
    for k in run:
        if k not in ("status", "t_end"):
            assert np.array_equal(ee[k][~hit], run[k][~hit], equal_nan=True), k
    # against the oracle while the trajectories agree
    o = O.integrate(O.fput(N), x0, O.Run(dt=DT, T=20.0, indicators=full(O), gali_kmax=2,
                                         n_lyap=2 * N, sali_threshold=0.1), w0=w0, threads=8)
    g = P.integrate_ensemble(P.fput(N), x0, **dict(kw, T=20.0, sali_threshold=0.1))
    assert np.array_equal(g["label"], o["label"])
    assert np.array_equal(g["t_chaos"], o["t_chaos"], equal_nan=True)
    assert np.isfinite(g["t_chaos"]).sum() > 10
    assert np.abs(np.log10(g["sali_min"] / o["sali_min"])).max() < 1e-6


def test_resume_and_escape(env):
    torch, P, O = env
    print("case: resume and escape in the frame", flush=True)
    n = 93
    x0, w0 = chains(O, n, 4.0), S.deviation_vectors(8, n, 8, 2 * N)
    x0[17, 3] = np.nan
    r2 = float(np.quantile(np.sum(x0[:, :N] ** 2, axis=1)[np.arange(n) != 17], 0.9))
    mask = np.ones(n, np.uint8)
    mask[40] = 0
    kw = dict(dt=DT, T=10.0, indicators=full(O), gali_kmax=8, n_lyap=2 * N, renorm_every=16, w0=w0,
              mask=mask, escape_r2=r2)
    ref = P.integrate_ensemble(P.fput(N), x0, **kw)
    assert (ref["status"] == O.ST_ESCAPED).sum() > 5 and (ref["status"] == O.ST_OK).sum() > 5
    with P.Ensemble(P.fput(N), x0, steps_per_launch=48, **kw) as e:
        e.advance(160)
        keep = (np.arange(n) % 3 != 1).astype(np.uint8)
        with e.subset(keep) as s:
            s.advance()
            sub = s.results()
        e.advance(400)
        e.advance(500)
        r = e.results()
    kept = (keep == 1) & (mask == 1)
    for k in ref:
        assert np.array_equal(ref[k], r[k], equal_nan=True), k
        assert np.array_equal(ref[k][kept], sub[k], equal_nan=True), k
