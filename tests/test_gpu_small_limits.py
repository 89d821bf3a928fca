"""The one-lane and one-row kernels, which ensembles beyond the size limits of
the small-ensemble kernels run on.

The small-ensemble kernels take the operations of the general ones in their
order, so the same orbits give the same bits on either side of a limit, and
an ensemble may cross one through a subset.  Every large ensemble here holds
more active orbits (masked ones do not count) than the limit of its form.
The block size and launch splits, which only the general kernels take
up, change nothing.
"""
import numpy as np
import pytest

import seeded_inputs as S

pytestmark = pytest.mark.gpu

# most active orbits of the small-ensemble kernels
PAIR, QUAD, QUAD_DP, ROW, ROW_RK, SPLIT = 32768, 32768, 16384, 4096, 8192, 2048
N_SMALL = 77  # an odd number of orbits in the last wavefront of every form


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available()
    import paper_2507_00622_amd as P
    from oracle import oracle as O
    return torch, P, O


def states(P, O, name, n):
    if name == "hh":  # E = 0.2: some orbits escape
        rng = np.random.default_rng(8)
        x, m = O.hh_points(0.2, rng.uniform(-0.3, 0.6, 2 * n), rng.uniform(-0.4, 0.4, 2 * n))
        return P.henon_heiles(), x[m == 1][:n]
    if name.startswith("quartic"):
        N = int(name[-1])
        return P.quartic(N, 0.1), O.quartic_ic(O.quartic(N, 0.1), S.quartic_draws(9, n, N))
    if name.startswith("harmonic"):
        N = int(name[-1])
        return P.harmonic([1.0, 1.3, 0.7][:N]), np.random.default_rng(3).normal(size=(n, 2 * N))
    if name.startswith("fput"):
        N = int(name[4:])
        return P.fput(N), O.fput_ic(O.fput(N), S.fput_mode_draws(40 + N, n))
    return P.double_pendulum(0.7, 2.5), S.dp_states(4, n, np.pi, 1.0)


def tensor(env, a):
    return env[0].as_tensor(np.ascontiguousarray(a), device="cuda:0")


def inputs(env, name, m, limit):
    """n orbits with a masked and a non-finite one, and repetitions of them
    with more than `limit` active orbits."""
    torch, P, O = env
    sys_, x0 = states(P, O, name, N_SMALL)
    n = len(x0)
    w0 = S.deviation_vectors(31, n, m, x0.shape[1])
    mask = np.ones(n, np.uint8)
    mask[n // 3] = 0
    x0 = x0.copy()
    x0[n // 2, 0] = np.nan
    rep = limit // (n - 1) + 1
    assert n - 1 <= limit < rep * int(mask.sum())
    return sys_, (x0, mask, w0), (np.tile(x0, (rep, 1)), np.tile(mask, rep),
                                  np.tile(w0, (rep, 1, 1)))


def same(env, a, b, what=""):
    for k in a:
        x, y = a[k].cpu().numpy(), b[k].cpu().numpy()
        assert np.array_equal(x, y, equal_nan=True), (what, k)


def compare(env, name, m, limit, **kw):
    """The small ensemble against the first and last copy in the large one,
    and against a subset of the large one taken half way."""
    torch, P, O = env
    sys_, small, big = inputs(env, name, m, limit)
    n = len(small[0])
    t = [tensor(env, a) for a in small]
    T = [tensor(env, a) for a in big]
    a = P.integrate_ensemble(sys_, t[0], mask=t[1], w0=t[2], **kw)
    K = kw["renorm_every"]
    half = int(round(kw["T"] / kw["dt"])) // (2 * K) * K
    with P.Ensemble(sys_, T[0], mask=T[1], w0=T[2], **kw) as e:
        e.advance(half)
        keep = torch.zeros(len(T[1]), dtype=torch.uint8, device=T[1].device)
        keep[:n] = 1
        with e.subset(keep) as s:
            s.advance()
            c = s.results()
        e.advance()
        b = e.results()
    same(env, a, {k: v[:n] for k, v in b.items()}, "first copy")
    same(env, a, {k: v[-n:] for k, v in b.items()}, "last copy")
    act = t[1] == 1
    same(env, {k: v[act] for k, v in a.items()}, c, "subset")
    assert a["status"][n // 2].item() == O.ST_NONFINITE
    if name == "hh" and kw.get("early_exit"):
        assert {O.ST_ESCAPED, O.ST_EXITED} <= set(a["status"].tolist())


def pair_forms(O, name):
    esc = 4.0 if name == "hh" else 0.0
    yield dict(indicators=O.IND_SALI | O.IND_LD | O.IND_ENERGY, renorm_every=7, escape_r2=esc,
               early_exit=True, sali_threshold=0.02)
    yield dict(indicators=O.IND_GALI, renorm_every=10, escape_r2=esc)
    yield dict(indicators=O.IND_SALI | O.IND_LD, renorm_every=1, escape_r2=esc)


LANE = ["hh", "quartic1", "quartic2", "quartic3", "harmonic1", "harmonic2", "harmonic3"]


@pytest.mark.parametrize("name", LANE)
def test_two_lanes_against_one(env, name):
    torch, P, O = env
    for kw in pair_forms(O, name):
        print(f"case: two lanes against one, {name} {kw}", flush=True)
        compare(env, name, 2, PAIR, dt=0.02, T=15.0, **kw)


@pytest.mark.parametrize("integ", ["dop853", "dop853_adaptive"])
@pytest.mark.parametrize("name", LANE + ["dp"])
def test_four_lanes_against_one(env, name, integ):
    torch, P, O = env
    for kw in pair_forms(O, name):
        print(f"case: four lanes against one, {name} {integ} {kw}", flush=True)
        compare(env, name, 2, QUAD_DP if name == "dp" else QUAD, dt=0.05, T=15.0,
                integrator=integ, **kw)


# the headline's set (SALI, GALI_2, four exponents: M = 6), sets without a
# Lyapunov part, and the largest of the three-dof systems (M = 12)
@pytest.mark.parametrize("integ", ["yoshida4", "dop853"])
@pytest.mark.parametrize("name,m,n_l", [("hh", 2, 4), ("hh", 4, 0), ("hh", 2, 1), ("dp", 2, 4),
                                        ("harmonic3", 2, 6), ("quartic3", 6, 6)])
def test_lane_per_vector_against_one(env, name, m, n_l, integ):
    torch, P, O = env
    if name == "dp" and integ == "yoshida4":
        pytest.skip("no Yoshida-4 for the double pendulum")
    print(f"case: a lane per vector against one lane, {name} {m}+{n_l} {integ}", flush=True)
    ind = O.IND_SALI | O.IND_GALI | O.IND_LD | O.IND_ENERGY | (O.IND_LYAP if n_l else 0)
    for K in (1, 5, 10):  # Yoshida-4 rows need K (N - 1) >= 5
        compare(env, name, m, ROW if integ == "yoshida4" else ROW_RK, dt=0.05, T=12.0,
                integrator=integ, indicators=ind, renorm_every=K, gali_kmax=m, n_lyap=n_l,
                escape_r2=4.0 if name == "hh" else 0.0)


@pytest.mark.parametrize("integ", ["yoshida4", "dop853", "dop853_adaptive"])
@pytest.mark.parametrize("N,m", [(2, 4), (8, 3), (11, 2), (16, 4)])
def test_row_per_vector_against_one(env, N, m, integ):
    torch, P, O = env
    print(f"case: a row per vector against one row, N={N} m={m} {integ}", flush=True)
    for ind, K in ((O.IND_GALI | O.IND_SALI | O.IND_LD | O.IND_ENERGY, 1), (O.IND_GALI, 7)):
        compare(env, f"fput{N}", m, SPLIT, dt=0.05, T=6.0, integrator=integ, indicators=ind,
                gali_kmax=m, renorm_every=K)


# ensembles beyond the limits: launch splits, resume and every block size
@pytest.mark.parametrize("name,integ,m,n_l,limit", [
    ("hh", "yoshida4", 2, 0, PAIR), ("hh", "yoshida4", 2, 4, ROW),
    ("quartic3", "yoshida4", 2, 6, ROW), ("hh", "dop853", 2, 0, QUAD),
    ("hh", "dop853", 2, 4, ROW_RK), ("quartic3", "dop853", 2, 0, QUAD),
    ("quartic3", "dop853", 3, 0, ROW_RK), ("dp", "dop853", 2, 4, ROW_RK),
    ("hh", "dop853_adaptive", 2, 0, QUAD), ("dp", "dop853_adaptive", 2, 0, QUAD_DP)])
def test_resume_and_block_sizes_beyond_limits(env, name, integ, m, n_l, limit):
    torch, P, O = env
    print(f"case: resume and blocks, {name} {integ} {m}+{n_l}", flush=True)
    sys_, _, big = inputs(env, name, m, limit)
    x0, mask, w0 = (tensor(env, a) for a in big)
    kw = dict(dt=0.02, T=3.0, integrator=integ, renorm_every=7, gali_kmax=m, n_lyap=n_l,
              indicators=O.IND_SALI | O.IND_GALI | O.IND_LD | O.IND_ENERGY
              | (O.IND_LYAP if n_l else 0))
    ref = P.integrate_ensemble(sys_, x0, mask=mask, w0=w0, **kw)
    with P.Ensemble(sys_, x0, mask=mask, w0=w0, steps_per_launch=14, **kw) as e:
        for s in (28, 77, 150):
            e.advance(s)
        same(env, ref, e.results(), "resume")
    for block in (64, 128, 256):
        b = P.integrate_ensemble(sys_, x0, mask=mask, w0=w0, block_size=block, **kw)
        same(env, ref, b, block)
