"""Performance cases of the library: what its users have it do, through the
Python binding, on device tensors.

listed() names the cases, draw(rng) gives more of the same ranges,
prepare(case, seed) makes what a program holds before the call, run(state) is
one pass through the public entry points, work(case) the bytes and flops that
the pass cannot do without, and exact(case, seed) the results in plain torch
in 64 bits.  Flop counts follow the method as stated (FMA = 2; square roots,
divisions and logarithms are not counted).
"""
import math

import numpy as np
import torch

import paper_2507_00622_amd as P
from paper_2507_00622_amd import chx

DEV = "cuda"
F64 = torch.float64
K = 10  # renormalisation cadence: the library's default
# the window of the Henon-Heiles section x = 0 used throughout
Y0, Y1, PY0, PY1 = -0.4, 0.7, -0.45, 0.45
SALI_LD = chx.IND_SALI | chx.IND_LD
SALI_E = chx.IND_SALI | chx.IND_ENERGY
GALI_E = chx.IND_GALI | chx.IND_ENERGY
FULL = chx.IND_SALI | chx.IND_GALI | chx.IND_LYAP | chx.IND_LD | chx.IND_ENERGY
# what one pass may cost at most (flops of the method): the largest listed case
MOST_FLOPS = 8.0e11
MOST_STEPS = 20000


def listed():
    return [
        # a first look at a section: a coarse grid, where launches and the
        # chain of one orbit's steps count
        dict(name="section_small", kind="section", ny=32, npy=32, E=0.125, ind="sali_ld",
             integrator="yoshida4", dt=0.01, T=200.0),
        # the headline: a fine grid at the escape energy, every indicator in
        # one pass (SALI, GALI_2, four exponents, LD, energy)
        dict(name="section_spectrum", kind="section", ny=1024, npy=1024, E=1.0 / 6.0, ind="full",
             integrator="yoshida4", dt=0.01, T=30.0),
        # the same indicators with the paper's eighth-order solver
        dict(name="section_dop853", kind="section", ny=512, npy=512, E=0.125, ind="full",
             integrator="dop853", dt=0.02, T=20.0),
        # the timing figure of Henon-Heiles: section points with the adaptive
        # solver, SALI and energy, an ensemble that leaves the chip part idle
        dict(name="points_adaptive", kind="points", n=4093, E=0.125, tol=1e-10, T=200.0),
        # the timing figure of the double pendulum: states from rest
        dict(name="dp_fixed", kind="dp", n=65536, integrator="dop853", T=10.0),
        # FPU chains, the full spectrum and GALI_2..N: the large-N workload
        dict(name="fput16_spectrum", kind="fput_spectrum", N=16, n=65536, T=10.0),
        # the same with eight masses and a ragged ensemble
        dict(name="fput8_spectrum", kind="fput_spectrum", N=8, n=40001, T=20.0),
        # the timing figure of the FPU chain: 1000 states, GALI_4 and energy,
        # any number of masses
        dict(name="fput_sweep", kind="fput_sweep", N=11, n=1000, integrator="dop853_adaptive",
             T=100.0),
        # chaos indicators from the LDs of neighbouring orbits, no tangents
        dict(name="ldn_section", kind="ldn", ny=1024, npy=1024, E=0.125, T=20.0),
        # a mixed ensemble in one persistent launch sequence, early exit
        dict(name="batched_mixed", kind="batched", n_hh=262144, n_quartic=65536, n_fput=16384,
             T=400.0),
        # an epoch of the gate's training at its default batch
        dict(name="gate_train", kind="gate_train", n=1 << 20, batch=4096, epochs=1),
        # the gate on every accessible point of the 2048 x 2048 section grid
        dict(name="gate_infer", kind="gate_infer", n=3405516),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _time(rng, case, step, lo, hi):
    """A final time in [lo, hi], a whole number of `step`, within MOST_FLOPS."""
    T = rng.uniform(lo, hi)
    one = work(dict(case, T=step))["flops"]
    return step * max(1, int(min(T, MOST_STEPS * case.get("dt", step)) / step
                             if one * (T / step) <= MOST_FLOPS else MOST_FLOPS / one))


def draw(rng):
    kind = rng.choice(["section", "section", "points", "dp", "fput_spectrum", "fput_sweep",
                       "ldn", "batched", "gate_train", "gate_infer"])
    if kind == "section":
        c = dict(kind=kind, ny=_log_int(rng, 12, 1024), npy=_log_int(rng, 12, 1024),
                 E=rng.choice([0.125, 1.0 / 6.0]), ind=rng.choice(["sali_ld", "full"]),
                 integrator=rng.choice(["yoshida4", "dop853"]))
        c["dt"] = 0.01 if c["integrator"] == "yoshida4" else 0.02
        c["T"] = _time(rng, c, 0.02, 5.0, 30.0)
    elif kind == "points":
        c = dict(kind=kind, n=_log_int(rng, 256, 200000), E=rng.choice([0.125, 1.0 / 6.0]),
                 tol=rng.choice([1e-9, 1e-10, 1e-11]))
        c["T"] = _time(rng, c, 1.0, 20.0, 60.0)
    elif kind == "dp":
        c = dict(kind=kind, n=_log_int(rng, 256, 65536),
                 integrator=rng.choice(["dop853", "dop853_adaptive"]))
        c["T"] = _time(rng, c, 1.0, 4.0, 10.0)
    elif kind == "fput_spectrum":
        c = dict(kind=kind, N=rng.choice([8, 16]), n=_log_int(rng, 500, 65536))
        c["T"] = _time(rng, c, 1.0, 5.0, 20.0)
    elif kind == "fput_sweep":
        c = dict(kind=kind, N=rng.randint(2, 16), n=_log_int(rng, 250, 4000),
                 integrator=rng.choice(["dop853_adaptive", "yoshida4"]))
        c["T"] = _time(rng, c, 1.0, 20.0, 40.0)
    elif kind == "ldn":
        c = dict(kind=kind, ny=_log_int(rng, 24, 1024), npy=_log_int(rng, 24, 1024),
                 E=rng.choice([0.125, 1.0 / 6.0]))
        c["T"] = _time(rng, c, 1.0, 5.0, 20.0)
    elif kind == "batched":
        c = dict(kind=kind, n_hh=_log_int(rng, 4096, 262144), n_quartic=_log_int(rng, 1024, 65536),
                 n_fput=_log_int(rng, 256, 16384))
        c["T"] = _time(rng, c, 1.0, 100.0, 400.0)
    elif kind == "gate_train":
        c = dict(kind=kind, n=_log_int(rng, 20000, 1 << 20),
                 batch=rng.choice([1024, 2048, 4096, 8192]), epochs=1)
    else:
        c = dict(kind=kind, n=_log_int(rng, 100, 3405516))
    return c


# --- inputs ------------------------------------------------------------------------

def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * int(seed) + stream)
    return g


def _section(case, seed):
    """The section grid of the case: its window moved a little by the seed,
    as a user does who zooms or pans; inaccessible points masked."""
    u = torch.rand(2, generator=_gen(seed, 1), device=DEV, dtype=F64) * 1e-3
    y = torch.linspace(Y0, Y1, case["ny"], device=DEV, dtype=F64) + u[0]
    py = torch.linspace(PY0, PY1, case["npy"], device=DEV, dtype=F64) + u[1]
    y, py = y.repeat(case["npy"]), py.repeat_interleave(case["ny"])
    r = 2.0 * case["E"] - py * py - y * y + (2.0 / 3.0) * y ** 3
    ok = r >= 0.0
    x = torch.stack([torch.zeros_like(y), y, torch.where(ok, r, 0.0).sqrt(), py], 1)
    return x.contiguous(), ok.to(torch.uint8)


def _points(n, E, seed, stream=2):
    """n accessible points of the section, uniform in the window."""
    u = torch.rand(2 * n + 64, 2, generator=_gen(seed, stream), device=DEV, dtype=F64)
    y, py = Y0 + (Y1 - Y0) * u[:, 0], PY0 + (PY1 - PY0) * u[:, 1]
    r = 2.0 * E - py * py - y * y + (2.0 / 3.0) * y ** 3
    ok = (r >= 0.0).nonzero()[:n, 0]
    y, py, r = y[ok], py[ok], r[ok]
    return torch.stack([torch.zeros_like(y), y, r.sqrt(), py], 1).contiguous()


def _normals(shape, seed, stream):
    return torch.randn(shape, generator=_gen(seed, stream), device=DEV, dtype=F64)


def _fput_states(N, n, seed, stream=4):
    """The energy (0.1 to 10, quadratic part) in the two lowest normal modes."""
    u = torch.rand(n, 5, generator=_gen(seed, stream), device=DEV, dtype=F64)
    i = torch.arange(1, N + 1, device=DEV, dtype=F64)
    q, p = 0.0, 0.0
    for k in (1, 2):
        om = 2.0 * math.sin(k * math.pi / (2 * (N + 1)))
        ph = 2.0 * math.pi * u[:, k + 2]
        s = math.sqrt(2.0 / (N + 1)) * torch.sin(i * (k * math.pi / (N + 1)))
        q = q + (u[:, k] * torch.cos(ph) / om)[:, None] * s
        p = p + (u[:, k] * torch.sin(ph))[:, None] * s
    h2 = 0.5 * (u[:, 1] ** 2 + u[:, 2] ** 2)
    f = torch.sqrt((0.1 + 9.9 * u[:, 0]) / h2.clamp_min(1e-3))[:, None]
    return torch.cat([q * f, p * f], 1).contiguous()


def _quartic_states(n, seed, stream=5):
    """H = 1 of the three coupled quartic oscillators (eps = 0.1)."""
    d = _normals((n, 6), seed, stream)
    f = torch.rand(n, generator=_gen(seed, stream + 20), device=DEV, dtype=F64)
    q, p = d[:, :3], d[:, 3:]
    q2 = q * q
    v = 0.25 * (q2 * q2).sum(1) + 0.1 * (q2[:, 0] * q2[:, 1] + q2[:, 0] * q2[:, 2]
                                         + q2[:, 1] * q2[:, 2])
    q = q * (f / v)[:, None] ** 0.25
    p = p * torch.sqrt(2.0 * (1.0 - f) / (p * p).sum(1))[:, None]
    return torch.cat([q, p], 1).contiguous()


def _dp_states(n, seed):
    """States from rest, angles uniform on the torus."""
    u = torch.rand(n, 2, generator=_gen(seed, 6), device=DEV, dtype=F64)
    return torch.cat([(2.0 * u - 1.0) * math.pi, torch.zeros_like(u)], 1).contiguous()


def _gate_rows(n, seed):
    """Feature rows shaped like those of the section at t = 200 (y, p_y, p_x,
    LD/t, two growth rates) and labels that follow the growth rates, the
    overlap of the two classes included."""
    x = _points(n, 0.125, seed, 7)
    z = _normals((n, 4), seed, 8).float()
    lab = torch.rand(n, generator=_gen(seed, 9), device=DEV) < 0.58
    rate = torch.where(lab, 0.045 + 0.012 * z[:, 0], 0.022 + 0.006 * z[:, 0])
    f = torch.stack([x[:, 1].float(), x[:, 3].float(), x[:, 2].float(),
                     1.75 + 0.06 * z[:, 1] + 0.05 * lab, rate + 0.003 * z[:, 2],
                     rate + 0.003 * z[:, 3]], 1)
    return f.contiguous(), lab.to(torch.int8)


def _gate_params(seed):
    """He-normal weights, zero biases, in the library's flat layout."""
    g = torch.Generator()
    g.manual_seed(77 + int(seed))
    p = np.zeros(chx.GATE_NPARAM, np.float32)
    w1 = p[:4096].reshape(16, 256)
    w2 = p[4352:69888].reshape(256, 256)
    w3 = p[70144:74240].reshape(256, 16)
    w1[:6] = torch.randn(6, 256, generator=g).numpy() * math.sqrt(2.0 / 6.0)
    w2[:] = torch.randn(256, 256, generator=g).numpy() * math.sqrt(2.0 / 256.0)
    w3[:, :2] = torch.randn(256, 2, generator=g).numpy() * math.sqrt(2.0 / 256.0)
    return p


GATE_MEAN = np.array([0.15, 0.0, 0.3, 1.78, 0.035, 0.035], np.float32)
GATE_ISTD = np.array([3.7, 4.4, 6.5, 15.0, 65.0, 65.0], np.float32)


def prepare(case, seed):
    k = case["kind"]
    s = dict(case=case)
    if k == "section":
        s["x0"], s["mask"] = _section(case, seed)
        s["w0"] = _normals((case["ny"] * case["npy"], 2, 4), seed, 3)
    elif k == "points":
        s["x0"] = _points(case["n"], case["E"], seed)
        s["w0"] = _normals((case["n"], 2, 4), seed, 3)
    elif k == "dp":
        s["x0"] = _dp_states(case["n"], seed)
        s["w0"] = _normals((case["n"], 2, 4), seed, 3)
    elif k in ("fput_spectrum", "fput_sweep"):
        N = case["N"]
        s["x0"] = _fput_states(N, case["n"], seed)
        s["w0"] = _normals((case["n"], N if k == "fput_spectrum" else 4, 2 * N), seed, 3)
    elif k == "ldn":
        s["x0"], s["mask"] = _section(case, seed)
    elif k == "batched":
        T = case["T"]
        s["items"] = [dict(sys=P.henon_heiles(), x0=_points(case["n_hh"], 0.125, seed),
                           dt=0.01, T=T),
                      dict(sys=P.quartic(3, 0.1), x0=_quartic_states(case["n_quartic"], seed),
                           dt=0.01, T=T),
                      dict(sys=P.fput(16), x0=_fput_states(16, case["n_fput"], seed),
                           dt=0.02, T=T)]
        s["seed"] = int(seed)
    elif k == "gate_train":
        s["feat"], s["lab"] = _gate_rows(case["n"], seed)
        s["gate"] = P.Gate(seed)
        s["gate"].set(params=_gate_params(seed))
        s["seed"] = int(seed)
    else:
        s["feat"], _ = _gate_rows(case["n"], seed)
        s["gate"] = P.Gate(seed)
        s["gate"].set(_gate_params(seed), GATE_MEAN, GATE_ISTD)
    return s


# --- one pass -----------------------------------------------------------------------

def run(s):
    c = s["case"]
    k = c["kind"]
    if k == "section":
        return P.integrate_ensemble(P.henon_heiles(), s["x0"], mask=s["mask"], w0=s["w0"],
                                    dt=c["dt"], T=c["T"], integrator=c["integrator"],
                                    indicators=FULL if c["ind"] == "full" else SALI_LD)
    if k == "points":
        return P.integrate_ensemble(P.henon_heiles(), s["x0"], w0=s["w0"], dt=0.1, T=c["T"],
                                    integrator="dop853_adaptive", rtol=c["tol"], atol=c["tol"],
                                    indicators=SALI_E)
    if k == "dp":
        o = (dict(dt=0.02, integrator="dop853") if c["integrator"] == "dop853" else
             dict(dt=0.1, integrator="dop853_adaptive", rtol=1e-11, atol=1e-11))
        return P.integrate_ensemble(P.double_pendulum(), s["x0"], w0=s["w0"], T=c["T"],
                                    indicators=SALI_E, **o)
    if k == "fput_spectrum":
        return P.integrate_ensemble(P.fput(c["N"]), s["x0"], w0=s["w0"], dt=0.02, T=c["T"],
                                    indicators=chx.IND_GALI | chx.IND_LYAP | chx.IND_ENERGY,
                                    gali_kmax=c["N"])
    if k == "fput_sweep":
        o = (dict(dt=0.0025) if c["integrator"] == "yoshida4" else
             dict(dt=0.1, integrator="dop853_adaptive", rtol=1e-11, atol=1e-11))
        return P.integrate_ensemble(P.fput(c["N"]), s["x0"], w0=s["w0"], T=c["T"],
                                    indicators=GALI_E, gali_kmax=4, **o)
    if k == "ldn":
        return P.ld_indicators(P.henon_heiles(), s["x0"], 1e-3, dirs=[1, 3], mask=s["mask"],
                               dt=0.01, T=c["T"])
    if k == "batched":
        outs, _ = P.integrate_batched(s["items"], indicators=SALI_E, early_exit=True,
                                      seed=s["seed"])
        return outs
    if k == "gate_train":
        loss = s["gate"].train(s["feat"], s["lab"], epochs=c["epochs"], batch=c["batch"],
                               seed=s["seed"], reset_stats=True)
        p, m, v = s["gate"].get()
        return dict(loss=loss, params=p, mean=m, istd=v)
    p, conf = s["gate"].infer(s["feat"])
    return dict(p=p, confidence=conf)


# --- what a pass cannot do without ---------------------------------------------------

ACCESS = {0.125: 0.8115, 1.0 / 6.0: 0.9466}  # accessible share of the window


def _hh_step(m_s, n_l, ld, sali=True):
    """Yoshida-4 Henon-Heiles: the state 70, 44 per vector, LD 6; per
    checkpoint the SALI pair 44 and the Gram-Schmidt of n_l vectors."""
    mgs = sum(16 * j + 7 + 4 for j in range(n_l))
    return 70 + 44 * (m_s + n_l) + (6 if ld else 0) + ((44 if sali else 0) + mgs) / K


def _fput_step(N, n_l, m_g):
    """Yoshida-4 FPU chain: three springs, forces and kicks; 3 kicks of 6N
    and 3 drifts of 2N per vector; Gram-Schmidt and norms per checkpoint."""
    D = 2 * N
    mgs = sum(4 * D * j + 3 * D for j in range(n_l))
    return 3 * 14 * (N + 1) + 14 * N + 24 * N * (n_l + m_g) + (mgs + 3 * D * m_g) / K


def _dop_step(N, D, force, hess, m, adaptive):
    """DOP853: 12 stages, 50 non-zero a_ij and 8 weights (2 flops each) per
    component; force and Hessian-vector product per stage."""
    sums = (50 + 8 + (12 if adaptive else 0)) * 2 + 12
    return 12 * force + D * sums + m * (12 * hess + D * sums)


def work(case):
    k = case["kind"]
    if k in ("section", "ldn"):
        n_all = case["ny"] * case["npy"]
        n = ACCESS[case["E"]] * n_all
    if k == "section":
        full = case["ind"] == "full"
        m_s, n_l = 2, 4 if full else 0
        if case["integrator"] == "yoshida4":
            f = _hh_step(m_s, n_l, True)
        else:
            f = _dop_step(2, 4, 8, 10, m_s + n_l, False)
        steps = case["T"] / case["dt"]
        out = 32 + 8 + 4 + 1 + 24 + 16 + 8 + ((8 + 32 + 8) if full else 0)
        return dict(bytes=n_all * (32 + 1 + 64 + out), flops=n * steps * f)
    if k == "points":
        steps = case["T"] * 5.0 * (1e-10 / case["tol"]) ** 0.125
        return dict(bytes=case["n"] * (32 + 64 + 32 + 8 + 5 + 24 + 8 + 16 + 32),
                    flops=case["n"] * steps * _dop_step(2, 4, 8, 10, 2, True))
    if k == "dp":
        fixed = case["integrator"] == "dop853"
        steps = case["T"] * (50.0 if fixed else 20.0)
        return dict(bytes=case["n"] * (32 + 64 + 32 + 8 + 5 + 24 + 8 + 16 + 32),
                    flops=case["n"] * steps * _dop_step(2, 4, 177, 77, 2, not fixed))
    if k == "fput_spectrum":
        N, n = case["N"], case["n"]
        out = 16 * N + 8 + 4 + 8 * (N - 1) + 16 * N + 8 + 8 * N
        return dict(bytes=n * (16 * N + 16 * N * N + out),
                    flops=n * (case["T"] / 0.02) * _fput_step(N, 2 * N, N))
    if k == "fput_sweep":
        N, n = case["N"], case["n"]
        if case["integrator"] == "yoshida4":
            f, steps = _fput_step(N, 0, 4), case["T"] / 0.0025
        else:
            f, steps = _dop_step(N, 2 * N, 10 * (N + 1), 6 * N, 4, True), case["T"] * 9.0
        return dict(bytes=n * (16 * N + 64 * N + 16 * N + 12 + 24 + 8 + 32 + 32), flops=n * steps * f)
    if k == "ldn":
        # ten member orbits: five points, forward and backward
        return dict(bytes=n_all * (33 + 36), flops=10 * n * (case["T"] / 0.01) * 76)
    if k == "batched":
        st = case["T"] / 0.01
        f = (case["n_hh"] * st * _hh_step(2, 0, False) + case["n_quartic"] * st * 334
             + case["n_fput"] * (st / 2) * _fput_step(16, 0, 2))
        b = case["n_hh"] * 105 + case["n_quartic"] * 137 + case["n_fput"] * 553
        return dict(bytes=b, flops=f)
    if k == "gate_train":
        # 6-256-256-2 forward, three weight gradients, two activation gradients
        row = 2 * (3 * (6 * 256 + 256 * 256 + 256 * 2) - 6 * 256)
        n, e = case["n"], case["epochs"]
        return dict(bytes=n * 25 * (e + 1) + 3 * 4 * chx.GATE_NPARAM, flops=n * e * row)
    return dict(bytes=case["n"] * (24 + 8) + 2 * chx.GATE_NPARAM,
                flops=case["n"] * 2 * (6 * 256 + 256 * 256 + 256 * 2))


# --- the results in 64 bits, plain torch -----------------------------------------------
#
# Points are kept component-major: q, p of shape [N, n], vectors [m, N, n].

class _HH:
    N = 2

    def force(self, q):
        x, y = q
        return torch.stack([x + 2 * x * y, y - y * y + x * x])

    def hess(self, q, d):
        x, y = q
        return torch.stack([(1 + 2 * y) * d[:, 0] + 2 * x * d[:, 1],
                            2 * x * d[:, 0] + (1 - 2 * y) * d[:, 1]], 1)


class _FPUT:
    def __init__(self, N):
        self.N = N

    @staticmethod
    def _ext(q, dim):
        z = torch.zeros_like(q.narrow(dim, 0, 1))
        return torch.cat([q, z], dim) - torch.cat([z, q], dim)

    def force(self, q):
        d = self._ext(q, 0)
        f = d + d ** 3
        return f[:-1] - f[1:]

    def hess(self, q, v):
        kap = 1 + 3 * self._ext(q, 0) ** 2
        t = kap * self._ext(v, 1)
        return t[:, :-1] - t[:, 1:]


class _Separable:
    """The extended field of a separable system: x = (q, p), w [m, 2N, n]."""

    def __init__(self, sys):
        self.sys, self.N = sys, sys.N

    def field(self, x, w):
        N = self.N
        f = torch.cat([x[N:], -self.sys.force(x[:N])])
        return f, torch.cat([w[:, N:], -self.sys.hess(x[:N], w[:, :N])], 1)


class _DP:
    """The double pendulum (length and mass ratio 1); its derivative along a
    vector by a complex step."""

    @staticmethod
    def _f(x):
        t1, t2, p1, p2 = x
        s, c = torch.sin(t1 - t2), torch.cos(t1 - t2)
        D = 2.0 - c * c
        Q = p1 * p1 - 2.0 * c * p1 * p2 + 2.0 * p2 * p2
        g = s * (c * Q - p1 * p2 * D) / (D * D)
        return torch.stack([(p1 - c * p2) / D, (2.0 * p2 - c * p1) / D,
                            g - 2.0 * torch.sin(t1), -g - torch.sin(t2)])

    def field(self, x, w):
        h = 1e-40
        z = torch.complex(x.unsqueeze(1).expand(-1, w.shape[0], -1),
                          h * w.transpose(0, 1)).contiguous()
        return self._f(x), (self._f(z).imag / h).transpose(0, 1)


def _a(v):
    t = np.zeros((12, 12))
    for i, row in enumerate(v):
        for j, x in row.items():
            t[i, j] = x
    return t


# the published coefficients of DOP853 (Hairer, Norsett, Wanner, Solving ODEs I)
A = _a([
    {}, {0: 5.26001519587677318785587544488e-2},
    {0: 1.97250569845378994544595329183e-2, 1: 5.91751709536136983633785987549e-2},
    {0: 2.95875854768068491816892993775e-2, 2: 8.87627564304205475450678981324e-2},
    {0: 2.41365134159266685502369798665e-1, 2: -8.84549479328286085344864962717e-1,
     3: 9.24834003261792003115737966543e-1},
    {0: 3.7037037037037037037037037037e-2, 3: 1.70828608729473871279604482173e-1,
     4: 1.25467687566822425016691814123e-1},
    {0: 3.7109375e-2, 3: 1.70252211019544039314978060272e-1,
     4: 6.02165389804559606850219397283e-2, 5: -1.7578125e-2},
    {0: 3.70920001185047927108779319836e-2, 3: 1.70383925712239993810214054705e-1,
     4: 1.07262030446373284651809199168e-1, 5: -1.53194377486244017527936158236e-2,
     6: 8.27378916381402288758473766002e-3},
    {0: 6.24110958716075717114429577812e-1, 3: -3.36089262944694129406857109825,
     4: -8.68219346841726006818189891453e-1, 5: 2.75920996994467083049415600797e1,
     6: 2.01540675504778934086186788979e1, 7: -4.34898841810699588477366255144e1},
    {0: 4.77662536438264365890433908527e-1, 3: -2.48811461997166764192642586468,
     4: -5.90290826836842996371446475743e-1, 5: 2.12300514481811942347288949897e1,
     6: 1.52792336328824235832596922938e1, 7: -3.32882109689848629194453265587e1,
     8: -2.03312017085086261358222928593e-2},
    {0: -9.3714243008598732571704021658e-1, 3: 5.18637242884406370830023853209,
     4: 1.09143734899672957818500254654, 5: -8.14978701074692612513997267357,
     6: -1.85200656599969598641566180701e1, 7: 2.27394870993505042818970056734e1,
     8: 2.49360555267965238987089396762, 9: -3.0467644718982195003823669022},
    {0: 2.27331014751653820792359768449, 3: -1.05344954667372501984066689879e1,
     4: -2.00087205822486249909675718444, 5: -1.79589318631187989172765950534e1,
     6: 2.79488845294199600508499808837e1, 7: -2.85899827713502369474065508674,
     8: -8.87285693353062954433549289258, 9: 1.23605671757943030647266201528e1,
     10: 6.43392746015763530355970484046e-1}])
B = np.array([5.42937341165687622380535766363e-2, 0, 0, 0, 0, 4.45031289275240888144113950566,
              1.89151789931450038304281599044, -5.8012039600105847814672114227,
              3.1116436695781989440891606237e-1, -1.52160949662516078556178806805e-1,
              2.01365400804030348374776537501e-1, 4.47106157277725905176885569043e-2])
ER = np.array([0.1312004499419488073250102996e-1, 0, 0, 0, 0, -0.1225156446376204440720569753e1,
               -0.4957589496572501915214079952, 0.1664377182454986536961530415e1,
               -0.3503288487499736816886487290, 0.3341791187130174790297318841,
               0.8192320648511571246570742613e-1, -0.2235530786388629525884427845e-1])
BHH = np.zeros(12)
BHH[[0, 8, 11]] = (0.244094488188976377952755905512, 0.733846688281611857341361741547,
                   0.220588235294117647058823529412e-1)


def _comb(c, k):
    """sum_j c_j k_j over the stages with a weight"""
    j = np.nonzero(c)[0]
    r = k[j[0]] * float(c[j[0]])
    for i in j[1:]:
        r = torch.add(r, k[i], alpha=float(c[i]))
    return r


def _dop_stages(f, x, w, h, ld):
    kx, kw, g = [], [], 0.0
    for i in range(12):
        X, W = (x, w) if i == 0 else (x + h * _comb(A[i], kx), w + h * _comb(A[i], kw))
        a, b = f.field(X, W)
        kx.append(a)
        kw.append(b)
        if ld and B[i]:
            g = g + float(B[i]) * a.abs().sqrt().sum(0)
    return kx, kw, g


class _Marks:
    """Checkpoint bookkeeping: the SALI/GALI set back to unit length, SALI,
    Gram-Schmidt of the Lyapunov set."""

    def __init__(self, n, m_s, n_l, sali):
        z = torch.zeros(n, device=DEV, dtype=F64)
        self.m_s, self.n_l, self.sali = m_s, n_l, sali
        self.min, self.last = z + math.inf, z * math.nan
        self.tch = z * math.nan
        self.grow = torch.zeros(m_s + n_l, n, device=DEV, dtype=F64)

    def at(self, t, w):
        m = self.m_s
        r = w[:m].square().sum(1).sqrt()
        self.grow[:m] += r.log()
        w[:m] /= r[:, None]
        if self.sali:
            s = torch.minimum((w[0] + w[1]).square().sum(0), (w[0] - w[1]).square().sum(0)).sqrt()
            self.last = s
            self.min = torch.minimum(self.min, s)
            t = t if torch.is_tensor(t) else torch.full_like(s, t)
            self.tch = torch.where((s < 1e-8) & self.tch.isnan(), t, self.tch)
        for j in range(m, m + self.n_l):
            r = w[j].square().sum(0).sqrt()
            self.grow[j] += r.log()
            w[j] /= r
            if j + 1 < m + self.n_l:
                d = (w[j + 1:] * w[j]).sum(1)
                w[j + 1:] -= d[:, None] * w[j]
        return w

    def out(self, x, w, t, ld, gali):
        """The library's outputs (whole numbers and the energy error, which
        is a difference at rounding level, left out)."""
        o = dict(x_final=x.T.contiguous(), t_end=torch.full_like(x[0], t))
        if self.sali:
            o.update(sali_final=self.last, sali_min=self.min, t_chaos=self.tch)
        if self.m_s:
            o["ln_growth"] = self.grow[:self.m_s].T.contiguous()
        if self.n_l:
            o["lyap"] = (self.grow[self.m_s:] / t).T.contiguous()
        if ld is not None:
            o["ld"] = ld
        if gali:
            r = torch.linalg.qr(w[:gali].permute(2, 1, 0).contiguous(), mode="r")[1]
            d = r.diagonal(dim1=1, dim2=2).abs()
            o["gali"] = torch.cumprod(d, 1)[:, 1:].contiguous()
        return o


C0 = 1.0 / (2.0 - 2.0 ** (1.0 / 3.0))
C1 = 1.0 - 2.0 * C0


def _yoshida(sys, x, w, marks, dt, steps, ld, gali):
    """Yoshida-4 and its tangent map; checkpoints every K steps."""
    N = sys.N
    q, p = x[:N], x[N:]
    dq, dp = w[:, :N], w[:, N:]
    acc = None
    if ld:
        g = p.abs().sqrt().sum(0) + sys.force(q).abs().sqrt().sum(0)
        acc = torch.zeros_like(g)
    for s in range(1, steps + 1):
        F = sys.force(q)
        for c in (C0, C1, C0):
            p = p - 0.5 * c * dt * F
            if len(w):
                dp = dp - 0.5 * c * dt * sys.hess(q, dq)
                dq = dq + c * dt * dp
            q = q + c * dt * p
            F = sys.force(q)
            p = p - 0.5 * c * dt * F
            if len(w):
                dp = dp - 0.5 * c * dt * sys.hess(q, dq)
        if ld:
            n = p.abs().sqrt().sum(0) + F.abs().sqrt().sum(0)
            acc, g = acc + 0.5 * dt * (g + n), n
        if marks and (s % K == 0 or s == steps):
            w = marks.at(s * dt, torch.cat([dq, dp], 1))
            dq, dp = w[:, :N], w[:, N:]
    return marks.out(torch.cat([q, p]), w, steps * dt, acc, gali) if marks else acc


def _dop_fixed(f, x, w, marks, dt, steps, ld, gali):
    acc = torch.zeros_like(x[0]) if ld else None
    for s in range(1, steps + 1):
        kx, kw, g = _dop_stages(f, x, w, dt, ld)
        x, w = x + dt * _comb(B, kx), w + dt * _comb(B, kw)
        if ld:
            acc = acc + dt * g
        if s % K == 0 or s == steps:
            w = marks.at(s * dt, w)
    return marks.out(x, w, steps * dt, acc, gali)


def _dop_adaptive(f, x, w, marks, dt, T, tol, gali):
    """Adaptive DOP8(5), every orbit with its own step, meeting at the
    checkpoints (multiples of K dt and T)."""
    n, D = x.shape[1], x.shape[0] * (1 + w.shape[0])
    h = torch.full((n,), dt, device=DEV, dtype=F64)
    rej = torch.zeros(n, device=DEV, dtype=torch.bool)
    emax, elast = torch.zeros_like(h), torch.zeros_like(h)
    steps, s = int(round(T / dt)), 0
    while s < steps:
        nxt = min(steps, s + K)
        t, tb = torch.full_like(h, s * dt), nxt * dt
        while True:
            on = t < tb
            if not bool(on.any()):
                break
            last = t + 1.01 * h >= tb
            hh = torch.where(last, tb - t, h)
            hh = torch.where(on, hh, torch.zeros_like(hh))
            kx, kw, _ = _dop_stages(f, x, w, hh, False)
            e5 = e3 = 0.0
            xn, wn = x + hh * _comb(B, kx), w + hh * _comb(B, kw)
            for y, yn, k in ((x, xn, kx), (w, wn, kw)):
                sk = tol + tol * torch.maximum(y.abs(), yn.abs())
                a = (hh * _comb(ER, k) / sk).square()
                b = (hh * _comb(B - BHH, k) / sk).square()
                e5 = e5 + a.reshape(-1, n).sum(0)
                e3 = e3 + b.reshape(-1, n).sum(0)
            den = e5 + 0.01 * e3
            err = torch.where(den > 0, e5 / torch.sqrt(D * den), torch.zeros_like(den))
            fac = torch.clamp(err ** 0.125 / 0.9, max=1.0 / 0.333)
            ok = on & (err <= 1.0)
            up = hh / torch.clamp(fac, min=1.0 / 6.0)
            up = torch.where(rej, torch.minimum(up, hh), up)
            h = torch.where(ok, up, torch.where(on, hh / fac, h))
            rej = torch.where(on, ~ok, rej)
            emax = torch.where(ok, torch.maximum(emax, err), emax)
            elast = torch.where(ok, err, elast)
            x, w = torch.where(ok, xn, x), torch.where(ok, wn, w)
            t = torch.where(ok, torch.where(last, torch.full_like(t, tb), t + hh), t)
        w = marks.at(tb, w)
        s = nxt
    return marks.out(x, w, T, None, gali)


def _scatter(o, mask, x0):
    """Rows of the masked points: their state, time 0, NaN."""
    out = {}
    for k, v in o.items():
        full = torch.full((len(mask),) + v.shape[1:], math.nan, device=DEV, dtype=F64)
        if k == "t_end":
            full.zero_()
        if k == "x_final":
            full = x0.clone()
        full[mask] = v
        out[k] = full
    return out


def _too_long(steps, numbers, passes, every=0.0):
    """Whether about `passes` torch operations over `numbers` doubles a step
    take more than a dozen seconds."""
    return steps * (passes * (8e-6 + numbers * 2.4e1 / 2.5e12) + every) > 12.0


def _unit(w0):
    w = w0.permute(1, 2, 0).contiguous()
    return w / w.square().sum(1, keepdim=True).sqrt()


def _with_basis(w, n_l):
    if not n_l:
        return w
    D, n = w.shape[1], w.shape[2]
    e = torch.eye(D, device=DEV, dtype=F64)[:n_l, :, None].expand(-1, -1, n)
    return torch.cat([w, e])


def exact(case, seed):
    k = case["kind"]
    if k == "section":
        full = case["ind"] == "full"
        m_s, n_l = 2, 4 if full else 0
        n = int(ACCESS[case["E"]] * case["ny"] * case["npy"])
        steps = int(round(case["T"] / case["dt"]))
        rk = case["integrator"] == "dop853"
        if _too_long(steps, 4 * (m_s + n_l) * n, 130 if rk else 45, 30e-5 if full else 0):
            return None
        x0, mask = _section(case, seed)
        on = mask.bool()
        w = _with_basis(_unit(_normals((len(x0), 2, 4), seed, 3)[on]), n_l)
        marks = _Marks(w.shape[2], m_s, n_l, True)
        x = x0[on].T.contiguous()
        if rk:
            o = _dop_fixed(_Separable(_HH()), x, w, marks, case["dt"], steps, True, 2 * full)
        else:
            o = _yoshida(_HH(), x, w, marks, case["dt"], steps, True, 2 * full)
        return _scatter(o, on, x0)
    if k in ("points", "dp", "fput_sweep", "fput_spectrum"):
        n = case["n"]
        if k == "points":
            f, x0, m, tol = _Separable(_HH()), _points(n, case["E"], seed), 2, case["tol"]
        elif k == "dp":
            f, x0, m, tol = _DP(), _dp_states(n, seed), 2, 1e-11
        else:
            f, x0, tol = _Separable(_FPUT(case["N"])), _fput_states(case["N"], n, seed), 1e-11
            m = case["N"] if k == "fput_spectrum" else 4
        D = x0.shape[1]
        n_l = D if k == "fput_spectrum" else 0
        sali = k in ("points", "dp")
        numbers = n * D * (m + n_l)
        w = _with_basis(_unit(_normals((n, m, D), seed, 3)), n_l)
        marks = _Marks(n, m, n_l, sali)
        x = x0.T.contiguous()
        gali = 0 if sali else m
        if k == "fput_spectrum" or case.get("integrator") == "yoshida4":
            dt = 0.02 if k == "fput_spectrum" else 0.0025
            steps = int(round(case["T"] / dt))
            if _too_long(steps, numbers, 40, 1e-4 * n_l / K):
                return None
            return _yoshida(f.sys, x, w, marks, dt, steps, False, gali)
        if case.get("integrator") == "dop853":
            steps = int(round(case["T"] / 0.02))
            if _too_long(steps, numbers, 400):
                return None
            return _dop_fixed(f, x, w, marks, 0.02, steps, False, gali)
        # two to three times the attempts of one orbit: every interval waits
        # for its slowest
        if _too_long(int(case["T"] * (40 if k == "dp" else 15)), numbers,
                     400 if k == "dp" else 250):
            return None
        return _dop_adaptive(f, x, w, marks, 0.1, case["T"], tol, gali)
    if k == "ldn":
        x0, mask = _section(case, seed)
        on = mask.bool()
        steps = int(round(case["T"] / 0.01))
        if _too_long(steps, 20 * int(on.sum()), 30):
            return None
        x = x0[on]
        pts = [x]
        for c in (1, 3):
            for sg in (1e-3, -1e-3):
                y = x.clone()
                y[:, c] += sg
                pts.append(y)
        z = torch.stack(pts)
        flip = torch.tensor([1.0, 1.0, -1.0, -1.0], device=DEV, dtype=F64)
        z = torch.stack([z, z * flip]).reshape(-1, 4).T.contiguous()
        ld = _yoshida(_HH(), z, torch.empty(0, 4, z.shape[1], device=DEV, dtype=F64), None, 0.01,
                      steps, True, 0)
        L = ld.reshape(2, 5, -1).sum(0)
        a, up, dn = L[0], L[1::2], L[2::2]
        o = dict(ld=a, D=((a - up).abs() + (a - dn).abs()).sum(0) / (4 * a),
                 R=(1.0 - (up + dn).sum(0) / (4 * a)).abs(),
                 S=(up - 2 * a + dn).abs().sum(0) / (2 * a))
        return _scatter(o, on, x0)
    if k == "batched":
        return None  # 40000 steps of three ensembles: longer than wanted
    if k == "gate_train":
        return _exact_train(case, seed)
    f, _ = _gate_rows(case["n"], seed)
    z = (f.double() - torch.as_tensor(GATE_MEAN, device=DEV).double()) \
        * torch.as_tensor(GATE_ISTD, device=DEV).double()
    ps = [t.double() for t in _unflat(torch.as_tensor(_gate_params(seed), device=DEV))]
    p = torch.cat([_logits(ps, r).softmax(1)[:, 1] for r in z.split(1 << 18)])
    return dict(p=p, confidence=torch.maximum(p, 1.0 - p))


def _unflat(p):
    return (p[:4096].reshape(16, 256)[:6], p[4096:4352], p[4352:69888].reshape(256, 256),
            p[69888:70144], p[70144:74240].reshape(256, 16)[:, :2], p[74240:74242])


def _logits(ps, z):
    w1, b1, w2, b2, w3, b3 = ps
    gelu = torch.nn.functional.gelu
    return gelu(gelu(z @ w1 + b1) @ w2 + b2) @ w3 + b3


def _mix64(z):
    m = (1 << 64) - 1
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & m
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & m
    return z ^ (z >> 31)


def _exact_train(case, seed):
    """AdamW on the softmax cross-entropy in 64 bits, the library's epoch
    permutation i -> (a i + c) mod n.  The weights after an epoch follow the
    rounding of every batch before them and have no value of their own."""
    n, batch = case["n"], case["batch"]
    f, lab = _gate_rows(n, seed)
    f = f.double()
    mean, istd = f.mean(0), 1.0 / f.std(0, unbiased=False)
    z, lab = (f - mean) * istd, lab.long()
    ps = [t.clone().double().requires_grad_() for t in
          _unflat(torch.as_tensor(_gate_params(seed), device=DEV))]
    opt = torch.optim.AdamW(ps, lr=1e-3, betas=(0.9, 0.999), eps=1e-8, weight_decay=0.0)
    i = torch.arange(n, device=DEV)
    losses = []
    for ep in range(case["epochs"]):
        key = _mix64(int(seed) ^ _mix64(0x6A7E0000 + ep))
        a = 1 + _mix64(key) % (n - 1) if n > 1 else 1
        while math.gcd(a, n) != 1:
            a = a + 1 if a + 1 < n else 1
        order = (a * i + _mix64(key + 1) % n) % n
        total = 0.0
        for r in order.split(batch):
            l = torch.nn.functional.cross_entropy(_logits(ps, z[r]), lab[r])
            opt.zero_grad()
            l.backward()
            opt.step()
            total = total + l.detach() * len(r)
        losses.append(total / n)
    pad = lambda v: v.float().cpu().numpy()  # noqa: E731
    return dict(loss=torch.stack(losses).cpu().numpy(), params=None, mean=pad(mean),
                istd=pad(istd))
