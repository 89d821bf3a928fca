"""The frame form of the SALI/GALI set, as arithmetic: a model in numpy.

The set's coordinates c in the frame of the full Lyapunov set Q go from one
checkpoint to the next as c' = R c, Q' R = Phi Q the Gram-Schmidt of the
integrated frame.  Q' is orthonormal to 1e-16 times the condition of R only, but
it enters only where c' is measured, so that error does not add up, and
what a nearly singular R costs in Q' it costs in directions that the measured
vectors have lost as well.  So the form needs no bound on the step: SALI and
GALI stay as close to the extended-precision ones as those of the set
integrated in 64 bits, from steps that resolve the motion to coarse ones, and
for chains that blow up between two checkpoints (condition up to 1e35).
"""
import numpy as np
import pytest

import seeded_inputs as S

N, D, M = 8, 16, 8
W1 = 1.0 / (2.0 - 2.0 ** (1.0 / 3.0))
W0 = 1.0 - 2.0 * W1
C = (W1, W0, W1)
KICK = (W1 / 2, (W1 + W0) / 2, (W1 + W0) / 2, W1 / 2)


def springs(q, prm):
    k, al, be = prm
    d = np.diff(np.pad(q, ((0, 0), (1, 1))), axis=1)
    f = d * (k + d * (al + be * d))
    return f[:, :-1] - f[:, 1:], k + d * (2 * al + 3 * be * d)


def kick(V, kappa, h):
    h, kappa = V.dtype.type(h), kappa.astype(V.dtype)[:, None]
    a = np.pad(V[..., :N], ((0, 0), (0, 0), (1, 1)))
    kl, kr = kappa[..., :-1], kappa[..., 1:]
    V[..., N:] -= h * ((kl + kr) * a[..., 1:-1] - kl * a[..., :-2] - kr * a[..., 2:])


def gram_schmidt(V):
    """V's rows orthonormalised in place; returns R (columns: the old rows)."""
    n, m = V.shape[:2]
    R = np.zeros((n, m, m), V.dtype)
    for j in range(m):
        R[:, j, j] = np.sqrt((V[:, j] ** 2).sum(1))
        V[:, j] /= R[:, j, j][:, None]
        for k in range(j + 1, m):
            R[:, j, k] = (V[:, j] * V[:, k]).sum(1)
            V[:, k] -= R[:, j, k][:, None] * V[:, j]
    return R


def measure(X):
    """Unit length, then SALI and GALI_M (extended precision)."""
    X /= np.sqrt((X * X).sum(2))[..., None]
    U = X.astype(np.longdouble)
    sali = np.sqrt(np.minimum(((U[:, 0] + U[:, 1]) ** 2).sum(1), ((U[:, 0] - U[:, 1]) ** 2).sum(1)))
    R = gram_schmidt(U.copy())
    return sali, np.prod(R[:, range(M), range(M)], axis=1)


@pytest.mark.parametrize("prm,scale", [((1.0, 0.0, 1.0), 1.0), ((1.0, 0.25, 1.0), 4.0),
                                       ((1.0, 0.25, 0.0), 1.0), ((1.0, 0.25, 0.0), 4.0)])
@pytest.mark.parametrize("dt", [0.02, 0.1, 0.3, 0.5])
def test_frame_is_as_close_as_the_integrated_set(O, prm, scale, dt):
    K, n, checkpoints = 16, 12, 20
    x = scale * O.fput_ic(O.fput(N), S.fput_mode_draws(5, n))
    q, p = x[:, :N].copy(), x[:, N:].copy()
    w = S.deviation_vectors(7, n, M, D)
    w /= np.sqrt((w * w).sum(2))[..., None]
    plain, ext, c = w.copy(), w.astype(np.longdouble), w.copy()
    Q = np.tile(np.eye(D), (n, 1, 1))
    with np.errstate(all="ignore"):
        for cp in range(checkpoints):
            for _ in range(K):
                for i in range(4):
                    F, kappa = springs(q, prm)
                    p -= KICK[i] * dt * F
                    for V in (plain, ext, Q):
                        kick(V, kappa, KICK[i] * dt)
                    if i < 3:
                        q += C[i] * dt * p
                        for V in (plain, ext, Q):
                            V[..., :N] += V.dtype.type(C[i] * dt) * V[..., N:]
            c = np.matmul(c, gram_schmidt(Q).transpose(0, 2, 1))
            (sf, gf), (si, gi), (se, ge) = measure(c), measure(plain), measure(ext)
            ok = np.isfinite(q).all(1) & (np.abs(q).max(1) < 1e6)
            # every step rounds the 16 components of a vector of unit size
            tol = 16 * K * (cp + 1) * np.finfo(np.float64).eps
            for got, ref in ((sf, se), (gf, ge)):
                assert not np.isnan(got[ok]).any()
                assert (np.abs(got - ref)[ok] < tol).all(), cp
            # and no further off than the integrated set is allowed to be
            assert (np.abs(si - se)[ok] < tol).all() and (np.abs(gi - ge)[ok] < tol).all(), cp
            if not ok.any():  # steps too coarse for any of these chains
                break
