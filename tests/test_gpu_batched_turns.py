"""Turns (steps per launch) that the batched form chooses, and the autotuner's
costs behind them.

A turn reloads and requeues every orbit, so it must not be short where little
is packed anew by it: in short runs, next to a long run of another item,
without early exit, or for the sake of an item without orbits.  The results do
not depend on the turns.
"""
import numpy as np
import pytest

import seeded_inputs as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available()
    import paper_2507_00622_amd as P
    from oracle import oracle as O
    return torch, P, O


def hh(P, O, n, steps, **kw):
    y, py = S.section_points(21, 2 * n + 16)
    x, m = O.hh_points(0.125, y, py)
    return dict(sys=P.henon_heiles(), x0=x[m == 1][:n], dt=0.01, T=0.01 * steps, **kw)


def fput(P, O, n, steps):
    return dict(sys=P.fput(16), x0=O.fput_ic(O.fput(16), S.fput_mode_draws(22, n)), dt=0.02,
                T=0.02 * steps)


def run(env, items, early_exit=True, ind=17, **kw):
    torch, P, O = env
    outs, stats = P.integrate_batched(items, indicators=ind, seed=5, early_exit=early_exit, **kw)
    print("  stats:", stats, flush=True)
    return outs, stats


def plain(env, items, **kw):
    torch, P, O = env
    return [P.integrate_ensemble(i["sys"], i["x0"], mask=i.get("mask"), dt=i["dt"], T=i["T"],
                                 indicators=17, seed=5 + k, early_exit=True)
            for k, i in enumerate(items)]


# a graph replay is four launches; two replays at most for runs that one turn
# can carry
@pytest.mark.parametrize("n_hh,hh_steps,n_f,f_steps", [
    (200, 100, 200, 20000),    # a short lane item next to a long row item
    (2000, 40000, 4000, 20000),  # a long one, but the rows carry the work
    (3000, 1000, 0, 0),        # short lane runs alone
    (3000, 320, 50, 300)])
def test_turns_that_pack_nothing_are_long(env, n_hh, hh_steps, n_f, f_steps):
    torch, P, O = env
    print(f"case: turns, {n_hh} x {hh_steps} lanes, {n_f} x {f_steps} rows", flush=True)
    items = [hh(P, O, n_hh, hh_steps)] + ([fput(P, O, n_f, f_steps)] if n_f else [])
    outs, stats = run(env, items)
    assert stats["launches"] <= 8
    assert stats["steps_per_launch"] >= max(hh_steps, f_steps)
    for a, b in zip(outs, plain(env, items)):
        for k in a:
            assert np.array_equal(a[k], b[k], equal_nan=True), k


def test_item_without_orbits_sets_no_turn(env):
    torch, P, O = env
    print("case: turns, an item whose orbits are all masked", flush=True)
    empty = hh(P, O, 64, 30000)
    empty["mask"] = np.zeros(64, np.uint8)
    rows = fput(P, O, 400, 2000)
    _, alone = run(env, [rows])
    outs, both = run(env, [empty, rows])
    assert both["steps_per_launch"] == alone["steps_per_launch"]
    assert (outs[0]["status"] == O.ST_MASKED).all()
    _, none = run(env, [empty])
    assert none["launches"] <= 4


def test_turns_only_where_orbits_exit_early(env):
    torch, P, O = env
    print("case: turns with and without early exit", flush=True)
    items = [hh(P, O, 3000, 32000)]
    _, no = run(env, items, early_exit=False)
    outs, ee = run(env, items)
    assert no["steps_per_launch"] >= 32000
    assert ee["steps_per_launch"] == 1000  # 1/32 of the run, the smallest turn
    for a, b in zip(outs, plain(env, items)):
        for k in a:
            assert np.array_equal(a[k], b[k], equal_nan=True), k


def test_turn_time_of_few_orbits(env):
    torch, P, O = env
    print("case: a turn of few orbits takes about 200 ms at most", flush=True)
    _, st = run(env, [fput(P, O, 16, 2000)])
    # a step takes at least as long as one with a wavefront on every SIMD
    rows = 4 * torch.cuda.get_device_properties(0).multi_processor_count * 4
    assert st["steps_per_launch"] * st["cost_ps"][0] * 1e-12 * rows < 0.201
