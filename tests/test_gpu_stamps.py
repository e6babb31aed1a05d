"""Timing a phase of several launches stamps its first and last dispatch alone:
the step takes no longer than with a phase of one launch timed, and the phase's
time covers all its launches."""
import time

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)
L = pytest.importorskip("paper_1303_2653_amd.lbdps")


def us_per_step(sim, kernel, steps=200):
    sim.time_kernels([kernel])
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    sim.step(steps)
    torch.cuda.synchronize()
    us = (time.perf_counter() - t0) / steps * 1e6
    ms, n = sim.kernel_times()[kernel]
    sim.time_kernels([])
    assert n == steps
    return us, ms / n * 1e3


def test_timed_resolution_costs_no_more_than_a_timed_search():
    """A bed of two patch passes and the rest, in steps of some 60 us: with a pair
    of events on each of the three launches the step took 1.2 to 1.4 times as long
    as with one pair on the contact search."""
    sim = L.Sim(synth.bubble(), precision="fp32")
    sim.step(50)
    assert sim.row_stats()["plan"] == 2
    best = {k: (np.inf, 0.0) for k in ("resolve", "contacts")}
    for _ in range(5):
        for k in best:
            best[k] = min(best[k], us_per_step(sim, k))
    print(best, flush=True)
    assert best["resolve"][0] < 1.12 * best["contacts"][0]


@pytest.mark.parametrize("n,plan", [(1500, 0), (9000, 1), (90_000, 2), (400, 0)])
def test_resolution_time_covers_its_launches(n, plan):
    """The phases' times add up to most of the step's and not to more, by patches,
    in one workgroup and behind the tile stage."""
    cfg = synth.tiny(nx=300 if n > 9000 else 100, ny=300 if n > 9000 else 100, n=n, seed=6, bc=("periodic",) * 4,
                     g=(0.0, 0.0))
    for tile in (0, 1):
        sim = L.Sim(cfg, precision="fp32")
        sim.set_tuning(sphere_tile=tile)
        sim.step(5)
        assert sim.row_stats()["plan"] == (plan if tile == 0 else -1)
        sim.time_kernels(L.KERNELS)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        sim.step(50)
        torch.cuda.synchronize()
        wall = (time.perf_counter() - t0) * 1e3
        kt = sim.kernel_times()
        total = sum(ms for ms, _ in kt.values())
        print(n, tile, {k: round(ms / 50 * 1e3, 1) for k, (ms, _) in kt.items()}, "of", round(wall / 50 * 1e3, 1), flush=True)
        assert all(c == 50 for _, c in kt.values())
        assert 0.1 * wall < total < 1.02 * wall
        assert kt["resolve"][0] / 50 * 1e3 > (10.0 if plan else 2.0) or tile
