"""The courses that the collision stage takes through the neighbour rows, by the
bed's size, density and evenness: the whole bed in one workgroup, patches in one
or two passes, contact clusters, and the search by clusters after patches that
were too full.  Each bed is checked to take its course (lbdps_row_stats) and
against the oracle's sequential sweep, bit for bit, as in test_gpu_patches; a
batch against the same beds alone."""
import time

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)
L = pytest.importorskip("paper_1303_2653_amd.lbdps")
import oracle  # noqa: E402

PER, WALLED = ("periodic",) * 4, ("wall",) * 4
BED = ("periodic", "periodic", "inlet", "outlet")
WHOLE, ONE, TWO, CLUSTERS = 0, 1, 2, 3
FINAL = 4096  # particles the final workgroup holds in LDS


def layer(nx, ny, n, x, y, seed, bc=PER):
    """n spheres uniform in the part [0, x nx) x [0, y ny) of the lattice."""
    cfg = synth.tiny(nx=nx, ny=ny, n=1, seed=seed, bc=bc, g=(0.0, 0.0))
    u = synth.uniform(seed, 4 * n).reshape(-1, 4)
    return dict(cfg, pos=np.stack([x * nx * u[:, 0], y * ny * u[:, 1]], 1), vel=(u[:, 2:] - 0.5) * 1e-2)


def crowd(cfg, x0, y0, w, h, n, seed):
    """n more spheres in [x0, x0 + w) x [y0, y0 + h)."""
    u = synth.uniform(seed, 2 * n).reshape(-1, 2)
    more = np.stack([x0 + w * u[:, 0], y0 + h * u[:, 1]], 1)
    return dict(cfg, pos=np.concatenate([cfg["pos"], more]), vel=np.zeros((len(cfg["pos"]) + n, 2)))


def big(left):
    return left > FINAL


# name: (bed, plan, whether the row statistics are those of its course)
BEDS = {
    "whole": (lambda: synth.tiny(nx=42, ny=43, n=2048, seed=3, bc=WALLED), WHOLE, lambda s: s["left"] == 0),
    "one-pass": (lambda: synth.tiny(nx=101, ny=97, n=9000, seed=5, bc=PER), ONE,
                 lambda s: 0 < s["left"] < FINAL and s["full"] == 0),
    "two-passes": (lambda: synth.tiny(nx=300, ny=300, n=90_000, seed=6, bc=PER), TWO,
                   lambda s: 0 < s["left"] < FINAL and s["full"] == 0),
    # few contacts: clusters, one slot per lane and four
    "sparse": (lambda: synth.tiny(nx=301, ny=299, n=9000, seed=7, bc=WALLED, d=0.3), CLUSTERS, lambda s: not s["more"]),
    "sparse-540k": (lambda: synth.tiny(nx=1500, ny=1501, n=540_001, seed=8, bc=PER, d=0.3), CLUSTERS,
                    lambda s: not s["more"]),
    # clusters beyond a wavefront; and beyond a workgroup, for the final one
    "dense": (lambda: synth.tiny(nx=150, ny=150, n=70_000, seed=9, bc=PER), CLUSTERS, lambda s: not s["more"]),
    "percolating": (lambda: synth.tiny(nx=60, ny=70, n=23_000, seed=10, bc=PER), CLUSTERS, lambda s: s["more"]),
    # a clump in a wide periodic lattice
    "clump": (lambda: layer(300, 300, 16_000, 0.3, 0.3, 11), CLUSTERS, lambda s: not s["more"]),
    # patches several times as full as they were laid out for: one pass, two, and
    # with clusters that no wavefront holds
    "layer-one": (lambda: layer(200, 300, 37_000, 1.0, 0.2, 12), ONE,
                  lambda s: big(s["left"]) and s["full"] > 37_000 // 16),
    "layer-two": (lambda: layer(400, 700, 170_000, 1.0, 0.3, 13), TWO,
                  lambda s: big(s["left"]) and s["full"] > 170_000 // 16),
    "layer-percolating": (lambda: layer(200, 300, 37_000, 1.0, 0.13, 14), ONE,
                          lambda s: big(s["left"]) and s["more"]),
    # single rows of a patch with more than its workgroup looks at
    "crowded-row": (lambda: crowd(synth.tiny(nx=64, ny=64, n=18_000, seed=15, bc=WALLED, d=0.1), 20.0, 30.0, 16.0, 3.0,
                                  4800, 16), TWO, lambda s: s["left"] > 0),
}


def state(cfg, seed=31):
    """Positions held exactly in FP32 as well, and velocities."""
    rng = np.random.default_rng(seed)
    cell = np.floor(cfg["pos"]).astype(np.int32)
    off = np.minimum((cfg["pos"] - cell).astype(np.float32), np.float32(0.99999994))
    vel = ((rng.random(off.shape) - 0.5) * 2e-2).astype(np.float32)
    return cell, off, cell.astype(np.float64) + off, vel


@pytest.mark.parametrize("name", BEDS)
def test_course_and_result(name):
    make, plan, course = BEDS[name]
    cfg = make()
    cell, off, pos, v32in = state(cfg)
    vel = v32in.astype(np.float64)
    cfg = dict(cfg, pos=pos, vel=vel)
    print("bed", name, "particles", len(pos), flush=True)
    p = oracle.make_params(cfg)
    pairs = oracle.contacts(p, pos)
    v64, nc = oracle.resolve(p, pos, vel, pairs)
    v64, nw = oracle.walls(p, pos, v64)
    pairs32, v32, nc32, nw32 = oracle.collide_f32(p, cell, off, v32in)
    for prec, ref, want in (("fp64", v64, (len(pairs), nc, nw)), ("fp32", v32, (len(pairs32), nc32, nw32))):
        gpu = L.Sim(cfg, precision=prec)
        for again in range(2):  # the second time on the state as it was: nothing is left over from the first
            gpu.set_state(None, pos, vel)
            gpu.collide_particles()
            got, c, s = gpu.particles()["vel"], gpu.counters(), gpu.row_stats()
            print(prec, s, flush=True)
            assert s["plan"] == plan and course(s), (name, prec, s)
            assert (c["pairs"], c["collisions"], c["walls"]) == want, (name, prec, again, c, want)
            assert np.array_equal(got, ref.astype(np.float64)), (name, prec, again)
        gpu.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_batch_of_all_courses(prec):
    """Beds of every course in one batch; with one of four beds that needs a second
    pass, the first lists what it leaves."""
    small = dict(bc=PER, g=(0.0, 0.0), vel_scale=5e-3)
    t = synth.tiny
    mixed = [t(nx=30, ny=31, n=700, seed=22, **small), t(nx=90, ny=60, n=6000, seed=23, **small),
             t(nx=70, ny=71, n=16_000, seed=24, **small), layer(200, 300, 37_000, 1.0, 0.2, 12),
             layer(300, 300, 16_000, 0.3, 0.3, 11)]
    listed = [t(nx=216, ny=208, n=90_000, seed=25, **small)] + [t(nx=60 + i, ny=50, n=3000, seed=26 + i, **small)
                                                               for i in range(4)]
    for kind, cfgs in (("mixed", mixed), ("listed", listed)):
        cfgs = [dict(c, precision=prec) for c in cfgs]
        print("batch", kind, prec, [len(c["pos"]) for c in cfgs], flush=True)
        batch = L.Batch(cfgs)
        batch.step(2)
        stats = [b.row_stats() for b in batch.beds]
        print(stats, flush=True)
        if kind == "mixed":
            assert [s["plan"] for s in stats] == [WHOLE, ONE, CLUSTERS, ONE, CLUSTERS]
            assert big(stats[3]["left"])
        else:
            assert {s["plan"] for s in stats} == {TWO}
            assert big(stats[0]["left"]) and 0 < stats[0]["left2"] < FINAL  # the second pass was needed ...
            assert all(0 < s["left"] < FINAL and s["left2"] == 0 for s in stats[1:])  # ... by this bed alone
        for i, c in enumerate(cfgs):
            one = L.Sim(c, precision=prec)
            one.step(2)
            for x, y in zip(batch.beds[i].state()[:3], one.state()[:3]):
                assert np.array_equal(x, y), (kind, prec, i)
            assert batch.beds[i].counters() == one.counters(), (kind, prec, i)
            one.close()


@pytest.mark.parametrize("name,nx,n,part,limit", [
    ("dense", 316, 400_000, (1.0, 1.0), 3000.0),   # 1 300 us in list order, 5 600 in one workgroup from memory
    ("clump", 1000, 200_000, (0.3, 0.3), 400.0),   # 140 us by clusters, 811 in patches that are too full
    ("sparse", 2000, 400_000, (1.0, 1.0), 150.0),  # 20 us by clusters, 324 in patches that are nearly empty
])
def test_stage_time(name, nx, n, part, limit):
    """Beds that no layout of patches suits are not much slower by it (us per
    stage; the limits are more than twice what the stage takes, and half of what
    it took by patches)."""
    cfg = layer(nx, nx, n, *part, 41, WALLED if name == "sparse" else PER)
    if name == "sparse":
        cfg["d"] = 0.1
    cfg["pos"] = cfg["pos"][synth.cell_order(cfg["pos"], nx)]
    gpu = L.Sim(dict(cfg, vel=np.zeros_like(cfg["pos"])), precision="fp32")
    best = np.inf
    for _ in range(5):
        gpu.collide_particles()
        gpu.counters()
        t0 = time.perf_counter()
        for _ in range(10):
            gpu.collide_particles()
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t0) * 1e5)
    print(name, "us per stage", best, flush=True)
    assert best < limit


@pytest.mark.parametrize("name", ["whole", "one-pass", "two-passes", "sparse", "dense", "layer-one", "layer-two"])
def test_contact_overflow_in_every_course(name):
    """One particle with more contacts than a row holds: nothing is resolved, every
    kernel ends, LBDPS_E_CAPACITY is reported, and the bed without it goes on."""
    make, plan, _ = BEDS[name]
    cfg = make()
    nx, ny, d = cfg["nx"], cfg["ny"], cfg["d"]
    vel = np.zeros((len(cfg["pos"]), 2))
    u = synth.uniform(5, 80).reshape(-1, 2)
    at = np.array([0.5 * nx, 0.1 * ny]) + 0.3 * d * (u - 0.5)
    pos = cfg["pos"].copy()
    pos[:: len(pos) // 40][:40] = at  # 40 spheres within half a diameter, the number as it was
    print(name, len(pos), flush=True)
    sim = L.Sim(dict(cfg, vel=vel), precision="fp32")
    sim.set_state(None, pos, vel)
    sim.collide_particles()
    with pytest.raises(L.LbdpsError) as e:
        sim.counters()
    assert e.value.status == L.LBDPS_E_CAPACITY
    assert sim.row_stats()["plan"] == plan
    assert (sim.particles()["vel"] == 0).all()
    sim.set_state(None, cfg["pos"], vel)
    sim.collide_particles()
    assert sim.counters()["pairs"] > 0
