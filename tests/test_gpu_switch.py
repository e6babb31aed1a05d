"""One context that goes from one course of the collision stage to another: the
tile stage, clusters, patches and the final workgroup share scratch arrays, and
each leaves them as the others can take them."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)
L = pytest.importorskip("paper_1303_2653_amd.lbdps")

PER = ("periodic",) * 4


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_switching_courses(prec):
    """Beds of one lattice with 700 to 16 000 spheres (whole, patches, clusters that
    percolate), each by rows and by tiles, in turn on one context: the state after
    two steps equals a fresh context's, bit for bit."""
    beds = [synth.tiny(nx=60, ny=61, n=n, seed=n, bc=PER, g=(0.0, 0.0), vel_scale=5e-3) for n in (16_500, 3000, 700)]
    ref, plans = [], []
    for b in beds:
        one = L.Sim(b, precision=prec)
        one.step(2)
        ref.append(one.state()[:3] + (one.counters(),))
        plans.append(one.row_stats()["plan"])
        one.close()
    assert plans == [3, 1, 0], plans
    sim = L.Sim(beds[0], precision=prec)  # the largest: its workspace holds the others
    for turn in range(2):
        for tile in (0, 1, 0, 2):
            for i, b in enumerate(beds):
                print("turn", turn, "tile", tile, "particles", len(b["pos"]), flush=True)
                sim.set_tuning(sphere_tile=tile)
                sim.set_state(None, b["pos"], b["vel"])
                sim.step(2)
                got = sim.state()[:3] + (sim.counters(),)
                for x, y in zip(got[:3], ref[i][:3]):
                    assert np.array_equal(x, y), (turn, tile, i)
                assert got[3] == ref[i][3], (turn, tile, i)
                pairs = sim.pairs()
                assert pairs[1] == got[3]["pairs"]
