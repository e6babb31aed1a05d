"""The autotuner times only shapes that have an effect: the cluster-resolution
shapes act behind the LDS tile stage alone, so a bed that keeps the rows, and a
batch, which has no tile stage, keep the shapes they had and advance by the steps
of the other candidates."""
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)
L = pytest.importorskip("paper_1303_2653_amd.lbdps")

LISTS, GROUPS = 3, 777  # no candidate


@pytest.mark.parametrize("n", [60, 40_000])
def test_single_bed(n):
    cfg = synth.tiny(nx=200, ny=200, n=n, seed=4, bc=("periodic",) * 4, g=(0.0, 0.0), vel_scale=1e-3)
    sim = L.Sim(cfg, precision="fp32")
    sim.set_tuning(cluster_lists=LISTS, cluster_groups_max=GROUPS)
    t = sim.autotune(2)
    steps = sim.state()[3]
    print(n, t, steps, flush=True)
    if t["sphere_tile"] == 0:
        assert (t["cluster_lists"], t["cluster_groups_max"]) == (LISTS, GROUPS)
        assert steps == 2 * 2 * (4 + 3)
    else:
        assert (t["cluster_lists"], t["cluster_groups_max"]) != (LISTS, GROUPS)
        assert steps == 2 * 2 * (4 + 9 + 3)
    assert sim.tuning() == t


def test_batch(tmp_path):
    cfgs = [synth.tiny(nx=40 + i, ny=50, n=n, seed=4 + i, bc=("periodic",) * 4, g=(0.0, 0.0), vel_scale=1e-3,
                       precision="fp32") for i, n in enumerate((500, 2600, 5000))]
    path = tmp_path / "tune.txt"
    batch = L.Batch(cfgs)
    before = [b.tuning() for b in batch.beds]
    after = batch.autotune(2, path)
    for a, b, bed in zip(before, after, batch.beds):
        assert {k: v for k, v in a.items() if k != "drag_tile"} == {k: v for k, v in b.items() if k != "drag_tile"}
        assert bed.state()[3] == 2 * 2 * 3
    # a file with other shapes, as one written before them, is read as it is
    lines = path.read_text().splitlines()
    assert len(lines) == 4
    path.write_text("\n".join([lines[0]] + [f"{c} {LISTS} {GROUPS} 2" for c in range(3)]) + "\n")
    other = L.Batch(cfgs)
    for t in other.autotune(2, path):
        assert (t["cluster_lists"], t["cluster_groups_max"], t["drag_tile"]) == (LISTS, GROUPS, 2)
    assert all(b.state()[3] == 0 for b in other.beds)
