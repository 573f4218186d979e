"""Plans are timed on the binning that renders will take, and the digit widths
of the sorts are searched only where renders sort."""
import pytest

from paper_2603_15186_amd.synth import workloads as W, yaw_camera

pytestmark = pytest.mark.gpu
pytest.importorskip("torch")


@pytest.mark.parametrize("binning", [0, 1])
def test_digit_widths(binning):
    from paper_2603_15186_amd import hgs
    scene, cams = W.plan2m(scale=0.005, n_poses=1)
    r = hgs.Renderer(0)
    r.load_scene(scene)
    r.set_option(hgs.HGS_OPT_BINNING, binning)
    r.set_cameras([yaw_camera(160, 90, 112.0, cams[0].position, 0.3)])
    tuned = [r.autotune(reps=1) for _ in range(3)]
    assert r.route()["lists"] == (binning == 0)
    assert all(6 <= p["sort_digit_bits"] <= 11 for p in tuned)
    if binning == 0:
        assert all(p["sort_digit_bits"] == 8 for p in tuned)
    r.close()
