"""The kernel that bench.py names in its roofline block follows from the library's dispatch rules."""
import pytest

import bench


@pytest.mark.parametrize("tau, longest, lanes, name", [
    (4, 40, 1, "k_verify_auto"), (4, 47, 1, "k_verify_auto"), (1, 48, 1, "k_verify_auto, k_verify_segs"),
    (4, 40, 2, "k_verify_segs"), (5, 40, 1, "k_verify_segs"), (8, 120, 1, "k_verify_segs")])
def test_list_kernel(tau, longest, lanes, name):
    assert bench.list_kernel(tau, longest, lanes) == name


def test_lane_cands(tmp_path):
    path = tmp_path / "tune.txt"
    assert bench.lane_cands(str(path), 2, 6) == 1 and bench.lane_cands(None, 2, 6) == 1
    path.write_text("# passjoin tune cache v3\ngfx950 2 6 32 4 32 8 2 1 0.5\n"
                    "# passjoin tune cache v4: arch tau\ngfx950 4 6 32 4 32 8 2 1 0.5\n")
    assert bench.lane_cands(str(path), 2, 6) == 1
    assert bench.lane_cands(str(path), 4, 6) == 2 and bench.lane_cands(str(path), 4, 5) == 1
