"""bench.py's roofline record (no GPU): it follows the launches that the library
reports, and its measured traffic is keyed by everything the traffic depends on."""
import os
import shutil
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402

ALGORITHMIC = 2 * 19 * 4 * 256 * 256 * 128   # one read and one write of the populations


def test_two_step_traffic_is_close_to_one_read_and_one_write():
    # neighbouring slabs read each other's border rows: more than the bytes of a
    # pass, less than those of two single steps
    for key, traffic in bench.TWO_STEP_TRAFFIC.items():
        assert len(key) == 16
        assert 1.0 <= traffic / ALGORITHMIC < 1.25


def test_the_record_names_the_kernel_that_ran():
    two = bench.headline_roofline(ALGORITHMIC, 250, 500, 68.0, {"flags": 24})
    one = bench.headline_roofline(ALGORITHMIC, 500, 500, 98.0, {"flags": 24})
    assert two["kernel"].startswith("k_two_step") and one["kernel"].startswith("k_step<")
    assert two["launches"] == 250 and one["launches"] == 500
    assert abs(one["achieved"] - ALGORITHMIC / 196e-6 / 1e9) < 0.1
    assert two["traffic"] in (None, bench.TWO_STEP_TRAFFIC.get(two["kernel_source_hash"]))
    assert one["traffic"] in (None, bench.MEASURED_TRAFFIC.get(one["kernel_source_hash"]))


def test_the_hash_covers_the_choice_of_patches(tmp_path, monkeypatch):
    csrc = tmp_path / "paper_2206_00366_amd" / "csrc"
    csrc.mkdir(parents=True)
    for f in bench.KERNEL_SOURCES:
        shutil.copy(os.path.join(ROOT, "paper_2206_00366_amd", "csrc", f), csrc / f)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    before = bench.kernel_source_hash()
    p = csrc / "sweep_plan.hpp"
    p.write_text(p.read_text().replace("columns / w", "columns / w / 2"))
    assert bench.kernel_source_hash() != before
