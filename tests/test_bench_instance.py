"""What bench.py says a stage runs follows the layout that the library reports
(host only)."""

import os

import pytest

native = pytest.importorskip("paper_2410_21607_amd.native")

from test_bench_host import CALIB, COLS, _write  # noqa: E402

OWN = "void sem::k_stage_own<5, 4>(sem::DevMesh)"


def test_stage_instance_follows_the_reported_layout():
    import bench
    inst = bench.stage_instance
    assert inst(4, 4, 0, 0, True, False) == "k_stage_own<5, "
    # a named chunk or order, or a mesh beyond the owner kernel's limits
    assert inst(4, 4, 0, 4, True, False) == "k_stage_columns<5, 4, double, false, false, 0>"
    assert inst(7, 2, 3, 2, True, False) == "k_stage_columns<8, 2, double, false, false, 2>"
    assert inst(7, 1, 0, 1, True, False) == "k_stage_columns<8, 1, double, false, false, 0>"
    # float and dissipation leave it in the default layout too
    assert inst(4, 4, 0, 0, False, False) == "k_stage_columns<5, 4, float, false, false, 1>"
    assert inst(4, 4, 0, 0, True, True) == "k_stage_columns<5, 4, double, false, true, 0>"
    assert inst(4, 4, 0, 0, False, True) == "k_stage_columns<5, 4, float, false, false, 1>"
    assert inst(4, 4, 1, 2, True, False) is None


def test_stage_launches_name_what_ran():
    import bench
    text = bench.stage_launches
    assert "owner kernel, one launch" in text(0, 0, True, False, False)
    assert "side columns" in text(0, 0, True, False, True)
    assert text(0, 4, True, False, False) == text(0, 0, False, False, False) == "fused stage (column passes)"
    assert text(0, 0, True, True, True) == "fused stage (column passes + hanging pass)"
    assert "block passes" in text(1, 2, True, False, False)


def test_owner_traffic_is_one_launch_on_a_periodic_mesh_only(tmp_path, monkeypatch):
    if not os.path.exists(native.LIB_PATH):
        pytest.skip("libsem.so not built")
    import bench
    from paper_2410_21607_amd.api import sem_mesh_plan
    from synth import cases
    info = sem_mesh_plan(cases.get("vortex_8x8x4_n4"))[0]
    calib = 5 * info["n_h"] * info["ldz"] * 8 / 1024
    _write(tmp_path / "f.csv", "FETCH_SIZE", [(CALIB, calib)] * 5 + [(OWN, 300.0)] * 9 + [(COLS, 1.0)] * 3)
    _write(tmp_path / "w.csv", "WRITE_SIZE", [(CALIB, calib)] * 5 + [(OWN, 100.0)] * 9 + [(COLS, 1.0)] * 3)
    args = (str(tmp_path / "f.csv"), str(tmp_path / "w.csv"), "vortex_8x8x4_n4")
    out = bench.traffic_from_counters(*args, out_dir=str(tmp_path))
    assert out["launches_per_stage"] == 1 and out["hbm_bytes_per_stage"] == pytest.approx(1024 * 400.0)
    # walls: the side columns' launch and their sums belong to the stage
    walls = dict(cases.get("vortex_8x8x4_n4"), periodic_y=False)
    monkeypatch.setattr(cases, "get", lambda name, **kw: walls)
    with pytest.raises(ValueError, match="periodic"):
        bench.traffic_from_counters(*args, out_dir=str(tmp_path))
