"""The roofline entry of bench.py (no GPU): every figure is per time step, whatever a
launch advances."""
import json
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402

CFG = dict(tile_rows=4, persist_blocks_per_cu=4, graph_steps=64, fp64_arith=0, chunk_rows=8)


@pytest.mark.parametrize("model,schedule,steps,kernel,bound,moved", [
    ("binary", 6, 3, "lb_block_bin", "valu", 64 / 3),
    ("vdw", 4, 4, "lb_block_vdw", "valu", 72 / 4),
    ("binary", 5, 2, "lb_wide2_bin", "hbm", 80 / 2),
    ("vdw", 5, 2, "lb_wide2_vdw", "hbm", 72 / 2),
    ("binary", 4, 1, "lb_wide_bin", "hbm", 80),
    ("vdw", 3, 1, "lb_strip_vdw", "hbm", 72),
    ("vdw", 1, 1, "lb_step_kernel_vdw_4", "hbm", 72),
])
def test_figures_are_per_step(monkeypatch, model, schedule, steps, kernel, bound, moved):
    asked = []
    monkeypatch.setattr(bench, "traffic_from_profiles", lambda *a: asked.append(a) or 1200)
    cfg = dict(CFG, schedule=schedule)
    r = bench.roofline(model, cfg, "sweep", 10_000_000, 100.0, steps, 6000.0)
    assert asked == [(kernel, "sweep", cfg)]
    assert r["kernel"] == kernel and r["bound"] == bound and r["steps_per_launch"] == steps
    assert r["traffic"] == 1200 // steps and r["kernel_us"] == 100.0
    # 10 M updates in 100 us: 100 updates per ns
    assert r["achieved"] == pytest.approx(100.0 * bench.BYTES_PER_LUP[model])
    assert r["frac_of_stored_bytes"] == pytest.approx(100.0 * moved / bench.HBM_PEAK_GBS, abs=1e-4)


def test_no_traffic_without_a_summary(monkeypatch):
    monkeypatch.setattr(bench, "traffic_from_profiles", lambda *a: None)
    assert bench.roofline("binary", dict(CFG, schedule=6), "sweep", 1, 0.0, 3, 6000.0)["traffic"] is None


@pytest.mark.parametrize("name,schedule,steps,lo,hi", [("lb_block_bin_sweep_counters.json", 6, 3, 0.25, 0.35),
                                                       ("lb_block_vdw_vdw16k_counters.json", 4, 4, 0.3, 0.45)])
def test_committed_summaries_of_the_tile_kernels(name, schedule, steps, lo, hi):
    """Their launch shape and steps per launch, every command a rocprofv3 call of
    committed files, and a launch that moves a fraction of its steps' algorithmic
    bytes (a third and a quarter, and the halos)."""
    d = json.load(open(os.path.join(ROOT, "profiles", name)))
    assert d["launch"]["schedule"] == schedule and d["steps_per_launch"] == steps
    assert d["kernel"].startswith(bench.step_kernel("binary" if schedule == 6 else "vdw", d["launch"]))
    assert lo < d["hbm_bytes_per_launch"] / d["algorithmic_bytes_per_launch"] < hi
    assert all(c.startswith(("cd ", "rocprofv3 ")) for c in d["commands"])
