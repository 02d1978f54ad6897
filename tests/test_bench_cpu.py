"""Host-side logic of bench.py: the size sweep's crossovers, the spread statistics of the timed
passes, and the single-GPU contract of the command line."""
import os
import subprocess
import sys

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


def _pt(n, res, same, mapped):
    return {"N": n, "bytes": n * 8192, "resident_GBps": res, "resident_same_buffer_GBps": same, "mapped_GBps": mapped}


def test_size_crossovers_synthetic_curve():
    # rates rise with size to a plateau; a repeated buffer beats rotated ones until the 4th point
    pts = [_pt(256, 500, 480, 40), _pt(512, 1000, 1100, 45), _pt(1024, 3000, 3600, 50),
           _pt(2048, 6000, 6100, 55), _pt(4096, 7000, 7050, 56), _pt(8192, 7200, 7200, 56)]
    c = bench.size_crossovers(pts)
    assert c["resident_plateau_GBps"] == 7200
    assert c["dispatch"]["N"] == 2048                  # first rate >= half the plateau (3600); 3000 is below
    assert c["mall"]["N"] == 2048                      # from here on same-buffer <= 1.02 x rotated
    assert c["largest_repeat_gain"]["bytes"] == 1024 * 8192   # 3600 / 3000
    assert abs(c["largest_repeat_gain"]["same_buffer_over_rotated"] - 1.2) < 1e-12
    assert c["mapped_equals_resident"] is None


def test_size_crossovers_dispatch_threshold_and_mapped():
    pts = [_pt(256, 100, 100, 120), _pt(512, 3600, 3600, 50), _pt(1024, 7200, 7200, 50)]
    c = bench.size_crossovers(pts)
    assert c["dispatch"]["N"] == 512                   # exactly half the plateau counts
    assert c["mapped_equals_resident"]["N"] == 256     # host-mapped at least as fast as resident
    assert c["mall"]["N"] == 256                       # no point where the repeat beats rotation by > 2 %


def test_size_crossovers_no_mall_when_last_point_repeats_faster():
    pts = [_pt(256, 1000, 1000, 40), _pt(512, 2000, 2100, 40)]
    assert bench.size_crossovers(pts)["mall"] is None


def test_spread_statistics():
    ms = [3.0, 1.0, 2.0, 5.0, 4.0]
    s = bench.spread(ms)
    assert s["n"] == 5 and s["median"] == 3.0
    assert s["iqr"] == [2.0, 4.0]
    lo, hi = s["ci95_median"]
    assert 1.0 <= lo <= 3.0 <= hi <= 5.0
    assert bench.spread(ms) == s                       # the bootstrap is seeded
    assert s["ms_per_token"] == ms                     # the passes in the order they ran


def test_spread_single_pass():
    s = bench.spread([7.25])
    assert s["median"] == 7.25 and s["iqr"] == [7.25, 7.25] and s["ci95_median"] == [7.25, 7.25]


def test_more_than_one_gpu_exits_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120, cwd=ROOT)
    assert r.returncode != 0
    assert "one GPU" in (r.stdout + r.stderr) or "1 GPU" in (r.stdout + r.stderr) or "single" in (r.stdout + r.stderr)


def test_oracle_threads_records_the_cap(monkeypatch):
    avail = len(os.sched_getaffinity(0))
    monkeypatch.delenv("OMP_NUM_THREADS", raising=False)
    assert bench.oracle_threads() == (avail, avail, None)
    if avail > 1:
        monkeypatch.setenv("OMP_NUM_THREADS", "1")
        assert bench.oracle_threads() == (1, avail, "OMP_NUM_THREADS=1")
    monkeypatch.setenv("OMP_NUM_THREADS", str(avail + 7))      # a cap above the cores is no cap
    assert bench.oracle_threads() == (avail, avail, None)


def test_size_crossovers_without_mapped_arm():
    pts = [{"N": n, "bytes": n * 8192, "resident_GBps": r, "resident_same_buffer_GBps": r}
           for n, r in ((256, 500), (512, 4000), (1024, 7000))]
    c = bench.size_crossovers(pts)
    assert c["dispatch"]["N"] == 512 and c["mapped_equals_resident"] == "not measured"


def test_probe_and_gemv_oracle_baselines_on_small_inputs():
    import synth
    buf = synth.grid_f32((1 << 16) + 3, seed=0, stream=1)
    r = bench.probe_cpu_baseline(buf)
    assert r["kind"] == "oracle" and r["sums_equal"] and r["value"] > 0 and r["single_thread"]["cores"] == 1
    assert r["cores"] >= 1 and r["cores_available"] >= r["cores"]
    W = [synth.normal16((64, 256), 0.02, "f16", seed=0, stream=5 + i) for i in range(3)]
    x = synth.normal16(256, 1.0, "f16", seed=0, stream=9)
    g = bench.gemv_cpu_baseline(W, x, "f16", 0.05, "three small matrices")
    assert g["value"] > 0 and g["single_thread"]["calls"] >= 1 and g["sample"].startswith("three small")


def test_measured_ceiling_second_denominator():
    rows = {"probe": {"resident_GBps": 7000.0, "roofline": {"achieved": 7000.0}},
            "gemv_f16": {"roofline": {"achieved": 3500.0}},
            "endpoints": {"GBps": {"resident": 1.0}}}
    pc = bench.measured_ceiling(7140.0, rows)
    assert pc["GBps"] == 7000.0 and pc["frac"] == 1.02
    assert rows["gemv_f16"]["frac_of_probe"] == 0.5
    assert "frac_of_probe" not in rows["probe"] and "frac_of_probe" not in rows["endpoints"]
    assert bench.measured_ceiling(7140.0, {"gemv_f16": {"roofline": {"achieved": 1.0}}}) is None


def test_result_line_is_one_short_line_with_the_whole_headline():
    """Every row present with all its figures: the line on stdout stays short and holds the headline."""
    import json
    sweep = {"GBps": 6893.123456789, "tokens_per_s": 1632.987654321, "roofline": {"traffic": 4229560908.5},
             "batched": [{"batch": b, "tokens_per_s": 7123.456789 * b, "note": "x" * 200} for b in (1, 2, 4, 8)],
             "batched_matrix_cores": [{"batch": b, "tokens_per_s": 17123.456789} for b in (1, 2, 4, 8, 16)]}
    rows = {"probe": {"resident_GBps": 7000.123456, "mapped_GBps": 55.123456, "roofline": {"note": "x" * 500}},
            "gemv_f16": {"us_per_gemv": 6.5123456, "GBps_per_dispatch": 5152.3, "one_launch_32_matrices_GBps": 6812.3},
            "llama8b_q4": sweep,
            "protocol": dict(sweep, one_launch_back_to_back={"GBps_at_median": 6912.3}, dispatches_12={"GBps_at_median": 5612.3}),
            "endpoints": {"GBps": {"map_pinned_in_place": 55.1, "resident": 6901.2, "copy_from_file_pages": 50.2, "copy_from_pinned": 52.3},
                          "alg2": {"choice": "resident", "theta_sweep": {}}},
            "ordering": {"results": {f"{w}/{d}": {"excess": {"event": {"median_ms": 0.0982}}} for w in ("mm", "small") for d in (2, 8, 32)}},
            "size_sweep": {"crossovers": {"resident_plateau_GBps": 7012.3}, "points": [{"resident_us": 3.4}] * 12},
            "bus": {"h2d_GBps": 57.3}}
    record = {"metric": "achieved GB/s (% of HBM peak) for decode-step GEMV sweep; tokens/s at batch 1", "value": 7204.11,
              "unit": "GB/s", "n_gpus": 1, "steps": 20, "warmup": 5, "ms_per_step": 19.3012, "higher_is_better": True,
              "scaling": "weak", "vs_baseline": None, "dtype": "bf16", "data": "synthetic", "config": {"step": "x" * 200},
              "tokens_per_s": 51.8, "hbm_frac": 0.9005, "roofline": {"bound": "hbm", "traffic": 141645873511.2},
              "probe_ceiling": {"GBps": 7000.1, "frac": 1.03, "note": "x" * 300},
              "cpu_baseline": {"value": 10.1, "unit": "GB/s", "cores": 16, "kind": "oracle", "sample": "x" * 300},
              "parity": {"worst_rel_l2": 1e-6, "rows": ["x"] * 100}, "passes": {"n": 5, "median": 19.3, "iqr": [19.2, 19.4],
              "ms_per_token": [19.3] * 5}, "rows": rows, "wall_s": 60.0}
    text = bench.short_line(record)
    assert "\n" not in text and len(text) <= bench.LINE_MAX
    line = json.loads(text)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline",
              "dtype", "data", "config"):
        assert line[k] == record[k], k
    assert set(line["rows"]) == set(rows)                       # all of them fit
    assert line["rows"]["llama8b_q4"]["matrix_cores16_tok_s"] == 17123.5 and line["passes"]["median"] == 19.3
    record["rows"]["endpoints"]["GBps"] = {"k" * 40 + str(i): 1.0 for i in range(60)}
    assert len(bench.short_line(record)) <= bench.LINE_MAX       # and a row that does not is left out
