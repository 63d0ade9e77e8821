"""Host-side checks of bench.py: the one-GPU contract, the workload it times and
the committed traffic record it reports (no GPU needed)."""

import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402
from paper_2609_33601_amd import jq, workloads  # noqa: E402


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in r.stderr


def test_headline_workload_is_the_flux_mlp_pair():
    up, down = workloads.FLUX_MLP.linears
    assert (up.M, up.K, up.N) == (4608, 3072, 12288) and up.bias_std is not None
    assert (down.M, down.K, down.N) == (9216, 12288, 3072) and down.bias_std is None
    assert workloads.FLUX_MLP.ops == 2 * (4608 * 3072 * 12288 + 9216 * 12288 * 3072)


@pytest.mark.skipif(not os.path.exists(jq.LIB_PATH), reason="libjq.so not built (run __graft_entry__.build())")
def test_packed_engine_is_labelled_by_the_kernel_that_runs():
    from tests.routes import route

    for wl in workloads.WORKLOADS.values():
        for l in wl.linears:
            r = route("w4a4", l.M, l.K, l.N)
            rows, dtype, peak = bench.packed_gemm(l, jq, 256)
            assert rows == r.rows
            assert (peak == bench.PEAK_FP6_TOPS) == dtype.startswith("E2M3") == (r.kernel == "wide"), l.name
    assert all(bench.packed_gemm(l, jq, 256)[2] == bench.PEAK_FP6_TOPS for l in workloads.FLUX_MLP.linears)


@pytest.mark.parametrize("linear", ["mlp_down", "mlp_up"])
def test_traffic_record_is_well_formed(linear):
    rec = json.load(open(bench.TRAFFIC_FILE))
    k = rec["kernels"][linear]
    assert len(rec["gemm_source_sha256"]) == 64
    # measured HBM bytes can only exceed what the kernel must move
    assert k["fetch_bytes"] + k["write_bytes"] >= k["algorithmic_bytes"] > 0
    # the scales come from a plain device copy of known size
    assert 0.5 < rec["fetch_scale"] < 4 and 0.5 < rec["write_scale"] < 4


def test_shared_input_linears_draw_identical_activations():
    # every workload linear marked as sharing its predecessor's input draws the same activations
    for wl in list(workloads.WORKLOADS.values()) + [workloads.FLUX_MLP]:
        bench.check_shared_inputs(list(wl.linears))
    gate, up = workloads.WORKLOADS["dllm_block"].linears[:2]
    assert up.shares_input and bench._x_key(gate) == bench._x_key(up)


def test_shared_input_mismatch_is_refused():
    import dataclasses

    gate, up = workloads.WORKLOADS["dllm_block"].linears[:2]
    with pytest.raises(ValueError):
        bench.check_shared_inputs([gate, dataclasses.replace(up, x_seed=up.x_seed + 1)])
    with pytest.raises(ValueError):
        bench.check_shared_inputs([dataclasses.replace(gate, K=2 * gate.K), up])
    with pytest.raises(ValueError):
        bench.check_shared_inputs([up])


def test_percentiles_interpolate_order_statistics():
    p = bench.percentiles([float(v) for v in range(11)])
    assert (p["median"], p["p10"], p["p90"], p["min"], p["max"]) == (5.0, 1.0, 9.0, 0.0, 10.0)


def test_group_fold_bound_uses_the_valu_peak():
    # 256 CUs x 4 SIMDs x 16 lanes x 2.4 GHz of non-packed fp32 VALU
    assert bench.PEAK_VALU_LANE_OPS == 256 * 4 * 16 * 2.4e9
    assert bench.GROUP_FOLD_VALU == {"int8": 5, "bf6": 3}


def test_line_keeps_its_values_and_stays_short():
    spread = {k: 270.62550187110901 for k in ("median", "p10", "p90", "min", "max")}
    rec = {"name": "dllm_block", "workload": "w" * 120, "layer": "W4A4 group128 (int8 engine)", "us_per_step": 1214.2512345,
           "effective_TOPS": 1131.88441, "pct_int8_peak": 22.6, "per_step_us": spread, "linears": [{"name": "x"}] * 4,
           "valu_fold_bound": {"frac": 0.5622126176289962}}
    out = {"metric": "m", "value": 3836.009971791953, "ms_per_step": 0.2720736026763916, "per_step_us": spread,
           "steps": 20, "vs_baseline": None, "kernels": [{"engine": "bf6", "avg_us": 1 / 3, "per_launch_us": spread}] * 8,
           "secondary": [rec] * 16}
    line = bench.short_line(out)
    assert line["value"] == out["value"] and line["ms_per_step"] == out["ms_per_step"] and line["steps"] == 20
    assert line["per_step_us"]["median"] == 270.626 and line["kernels"][0] == {"engine": "bf6", "avg_us": 0.333333}
    assert line["secondary"][0] == {"name": "dllm_block", "layer": rec["layer"], "us_per_step": 1214.25,
                                    "median_us": 270.626, "effective_TOPS": 1131.88, "fold_bound_frac": 0.562213}
    assert len(json.dumps(line["secondary"])) < 3500
    assert bench.short_line({**out, "secondary": None})["secondary"] is None
