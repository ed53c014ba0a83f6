"""The host side of bench.py, without a GPU: the one-GPU contract, the HBM
traffic figure that follows the kernel source, and the CPU oracle legs."""
from __future__ import annotations

import os
import re
import shutil
import sys

import pytest

import bench
import seeded_inputs as si


def test_more_than_one_gpu_exits_with_a_message(monkeypatch, capsys):
    monkeypatch.setattr(sys, "argv", ["bench.py", "--gpus", "2"])
    with pytest.raises(SystemExit) as e:
        bench.main()
    assert e.value.code == 2
    assert "one GPU" in capsys.readouterr().err


def _recorded(path):
    """The kernel source hash a committed summary records, or None."""
    m = re.search(r"kernel_source_sha256:\s*([0-9a-f]{64})", open(path).read())
    return m and m.group(1)


def test_traffic_is_reported_only_for_the_profiled_kernel_source(monkeypatch, tmp_path):
    text = open(bench.TRAFFIC_SUMMARY).read()
    value = float(re.search(r"traffic_bytes_per_launch:\s*([0-9.eE+]+)", text).group(1))
    recorded = re.search(r"kernel_source_sha256:\s*([0-9a-f]{64})", text).group(1)
    if recorded != bench.kernel_source_sha256():   # measured before a kernel change
        assert bench.committed_traffic() is None
    # the source the counters were taken on gets their figure ...
    monkeypatch.setattr(bench, "kernel_source_sha256", lambda: recorded)
    assert bench.committed_traffic() == value
    monkeypatch.undo()
    # the counter summary is for the current kernel source; any other source
    # (here: one more comment line) gets no traffic figure
    src = tmp_path / "kernel.hip"
    shutil.copy(bench.KERNEL_SOURCE, src)
    with open(src, "a") as f:
        f.write("// edited\n")
    monkeypatch.setattr(bench, "KERNEL_SOURCE", str(src))
    assert bench.committed_traffic() is None


@pytest.mark.parametrize("workload", sorted(bench.TRAFFIC_SUMMARIES))
def test_traffic_summary_gives_its_workloads_bytes(monkeypatch, workload):
    """A workload with a counter summary gets its traffic figure on the source that it
    was measured on, at least the algorithmic bytes (Q, K, V read once, O and lse
    written once)."""
    recorded = _recorded(os.path.join(bench.PROFILES, bench.TRAFFIC_SUMMARIES[workload]))
    monkeypatch.setattr(bench, "kernel_source_sha256", lambda: recorded)
    w = si.WORKLOADS[workload]
    es = 1 if w.dtype == "e4m3" else 2
    alg = (w.B * w.N * (w.H * w.d + w.kv_heads * (w.d + w.d_v)) * es
           + w.B * w.H * w.N * (2 * w.d_v + 4))
    t = bench.committed_traffic(workload)
    assert t is not None and 0.99 * alg <= t <= 4 * alg, (t, alg)


def test_no_traffic_without_a_summary():
    assert bench.committed_traffic("mha_b1_h2_n128_d64_f16") is None


def test_profile_summaries_are_of_one_kernel_source():
    """The committed rocprofv3 summaries that record a kernel source hash record the same
    one: once some are measured again after a kernel change, none is left behind."""
    recorded = {name: _recorded(os.path.join(bench.PROFILES, name)) for name in sorted(os.listdir(bench.PROFILES))}
    recorded = {name: sha for name, sha in recorded.items() if sha}
    assert len(recorded) >= 2 and len(set(recorded.values())) == 1, recorded
    if bench.kernel_source_sha256() not in recorded.values():
        pytest.skip("the summaries predate the current kernel source")


def test_cpu_baseline_reports_the_oracle_on_host_cores():
    w = si.WORKLOADS["mha_b1_h2_n128_d64_f16"]
    q, k, v = w.inputs()
    r = bench.cpu_baseline(w, q, k, v)
    affinity, usable = bench.usable_cpus()
    assert r["kind"] == "oracle" and r["unit"] == "TFLOPS"
    assert r["cores"] == usable and r["cores_in_affinity"] == affinity and r["value"] > 0
    assert 1 <= usable <= affinity == len(os.sched_getaffinity(0))
    assert "2 of 2 (batch, head) slices" in r["sample"]


def test_cpu_single_core_times_whole_small_workloads():
    r = bench.cpu_single_core(names=("mha_b1_h2_n128_d64_f16",))
    assert set(r) == {"mha_b1_h2_n128_d64_f16"}
    assert r["mha_b1_h2_n128_d64_f16"]["seconds"] >= 0
    assert r["mha_b1_h2_n128_d64_f16"]["gflops"] > 0


def test_rocm_smi_json_gives_clock_and_power():
    """The sampler reads SCLK and a package-power key (rocm-smi JSON)."""
    import json
    text = json.dumps({"card0": {"sclk clock speed:": "(1804Mhz)",
                                 "Current Socket Graphics Package Power (W)": "1397.0"},
                       "system": {"Driver version": "6.x"}})
    assert bench.SclkSampler.parse(text) == (1804, 1397.0)
    assert bench.SclkSampler.parse(json.dumps({"card0": {}})) == (None, None)
