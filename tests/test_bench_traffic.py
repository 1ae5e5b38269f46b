"""bench.py --traffic-from on made-up counter files: which dispatches are filter steps, and
a step's bytes where it is several dispatches (one per group of vectors)."""

import csv
import json

import pytest

import bench

NS = "void hkp::(anonymous namespace)::"
STEP = NS + "stencil_pipe_kernel<float, float, float, 1, true, 32, 2, 6, false>(hkp::KArgs<float>)"
LAST = NS + "stencil_pipe_kernel<float, float, double, 1, true, 32, 2, 6, false>(hkp::KArgs<float>)"
OTHERS = [NS + "stencil_pipe_kernel<float, void, float, 1, true, 32, 2, 6, false>(hkp::KArgs<float>)",
          NS + "stencil_kernel<double, double, double, 1, true, 2, 6>(hkp::KArgs<double>)",
          NS + "rotate_kernel<40, true>(double*)"]


def _counters(path, counter, per_step):
    """A 1 GiB copy, then two steps of two groups each, among other kernels."""
    with open(path, "w", newline="") as f:
        w = csv.writer(f)
        w.writerow(["Kernel_Name", "Counter_Name", "Counter_Value"])
        w.writerow(["__amd_rocclr_copyBuffer", counter, 1 << 19])   # reads half of the truth
        for name in (STEP, STEP, LAST, LAST):
            w.writerow([name, counter, per_step / 2])
            for other in OTHERS:
                w.writerow([other, counter, 7])
        w.writerow([STEP, "SQ_WAVES", 5])


@pytest.mark.parametrize("warmup", [0, 1])
def test_a_step_is_the_sum_of_its_groups(tmp_path, monkeypatch, capsys, warmup):
    fetch, write, out = tmp_path / "f.csv", tmp_path / "w.csv", tmp_path / "t.json"
    _counters(fetch, "FETCH_SIZE", 3000)
    _counters(write, "WRITE_SIZE", 1000)
    line = {"steps": 1, "warmup": warmup,
            "roofline": {"algorithmic_bytes_per_launch": 4.0e6, "launches": 2 // (1 + warmup)}}
    log = tmp_path / "log"
    log.write_text("[bench] text\n" + json.dumps(line) + "\n")
    monkeypatch.setattr(bench, "TRAFFIC_JSON", str(out))
    bench.traffic_from(str(fetch), str(write), "2,4,1", 40, "fp32", str(log))
    e = json.loads(out.read_text())["by_launch"]["2,4,1/nb40"]
    assert (e["dispatches"], e["steps"]) == (4, 2)
    assert e["hbm_bytes_per_launch"] == pytest.approx(2 * 1024 * 4000)   # copy factor 2
    assert e["ratio"] == pytest.approx(2 * 1024 * 4000 / 4.0e6)
    assert bench._traffic_for(bench._src_hash(), "2,4,1/nb40", 4.0e6) == \
        pytest.approx(2 * 1024 * 4000)
    assert bench._traffic_for("another source", "2,4,1/nb40", 4.0e6) is None


def test_step_kernels_by_precision():
    assert bench._recurrence_step(STEP, "fp32") and bench._recurrence_step(LAST, "fp32")
    assert [bench._recurrence_step(n, "fp32") for n in OTHERS] == [False] * 3
    assert [bench._recurrence_step(n, "fp64") for n in OTHERS] == [False, True, False]
    assert bench._recurrence_step(STEP.replace("<float, float, float", "<double, double, double"),
                                  "fp64")
