"""Host-side checks of bench.py that need no GPU: the traffic figure of the roofline object is read from the
rocprofv3 counter summary that measured it, so the summary must be there and carry the line the parser wants;
a multi-GPU request is refused with a message."""
import os
import re
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_traffic_is_read_from_the_committed_counter_summary():
    sys.path.insert(0, ROOT)
    import bench
    text = open(bench.TRAFFIC_PROFILE).read()
    assert "rocprofv3 --pmc FETCH_SIZE" in text and "rocprofv3 --pmc WRITE_SIZE" in text      # the commands that made it
    v = bench.traffic_from_profile()
    assert isinstance(v, int)
    # between the algorithmic bytes of the gate|up launch at 8192 rows (0.47 GB) and ten times that
    assert 0.4e9 < v < 5e9
    m = re.search(r"(\d+(?:\.\d+)?) MB read \+ (\d+(?:\.\d+)?) MB written per launch", text)
    assert m and abs((float(m.group(1)) + float(m.group(2))) * 1e6 - v) < 0.01 * v        # the line agrees with the table above it


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode != 0 and "one GPU" in r.stderr


def test_the_result_line_is_short():
    """With as many samples as the default run makes, each with its per-kernel split, the line stays below 8 KB, headline first."""
    sys.path.insert(0, ROOT)
    import json
    import bench
    row = {"M": 8192, "M_over_N": 1.0, "ms": 90.1234, "rows_per_s": 90909, "kernels": {str(i): {"us": 1234.5, "mfma_frac": 0.1234, "hbm_frac": 0.1234}
                                                                                      for i in range(10)},
           "gemm_mfma_frac": 0.1234, "gemm_hbm_frac": 0.1234}
    out = {"metric": "m" * 80, "value": 1.0, "config": {"workload": "w" * 900}, "roofline": {"per_kernel": row["kernels"], "note": "n" * 700},
           "cpu_baseline": {"sample": "s" * 1200}, "achievable": {"note": "a" * 500}, "latency_vs_active_fraction": {k: "l" * 400 for k in "abc"},
           "sweep": {k: [row] * 7 for k in ("c5", "c4", "c3")}, "c2": {"workload": "x" * 100, "sweep": [row] * 5}}
    line = json.dumps(bench.short(out))
    assert len(line) < 8000 and line.startswith('{"metric"') and len(json.dumps(out)) > 2 * len(line)
    assert bench.short(dict(out, c2=None))["c2"] is None
    assert [r["M"] for r in bench.short(out)["sweep"]["c4"]] == [8192] * 7
