"""bench.py's command line on a machine without a GPU: more than one GPU is
refused with a message, the per-set constants describe the kernels, the
roofline names the kernel the library launches for each workload, and a stage
that does not run is priced as none."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in r.stderr
    assert r.stdout == ""


def test_set_constants():
    sys.path.insert(0, ROOT)
    import bench
    s12, a15 = bench.SETS["s12"], bench.SETS["a15"]
    assert (s12["r"], s12["products"], s12["plane_bytes"]) == (12, 36, 30)
    assert (a15["r"], a15["products"], a15["plane_bytes"]) == (15, 15, 15)
    assert s12["cres_bytes"] == 12 * 2 and a15["cres_bytes"] == 15


def test_committed_counters_are_plausible():
    """The rocprofv3 counter summaries bench.py reads for roofline.traffic and
    roofline_deconstruct.measured_*: square workload, byte counts at least the
    algorithmic ones (planes read once per GEMM launch; FP64 read, planes
    written and one exponent-scan read per call), and taken on the current
    kernel sources (else skipped: the bench then reports null)."""
    sys.path.insert(0, ROOT)
    import bench
    import workloads
    w = workloads.WORKLOADS["square"]
    stale = []
    for name, cfg in bench.SETS.items():
        path = bench.COUNTER_FILES[name]
        kv = dict(line.split(":", 1) for line in open(path) if ":" in line and not line.startswith("#"))
        kv = {k.strip(): v.strip() for k, v in kv.items()}
        assert kv["workload"] == "square"
        planes = cfg["plane_bytes"] * (w.m * w.k + w.k * w.n)
        assert float(kv["hbm_bytes_per_launch"]) >= planes
        if bench.measured_traffic(w, name) is None:
            stale.append(path)
    kv = dict(line.split(":", 1) for line in open(bench.DEC_COUNTERS) if ":" in line and not line.startswith("#"))
    kv = {k.strip(): v.strip() for k, v in kv.items()}
    for name, cfg in bench.SETS.items():
        alg = (8 + cfg["plane_bytes"] + 8) * (w.m * w.k + w.k * w.n)
        assert 0.95 * alg <= float(kv[f"hbm_bytes_per_call_{name}"]) <= 1.5 * alg
    if bench.measured_deconstruction(w, "s12", 0.2, 1.0)["measured_bytes"] is None:
        stale.append(bench.DEC_COUNTERS)
    if stale:
        import pytest
        pytest.skip(f"counter summaries taken on older kernel sources: {stale}")


def test_gemm_kernel_names(monkeypatch):
    """The kernel named in the roofline object follows the library's rule:
    the persistent forms at an even count of 2-16 K stages with at least two
    tiles per CU (256 CUs here), the grid of one block per tile otherwise."""
    import types

    import torch
    sys.path.insert(0, ROOT)
    import bench
    import workloads
    monkeypatch.setattr(torch.cuda, "get_device_properties",
                        lambda i: types.SimpleNamespace(multi_processor_count=256))
    s12, a15 = bench.SETS["s12"], bench.SETS["a15"]
    W = workloads.WORKLOADS
    assert bench.gemm_kernel_name(W["hpl"], s12) == "residue_gemm_persistent_kernel<int16>"
    assert bench.gemm_kernel_name(W["hpl"], a15) == "residue_gemm_bytes_persistent_kernel<int8>"
    for name in ("square", "ragged", "reach", "tiny"):
        assert bench.gemm_kernel_name(W[name], s12) == "residue_gemm_kernel<int16>", name
        assert bench.gemm_kernel_name(W[name], a15) == "residue_gemm_bytes_kernel<int8>", name


def test_one_launch_rule_is_the_library_s():
    """bench.one_launch follows the library's rule (dispatch.hpp) on both
    sides of its line; beyond it fused(w) the storage-mode rule, and joint(w)
    the joint launches'."""
    import itertools
    sys.path.insert(0, ROOT)
    sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
    import bench
    import workloads
    from routes import route, rules
    sizes = (1, 31, 64, 300, 512, 1023, 1024, 2049, 6000, 40000)
    seen = set()
    for m, n, k in itertools.product(sizes, sizes, (1, 64, 65, 300, 640, 768, 1000, 4096, 4097)):
        w = workloads.Workload("x", m, n, k, 1.0, 1)
        want = route(m, n, k)
        seen.add(want)
        assert bench.one_launch(w) == (want == "one"), (m, n, k)
        assert want == "one" or bench.fused(w) == (want == "fused"), (m, n, k)
        if want == "staged":
            assert bench.joint(w) == bool(rules().rule_both_at_once(m, n, k, -(-k // 128) * 128, 1 << 40)), (m, n, k)
    assert seen == {"one", "fused", "staged"}


def test_stages_that_do_not_run_are_not_priced():
    """The tiny workload runs as one kernel: its event gaps, zero or not, are
    no scan, deconstruction or reconstruction rates."""
    sys.path.insert(0, ROOT)
    import bench
    import workloads
    w, cfg = workloads.WORKLOADS["tiny"], bench.DGEMM["s12"]
    for stages in ([0.0, 0.0, 0.007, 0.0], [0.002, 0.002, 0.007, 0.002]):
        rt = bench.rates(w, cfg, 0.01, stages)
        for r in (bench.dec_roofline(w, cfg, rt, *stages[:2]), bench.rec_roofline(w, rt)):
            assert r["achieved"] is None and r["frac"] is None and "one kernel" in r["note"]
        r = bench.gemm_roofline(w, cfg, rt)
        assert r["kernel"] == "one_kernel" and r["achieved"] == round(2 * 15 * 64 ** 3 / 0.007e-3 / 1e12, 2)
    w = workloads.WORKLOADS["reach"]
    rt = bench.rates(w, cfg, 0.05, [0.007, 0.02, 0.02, 0.006])
    assert bench.dec_roofline(w, cfg, rt, 0.007, 0.02)["achieved"] > 0 and bench.rec_roofline(w, rt)["achieved"] > 0
