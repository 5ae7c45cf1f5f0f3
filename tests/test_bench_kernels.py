"""The benchmark names kernels that the library has, and prices none of them
above its peak."""
import os
import subprocess

import pytest

import bench
from paper_2405_12964_amd import build


@pytest.fixture(scope="module")
def symbols():
    if not os.path.exists(build.LIB):
        pytest.skip("library not built")
    return subprocess.run(["nm", "-C", build.LIB], capture_output=True, text=True, check=True).stdout.replace(" ", "")


def test_named_kernels_exist(symbols):
    names = [bench.walk_kernel_name(dim, kind, stage) for dim in (2, 3) for kind in (0, 1) for stage in (0, 1, 2)]
    names += [bench.walk_kernel_name(3, 1, 0, cv=True), bench.walk_kernel_name(2, 1, 2, group=True)]
    names += ["wost_kernel<float,1>", "wost3_kernel<float,1>", "implicit_kernel<float,1>", "adjoint_kernel<float,2>"]
    for name in names:
        assert f"dwos::{name}(" in symbols, name


def test_traffic_lookup(monkeypatch, tmp_path):
    f = tmp_path / "t.txt"
    f.write_text(f"# sources_sha256: {bench.sources_sha256()}\n# nested_walks_per_terminal: 1\n"
                 "traffic_bytes_per_launch walk_kernel<float,3,0,0,false,false> 1.0e+09\n"
                 "traffic_bytes_per_launch walk_kernel<float,3,1,0,false,true> 2.0e+09\n"
                 "traffic_bytes_per_launch walk_kernel<float,3,1,0,false,false> 3.0e+09\n")
    monkeypatch.setitem(bench.TRAFFIC_FILES, "c3", str(f))
    assert bench.measured_traffic(bench.walk_kernel_name(3, 1, 0), 1, "c3") == 3e9
    assert bench.measured_traffic(bench.walk_kernel_name(3, 0, 1), 1, "c3") == 1e9
    assert bench.measured_traffic(bench.walk_kernel_name(2, 1, 0), 1, "c3") is None
    assert bench.measured_traffic(bench.walk_kernel_name(3, 1, 0), 2, "c3") is None


def test_roofline_of_the_default_workload(monkeypatch):
    """The default workload's counters and launch time: more bytes than HBM could
    deliver, which the caches serve, and a share of the arithmetic peak."""
    monkeypatch.setattr(bench, "probe_gather", lambda b: {"working_set_bytes": b})
    steps = 743877826 * 20
    tot = dict(steps=steps, nodes=10.851 * steps, prims=4.941 * steps)
    info = dict(node_bytes=5973024, prim_bytes=9600576)
    r = bench.roofline_3d(bench.walk_kernel_name(3, 1, 0), 1841.6, 20, tot, 1.4e11, info)
    assert r["cache_reads"]["GBs"] * 1e9 > bench.PEAK_HBM
    assert r["bound"] == "alu" and 0 < r["frac"] < 1 and 0 < r["hbm_frac"] < 1
    assert abs(r["frac"] - r["achieved"] / r["peak"]) < 1e-12
