"""Rules by which the host code picks kernels and launch shapes, from its own
headers compiled as a host program (no GPU)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    exe = str(tmp_path_factory.mktemp("host_rules") / "host_rules")
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature",
                    "-Xclang", "-packed-fp32-ops", "-o", exe, os.path.join(HERE, "host_rules.hip")],
                   check=True, capture_output=True, text=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    return {k: int(v) for k, v in (line.split() for line in out.splitlines())}


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_dual_launch_needs_the_cache_at_both_positions(rules, precision):
    # 3 reads the exchange cache, 2 the spline, 0 the positions
    assert rules[precision + "_cache_at_both"] == rules[precision + "_cache_single"] == 3
    assert rules[precision + "_cache_at_first"] == rules[precision + "_cache_at_second"] == 0
    assert rules[precision + "_spline_cache_at_first"] == (2 if precision == "fp32" else 0)


def test_bucket_sort_launch_is_within_the_device_limit(rules):
    # at most 2^32 - 1 threads in a launch: cells (two per atom) and lattice rows
    # times colours can be 2^26 and more
    for nbucket in (1, 5, 16384, 1 << 26, 1 << 30):
        threads = rules[f"sort_threads_{nbucket}"]
        assert 64 <= threads < 1 << 32 and threads >= 64 * min(nbucket, 16384)


def test_slot_groups_are_bounded_and_cover_the_row(rules):
    for rows in (1, 5, 6, 63, 80, 640, 641, 400000):
        slots, groups = rules[f"slots_{rows}"], rules[f"groups_{rows}"]
        assert slots % 5 == 0 and slots * groups >= rows and groups <= 128
        assert slots == 5 or rows > 640            # one round per group up to there


def test_benchmark_reports_the_default_lanes(rules):
    import sys
    sys.path.insert(0, os.path.dirname(HERE))
    import bench
    for prec in (bench.sl.SL_FP64, bench.sl.SL_FP32):
        for jc in (-1, 1):
            for m in (1, 3000, 3001, 70000, 70001, 108000):
                assert rules[f"spin_lanes_{prec}_{jc}_{m}"] == bench.default_spin_lanes(prec, m, jc > 0)
    for n in (1, 12000, 12001, 120000, 120001, 432000):
        assert rules[f"force_lanes_{n}"] == bench.default_force_lanes(n)


@pytest.mark.parametrize("system", ["small", "middle", "middle_fp32", "large", "frozen", "soc"])
def test_autotuner_tries_the_default_and_no_shape_twice(rules, system):
    r = {k[len(system) + 1:]: v for k, v in rules.items() if k.startswith(system + "_")}
    assert r["default_first"] == 1
    assert r["default_one_workgroup"] == (1 if system == "small" else 0)
    # every lane count, with the cache and without (with the spin-orbit terms none is
    # read); the default may be one of them
    assert r["distinct"] == r["count"] >= (4 if system == "soc" else 8)
    assert r["cached"] == 0 if system == "soc" else r["cached"] >= 4


@pytest.mark.parametrize("n", [1, 12000, 12001, 120000, 120001, 432000])
def test_force_lanes_that_are_set_are_those_that_run(rules, n):
    for lanes in (1, 2, 4, 8):
        for overlap in (-1, 1):
            assert rules[f"force_lanes_{n}_set_{lanes}_{overlap}"] == lanes
    assert rules[f"force_lanes_{n}_split"] == 1


@pytest.mark.parametrize("precision", [0, 1])
def test_cache_without_memory_is_off_until_set_again(rules, precision):
    assert [rules[f"cache_{precision}_{k}"] for k in ("on", "failed", "set_again")] == [1, 0, 1]


def test_benchmark_names_the_launches_that_ran():
    import sys
    sys.path.insert(0, os.path.dirname(HERE))
    import bench
    f64, f32 = bench.sl.SL_FP64, bench.sl.SL_FP32
    default = dict(spin_lanes=2, force_lanes=1, jcache=0)
    assert bench.launch_shape(default, f64, 432000, 4, 10) == (1, 1, True)
    assert bench.launch_shape(default, f32, 432000, 4, 10) == (4, 1, True)
    assert bench.launch_shape(default, f64, 16000, 4, 0) == (4, 4, False)
    assert bench.launch_shape(dict(spin_lanes=8, force_lanes=0, jcache=-1), f64, 16000, 4, 0) == (8, 4, False)
    assert bench.launch_shape(dict(spin_lanes=2, force_lanes=1, jcache=1), f64, 432000, 4, 10) == (2, 1, True)
