"""Host-side checks of the benchmark's bookkeeping (no GPU): how the N_T - 1
steps after the half step split into launches, the algorithmic bytes priced
on them, the remainder-free N_T used to time the K-step kernel alone, and
the refusal of more than one GPU."""

import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


@pytest.mark.parametrize("nt,fuse,expect", [
    (63, 4, [4] * 15 + [2]),        # the 1024^2 benchmark workload
    (63, 2, [2] * 31),
    (64, 4, [4] * 15 + [3]),
    (66, 4, [4] * 16 + [1]),
    (5, 3, [3, 1]),
    (3, 4, [2]),
    (6, 1, [1] * 5),
])
def test_step_launches_split_like_the_library(nt, fuse, expect):
    """K-step launches while K or more steps are left, then one shorter
    multi-step launch for two or three steps, or one single step."""
    got = bench.step_launches(nt, fuse)
    assert got == expect
    assert sum(got) == nt - 1


@pytest.mark.parametrize("nt", [4, 9, 63, 64, 65, 66, 121])
@pytest.mark.parametrize("fuse", [2, 3, 4])
def test_remainder_free_nt_gives_only_k_step_launches(nt, fuse):
    nt_k = fuse * ((nt - 1 + fuse - 1) // fuse) + 1
    assert nt_k >= nt and nt_k - nt < fuse
    assert set(bench.step_launches(nt_k, fuse)) == {fuse}


def test_phase_bytes_price_each_launch():
    nodes = 1047552
    b, n = bench.phase_bytes(2, "f64", 4, 63, nodes)
    assert n == 16
    assert b == 16 * bench.BYTES_PER_MULTI_LAUNCH["f64"] * nodes
    b1, n1 = bench.phase_bytes(2, "f64", 1, 63, nodes)
    assert n1 == 62 and b1 == 62 * bench.BYTES_PER_LUP[(2, "f64", 1)] * nodes
    # a single-step remainder is priced at the single step's bytes
    b2, n2 = bench.phase_bytes(2, "f32c", 4, 66, nodes)
    assert n2 == 17
    assert b2 == (16 * bench.BYTES_PER_MULTI_LAUNCH["f32c"] + bench.BYTES_PER_LUP[(2, "f32c", 1)]) * nodes


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in r.stderr


@pytest.mark.parametrize("nx,nrows,nt", [(1024, 1024, 63), (64, 64, 141), (611, 373, 90), (2, 2, 3)])
def test_register_tile_is_the_librarys(nx, nrows, nt):
    """Wavefronts, rows and steps per launch come from the library: a shape its
    kernels are built for, with inner rows left."""
    nw, r, h = bench.register_tile(nx, nrows, nt)
    assert (nw, r) in ((4, 4), (8, 3), (8, 4)) and 3 <= h <= min(12, nw * r // 2 - 1)


def test_traffic_is_read_for_the_kernel_that_runs(tmp_path, monkeypatch):
    """Counters count for the tiling and for the kernel sources they were taken with."""
    (tmp_path / "profiles").mkdir()
    csrc = tmp_path / "paper_2205_12344_amd" / "csrc"
    csrc.mkdir(parents=True)
    for family in bench.KERNEL_SOURCES:
        for f in bench.KERNEL_SOURCES[family]:
            (csrc / f).write_text(f)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    (tmp_path / "profiles" / "march3d_f64_cube256_counters.txt").write_text(
        f"kernel_source_hash: {bench.kernel_source_hash('3dmarch')}\ntraffic_bytes_per_launch[0,0]: 123\n")
    assert bench.read_traffic("march3d_f64_cube256", (0, 0), "3dmarch") == 123.0
    assert bench.read_traffic("march3d_f64_cube256", (6, 32), "3dmarch") is None
    (csrc / "kernels3d_k2.hip").write_text("changed")
    assert bench.read_traffic("march3d_f64_cube256", (0, 0), "3dmarch") == 123.0
    (csrc / "kernels3d_march.hip").write_text("changed")
    assert bench.read_traffic("march3d_f64_cube256", (0, 0), "3dmarch") is None


def test_kernel_sources_exist():
    for files in bench.KERNEL_SOURCES.values():
        for f in files:
            assert os.path.exists(os.path.join(ROOT, "paper_2205_12344_amd", "csrc", f)), f
