"""Device helpers compiled for the host and run on the CPU (no GPU needed).

``tests/host/trace_clamp.hip`` checks the clamp the attention kernels apply to
trace offsets read from device memory (every addressed trace stays inside the
packed buffers and within max_seqlen; valid offsets pass unchanged) and the
tile-classifier switches of the ``*_ex`` calls.  ``tests/host/stager_bounds.hip``
checks the addressing of every staged tile: each LDS slot written once, every
source read inside the trace's rows, and rows inside the trace copied
unchanged through the swizzle.  ``tests/host/decode_plan.hip`` checks that the
paged decode's units fit its grid and workspace, ``tests/host/launch_grids.hip`` how
the runs of a slot list are shared out to workgroups and the limit of the
backward's preprocess."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or ("/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else None)


@pytest.mark.skipif(HIPCC is None, reason="hipcc not available")
def test_trace_clamp_and_class_switches(tmp_path):
    exe = str(tmp_path / "trace_clamp")
    cmd = [HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2609_35750_amd", "csrc"), os.path.join(ROOT, "tests", "host", "trace_clamp.hip"),
           "-o", exe]
    subprocess.run(cmd, check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr


def _build_and_run(tmp_path, src, name):
    exe = str(tmp_path / name)
    cmd = [HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2609_35750_amd", "csrc"), os.path.join(ROOT, "tests", "host", src), "-o", exe]
    subprocess.run(cmd, check=True, capture_output=True, text=True)
    return subprocess.run([exe], capture_output=True, text=True, timeout=120)


@pytest.mark.skipif(HIPCC is None, reason="hipcc not available")
def test_tile_copy_addressing(tmp_path):
    r = _build_and_run(tmp_path, "stager_bounds.hip", "stager_bounds")
    assert r.returncode == 0 and r.stdout.rstrip().endswith("ok"), r.stdout + r.stderr


@pytest.mark.skipif(HIPCC is None, reason="hipcc not available")
def test_decode_units_fit(tmp_path):
    r = _build_and_run(tmp_path, "decode_plan.hip", "decode_plan")
    assert r.returncode == 0 and r.stdout.rstrip().endswith("ok"), r.stdout + r.stderr


@pytest.mark.skipif(HIPCC is None, reason="hipcc not available")
def test_launch_grids(tmp_path):
    r = _build_and_run(tmp_path, "launch_grids.hip", "launch_grids")
    assert r.returncode == 0 and r.stdout.rstrip().endswith("ok"), r.stdout + r.stderr


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_block_manager_out_of_memory(tmp_path):
    """Host only: a failed allocation in an append gives an error and leaves the manager as it was."""
    exe = str(tmp_path / "bm_memory")
    csrc = os.path.join(ROOT, "paper_2609_35750_amd", "csrc")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", csrc, os.path.join(ROOT, "tests", "host", "bm_memory.cpp"),
                    os.path.join(csrc, "kvs_cache.cpp"), "-o", exe], check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.rstrip().endswith("ok"), r.stdout + r.stderr
