"""The library's host code against a HIP runtime that runs nothing
(host/fake_hip.cpp): what it allocates, frees and launches, and when."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(ROOT, "paper_2403_04053_amd", "libpstd.so")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(LIB):
        pytest.skip("libpstd.so is not built")
    exe = str(tmp_path_factory.mktemp("host") / "fake_hip")
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-Wno-unused-result", os.path.join(HERE, "host", "fake_hip.cpp"), "-I",
                    os.path.join(ROOT, "include"), "-I", os.path.join(ROCM, "include"), "-o", exe, LIB,
                    "-Wl,-rpath," + os.path.dirname(LIB), "-Wl,-rpath," + os.path.join(ROCM, "lib"),
                    "-Wl,--allow-shlib-undefined"], check=True)
    return exe


@pytest.mark.parametrize("what", ["far_field_captured", "batch_rebuild", "batch_short_runs", "timed_launches"])
def test_host_code(program, what):
    p = subprocess.run([program, what], capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, p.stdout[-4000:] + p.stderr[-2000:]


def test_row_entries_of_every_tile_shape(tmp_path):
    exe = str(tmp_path / "row_entries")
    subprocess.run(["hipcc", "-std=c++17", "--offload-host-only", "-I",
                    os.path.join(ROOT, "paper_2403_04053_amd", "csrc"), os.path.join(HERE, "host", "row_entries.hip"),
                    "-o", exe], check=True, env=dict(os.environ, TMPDIR=str(tmp_path)))
    p = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0, p.stdout
