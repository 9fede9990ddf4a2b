"""The memory kept between index builds, its book-keeping on the CPU: index_memory.cpp compiled against a made-up
runtime that only counts (so that blocks of gigabytes cost nothing)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    folder = tmp_path_factory.mktemp("index_memory")
    os.makedirs(folder / "hip")
    with open(folder / "hip" / "hip_runtime.h", "w") as f:
        f.write('#include "%s"\n' % os.path.join(HOST, "hip_runtime_stub.h"))
    out = str(folder / "check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-pthread", "-Wall", "-I", str(folder),
                    "-I", os.path.join(ROOT, "paper_2309_15479_amd", "csrc"),
                    os.path.join(HOST, "index_memory_check.cpp"), "-o", out], check=True)
    return out


@pytest.mark.parametrize("check", ["reuse", "no_exceptions", "slack", "limit", "scratch_limit", "out_of_memory", "threads"])
def test_index_memory(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
