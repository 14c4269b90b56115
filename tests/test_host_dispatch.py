"""What the host code chooses and asks memory for, without a GPU: libann.so against HIP functions that only note what is called
(tests/host_dispatch/calls.c)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    from paper_2512_02278_amd import ann

    ann.lib()  # raises if it has not been built
    exe = tmp_path_factory.mktemp("dispatch") / "calls"
    package = os.path.dirname(ann.LIB_PATH)
    subprocess.run(["gcc", "-std=gnu11", "-O1", "-Wall", "-rdynamic", "-I", os.path.join(ROOT, "include"), "-I", "/opt/rocm/include",
                    os.path.join(ROOT, "tests", "host_dispatch", "calls.c"), "-o", str(exe), ann.LIB_PATH, f"-Wl,-rpath,{package}",
                    "-Wl,-rpath,/opt/rocm/lib", "-Wl,--allow-shlib-undefined"], check=True)
    return exe


@pytest.mark.parametrize("scenario", ["scratch", "stand_ins", "searched_anew", "bytes_read", "ranked", "hash"])
def test_dispatch(program, scenario):
    r = subprocess.run([str(program), scenario], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and f"{scenario} ok" in r.stdout, r.stdout + r.stderr
