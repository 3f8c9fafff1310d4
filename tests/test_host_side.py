"""The library's host side (scratch, launches, graph cache) on a stand-in HIP
runtime: no GPU, no kernels, allocations refused where a check says so."""

import glob
import os
import subprocess

import pytest

from paper_1208_0277_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(build.HERE, "csrc")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    """The check program: the host halves of the device library's sources (the
    server aside), linked with the stand-in instead of the runtime."""
    d = tmp_path_factory.mktemp("host")
    sources = [f for f in sorted(glob.glob(os.path.join(CSRC, "*.hip"))) if not f.endswith("sccg_serve.hip")]
    inc = ["-I", os.path.join(build.ROOT, "include"), "-I", CSRC]
    sources += [os.path.join(HERE, f) for f in ("host_hip.cpp", "host_check.cpp")]
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17", *inc, "-c",
                    *sources], check=True, cwd=d)
    exe = d / "host_check"
    # the device code that the objects refer to is not there
    subprocess.run(["g++", "-no-pie", "-o", str(exe), *sorted(glob.glob(str(d / "*.o"))), "-Wl,--unresolved-symbols=ignore-all", "-pthread"],
                   check=True)
    return str(exe)


@pytest.mark.parametrize("name", ["join_out_of_memory", "join_launch_sizes", "errors_are_reported_once", "tiles_out_of_memory",
                                  "tiles_tried_again_with_new_parameters", "graph_of_repeated_arguments", "launches_within_a_dispatch",
                                  "lists_hold_their_pairs"])
def test_host_side(check, name):
    r = subprocess.run([check, name], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
