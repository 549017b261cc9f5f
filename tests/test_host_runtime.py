"""The library's host code (scratch memory, graph cache, launch shapes) on a HIP
runtime that only keeps account (host_runtime.cpp): no GPU, nothing computed."""
import os
import subprocess

import pytest

from paper_2407_07463_amd import _build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("host_runtime")
    objs = []
    for src in ("api", "advect", "batched"):
        objs.append(str(d / f"{src}.o"))
        subprocess.run([_build.HIPCC, *_build.HIP_FLAGS, "--cuda-host-only", "-x", "hip", "-c",
                        os.path.join(_build.CSRC, src + ".hip"), "-o", objs[-1]], check=True)
    exe = str(d / "host_runtime")
    # (the kernels' code is not linked: nothing follows the pointer to it)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-Wno-return-type-c-linkage",
                    "-I" + os.path.join(os.path.dirname(os.path.dirname(_build.HIPCC)), "include"), "-I" + _build.INCLUDE,
                    os.path.join(HERE, "host_runtime.cpp"), *objs, "-Wl,--unresolved-symbols=ignore-all", "-o", exe], check=True)
    return exe


def _holds(program, scenario):
    r = subprocess.run([program, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


def test_graph_after_failed_growth(program):
    _holds(program, "graph_after_failed_growth")


def test_call_after_no_memory(program):
    _holds(program, "call_after_no_memory")


def test_captured_third_copy(program):
    _holds(program, "captured_third_copy")


def test_third_copy_given_back(program):
    _holds(program, "third_copy_given_back")


def test_third_copy_leaves_room(program):
    _holds(program, "third_copy_leaves_room")


def test_tuning_holds_untuned(program):
    _holds(program, "tuning_holds_untuned")


def test_tuning_on_equal_fields(program):
    _holds(program, "tuning_on_equal_fields")
