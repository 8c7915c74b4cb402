"""Host logic of the library (memory, streams, threads, errors) on the CPU: the built library is
linked with a program that brings a HIP runtime of its own (tests/host/fake_hip.cpp), so its
kernels do nothing and its host code runs as it does on a device."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")
LIBDIR = os.path.join(ROOT, "paper_2006_16117_amd")
LIB = os.path.join(LIBDIR, "libsimm.so")

pytestmark = [pytest.mark.skipif(not os.path.exists(LIB), reason="library not built"),
              pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")]


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "host_cases")
    cmd = ["g++", "-std=c++17", "-O1", "-rdynamic", "-pthread", "-I", os.path.join(ROOT, "include"), "-I", HOST,
           os.path.join(HOST, "host_cases.cpp"), os.path.join(HOST, "fake_hip.cpp"), LIB, f"-Wl,-rpath,{LIBDIR}",
           "-Wl,--allow-shlib-undefined", "-ldl", "-o", exe]
    out = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert out.returncode == 0, out.stdout
    return exe


@pytest.mark.parametrize("case", ["batch_keeps_nothing", "kept_while_a_quarter_is_free",
                                  "sizes_in_use_are_kept", "factors_ahead_fit",
                                  "blocks_have_the_size_asked_for", "spikes_with_less_scratch",
                                  "whole_factor_where_it_fits", "three_at_once", "helpers_free_nothing",
                                  "threads_side_by_side", "no_threads", "no_host_memory"])
def test_host_case(program, case):
    out = subprocess.run([program, case], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert out.returncode == 0, f"exit status {out.returncode}\n{out.stdout}"
