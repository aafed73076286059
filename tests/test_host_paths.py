"""Host paths of libcorr against a stand-in for the HIP runtime (fake_hip.cpp):
what happens between the queueing of GPU work and its end, on the CPU."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_0906_1887_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"
INC = ["-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I", HERE]


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    from paper_0906_1887_amd import build
    tmp = str(tmp_path_factory.mktemp("host_paths"))
    objs = [os.path.join(build.BUILD, "corr_" + os.path.splitext(s)[0] + ".o") for s in build.SOURCES]
    newest = max(os.path.getmtime(os.path.join(CSRC, f)) for f in os.listdir(CSRC))
    if not all(os.path.exists(o) and os.path.getmtime(o) >= newest for o in objs):
        build.build()
    for name in ("fake_hip", "host_paths"):
        o = os.path.join(tmp, name + ".o")
        cmd = [HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-g", "-Wall", *INC,
               "-c", os.path.join(HERE, name + ".cpp"), "-o", o]
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-4000:]
        objs.append(o)
    out = os.path.join(tmp, "host_paths")
    r = subprocess.run(["/opt/rocm/llvm/bin/clang++", "-o", out, *objs, "-lpthread"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return out


def run(exe, scenario):
    r = subprocess.run([exe, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr[-4000:]


def test_dump_refuses_a_destination_that_is_too_small(exe):
    run(exe, "dump_range")


def test_dump_that_fails_waits_for_what_it_queued(exe):
    run(exe, "dump_failed_in_flight")


def test_submission_goes_on_while_fills_run(exe):
    run(exe, "submit_never_blocks")


def test_a_job_runs_while_the_next_one_is_filled(exe):
    run(exe, "fills_overlap")


def test_an_error_left_by_a_fill_fails_no_job(exe):
    run(exe, "error_of_a_fill")
