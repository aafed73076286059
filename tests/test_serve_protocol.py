"""The serving queue's claim and publish protocols in every order in which their
loads and stores can take effect (tests/serve_model.cpp, on the CPU): one update
under running workgroups, for a slot's next job with fewer, more or as many
items, and for lists whose places move."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRC = os.path.join(HERE, "serve_model.cpp")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("serve") / "serve_model")
    r = subprocess.run(["/opt/rocm/bin/hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-O2", "-Wall",
                        "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_0906_1887_amd", "csrc"), SRC, "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


@pytest.mark.parametrize("scenario", ["shrinking", "growing", "equal", "moved", "longer", "shorter"])
def test_every_order_of_one_update(model, scenario):
    r = subprocess.run([model, scenario], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[1]) > 10       # executions: the orders were tried
