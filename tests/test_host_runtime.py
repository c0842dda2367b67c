"""The library's host code -- which device it works on, what it does with memory when a call fails -- without a GPU: the
built libctkvr.so against a stand-in for the HIP runtime (host_runtime/fake_hip.cpp), one process per scenario."""
import os
import subprocess
import sys

import pytest

from tests.host_runtime.scenarios import SCENARIOS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("fake_hip") / "libfake_hip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-o", lib, os.path.join(ROOT, "tests", "host_runtime", "fake_hip.cpp")],
                   check=True)
    return lib


@pytest.mark.parametrize("name", SCENARIOS)
def test_host_code(fake, name):
    r = subprocess.run([sys.executable, "-m", "tests.host_runtime.scenarios", name, fake], cwd=ROOT, capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0 and r.stdout.endswith("ok\n"), r.stdout + r.stderr
