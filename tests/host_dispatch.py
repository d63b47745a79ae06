"""Runs a program against libsk.so over the fake HIP runtime (tests/host), in a
process of its own: no GPU, no torch."""
import os
import subprocess
import sys
import textwrap

import pytest

from paper_1808_10365_amd import _build

HOST = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host")


@pytest.fixture(scope="module")
def dispatch(tmp_path_factory):
    d = tmp_path_factory.mktemp("fake")
    fake = str(d / "libfake_hip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", os.path.join(HOST, "fake_hip.cpp"), "-o", fake,
                    "-lpthread"], check=True)

    def run(program: str):
        path = d / "program.py"
        path.write_text(textwrap.dedent(program))
        r = subprocess.run([sys.executable, os.path.join(HOST, "run.py"), fake, _build.LIB, str(path)],
                           capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr
        return r.stdout
    return run
