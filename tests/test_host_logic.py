"""Host side of the library on a HIP runtime that does nothing (fake_hip.c),
without a GPU: what the entry points allocate, which class streams they take,
and what they leave behind when a launch fails."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    from paper_2406_03121_amd import build as hipbuild
    if not os.path.exists(hipbuild.LIB):
        hipbuild.build()
    so = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-pthread", os.path.join(HERE, "fake_hip.c"), "-o", so], check=True)
    return so


def run(fake, case):
    r = subprocess.run([sys.executable, os.path.join(HERE, "fake_hip_cases.py"), fake, case], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr


def test_noalloc_creates_nothing(fake):
    run(fake, "noalloc_creates_nothing")


def test_class_streams_per_caller(fake):
    run(fake, "streams_per_caller")


def test_class_streams_per_device(fake):
    run(fake, "streams_per_device")


def test_gradient_waits_for_its_copy(fake):
    run(fake, "gradient_waits_for_its_copy")


def test_xc_buffers_stay(fake):
    run(fake, "xc_buffers_stay")


def test_tensor_workspace(fake):
    run(fake, "tensor_workspace")
