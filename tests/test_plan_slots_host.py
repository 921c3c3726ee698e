"""The pinned slots of skrull_attn_plan when the runtime fails: its host code, compiled for the host only, on top of a
runtime that the test makes up (plan_slots.hip).  No GPU."""
import os
import shutil
import subprocess

import pytest

from paper_2505_19609_amd import build

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan_slots")
    objects = []
    for src in (os.path.join(build.CSRC, "api.hip"), os.path.join(HERE, "plan_slots.hip")):
        objects.append(str(d / (os.path.basename(src) + ".o")))
        subprocess.run(["hipcc", *build.FLAGS, "-w", "--cuda-host-only", "-c", src, "-o", objects[-1]], check=True)
    # (what the cases do not call stays undefined, the device code of api.hip among it)
    subprocess.run(["g++", "-no-pie", "-Wl,--unresolved-symbols=ignore-all", "-o", str(d / "program"), *objects, "-lpthread"],
                   check=True)
    return str(d / "program")


@pytest.mark.parametrize("case", ["wait_fails", "launch_fails", "failures_use_up_no_slots", "memory_is_coherent", "memory_comes_later"])
def test_slots(program, case):
    r = subprocess.run([program, case], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
