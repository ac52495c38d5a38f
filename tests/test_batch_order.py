"""Stream ordering of the batch scheduler, on the host: ``ns_batch.hip`` linked
with ``batch_order.cpp``, which stands in for the HIP runtime and the stage
kernels and checks that a member's steps follow each other whatever streams the
caller passes."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_steps_of_a_member_are_ordered(tmp_path):
    objs = []
    for name, src in (("batch.o", os.path.join(ROOT, "paper_1709_09713_amd", "csrc", "ns_batch.hip")),
                      ("order.o", os.path.join(HERE, "batch_order.cpp"))):
        obj = str(tmp_path / name)
        subprocess.check_call([HIPCC, "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17",
                               "-fPIC", "-w", "-I" + os.path.join(ROOT, "include"), "-c", src, "-o", obj])
        objs.append(obj)
    exe = str(tmp_path / "batch_order")
    subprocess.check_call(["g++", "-o", exe, *objs])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout + out.stderr
