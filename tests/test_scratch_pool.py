"""Who may use which scratch memory, on the CPU: the library's own code for it, linked with a model of the HIP runtime (scratch_pool_check.cpp)."""
import os
import subprocess

from paper_2603_06731_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_launches_that_share_scratch_memory_are_ordered(tmp_path):
    obj, main, exe = (str(tmp_path / n) for n in ("scratch.o", "check.o", "check"))
    for src, out in ((os.path.join(build.CSRC, "scratch.hip"), obj), (os.path.join(HERE, "scratch_pool_check.cpp"), main)):
        subprocess.check_call([build.HIPCC, "-x", "hip", "--offload-host-only", *build.FLAGS, "-c", src, "-o", out], stderr=subprocess.DEVNULL)
    subprocess.check_call(["g++", obj, main, "-o", exe])
    subprocess.check_call([exe])
