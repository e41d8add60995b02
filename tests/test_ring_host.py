"""The upload ring of the kernels' tables, compiled for the host with the HIP calls replaced
(tests/native/ring_lifetime.cpp)."""
import os
import subprocess

from paper_1908_06043_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_tables_stay_whole_until_their_launch(tmp_path):
    obj, exe = str(tmp_path / "ring.o"), str(tmp_path / "ring")
    src = os.path.join(HERE, "native", "ring_lifetime.cpp")
    subprocess.run([build.hipcc(), "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1", "-fPIC", "-w", "-c", src, "-o", obj,
                    "-I", build.INCLUDE, "-I", build.CSRC], check=True, capture_output=True, text=True)
    subprocess.run(["g++", obj, "-o", exe], check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
