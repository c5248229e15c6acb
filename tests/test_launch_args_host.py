"""Host: the kernel launchers refuse filter lengths that no kernel has (compiled against the library's internal header and
linked with it; run only where no device could take a launch)."""
import os
import shutil
import subprocess

import pytest

from paper_2507_02401_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2507_02401_amd")


@pytest.mark.skipif(os.path.exists("/dev/kfd"), reason="made-up addresses: only where no launch can follow")
def test_lengths_without_a_kernel_are_refused(lib, tmp_path):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("g++ or the ROCm headers are missing")
    exe = str(tmp_path / "launch_check")
    so = os.path.join(os.path.dirname(os.path.abspath(_lib.__file__)), "libeswave.so")
    cmd = [gxx, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{os.path.join(ROOT, 'include')}",
           f"-I{os.path.join(PKG, 'csrc')}", os.path.join(ROOT, "tests", "native", "launch_check.cpp"), so, "-L/opt/rocm/lib",
           "-lamdhip64", "-lhipfft", f"-Wl,-rpath,{os.path.dirname(so)}", "-Wl,-rpath,/opt/rocm/lib", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("ok"), (r.returncode, r.stdout, r.stderr[-500:])
