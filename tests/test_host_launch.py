"""Rules of the scalar path's launch that are decided on the host, checked without a GPU against the built library."""
import os
import shutil
import subprocess

import paper_2412_08902_amd.binding as hc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_a_mask_is_applied_or_refused(tmp_path):
    hc.load_library()
    pkg = os.path.join(ROOT, "paper_2412_08902_amd")
    exe = tmp_path / "mask_driver"
    r = subprocess.run([shutil.which("g++"), "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(pkg, "csrc"),
                        "-I", "/opt/rocm/include", os.path.join(ROOT, "tests", "host_sanitize", "mask_driver.cpp"), "-o", str(exe),
                        os.path.join(pkg, "libhcspmm.so"), "-Wl,-rpath," + pkg, "-Wl,-rpath-link,/opt/rocm/lib", "-L", "/opt/rocm/lib", "-lamdhip64"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    # no device is visible: nothing can be launched, on whatever machine this runs
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", LD_LIBRARY_PATH="/opt/rocm/lib:" + os.environ.get("LD_LIBRARY_PATH", ""))
    r = subprocess.run([str(exe)], capture_output=True, text=True, env=env, timeout=120)
    assert r.returncode == 0 and "mask driver: ok" in r.stdout, (r.stdout[-2000:], r.stderr[-4000:])
