"""The staging ring under threads and failed launches (CPU; see staging_threads.cpp)."""
import os
import re
import subprocess

from paper_2608_10402_amd.build import _hipcc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_10402_amd", "csrc")
INC = ["-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I", "/opt/rocm/include"]


def _run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (cmd[0], r.stdout[-2000:], r.stderr[-2000:])
    return r.stdout


def test_staging_ring_under_threads(tmp_path):
    obj, exe = str(tmp_path / "api.o"), str(tmp_path / "staging")
    _run([_hipcc(), "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", *INC,
          "-c", os.path.join(CSRC, "tide_api.hip"), "-o", obj])
    # the device code that a full compile would embed
    fatbin = re.findall(r"\b__hip_fatbin\w*", _run(["nm", "-u", obj]))
    _run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", *INC,
          os.path.join(ROOT, "tests", "staging_threads.cpp"), os.path.join(CSRC, "plan.cpp"), obj,
          *["-Wl,--defsym=%s=0" % s for s in fatbin], "-o", exe, "-pthread"])
    assert _run([exe]).strip() == "ok"
