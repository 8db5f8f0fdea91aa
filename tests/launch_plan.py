"""The launch plan that a call makes (make_plan of csrc/t3_api.hip) for a device of 256 compute units; no GPU needed."""
import ctypes
import os
import subprocess
import tempfile

from paper_2401_16677_amd import build as hip_build

_lib = None


def lib():
    global _lib
    if _lib is None:
        with tempfile.TemporaryDirectory() as d:
            so = os.path.join(d, "plan_host.so")
            subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *hip_build.HIPCC_FLAGS, "-w", "-shared", "-I",
                            os.path.join(hip_build.ROOT, "include"), "-I", hip_build.CSRC,
                            os.path.join(hip_build.ROOT, "tests", "plan_host.hip"), "-o", so, "-L", hip_build.HERE, "-l:libt3.so",
                            "-Wl,-rpath," + hip_build.HERE], check=True, stderr=subprocess.DEVNULL)
            _lib = ctypes.CDLL(so)
    return _lib


def plan(p, call, before=0):
    """The plan's bytes; `before`: what every byte of its memory held."""
    out = ctypes.create_string_buffer(lib().plan_bytes())
    status = lib().make(ctypes.byref(p), call, before, out)
    assert status == 0, status
    return out.raw
