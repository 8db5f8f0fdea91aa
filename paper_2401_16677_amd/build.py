"""Compile the HIP sources into paper_2401_16677_amd/libt3.so for gfx950 (in-tree)."""
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libt3.so")
BUILD_DIR = os.path.join(HERE, "_build")
# Translation units: (source, object, defines).  t3_gemm_launch.hip is compiled once per mode (0 plain
# GEMM, 1 fused) and operand layout, so that the kernel instantiations compile in parallel.
UNITS = [("t3_api.hip", "t3_api.o", [])] + [
    ("t3_gemm_launch.hip", f"{fn}.o",
     [f"-DT3_LAUNCHER={fn}", f"-DT3_MODE={mode}", f"-DT3_BKN={kn}", f"-DT3_AKM={km}"])
    for fn, mode, kn, km in [
        ("launch_fused", 1, 0, 0), ("launch_fused_kn", 1, 1, 0),
        ("launch_fused_km", 1, 0, 1), ("launch_fused_km_kn", 1, 1, 1),
        ("launch_gemm_nk", 0, 0, 0), ("launch_gemm_kn", 0, 1, 0),
        ("launch_gemm_km", 0, 0, 1), ("launch_gemm_km_kn", 0, 1, 1)]] + [
    ("t3_small_launch.hip", f"{fn}.o", [f"-DT3_LAUNCHER={fn}", f"-DT3_MODE={mode}"])
    for fn, mode in [("launch_small_fused", 1), ("launch_small_gemm", 0)]] + [
    ("t3_wide_launch.hip", f"{fn}.o",
     [f"-DT3_LAUNCHER={fn}", f"-DT3_MODE={mode}", f"-DT3_BKN={kn}", f"-DT3_AKM={km}", f"-DT3_OVERLAP={overlap}"])
    for fn, mode, kn, km, overlap in [
        ("launch_wide_fused", 1, 0, 0, 0), ("launch_wide_fused_kn", 1, 1, 0, 0),
        ("launch_wide_fused_km", 1, 0, 1, 0), ("launch_wide_fused_km_kn", 1, 1, 1, 0),
        ("launch_wide_overlap", 1, 0, 0, 1), ("launch_wide_overlap_kn", 1, 1, 0, 1),
        ("launch_wide_overlap_km", 1, 0, 1, 1), ("launch_wide_overlap_km_kn", 1, 1, 1, 1),
        ("launch_wide_gemm_nk", 0, 0, 0, 0), ("launch_wide_gemm_kn", 0, 1, 0, 0),
        ("launch_wide_gemm_km", 0, 0, 1, 0), ("launch_wide_gemm_km_kn", 0, 1, 1, 0)]]
DEPS = ["t3_api.hip", "t3_gemm_launch.hip", "t3_small_launch.hip", "t3_wide_launch.hip", "t3_choice.h", "t3_div.h", "t3_device.h", "t3_gemm.h",
        "t3_small.h", "t3_wide.h", "t3_aux.h", "t3_launch.h"]
JOBS = 8

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-mllvm", "-pragma-unroll-threshold=1000000",
    "-Wall", "-Wno-unused-command-line-argument",
]


def up_to_date():
    if not os.path.exists(LIB):
        return False
    t = os.path.getmtime(LIB)
    deps = [os.path.join(CSRC, d) for d in DEPS] + [os.path.join(ROOT, "include", "t3.h")]
    return all(os.path.getmtime(d) <= t for d in deps)


def build(force=True, extra_flags=()):
    if not force and up_to_date():
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(BUILD_DIR, exist_ok=True)
    objects = [os.path.join(BUILD_DIR, obj) for _, obj, _ in UNITS]

    def compile_unit(unit):
        src, obj, defines = unit
        subprocess.run([hipcc, *HIPCC_FLAGS, *extra_flags, *defines, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        "-c", os.path.join(CSRC, src), "-o", os.path.join(BUILD_DIR, obj)], check=True)

    with ThreadPoolExecutor(JOBS) as pool:
        list(pool.map(compile_unit, UNITS))
    subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objects], check=True)
    return LIB


C_CLIENT_SRC = os.path.join(ROOT, "tests", "c_abi_client.c")
C_CLIENT = os.path.join(ROOT, "tests", "c_abi_client")


def build_c_client(force=True):
    """Compile tests/c_abi_client.c, a plain C11 user of include/t3.h, with gcc against the
    built library and the HIP runtime (it is run by the GPU tests)."""
    if not force and os.path.exists(C_CLIENT) and \
            os.path.getmtime(C_CLIENT) >= max(os.path.getmtime(C_CLIENT_SRC), os.path.getmtime(LIB)):
        return C_CLIENT
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    cmd = ["gcc", "-std=c11", "-O1", "-Wall", "-Werror", "-D__HIP_PLATFORM_AMD__",
           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(rocm, "include"),
           C_CLIENT_SRC, "-o", C_CLIENT, "-L", HERE, "-l:libt3.so",
           "-L", os.path.join(rocm, "lib"), "-lamdhip64",
           "-Wl,-rpath,$ORIGIN/../paper_2401_16677_amd", "-Wl,-rpath," + os.path.join(rocm, "lib")]
    subprocess.run(cmd, check=True)
    return C_CLIENT


if __name__ == "__main__":
    print(build())
    print(build_c_client())
