"""What a call of the library launches (kernel, workgroup tile, balanced tail), asked of the header that
decides it; no GPU needed.  The decision is compiled from csrc/t3_choice.h as the library's is."""
import ctypes
import os
import subprocess
import tempfile
from typing import NamedTuple

from paper_2401_16677_amd import binding as t3
from paper_2401_16677_amd import build as hip_build

GENERAL, WIDE, SMALL, REDUCTION = range(4)
FUSED, GEMM, REDUCE = range(3)
CUS = 256


class Shape(NamedTuple):
    kernel: int
    tile_m: int
    tile_n: int
    tpc: int
    begin: int
    limit: int
    blocks: int
    resident: int
    tail_r: int
    tail_q: int


class CopyShape(NamedTuple):
    """The all-gather step: lanes per row, 16-byte pieces per lane and batch, those in flight at once, workgroups."""
    team: int
    batch: int
    in_flight: int
    workgroups: int


_lib = None


def lib():
    global _lib
    if _lib is None:
        with tempfile.TemporaryDirectory() as d:
            so = os.path.join(d, "kernel_choice.so")
            subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                            os.path.join(hip_build.ROOT, "include"), "-I", hip_build.CSRC,
                            os.path.join(hip_build.ROOT, "tests", "kernel_choice.cpp"), "-o", so], check=True)
            _lib = ctypes.CDLL(so)
    return _lib


def launch_shape(p, call=FUSED, cus=CUS):
    tracked = (p.tile_m, p.tile_n) if p.tile_m else t3.t3_default_tile(p)
    out = (ctypes.c_int64 * 10)()
    lib().launch_shape(ctypes.byref(p), call, *tracked, cus, out)
    return Shape(*out)


def copy_shape(M, W, cus=CUS):
    out = (ctypes.c_int64 * 4)()
    lib().copy_shape(ctypes.c_int64(M), ctypes.c_int64(W), cus, out)
    return CopyShape(*out)


def start_offsets(p, call=FUSED, cus=CUS):
    """Phase groups and the window they start over, in ns."""
    tracked = (p.tile_m, p.tile_n) if p.tile_m else t3.t3_default_tile(p)
    out = (ctypes.c_double * 2)()
    lib().start_offsets(ctypes.byref(p), call, *tracked, cus, out)
    return tuple(out)


def tile_places(p, call=FUSED, cus=CUS, now=1e9):
    """(stage, row, column) of every grid position where tiles are put in a line, else None; columns of a band."""
    shape = launch_shape(p, call, cus)
    tracked = (p.tile_m, p.tile_n) if p.tile_m else t3.t3_default_tile(p)
    out = (ctypes.c_int32 * (3 * max(shape.blocks, 1)))()
    lib().tile_places.argtypes = [ctypes.c_void_p] + [ctypes.c_int] * 4 + [ctypes.c_double, ctypes.c_void_p]
    width = lib().tile_places(ctypes.byref(p), call, *tracked, cus, now, ctypes.byref(out))
    return ([tuple(out[3 * i:3 * i + 3]) for i in range(shape.blocks)], 1 << (width - 1)) if width else (None, 0)


def tile_order(p, call=FUSED, cus=CUS, xcds=8):
    """What the library decides: columns of a band of tiles in a line, or 0 stage by stage; blocks a stage is cut into by rows (0: runs),
    tile rows and columns of one."""
    tracked = (p.tile_m, p.tile_n) if p.tile_m else t3.t3_default_tile(p)
    blocks = (ctypes.c_int32 * 3)()
    width = lib().tile_order(ctypes.byref(p), call, *tracked, cus, xcds, blocks)
    return width, tuple(blocks)


def column_overlap(p, call=FUSED, cus=CUS):
    tracked = (p.tile_m, p.tile_n) if p.tile_m else t3.t3_default_tile(p)
    return lib().column_overlap(ctypes.byref(p), call, *tracked, cus)


def column_align(p, tile_n, call=FUSED):
    return lib().column_align(ctypes.byref(p), call, tile_n)
