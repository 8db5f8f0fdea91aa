"""CPU-only checks of the launch plan (csrc/t3_api.hip)."""
import pytest

from paper_2401_16677_amd import binding as t3
from tests.launch_plan import plan
from tests.launch_shape import FUSED, GEMM, GENERAL, REDUCE, REDUCTION, SMALL, WIDE, launch_shape


@pytest.mark.parametrize("call,kernel,sizes,kw", [
    (FUSED, GENERAL, (4096, 12288, 1536, 8), dict(tile_begin=1)),
    (FUSED, GENERAL, (4096, 12288, 1536, 8), dict(flags=t3.T3_FLAG_TWO_WRITERS, split_k=2)),
    (FUSED, SMALL, (24, 12288, 1536, 8), {}),
    (FUSED, WIDE, (4096, 12288, 1536, 8), {}),
    (FUSED, WIDE, (2048, 20480, 10240, 8), dict(flags=t3.T3_FLAG_FWD_DIRECT)),
    (GEMM, GENERAL, (163840, 2048, 8192, 4), dict(a_layout=t3.T3_A_KM)),
    (GEMM, SMALL, (24, 12288, 1536, 8), {}),
    (GEMM, WIDE, (2048, 20480, 10240, 8), {}),
    (REDUCE, REDUCTION, (4096, 12288, 1536, 8), {}),
])
def test_a_plan_depends_on_the_call_alone(call, kernel, sizes, kw):
    """No byte of it is what its memory held before, an earlier call's plan for one."""
    M, N, K, tp = sizes
    p = t3.problem(M, N, K, tp, 3 % tp, 256, 256, **kw)
    assert launch_shape(p, call).kernel == kernel
    clean = plan(p, call)
    for before in (0xFF, 0x5A):
        again = plan(p, call, before)
        assert again == clean, [i for i, (a, b) in enumerate(zip(again, clean)) if a != b]
