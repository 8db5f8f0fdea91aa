"""CPU-only checks of which kernel serves a call, on which workgroup tile (csrc/t3_choice.h)."""
import ctypes

import numpy as np
import pytest

from paper_2401_16677_amd import binding as t3
from tests.launch_shape import lib as choice_lib
from tests.launch_shape import FUSED, GEMM, GENERAL, REDUCE, REDUCTION, SMALL, WIDE, column_align, column_overlap, copy_shape, launch_shape, start_offsets, tile_order, tile_places


def _problem(M, W, K, tp, layout="nk", **kw):
    return t3.problem(M, W * tp, K, tp, 0, b_layout=t3.T3_B_KN if "kn" in layout else t3.T3_B_NK,
                      a_layout=t3.T3_A_KM if "km" in layout else t3.T3_A_MK, **kw)


@pytest.mark.parametrize("call", [FUSED, GEMM, REDUCE])
def test_tile_and_tail_follow_the_device(call):
    """The tile is chosen, and the workgroups and the balanced tail counted, for the compute units there are."""
    p = _problem(2048, 2560, 10240, 8)
    whole, half = launch_shape(p, call, 256), launch_shape(p, call, 128)
    assert whole.resident == 256 and half.resident == 128
    if call == REDUCE:
        assert whole.kernel == half.kernel == REDUCTION
        few = _problem(64, 256, 64, 8)
        assert launch_shape(few, REDUCE, 16).tile_m > launch_shape(few, REDUCE, 256).tile_m
    else:
        assert (whole.kernel, whole.tile_m, whole.tile_n, whole.tail_r, whole.tail_q) == (WIDE, 256, 256, 128, 2)
        assert (half.tail_r, half.tail_q) == (0, 0) and half.blocks == 640      # five whole rounds
        # a problem of one round on 256 units is several on 64, and takes larger tiles there
        few = _problem(1024, 512, 1536, 8)
        a, b = launch_shape(few, call, 256), launch_shape(few, call, 64)
        assert a.tile_m * a.tile_n < b.tile_m * b.tile_n


def test_random_problems_are_covered_once():
    """Workgroup tiles of a random problem: the range covers whole steps of the tracked one, the
    balanced tail splits what the last round leaves, and ranges that cut a step stay in tracked tiles."""
    rng = np.random.default_rng(5)
    for _ in range(400):
        tp = int(rng.choice([1, 2, 3, 8, 16, 32]))
        layout = str(rng.choice(["nk", "kn", "km_kn"]))
        M, W = int(rng.integers(1, 700)) * 8, int(rng.integers(1, 200)) * 8
        K = int(rng.integers(1, 40)) * 64 if layout != "nk" else int(rng.integers(1, 300)) * 8
        p = _problem(M, W, K, tp, layout)
        tpc = t3.t3_tiles_per_chunk(p)
        lo = int(rng.integers(0, tp))
        hi = int(rng.integers(lo + 1, tp + 1))
        cut = bool(rng.integers(0, 2)) and tpc > 1
        p = _problem(M, W, K, tp, layout, tile_begin=lo * tpc + cut, tile_limit=hi * tpc)
        for call in (FUSED, GEMM, REDUCE):
            s = launch_shape(p, call)
            Mt, Wt = -(-M // s.tile_m), -(-W // s.tile_n)
            assert s.tpc == Mt * Wt
            if cut:
                assert (s.tile_m, s.tile_n) == t3.t3_default_tile(p) and (s.begin, s.limit) == (lo * tpc + 1, hi * tpc)
            else:
                assert (s.begin, s.limit) == (lo * s.tpc, hi * s.tpc) and s.blocks == (hi - lo) * s.tpc
            assert (s.kernel, s.tile_m, s.tile_n) != (SMALL, 32, 64) or layout.endswith("kn"), p
            if s.tail_r:
                assert s.kernel == WIDE and s.tail_q * s.resident + s.tail_r == s.blocks and 2 * s.tail_r <= s.resident


# One problem for every kernel and workgroup tile there is.
@pytest.mark.parametrize("M,W,K,tp,layout,want", [
    (4096, 1536, 1536, 8, "nk", (WIDE, 256, 256)),
    (1536, 1536, 4096, 8, "km_kn", (WIDE, 256, 192)),
    (512, 512, 4096, 32, "nk", (WIDE, 256, 128)),
    (4096, 1536, 1536, 1, "nk", (WIDE, 128, 192)),
    (2048, 512, 1536, 8, "nk", (WIDE, 128, 128)),
    (64, 384, 128, 32, "nk", (SMALL, 64, 64)),
    (8, 384, 4096, 32, "kn", (SMALL, 32, 64)),
    (256, 256, 256, 4, "nk", (SMALL, 32, 32)),
    (8, 384, 65536, 32, "nk", (SMALL, 32, 32)),      # (32 x 64 is not built for B stored N x K)
    (8, 384, 65536, 32, "km", (SMALL, 32, 32)),
])
def test_every_tile_has_a_problem(M, W, K, tp, layout, want):
    s = launch_shape(_problem(M, W, K, tp, layout))
    assert (s.kernel, s.tile_m, s.tile_n) == want


def test_problems_of_the_gpu_tests_get_the_tiles_they_are_meant_for():
    from tests.test_gpu_workgroup_tiles import MODES, PICKED_MODES, picked_range
    for case, mode in PICKED_MODES:
        M, W, K, tp, layout, _, tile, tail_r = case
        begin, limit = picked_range(case)
        p = _problem(M, W, K, tp, layout, tile_begin=begin, tile_limit=limit, flags=MODES[mode])
        s = launch_shape(p, GEMM if mode == "unfused" else FUSED)
        assert (s.kernel, s.tile_m, s.tile_n, s.tail_r) == (SMALL if tile == (32, 64) else WIDE, *tile, tail_r), (case, mode)


def test_cases_by_rounds_of_the_gpu_tests_are_what_they_say():
    from tests.test_gpu_workgroup_tiles import ROUNDS
    for M, W, K, tp, layout, tile, tiles in ROUNDS:
        for call in (FUSED, GEMM):
            s = launch_shape(_problem(M, W, K, tp, layout), call)
            assert (s.kernel, s.tile_m, s.tile_n, s.blocks) == (SMALL, *tile, tiles), (M, W, K, tp)


def test_granule_cases_of_the_gpu_tests_are_what_they_say():
    from tests.test_gpu_workgroup_tiles import GRANULE_MODES
    for case, mode in GRANULE_MODES:
        M, W, K, tp, layout, tile, tail_r, early = case
        p = _problem(M, W, K, tp, layout, flags=t3.T3_FLAG_FWD_BF16 if mode == "bf16_copy" else 0)
        call = GEMM if mode == "unfused" else FUSED
        s = launch_shape(p, call)
        assert (s.kernel, s.tile_m, s.tile_n, s.tail_r) == (WIDE, *tile, tail_r), (case, mode)
        assert column_align(p, s.tile_n, call) == (15 if early else 0), (case, mode)


def test_general_kernel():
    p = _problem(4096, 1536, 1536, 8, tile_m=256, tile_n=256, tile_begin=1)
    assert launch_shape(p).kernel == GENERAL                     # a range that cuts a step
    p = _problem(4096, 1536, 1536, 8, tile_m=128, tile_n=128, flags=t3.T3_FLAG_TWO_WRITERS)
    s = launch_shape(p)
    assert (s.kernel, s.tile_m, s.tile_n) == (GENERAL, 128, 128)
    assert launch_shape(p, GEMM).kernel == WIDE                  # (the plain GEMM has no second writer)


@pytest.mark.parametrize("M,W,K,tp,layout,wide", [
    (160000, 512, 8192, 4, "nk", True),          # A of 2.4 GiB
    (512, 16384, 10240, 8, "nk", True),          # B of 2.5 GiB
    (65536, 1536, 1536, 8, "nk", True),          # R of 3 GiB
    (65536, 1536, 1536, 8, "km_kn", True),       # R of 3 GiB, operands small
    (512, 16384, 10240, 8, "kn", False),         # B of 2.5 GiB, stored K x N
    (163840, 512, 8192, 4, "km", False),         # A of 2.5 GiB, stored K x M
])
def test_arrays_of_more_than_2_gib(M, W, K, tp, layout, wide):
    """Only a transposed operand past 2 GiB keeps a problem from the wide-tile kernel."""
    for call in (FUSED, GEMM):
        assert (launch_shape(_problem(M, W, K, tp, layout), call).kernel == WIDE) == wide


def test_division_without_dividing():
    """Numbers below 2^31 by 1 .. 2^31 - 1: edges of every power of two and of the quotients, and random ones."""
    rng = np.random.default_rng(9)
    near = np.unique(np.clip((2 ** np.arange(31, dtype=np.int64))[:, None] + np.arange(-3, 4), 1, 2 ** 31 - 1))
    d = np.concatenate([np.repeat(near, 40), rng.integers(1, 2 ** 31, 20000), rng.integers(1, 3000, 20000)])
    n = rng.integers(0, 2 ** 31, d.size)
    n[::3] = np.clip(n[::3] // d[::3] * d[::3] - rng.integers(0, 2, n[::3].size), 0, 2 ** 31 - 1)
    n[:near.size] = 2 ** 31 - 1
    u32 = [np.ascontiguousarray(x, dtype=np.uint32) for x in (n, d, np.zeros(d.size))]
    choice_lib().divide(*[x.ctypes.data_as(ctypes.c_void_p) for x in u32], d.size)
    assert np.array_equal(u32[2], n // d)


def test_columns_start_at_granules_where_the_grid_has_room():
    """Every column of a chunk falls to one tile, no tile is wider than it is, and none but a chunk's first
    starts inside a 64-byte granule."""
    aligned = 0
    for layout, step in (("nk", 4), ("kn", 8)):
        for W in range(step, 1100, step):
            p = _problem(512, W, 256, 8, layout)
            for bn in (128, 192, 256):
                mask = column_align(p, bn)
                assert mask in (0, 15) and column_align(p, bn, GEMM) == mask
                # (sizes alone decide: nothing is known of the buffer, and its rows may be padded)
                padded = _problem(512, W, 256, 8, layout, ldr=8 * W + 4, ldc=8 * W + 4)
                assert column_align(padded, bn) == column_align(padded, bn, GEMM) == mask
                assert column_align(_problem(512, W, 256, 8, layout, flags=t3.T3_FLAG_FWD_DIRECT), bn) == 0
                if not mask:
                    continue
                aligned += 1
                for c in range(8):
                    shift = c * W & mask
                    starts = [j * bn - (shift if j else 0) for j in range(-(-W // bn))] + [W]
                    assert all(0 < b - a <= bn for a, b in zip(starts, starts[1:])), (W, bn, c)
                    assert all((c * W + a) % 16 == 0 and a % step == 0 for a in starts[1:-1]), (W, bn, c)
    assert aligned > 100


def test_all_gather_step_shapes():
    """The workgroups hold all rows, one of them no more than it needs; the cases of the GPU test reach every kernel there is."""
    from tests.test_gpu_parity import COPIES
    kinds = {(256, 1, 1), (256, 8, 8), (64, 4, 4), (64, 4, 1), (64, 8, 8), (64, 8, 2), (64, 8, 1), (16, 4, 4), (4, 4, 4)}
    assert {copy_shape(M, W)[:3] for M, W in COPIES} == kinds
    rng = np.random.default_rng(12)
    for _ in range(2000):
        M, W = int(2 ** rng.uniform(0, 18)), 4 * int(2 ** rng.uniform(0, 12))
        for cus in (64, 256):
            s = copy_shape(M, W, cus)
            assert s[:3] in kinds and (s.workgroups - 1) * (256 // s.team) < M <= s.workgroups * (256 // s.team)
            assert s.in_flight == s.batch or 4 * cus <= s.workgroups <= 8 * cus


DIRECT = t3.T3_FLAG_FWD_DIRECT


@pytest.mark.parametrize("M,W,K,tp,call,flags,tile,want", [
    # 256 x 256 tiles: direct from two rounds on, by copy from three, or eight slabs
    (8192, 1024, 192, 4, FUSED, DIRECT, (256, 256), (4, 12000)),
    (8192, 1024, 192, 4, FUSED, 0, (256, 256), (4, 4000)),
    (8192, 1024, 512, 4, FUSED, 0, (256, 256), (4, 12000)),
    (4096, 1536, 192, 8, FUSED, 0, (256, 256), (4, 12000)),
    (4096, 1536, 128, 8, FUSED, 0, (256, 256), (4, 4000)),              # two slabs
    (4096, 1536, 128, 8, FUSED, DIRECT, (256, 256), (4, 12000)),
    (16384, 1024, 704, 8, FUSED, 0, (256, 256), (4, 12000)),            # eight rounds, 11 slabs
    (16384, 1024, 768, 8, FUSED, 0, (256, 256), (8, 16000)),            # 12
    (4096, 1536, 768, 8, FUSED, DIRECT, (256, 256), (4, 12000)),        # three rounds
    (4096, 1536, 4032, 8, FUSED, DIRECT, (256, 256), (4, 12000)),
    (4096, 1536, 4096, 8, FUSED, DIRECT, (256, 256), (0, 0)),
    # 256 x 192
    (8192, 576, 448, 8, FUSED, DIRECT, (256, 192), (4, 4000)),
    (8192, 576, 512, 8, FUSED, DIRECT, (256, 192), (4, 12000)),
    (14748, 576, 1152, 4, FUSED, DIRECT, (256, 192), (4, 6000)),        # less than three rounds
    (16384, 576, 384, 8, FUSED, DIRECT, (256, 192), (4, 12000)),        # six
    (8192, 1152, 1152, 16, FUSED, DIRECT, (256, 192), (8, 16000)),
    (4460, 1152, 1024, 16, FUSED, DIRECT, (256, 192), (4, 12000)),      # 6.75
    # the plain GEMM: half a tile time unless there are rounds enough
    (8192, 572, 200, 8, GEMM, 0, (256, 192), (4, 256 * 192 * 200 / 6250)),
    (4096, 1536, 192, 8, GEMM, 0, (256, 256), (4, 256 * 256 * 192 / 6250)),
    (16384, 512, 512, 8, GEMM, 0, (256, 256), (4, 12000)),              # four
    (16384, 512, 448, 8, GEMM, 0, (256, 256), (4, 256 * 256 * 448 / 6250)),
    (16384, 1536, 256, 4, GEMM, 0, (256, 256), (4, 12000)),             # six
    (16384, 1536, 192, 4, GEMM, 0, (256, 256), (4, 256 * 256 * 192 / 6250)),
    (4096, 1536, 1536, 8, GEMM, 0, (256, 256), (4, 12000)),
    # an eighth of the columns past the chunk's end; one round; smaller tiles
    (8192, 388, 200, 8, FUSED, 0, (256, 256), (4, 256 * 256 * 200 / 6250)),
    (4096, 512, 1536, 8, FUSED, 0, (256, 256), (0, 0)),
    (8728, 144, 256, 8, FUSED, 0, (128, 192), (4, 128 * 192 * 256 / 6250)),
])
def test_start_up_offsets(M, W, K, tp, call, flags, tile, want):
    p = _problem(M, W, K, tp, flags=flags)
    assert launch_shape(p, call)[1:3] == tile
    assert start_offsets(p, call) == pytest.approx(want)
    off_granules = _problem(M, W, K, tp, flags=flags, ldr=W * tp + 4, ldc=W * tp + 4)
    few = launch_shape(p, call).blocks // 256 < (3 if call == FUSED and flags & DIRECT else 6)
    if few and want[0]:                          # (rows off 64-byte granules)
        want = (4, min(12000, tile[0] * tile[1] * K / 6250))
    assert start_offsets(off_granules, call) == pytest.approx(want)


def test_tiles_in_a_line():
    """Every tile once, its stage no further than two rounds from its place in the issue order; a band is no larger than a round or
    lies inside a stage."""
    rng = np.random.default_rng(11)
    lines = 0
    for _ in range(600):
        col = 32
        M, W, K = (int(round(np.exp(rng.uniform(np.log(a), np.log(b))))) for a, b in ((128, 16384), (32, 4096), (256, 4096)))
        p = _problem(M, max(col, W // col * col), K // 8 * 8, int(rng.integers(1, 33)))
        call, cus = int(rng.choice([FUSED, GEMM])), int(rng.choice([256, 256, 64, 20, 7]))
        shape = launch_shape(p, call, cus)
        if shape.kernel != WIDE or not 0 < shape.blocks <= 40000:
            continue
        places, width = tile_places(p, call, cus)
        assert places is not None
        lines += 1
        Mt = -(-M // shape.tile_m)
        Wt = shape.tpc // Mt
        assert sorted(places) == [(s, r, c) for s in range(shape.blocks // shape.tpc) for r in range(Mt) for c in range(Wt)]
        round_ = min(shape.blocks, shape.resident)
        assert width == 1 or Mt * width <= round_ or Wt % width == 0
        for i, (s, _, _) in enumerate(places):
            assert s * shape.tpc - 2 * round_ <= i < (s + 1) * shape.tpc + 2 * round_
    assert lines > 150


def test_chunks_in_a_line_are_complete_no_more_than_a_round_later():
    """As the header has it: a tile is worked on in its stage, or a round from where it would be in issue order, and so is a chunk's last."""
    rng = np.random.default_rng(12)
    later, chunks = 0, 0
    for _ in range(400):
        M, W, K = (int(round(np.exp(rng.uniform(np.log(a), np.log(b))))) for a, b in ((128, 16384), (32, 4096), (256, 4096)))
        p = _problem(M, max(4, W // 4 * 4), K // 8 * 8, int(rng.integers(1, 33)), flags=DIRECT)
        shape = launch_shape(p)
        if shape.kernel != WIDE or not 0 < shape.blocks <= 40000 or not tile_order(p)[0]:
            continue
        places, _ = tile_places(p)
        Mt = -(-M // shape.tile_m)
        index = np.array([s * shape.tpc + c * Mt + r for s, r, c in places])         # issue index of every position
        here, there = np.arange(index.size) // shape.resident, index // shape.resident
        inside = np.arange(index.size) // shape.tpc == index // shape.tpc
        assert np.all(inside | (abs(here - there) <= 1)), p
        ends = np.array([here[index // shape.tpc == s].max() for s in range(index.size // shape.tpc)])
        due = (np.arange(1, ends.size + 1) * shape.tpc - 1) // shape.resident
        assert np.all(ends <= due + 1), p
        later, chunks = later + int((ends > due).sum()), chunks + ends.size
    assert 0 < later < 0.05 * chunks


def test_which_tiles_are_put_in_a_line():
    in_line = lambda p, call=FUSED, now=1e9: tile_places(p, call, now=now)[0] is not None
    wide = (2048, 2560, 10240, 8)                # a balanced tail: 8 bands of 256 rows in a line, in runs of 16
    assert in_line(_problem(*wide, flags=DIRECT)) and in_line(_problem(*wide))
    assert in_line(_problem(*wide), now=8 * 256 / 0.84) and not in_line(_problem(*wide), now=8 * 256 / 0.86)
    assert tile_places(_problem(*wide))[1] == 4
    whole = _problem(2048, 2048, 4096, 8)        # none: 12 in runs of 32
    assert in_line(whole, now=12 * 256 / 0.84) and not in_line(whole, now=12 * 256 / 0.86)
    assert not in_line(_problem(534, 1048, 192, 2, flags=DIRECT)) and in_line(_problem(534, 1048, 256, 2, flags=DIRECT))
    assert not in_line(_problem(2131, 464, 640, 16)) and in_line(_problem(2131, 464, 640, 16, flags=DIRECT))
    assert in_line(_problem(2131, 448, 640, 16)) and in_line(_problem(2131, 464, 640, 16), GEMM)


def test_overlap_cases_of_the_gpu_tests_are_what_they_say():
    from tests.test_gpu_workgroup_tiles import OVERLAPS
    for M, W, K, tp, layout, bf16, tile, tail, columns in OVERLAPS:
        p = _problem(M, W, K, tp, layout, flags=DIRECT | (t3.T3_FLAG_FWD_BF16 if bf16 else 0), ldr=W * tp + 4)
        s = launch_shape(p, FUSED)
        assert (s.kernel, (s.tile_m, s.tile_n), s.tail_r, column_overlap(p)) == (WIDE, tile, tail, columns), (M, W, K, tp)
        assert column_overlap(_problem(M, W, K, tp, layout)) == 0 and column_overlap(p, GEMM) == 0


@pytest.mark.parametrize("name,order,blocks", [
    # tile columns of a band (0: stage by stage), blocks a stage is cut into by rows, tile rows and columns of one
    ("gpt3_outproj", 0, (4, 4, 3)),
    ("gpt3_fc2", 0, (4, 4, 3)),
    ("wide_fc2", 4, (4, 2, 5)),
    ("hightp_outproj", 0, (8, 4, 6)),
    ("palm_outproj_tp32", 8, (8, 1, 3)),
    ("tnlg_fc2_tp8", 0, (8, 4, 3)),
    ("megagpt2_fc2_tp8", 0, (8, 8, 2)),
])
def test_order_of_the_named_workloads(name, order, blocks):
    """As the library decides it: from the blocks a stage would be cut into otherwise, and what an XCD pulls for them."""
    from paper_2401_16677_amd import workloads as wl
    w = wl.WORKLOADS[name]
    p = _problem(w.M, w.N // w.tp, w.K, w.tp, flags=DIRECT)
    assert tile_order(p) == (order, blocks)
    assert tile_order(p, xcds=4)[1] == (0, 0, 0)             # (runs on a device of other XCDs)


@pytest.mark.parametrize("sizes,order,blocks", [
    ((700, 128, 392, 16), 4, (0, 0, 0)),                     # runs, several stages a round
    ((8689, 840, 1120, 4), 4, (0, 0, 0)),
    ((841, 264, 5328, 32), 1, (4, 1, 1)),                    # blocks of one tile
    ((2048, 640, 4096, 32), 4, (8, 1, 3)),                   # of one row
    ((2048, 2816, 4096, 8), 4, (8, 1, 11)),
    ((4096, 2048, 2048, 4), 0, (4, 4, 4)),                   # square ones
])
def test_order_by_what_an_xcd_pulls(sizes, order, blocks):
    assert tile_order(_problem(*sizes, flags=DIRECT)) == (order, blocks)


@pytest.mark.parametrize("K,fused,gemm", [(1536, 4, 0), (4096, 4, 0), (4160, 4, 4), (10240, 4, 4)])
def test_plain_gemm_keeps_its_rows_of_a(K, fused, gemm):
    """Blocks of 2 x 5 tiles over two and a half rounds, a balanced tail: A rows that fit an XCD's L2 are pulled once by the plain GEMM."""
    p = _problem(2048, 2560, K, 8, flags=DIRECT)
    assert (tile_order(p)[0], tile_order(p, GEMM)[0]) == (fused, gemm)
    no_tail = _problem(2048, 2560, K, 8, tile_limit=3 * t3.t3_tiles_per_chunk(p))
    assert tile_order(no_tail)[0] == tile_order(no_tail, GEMM)[0]


def test_line_cases_of_the_gpu_tests_are_what_they_say():
    from tests.test_gpu_workgroup_tiles import LINE_MODES, MODES, line_range
    larger = 0
    for case, mode in LINE_MODES:
        M, W, K, tp, layout, first, _, tile, tail, overlap, width, rest = case
        p = _problem(M, W, K, tp, layout, flags=MODES[mode], tile_begin=line_range(case))
        call = GEMM if mode == "unfused" else FUSED
        s = launch_shape(p, call)
        assert (s.kernel, (s.tile_m, s.tile_n), s.tail_r, s.begin) == (WIDE, tile, tail, first * s.tpc), (case, mode)
        assert tile_order(p, call)[0] == width and s.blocks // -(-M // s.tile_m) % width == rest, (case, mode)
        assert column_overlap(p, call) == (overlap if mode in ("direct", "bf16") else 0), (case, mode)
        larger += -(-M // s.tile_m) * width > s.resident
    assert larger >= 2
