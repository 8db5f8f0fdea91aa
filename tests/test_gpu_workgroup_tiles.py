"""GPU parity of the kernels and workgroup tiles that the library picks by size: few tokens and
narrow chunks (32 and 64 wide tiles, K split over wavefronts), chunks that fit no tile, K of a few
slabs only (fewer than the pipeline of the large tiles is deep, or just enough for a tile's count
to be put off into the next tile), ragged K, every operand layout.

Small-integer inputs make fp32 accumulation exact in any order: R, the slots and C must equal the
fp64 oracle bit for bit, whatever tile is picked."""
import numpy as np
import pytest

from paper_2401_16677_amd import binding as t3
from paper_2401_16677_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "needs a GPU"
    from tests import gpu_harness
    return gpu_harness


def _check(gpu, oracle, M, W, K, tp, mode, layout="nk", unfused=False, tile=None, begin=0, limit=-1, ldr_pad=4):
    N, rank = W * tp, (M + W) % tp
    print(f"M={M} W={W} K={K} tp={tp} rank={rank} mode={mode} layout={layout}", flush=True)
    kn, km = layout.endswith("kn"), layout.startswith("km")
    direct, bf16, step0 = not mode.endswith("copy"), mode.startswith("bf16"), mode.startswith("step0")
    a, b, inc = wl.make_integer_inputs(M, N, K, seed=M + 3 * W + 7 * K)
    tile = tile or t3.t3_default_tile(t3.problem(M, N, K, tp, rank, 0, 0))
    init = np.full((tp - 1, M, W), gpu.SENTINEL_BF16 if bf16 else gpu.SENTINEL, np.uint16 if bf16 else np.float32)
    want = oracle.fused_path(a, b, inc, tp, rank, *tile, fwd_direct=direct, fwd_bf16=bf16,
                             step0_store_only=step0, fwd_init=init, tile_begin=begin, tile_limit=limit)
    flags = (t3.T3_FLAG_FWD_DIRECT if direct else 0) | (t3.T3_FLAG_FWD_BF16 if bf16 else 0) | \
            (t3.T3_FLAG_STEP0_STORE_ONLY if step0 else 0)
    # a launch before the one that is checked: the words its tiles are counted in must be back to zero
    got = gpu.run_gpu(a, b, inc, tp, rank, tile, flags=flags, unfused=unfused or mode == "unfused", ldr_pad=ldr_pad,
                      lda_pad=8, b_kn=kn, a_km=km, launches_before=1, tile_begin=begin, tile_limit=limit)
    for name in ("R", "fwd"):
        bad = np.argwhere(got[name] != want[name])
        assert bad.size == 0, f"{name}: {bad.shape[0]} mismatches, first at {tuple(bad[0])}"
    assert np.all(got["R_pad"] == 123.0)
    if mode == "unfused" and (begin, limit) == (0, -1):      # (a range leaves the rest of C alone; its sums are in R)
        assert np.array_equal(got["C"], oracle.gemm_rows(a, b).astype(np.float32))
    assert np.array_equal(got["counter"], want["counter"]) and np.array_equal(got["ready"], want["ready"])
    n = want["queue_len"]
    assert got["queue_len"] == n and set(got["queue"][:n].tolist()) == set(want["queue"][:n].tolist())
    assert got["error"] == 0


@pytest.mark.parametrize("mode", ["direct", "copy", "bf16", "unfused", "step0"])
@pytest.mark.parametrize("M,W,K,tp", [
    (1, 8, 8, 2),           # one row, no full K-slab
    (7, 72, 56, 3),
    (24, 200, 328, 5),      # five slabs and a ragged one over four wavefronts
    (33, 40, 64, 4),        # one row and 8 columns past a 32-wide tile
    (65, 136, 456, 2),
    (96, 1544, 200, 2),     # three slabs: fewer than wavefronts
])
def test_few_tokens(gpu, oracle, M, W, K, tp, mode):
    _check(gpu, oracle, M, W, K, tp, mode)


@pytest.mark.parametrize("layout", ["kn", "km_kn"])
@pytest.mark.parametrize("M,W,K,tp", [(8, 8, 64, 2), (40, 72, 320, 3), (72, 200, 576, 2)])
def test_few_tokens_transposed(gpu, oracle, M, W, K, tp, layout):
    _check(gpu, oracle, M, W, K, tp, "direct", layout)


# The small-tile kernel with exactly as many tiles as the chip holds at once, and with more: the latter take the argument another
# way.  M, W, K, tp, layout, workgroup tile, tiles.  (A test without a GPU checks the last two.)
ROUNDS = [
    (8, 1000, 64, 16, "nk", (32, 32), 512),
    (8, 1000, 64, 16, "km_kn", (32, 32), 512),
    (8, 2072, 784, 8, "nk", (32, 32), 520),
    (8, 2072, 1024, 8, "kn", (32, 32), 520),
    (8, 2072, 1472, 8, "km_kn", (32, 32), 520),
    (8, 2072, 2048, 8, "km_kn", (32, 64), 264),
    (40, 968, 64, 16, "nk", (64, 64), 256),
    (40, 2072, 1472, 8, "nk", (64, 64), 264),
    (40, 2072, 1472, 8, "kn", (64, 64), 264),
    (520, 8, 2048, 32, "km_kn", (64, 64), 288),
]


@pytest.mark.parametrize("mode", ["direct", "copy", "bf16", "unfused"])
@pytest.mark.parametrize("M,W,K,tp,layout,tile,tiles", ROUNDS)
def test_few_tokens_by_rounds(gpu, oracle, M, W, K, tp, layout, tile, tiles, mode):
    _check(gpu, oracle, M, W, K, tp, mode, layout)


# K: slabs of 64 from one to eight, whole and ragged.  Chunk widths: one 192 and one 256 column tile, the
# same and 4 or 8 columns more or less.
@pytest.mark.parametrize("K", [64, 128, 136, 192, 200, 256, 264, 328, 384, 392, 512])
@pytest.mark.parametrize("M,W,tp", [(4088, 384, 8), (4096, 260, 8), (2050, 1020, 8), (1030, 532, 4)])
def test_short_k(gpu, oracle, M, W, tp, K):
    _check(gpu, oracle, M, W, K, tp, "direct")


@pytest.mark.parametrize("mode", ["copy", "bf16", "unfused", "step0"])
@pytest.mark.parametrize("K", [128, 200, 520])
@pytest.mark.parametrize("M,W,tp", [(4088, 384, 8), (2050, 1016, 8)])
def test_short_k_modes(gpu, oracle, M, W, tp, K, mode):
    _check(gpu, oracle, M, W, K, tp, mode)


@pytest.mark.parametrize("layout", ["kn", "km_kn"])
@pytest.mark.parametrize("K", [64, 128, 192, 256, 384, 576])
@pytest.mark.parametrize("M,W,tp", [(4088, 384, 8), (2056, 1032, 8), (2048, 32, 32)])
def test_short_k_transposed(gpu, oracle, M, W, tp, K, layout):
    _check(gpu, oracle, M, W, K, tp, "direct", layout)


# The reduction's own tiles: parts of a chunk of 256 columns or fewer, few and many rows per workgroup, the
# last ones ragged, chunks narrower than a wavefront's 16-byte pieces.
@pytest.mark.parametrize("mode", ["direct", "copy", "bf16", "step0"])
@pytest.mark.parametrize("M,W,tp", [(1, 8, 2), (5, 264, 3), (1148, 512, 8), (2051, 8, 2), (4097, 536, 4)])
def test_reduction(gpu, oracle, M, W, tp, mode):
    _check(gpu, oracle, M, W, 64, tp, mode, unfused=True)


@pytest.mark.parametrize("M,W,tp", [(3, 4, 2), (2500, 532, 4), (600, 20, 40)])
def test_reduction_fp32_columns(gpu, oracle, M, W, tp):
    _check(gpu, oracle, M, W, 64, tp, "unfused")


# A range that cuts a ring step keeps the tracked tile: several batches of 1024 pieces of 16 bytes, the next one requested
# while one leaves.  Rows and columns of the last tiles: less than one batch, one to sixteen, whole and with a remainder.
@pytest.mark.parametrize("mode", ["direct", "copy", "bf16", "step0"])
@pytest.mark.parametrize("M,W,tp,tile", [
    (300, 264, 3, (128, 128)),       # 4 batches; 44 rows, 8 columns: one, ragged
    (261, 512, 2, (256, 256)),       # 16 batches; 5 rows: less than one
    (96, 384, 3, (256, 128)),        # 3 batches
    (1024, 536, 4, (128, 256)),      # 8 batches; 24 columns: one, ragged
])
def test_reduction_of_a_cut_range(gpu, oracle, M, W, tp, tile, mode):
    tpc = t3.t3_tiles_per_chunk(t3.problem(M, W * tp, 64, tp, 0, *tile))
    for begin, limit in ((1, tpc * tp), (0, tpc * tp - 1)):
        _check(gpu, oracle, M, W, 64, tp, mode, unfused=True, tile=tile, begin=begin, limit=limit)


# What the choice by size picks and nothing above reaches: the wide-tile kernel's 256 x 128 and 128 x 192 tiles (three LDS
# stages), balanced tails on every tile that has them, and 32 x 64.  (Which tile each problem gets is checked
# without a GPU as well.)  M, W, K, tp, layout, one ring step only, workgroup tile, tiles the tail splits.
PICKED = [
    # more tiles than workgroups; four to seven K-slabs, whole and ragged: a tile's count is put off into the next one's loop
    (6432, 280, 200, 5, "nk", False, (128, 192), 0),
    (533, 528, 264, 32, "nk", False, (128, 192), 0),
    (522, 544, 320, 32, "nk", False, (128, 192), 0),
    (4448, 136, 384, 16, "nk", False, (128, 192), 0),
    (4344, 136, 392, 16, "nk", False, (128, 192), 0),
    (8728, 144, 256, 8, "km", False, (128, 192), 0),
    (544, 520, 320, 32, "km_kn", False, (128, 192), 0),
    (8368, 136, 320, 8, "kn", False, (128, 192), 0),
    (4096, 1536, 1536, 2, "nk", True, (128, 192), 0),       # one tile per compute unit
    (6928, 40, 4104, 16, "nk", False, (256, 128), 0),
    (3112, 56, 4096, 32, "nk", False, (256, 128), 0),
    (7944, 8, 4096, 32, "km", False, (256, 128), 0),
    (3352, 48, 4096, 32, "km_kn", False, (256, 128), 0),
    (7432, 64, 4096, 16, "kn", False, (256, 128), 0),
    # balanced tails: halves of four K-slabs, the second one with a ragged slab more
    (4104, 136, 520, 16, "nk", False, (256, 192), 16),
    (4128, 136, 512, 16, "km", False, (256, 192), 16),
    (4488, 136, 512, 16, "kn", False, (256, 192), 32),
    (4552, 136, 512, 16, "km_kn", False, (256, 192), 32),
    (4200, 128, 520, 16, "nk", False, (256, 128), 16),
    (4936, 8, 4096, 32, "km", False, (256, 128), 128),
    (4704, 128, 1024, 16, "kn", False, (256, 128), 48),
    (4104, 128, 512, 16, "km_kn", False, (256, 128), 16),
    (4104, 136, 520, 8, "nk", False, (128, 192), 8),
    (2088, 136, 512, 16, "km", False, (128, 192), 16),
    (2080, 136, 512, 16, "kn", False, (128, 192), 16),
    (2400, 136, 512, 16, "km_kn", False, (128, 192), 48),
    # rows of a few tokens, the last columns ragged
    (8, 392, 2816, 32, "kn", False, (32, 64), 0),
    (24, 264, 1920, 32, "km_kn", False, (32, 64), 0),
    (136, 40, 2048, 32, "km_kn", False, (32, 64), 0),
]
MODES = {"direct": t3.T3_FLAG_FWD_DIRECT, "copy": 0, "bf16": t3.T3_FLAG_FWD_DIRECT | t3.T3_FLAG_FWD_BF16,
         "step0": t3.T3_FLAG_FWD_DIRECT | t3.T3_FLAG_STEP0_STORE_ONLY, "unfused": t3.T3_FLAG_FWD_DIRECT}
# all modes where both operands are K-contiguous (no bfloat16 slots with a tail), the two kernels there are in every layout
PICKED_MODES = [(case, mode) for case in PICKED for mode in MODES
                if (case[4] == "nk" or case[6] == (32, 64) or mode in ("direct", "unfused")) and not (case[7] and mode == "bf16")]


def picked_range(case):
    M, W, K, tp, _, one_step, _, _ = case
    tpc = t3.t3_tiles_per_chunk(t3.problem(M, W * tp, K, tp, 0, 0, 0))
    return (tpc, 2 * tpc) if one_step else (0, -1)


@pytest.mark.parametrize("case,mode", PICKED_MODES)
def test_picked_tiles(gpu, oracle, case, mode):
    M, W, K, tp, layout, _, _, _ = case
    begin, limit = picked_range(case)
    _check(gpu, oracle, M, W, K, tp, mode, layout, begin=begin, limit=limit)


# Chunks that do not start at 64-byte granules of R and C: tile columns start early, at granules, where the last one has columns
# to spare: 12 for chunk widths that are multiples of 4, 8 for multiples of 8.  M, W, K, tp, layout, workgroup tile, tiles a balanced
# tail splits, whether they do.  (A test without a GPU checks the last three.)
GRANULES = [
    (1032, 564, 200, 12, "nk", (256, 192), 0, True),         # 12 to spare
    (1032, 568, 200, 12, "nk", (256, 192), 0, True),         # 8, and a width that is a multiple of 8
    (1032, 572, 200, 12, "nk", (256, 192), 0, False),        # 4
    (4100, 532, 520, 8, "nk", (256, 192), 0, True),
    (1304, 948, 520, 12, "nk", (256, 192), 104, True),
    (520, 564, 200, 12, "nk", (128, 192), 0, True),
    (1032, 568, 520, 12, "nk", (128, 192), 68, True),
    (520, 372, 200, 5, "nk", (128, 128), 0, True),
    (520, 500, 200, 32, "nk", (256, 256), 0, True),
    (520, 508, 200, 32, "nk", (256, 256), 0, False),
    (1304, 1012, 520, 12, "nk", (256, 256), 32, True),
    (4104, 244, 2048, 8, "nk", (256, 128), 16, True),
    (520, 952, 576, 16, "kn", (256, 192), 0, True),
    (1032, 568, 576, 12, "kn", (128, 192), 68, True),
    (4104, 248, 2048, 8, "kn", (256, 128), 16, True),
    (520, 948, 576, 16, "km", (256, 192), 0, True),
    (1304, 1012, 576, 12, "km", (256, 256), 32, True),
    (1304, 244, 4096, 12, "km", (256, 128), 0, True),
    (520, 952, 576, 16, "km_kn", (256, 192), 0, True),
    (520, 504, 576, 32, "km_kn", (256, 256), 0, True),
    (520, 376, 576, 5, "km_kn", (128, 128), 0, True),
]
# (bfloat16 slots hold multiples of 8 columns, and have no balanced tail)
GRANULE_MODES = [(case, mode) for case in GRANULES for mode in ("copy", "bf16_copy", "unfused", "step0_copy")
                 if mode != "bf16_copy" or (case[1] % 8 == 0 and not case[6])]


@pytest.mark.parametrize("case,mode", GRANULE_MODES)
def test_columns_start_at_granules(gpu, oracle, case, mode):
    M, W, K, tp, layout, _, _, _ = case
    _check(gpu, oracle, M, W, K, tp, mode, layout, ldr_pad=16 + -W * tp % 16)


@pytest.mark.parametrize("M,W,K,tp,layout", [(4100, 532, 520, 8, "nk"), (2050, 500, 1536, 16, "nk"), (2056, 1016, 576, 8, "kn")])
def test_results_do_not_depend_on_where_the_buffers_start(gpu, M, W, K, tp, layout):
    """Real-valued inputs: the sums of a call depend on its sizes alone, to the last bit, not on the address or the leading
    dimension of C or R."""
    import torch
    N, kn = W * tp, layout.endswith("kn")
    g = torch.Generator("cuda").manual_seed(W)
    A = torch.randn(M, K, generator=g, device="cuda").to(torch.bfloat16)
    B = torch.randn(*((K, N) if kn else (N, K)), generator=g, device="cuda").to(torch.bfloat16)
    inc = torch.randn(M, N, generator=g, device="cuda")
    track = torch.zeros(t3.t3_track_words(tp), dtype=torch.int32, device="cuda")
    t3.t3_track_reset(tp, track)
    first = None
    for ld, off in ((N, 0), (N, 4), (N + 4, 0), (N + 16, 8)):
        print(f"M={M} W={W} K={K} tp={tp} {layout} ld={ld} offset={off}", flush=True)
        C, R = (torch.zeros(M * ld + off, device="cuda")[off:].view(M, ld) for _ in range(2))
        R[:, :N] = inc
        fwd = torch.zeros(tp - 1, M, W, device="cuda")
        p = t3.problem(M, N, K, tp, 1, b_layout=t3.T3_B_KN if kn else t3.T3_B_NK, ldr=ld, ldc=ld)
        t3.t3_gemm(p, A, B, C)
        t3.t3_gemm_rs_fused(p, A, B, R, fwd, track)
        torch.cuda.synchronize()
        got = [t.cpu().numpy().view(np.uint32) for t in (C[:, :N].contiguous(), R[:, :N].contiguous(), fwd)]
        first = first or got
        for name, x, y in zip(("C", "R", "fwd"), got, first):
            assert np.array_equal(x, y), (name, ld, off, int((x != y).sum()))


# Direct release of chunks whose rows start inside a 64-byte granule of their slot: tile columns overlap where the grid has columns
# to spare.  M, W, K, tp, layout, bfloat16 slots, workgroup tile, tiles a balanced tail splits, columns.  (A test without a GPU checks the last three.)
OVERLAPS = [
    (1032, 540, 200, 12, "nk", False, (256, 192), 0, 12),
    (1032, 536, 200, 12, "nk", False, (256, 192), 0, 8),
    (1030, 552, 200, 12, "nk", False, (256, 192), 0, 8),
    (1032, 564, 200, 12, "nk", False, (256, 192), 0, 0),     # 12 columns to spare for two cuts
    (1304, 908, 520, 12, "nk", False, (256, 192), 104, 12),
    (520, 548, 200, 12, "nk", False, (128, 192), 0, 12),
    (520, 372, 200, 5, "nk", False, (128, 128), 0, 0),
    (520, 356, 200, 5, "nk", False, (128, 128), 0, 12),
    (520, 500, 200, 32, "nk", False, (256, 256), 0, 12),
    (1304, 976, 520, 12, "nk", False, (256, 256), 32, 0),    # whole granules
    (1304, 980, 520, 12, "nk", False, (256, 256), 32, 12),
    (4104, 244, 2048, 8, "nk", False, (256, 128), 16, 12),
    (1032, 536, 200, 12, "nk", True, (256, 192), 0, 0),      # bfloat16: 24 columns a cut
    (1032, 528, 200, 12, "nk", True, (256, 192), 0, 16),
    (1032, 520, 200, 12, "nk", True, (256, 192), 0, 24),
    (520, 952, 576, 16, "kn", False, (256, 192), 0, 0),
    (520, 920, 576, 16, "kn", False, (256, 192), 0, 8),
    (520, 504, 576, 32, "km_kn", False, (256, 256), 0, 8),
]


@pytest.mark.parametrize("case", OVERLAPS)
def test_tile_columns_overlap(gpu, oracle, case):
    M, W, K, tp, layout, bf16 = case[:6]
    for mode in ("bf16",) if bf16 else ("direct", "step0"):
        _check(gpu, oracle, M, W, K, tp, mode, layout)


@pytest.mark.parametrize("M,W,K,tp,layout", [(1304, 908, 520, 12, "nk"), (2050, 500, 1536, 16, "nk"), (520, 920, 576, 16, "kn")])
def test_direct_results_do_not_depend_on_where_the_buffers_start(gpu, M, W, K, tp, layout):
    import torch
    N, kn = W * tp, layout.endswith("kn")
    g = torch.Generator("cuda").manual_seed(W)
    A = torch.randn(M, K, generator=g, device="cuda").to(torch.bfloat16)
    B = torch.randn(*((K, N) if kn else (N, K)), generator=g, device="cuda").to(torch.bfloat16)
    inc = torch.randn(M, N, generator=g, device="cuda")
    track = torch.zeros(t3.t3_track_words(tp), dtype=torch.int32, device="cuda")
    t3.t3_track_reset(tp, track)
    first = None
    for ld, off in ((N, 0), (N, 4), (N + 4, 0), (N + 16, 8)):
        print(f"M={M} W={W} K={K} tp={tp} {layout} ld={ld} offset={off}", flush=True)
        R = torch.zeros(M * ld + off, device="cuda")[off:].view(M, ld)
        R[:, :N] = inc
        fwd = torch.zeros((tp - 1) * M * W + off, device="cuda")[off:]
        p = t3.problem(M, N, K, tp, 1, b_layout=t3.T3_B_KN if kn else t3.T3_B_NK, ldr=ld, flags=t3.T3_FLAG_FWD_DIRECT)
        t3.t3_gemm_rs_fused(p, A, B, R, fwd, track)
        torch.cuda.synchronize()
        got = [t.cpu().numpy().view(np.uint32) for t in (R[:, :N].contiguous(), fwd)]
        first = first or got
        for name, x, y in zip(("R", "fwd"), got, first):
            assert np.array_equal(x, y), (name, ld, off, int((x != y).sum()))


# Tiles in a line: bands of one to eight tile columns, a last band of fewer, in one round and in several, with a balanced tail, with
# overlapping columns, bands larger than a round, ranges that begin at a later ring step.  M, W, K, tp, layout, first step, bfloat16 slots, workgroup
# tile, tiles the tail splits, columns of overlap, columns of a band, of the last one if it has fewer.  (A test without a GPU checks the last five.)
LINES = [
    (523, 16, 272, 32, "nk", 0, False, (128, 128), 0, 0, 1, 0),
    (712, 68, 296, 11, "nk", 0, False, (128, 128), 0, 0, 2, 1),
    (561, 160, 256, 11, "nk", 0, False, (128, 128), 0, 0, 4, 2),
    (2555, 16, 264, 15, "nk", 0, False, (128, 128), 0, 0, 8, 7),
    (4429, 16, 256, 15, "kn", 0, False, (128, 128), 0, 0, 8, 7),
    (4429, 16, 256, 18, "nk", 3, False, (128, 128), 0, 0, 8, 7),
    (2246, 160, 664, 15, "nk", 0, False, (128, 192), 14, 0, 4, 3),
    (2246, 160, 664, 18, "nk", 3, False, (128, 192), 14, 0, 4, 3),
    (2945, 208, 264, 11, "nk", 0, True, (256, 256), 0, 0, 4, 3),
    (535, 136, 256, 11, "nk", 0, True, (128, 128), 0, 24, 4, 2),
    (7464, 264, 512, 3, "km_kn", 0, False, (128, 192), 98, 8, 4, 2),
    (2208, 16, 512, 32, "km_kn", 1, False, (256, 128), 23, 0, 4, 3),
    (11112, 688, 512, 1, "km_kn", 0, False, (128, 192), 92, 0, 4, 0),
    (22752, 280, 320, 2, "km_kn", 0, False, (128, 192), 0, 8, 2, 0),
]
LINE_MODES = [(case, mode) for case in LINES for mode in ("direct", "copy", "unfused", "bf16")
              if (mode == "bf16") == case[6] and (mode != "copy" or case[1] % 32 == 0) and (mode != "unfused" or case[4] == "nk")]


def line_range(case):
    M, W, K, tp = case[:4]
    return case[5] * t3.t3_tiles_per_chunk(t3.problem(M, W * tp, K, tp, 0, 0, 0))


@pytest.mark.parametrize("case,mode", LINE_MODES)
def test_tiles_in_a_line(gpu, oracle, case, mode):
    M, W, K, tp, layout = case[:5]
    _check(gpu, oracle, M, W, K, tp, mode, layout, begin=line_range(case))
