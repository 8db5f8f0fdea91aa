"""The work a user of this library has it do, as a list of measurable cases.

A case is one pass of one tensor-parallel rank through the public entry points (`binding`):

  path = "direct"   t3_gemm_rs_fused, sums of forwarded chunks stored straight into their slot
  path = "copy"     t3_gemm_rs_fused in its default release mode (sums in R, triggered chunks
                    copied to their slots)
  path = "unfused"  t3_gemm followed by t3_rs_reduce
  path = "ring"     the whole all-reduce of one rank: one t3_gemm_rs_fused call per ring step
                    (tile ranges, the next chunk's partial could arrive in between), then the
                    tp - 1 steps of the all-gather from an upstream neighbour's buffer

M tokens, hidden size N cut into tp chunks, K = this rank's slice; layouts: "nk" (A M x K, B N x K,
the forward pass), "kn" (B stored K x N) and "km_kn" (A stored K x M, B stored K x N), both of the
backward pass; tile 0 x 0 is the library's own choice.
"""
import math

import torch

from paper_2401_16677_amd import binding as t3


def _case(name, M, N, K, tp, rank, tile=(0, 0), path="direct", layout="nk", fwd="fp32", step0=False,
          relu=False):
    c = {"M": M, "N": N, "K": K, "tp": tp, "rank": rank, "tile_m": tile[0], "tile_n": tile[1],
         "path": path, "layout": layout, "fwd": fwd, "step0_store": step0, "relu": relu}
    return c if name is None else {"name": name, **c}


def listed():
    return [
        # the smallest configuration: one short call, launch and host time count
        _case("tiny_outproj", 256, 1024, 256, 4, 0, (128, 128)),
        # a serving step: a few tokens against the whole output-projection slice, weight bound
        _case("decode_outproj", 24, 12288, 1536, 8, 3),
        # output projection of a training step or prefill, GPT-3 sized: at the ridge
        _case("gpt3_outproj", 4096, 12288, 1536, 8, 3, (256, 256)),
        # FC-2 behind a ReLU-like activation: matrix bound
        _case("gpt3_fc2", 4096, 12288, 6144, 8, 5, (256, 256), relu=True),
        # the largest configuration: wide model, tall K, tile count that is no whole number of rounds
        _case("wide_fc2", 2048, 20480, 10240, 8, 7, (128, 256)),
        # high TP degree, long sequence: the output's traffic dominates
        _case("hightp_outproj", 8192, 18432, 1152, 16, 9, (256, 256)),
        # mixed precision: bfloat16 on the wire, first chunk stored only, TP 32
        _case("palm_outproj_tp32_bf16", 2048, 18432, 576, 32, 30, fwd="bf16", step0=True),
        # default release mode on a model whose chunks (532 columns) fit no tile
        _case("tnlg_fc2_tp8_copy", 8192, 4256, 2128, 8, 6, path="copy", relu=True),
        # backward pass, input gradient of FC-1: B stored K x N
        _case("gpt3_fc1_dgrad", 4096, 12288, 6144, 8, 5, layout="kn"),
        # backward pass, weight gradient of the output projection reduced over data-parallel ranks
        _case("gpt3_outproj_wgrad", 1536, 12288, 4096, 8, 2, layout="km_kn"),
        # GEMM and reduction as two calls
        _case("megagpt2_fc2_tp8_unfused", 16384, 3072, 1536, 8, 2, path="unfused"),
        # a whole all-reduce, ring step by ring step
        _case("gpt3_outproj_ring", 4096, 12288, 1536, 8, 3, (256, 256), path="ring"),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: few tokens to the longest batch, narrow to wide models, short to long K."""
    while True:
        path = rng.choice(("direct", "direct", "direct", "copy", "unfused", "ring"))
        layout = rng.choice(("nk", "nk", "nk", "kn", "km_kn")) if path in ("direct", "copy") else "nk"
        fwd = rng.choice(("fp32", "fp32", "bf16")) if path in ("direct", "copy") else "fp32"
        tp = rng.choice((4, 8, 16) if path == "ring" else (2, 4, 8, 8, 16, 32))
        col = 8 if layout != "nk" or fwd == "bf16" else 4
        W = max(col, _logint(rng, 1024, 20480) // tp // col * col)
        N = W * tp
        M = _logint(rng, 8, 16384)
        K = _logint(rng, 128, 10240) // 8 * 8
        if layout != "nk":
            K = max(64, K // 64 * 64)
        if layout == "km_kn":
            M = max(8, M // 8 * 8)
        if 2.0 * M * N * K > 4e11 or M * N > 100e6:
            continue                                    # no dearer than the largest listed case
        tile = (0, 0)
        if M >= 512 and W >= 256 and rng.random() < 0.25:
            tile = rng.choice(((256, 256), (256, 128), (128, 256), (128, 128)))
        return _case(None, M, N, K, tp, rng.randrange(tp), tile, path, layout, fwd,
                     step0=rng.random() < 0.25, relu=rng.random() < 0.3)


def prepare(case, seed):
    """Inputs, output buffers and the call's description, as the caller's program keeps them.

    A, B ~ N(0, K^-1/2) in variance (so a sum has variance 1; half of A exact zeros after a
    ReLU), the incoming partial ~ N(0, tp - 1): what has passed up to tp - 1 ranks."""
    M, N, K, tp, rank = (case[k] for k in ("M", "N", "K", "tp", "rank"))
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    sigma = float(K) ** -0.25
    km, kn = case["layout"] == "km_kn", case["layout"] != "nk"
    A = torch.randn((K, M) if km else (M, K), generator=g, device=dev).mul_(sigma)
    if case["relu"]:
        A.clamp_(min=0.0)
    A = A.to(torch.bfloat16)
    B = torch.randn((K, N) if kn else (N, K), generator=g, device=dev).mul_(sigma).to(torch.bfloat16)
    R = torch.randn((M, N), generator=g, device=dev).mul_(math.sqrt(max(tp - 1, 1)))
    bf16 = case["fwd"] == "bf16"
    fwd = torch.zeros((tp - 1, M, N // tp), dtype=torch.bfloat16 if bf16 else torch.float32, device=dev)
    track = torch.zeros(t3.t3_track_words(tp), dtype=torch.int32, device=dev)
    t3.t3_track_reset(tp, track)
    flags = t3.T3_FLAG_FWD_BF16 if bf16 else 0
    if case["path"] in ("direct", "unfused", "ring"):
        flags |= t3.T3_FLAG_FWD_DIRECT
    if case["step0_store"]:
        flags |= t3.T3_FLAG_STEP0_STORE_ONLY

    def problem(**kw):
        return t3.problem(M, N, K, tp, rank, case["tile_m"], case["tile_n"],
                          b_layout=t3.T3_B_KN if kn else t3.T3_B_NK,
                          a_layout=t3.T3_A_KM if km else t3.T3_A_MK, flags=flags, **kw)

    st = {"path": case["path"], "p": problem(), "A": A, "B": B, "R": R, "fwd": fwd, "track": track}
    # what the tracker reports: counters and ready flags of its two banks, generation and error
    # (the order in which chunks were queued is the device's own)
    bank = 3 * tp + 2
    st["out"] = [R, fwd, track[:2 * tp], track[bank:bank + 2 * tp], track[2 * bank:2 * bank + 2]]
    if case["path"] == "unfused":
        st["C"] = torch.zeros((M, N), device=dev)
        st["out"].append(st["C"])
    if case["path"] == "ring":
        tpc = t3.t3_tiles_per_chunk(st["p"])
        st["steps"] = [problem(tile_begin=s * tpc, tile_limit=(s + 1) * tpc) for s in range(tp)]
        st["up"] = torch.randn((M, N), generator=g, device=dev).mul_(math.sqrt(tp))
    return st


def run(st):
    if st["path"] == "unfused":
        t3.t3_gemm(st["p"], st["A"], st["B"], st["C"])
        t3.t3_rs_reduce(st["p"], st["C"], st["R"], st["fwd"], st["track"])
    elif st["path"] == "ring":
        for p in st["steps"]:
            t3.t3_gemm_rs_fused(p, st["A"], st["B"], st["R"], st["fwd"], st["track"])
        for g in range(len(st["steps"]) - 1):
            t3.t3_ag_step(st["p"], g, st["up"], st["R"])
    else:
        t3.t3_gemm_rs_fused(st["p"], st["A"], st["B"], st["R"], st["fwd"], st["track"])
    return st["out"]


def work(case):
    M, N, K, tp = case["M"], case["N"], case["K"], case["tp"]
    W = N // tp
    out = 2 if case["fwd"] == "bf16" else 4
    incoming = 4 * M * (N - W if case["step0_store"] else N)
    own, slots = 4 * M * W, out * M * (N - W)
    b = 2 * M * K + 2 * N * K + incoming + own + slots
    if case["path"] == "copy":
        b += 4 * M * (N - W)            # the sums of forwarded chunks stay in R too
    if case["path"] == "unfused":
        b += 8 * M * N                  # C is handed from the one call to the other
    if case["path"] == "ring":
        b += 8 * M * (N - W)            # the gathered chunks, read and written
    return {"bytes": b, "flops": 2.0 * M * N * K}


def tolerance(case):
    # fp32 sums of up to 10240 products in some order; bfloat16 slots may round to the other
    # neighbour where the fp32 sums differ
    if case["fwd"] == "bf16":
        return {"rel": 2e-3, "max": 1e-2}
    return {"rel": 1e-5, "max": 1e-4}
