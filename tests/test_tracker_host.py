"""The chain behind a tile's count (track_finish of csrc/t3_device.h), played on the host in random orders: what the words
hold when a launch has ended, and that no addition is made, or waited for, that nothing depends on."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2401_16677_amd import binding as t3
from paper_2401_16677_amd import build as hip_build

EMPTY = 0xFFFFFFFF


@pytest.fixture(scope="module")
def play(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("tracker") / "tracker_host.so")
    flags = [f for f in hip_build.HIPCC_FLAGS if f != "-Wall"]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "-w", "--offload-host-only", "-shared", "-I",
                    os.path.join(hip_build.ROOT, "include"), "-I", hip_build.CSRC,
                    os.path.join(hip_build.ROOT, "tests", "tracker_host.hip"), "-o", so], check=True, stderr=subprocess.DEVNULL)
    return ctypes.CDLL(so).play


def _launch(play, words, P, rank, Mt, Wt, begin, limit, rng, sub=(1, 0), writers=1, step0=False, tracked=None):
    """One launch over issue positions [begin, limit); words are updated.  -> (zeros, round trips)."""
    tpc = Mt * Wt
    whole = writers == 1 and begin % tpc == 0 and limit % tpc == 0
    tiles = [(t // tpc, t % tpc % Mt, t % tpc // Mt) for t in range(begin, limit)]
    landings = tiles + [t for t in tiles for _ in range(writers - 1) if not (step0 and t[0] == 0)]
    order = rng.permutation(len(landings))
    flat = np.ascontiguousarray(np.array(landings, dtype=np.int32)[order])
    seen = np.zeros(2, np.int64)
    play(P, rank, Mt, Wt, int(whole), *sub, begin // tpc, writers - (1 if step0 else 0), writers, len(landings),
         tpc if tracked is None else tracked, flat.ctypes.data_as(ctypes.c_void_p), len(landings),
         words.ctypes.data_as(ctypes.c_void_p), seen.ctypes.data_as(ctypes.c_void_p))
    return seen


def _clear(P):
    words = np.zeros(t3.t3_track_words(P), np.uint32)
    for b in (0, 3 * P + 2):
        words[b + 2 * P:b + 3 * P] = EMPTY
    return words


@pytest.mark.parametrize("P,Mt,Wt,begin,limit,sub,writers,step0,tracked", [
    (4, 2, 1, 0, 8, (1, 0), 1, False, None),             # whole chunks
    (4, 2, 1, 0, 8, (1, 0), 1, False, 5),                # counted as five tracked tiles
    (8, 8, 4, 0, 256, (8, 0), 1, False, None),           # in groups
    (8, 16, 17, 0, 8 * 272, (32, 2), 1, False, None),
    (8, 8, 4, 64, 96, (8, 0), 1, False, None),           # one ring step
    (3, 3, 3, 1, 27, (1, 0), 1, False, None),            # ranges that cut a step
    (3, 3, 3, 0, 14, (1, 0), 1, False, None),
    (4, 3, 2, 0, 24, (1, 0), 2, False, None),            # two writers
    (4, 3, 2, 0, 24, (1, 0), 2, True, None),
    (4, 3, 2, 0, 24, (1, 0), 3, False, None),            # and K in two parts
    (1, 2, 2, 0, 4, (1, 0), 1, False, None),
])
def test_launches_played_on_the_host(play, P, Mt, Wt, begin, limit, sub, writers, step0, tracked):
    rng = np.random.default_rng(P + Mt * Wt + begin)
    words, bank, tpc = _clear(P), 3 * P + 2, Mt * Wt
    for launch in range(3):
        rank = int(rng.integers(0, P))
        own = (rank + P - 1) % P
        zeros, trips = _launch(play, words, P, rank, Mt, Wt, begin, limit, rng, sub, writers, step0, tracked)
        gen = int(words[2 * bank])
        assert gen == launch + 1 and words[2 * bank + 1] == 0
        now, other = words[(gen - 1 & 1) * bank:][:bank], words[(gen & 1) * bank:][:bank]
        steps = {s: sum(begin <= t < limit for t in range(s * tpc, (s + 1) * tpc)) for s in range(P)}
        landed = {s: n * (writers - 1 if step0 and s == 0 else writers) for s, n in steps.items()}
        want = np.zeros(P, np.uint32)
        done_chunks = [s for s, n in steps.items() if n == tpc]
        for s, n in landed.items():
            full = s in done_chunks and tracked is not None
            want[(rank + s) % P] = tracked * n // tpc if full else n
        assert np.array_equal(now[:P], want)
        complete = {(rank + s) % P for s in done_chunks}
        assert set(np.flatnonzero(now[P:2 * P]).tolist()) == complete
        queued = sorted(complete - {own})
        assert now[3 * P] == len(queued) and sorted(now[2 * P:2 * P + len(queued)].tolist()) == queued
        assert np.all(now[2 * P + len(queued):3 * P] == EMPTY) and now[3 * P + 1] == sum(landed.values())
        assert not other[:2 * P].any() and np.all(other[2 * P:3 * P] == EMPTY) and not other[3 * P:].any()
        assert not words[2 * bank + 2:].any()                    # the groups' words return to 0
        # one answer per landing, one more where every landing counts in `done`, one per group, one per chunk that
        # has anything to add, one for gen; nothing is added by itself that is nothing
        whole = writers == 1 and begin % tpc == 0 and limit % tpc == 0
        assert zeros == (1 if whole and own in complete else 0)
        n = sum(landed.values())
        groups = len(done_chunks) * sub[0] if sub[0] > 1 else 0
        assert trips == n * (1 if whole else 2) + groups + (len(done_chunks) if whole else len(queued)) + 1
