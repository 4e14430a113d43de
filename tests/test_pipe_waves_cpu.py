"""The pipelined step kernel's waves on the CPU (tests/emul/kvr_emul_waves.cpp):
csrc/kvr_trail.h unchanged, a routing wave, two evicting waves and helpers as
coroutines that are cut at any step and held back while the others go on,
against the oracle."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import paper_2601_18999_amd as K
from oracle import oracle as O
from streams import long_beside_short_stream
from workload import generate, small_spec

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "emul")


def build(tmp_path_factory, *flags):
    out = str(tmp_path_factory.mktemp("waves") / "libwaves.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-ffp-contract=off", "-fPIC", "-shared", *flags,
                           "-Wno-unknown-pragmas", "-o", out, os.path.join(HERE, "kvr_emul_waves.cpp")])
    lib = ctypes.CDLL(out)
    lib.emul_waves.restype = ctypes.c_int
    lib.emul_waves.argtypes = ([ctypes.POINTER(K.KvrConfig), ctypes.c_uint64] + [ctypes.c_void_p] * 8 +
                               [ctypes.c_uint32, ctypes.c_uint32, ctypes.c_int32, ctypes.c_uint64, ctypes.c_uint32,
                                ctypes.c_void_p])
    return lib


@pytest.fixture(scope="module")
def waves(tmp_path_factory):
    return build(tmp_path_factory)


def check(lib, s, W, B, update, ucap, nbuf, router, order, hold_draws=0, may_fail=False, **cfg):
    c = K.kvr_config_default(1, W, B, max(1, s.max_len), seed=order,
                             update={"nlms": 0, "rls": 1, "none": 2}[update], **cfg)
    arrays = [np.ascontiguousarray(s.tokens, np.int32), np.ascontiguousarray(s.offsets, np.uint64),
              np.ascontiguousarray(s.arrival_us, np.int64), np.ascontiguousarray(s.out_len, np.uint16)]
    route, hits, ah = np.zeros(s.n, np.int32), np.zeros(s.n, np.int32), np.zeros((s.n, W), np.int32)
    st = (K.KvrWorkerStats * W)()
    counts = np.zeros(6, np.uint64)
    rc = lib.emul_waves(ctypes.byref(c), s.n, *[a.ctypes.data for a in arrays], route.ctypes.data, hits.ctypes.data,
                        ah.ctypes.data, ctypes.cast(st, ctypes.c_void_p), ucap, nbuf,
                        {"lbgr": K.KVR_ROUTE_LBGR, "round_robin": K.KVR_ROUTE_ROUND_ROBIN}[router], order,
                        hold_draws, counts.ctypes.data)
    if may_fail and rc == 64:  # KVR_DEV_INTERNAL
        return None
    assert rc == 0, (order, rc)
    o = O.run(s, W, B, replica=0, all_hits=True, update=update, seed=order, router=router)
    np.testing.assert_array_equal(ah, o["all_hits"], err_msg=str(order))
    np.testing.assert_array_equal(route, o["route"])
    np.testing.assert_array_equal(hits, o["hits"])
    for i, got in enumerate(K._stats_dicts(st, W)):
        want = o["workers"][i]
        assert {k: got[k] for k in want} == want, (order, i)
    return counts


@pytest.mark.parametrize("block", range(3))
def test_waves_cut_anywhere_match_the_oracle(waves, block):
    """Random small instances, each under a random schedule."""
    rng = np.random.default_rng(70 + block)
    total = np.zeros(6, np.uint64)
    for case in range(24):
        s = generate(small_spec(n=int(rng.integers(20, 160)), groups=int(rng.integers(1, 8)),
                                prefix_len=(1, int(rng.integers(2, 40))), suffix_len=(1, int(rng.integers(2, 24))),
                                vocab=int(rng.integers(2, 12)), seed=1000 * block + case))
        W = int(rng.integers(1, 10))
        B = int(max(s.max_len, rng.integers(2, 260)))
        tight = {"arena_words": 3 * (B + 2 * s.max_len + 64)} if case % 4 == 3 else {}
        total += check(waves, s, W, B, ["nlms", "rls", "none"][case % 3], [8192, 4, 0][case % 3], 2 + case % 3,
                       ["round_robin", "lbgr"][case % 2], 100 * block + case, **tight)
    assert (total[[0, 2, 4, 5]] > 0).all(), total


@pytest.mark.parametrize("block", range(4))
def test_an_insertion_that_outlasts_the_next_seven(waves, block):
    """One long insertion beside short ones on other workers, with later
    queries' matches beside it: its record must stay while any of them may
    still read it, whichever wave is held back."""
    rng = np.random.default_rng(20 + block)
    total = np.zeros(6, np.uint64)
    for case in range(12):
        W, length = int(rng.integers(12, 16)), int(rng.integers(40, 200))
        s = long_beside_short_stream(rng, 12, W, length, 6)
        total += check(waves, s, W, length + int(rng.integers(0, length)), "nlms", [8192, 0][case % 2], 4 - case % 3,
                       "round_robin", 50 * block + case)
    assert (total > 0).all(), total


def test_draw_words_that_come_too_late(tmp_path_factory):
    """Draw words are waited for at most so long, and their room goes to later
    insertions, where a wave that is later still would write into theirs: such a run
    ends in an internal error, any other is right."""
    lib = build(tmp_path_factory, "-DKVR_AWAIT_POLLS=20000")
    ended = {True: 0, False: 0}
    for case in range(32):
        s = generate(small_spec(n=120, groups=6, prefix_len=(1, 8), suffix_len=(8, 30), vocab=30, seed=case))
        r = check(lib, s, 3 + case % 3, s.max_len + 30, "nlms", 8192, 4 - case % 3, "round_robin", case, hold_draws=100,
                  may_fail=True)
        ended[r is not None] += 1
    assert min(ended.values()) > 0, ended
