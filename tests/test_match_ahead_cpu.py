"""The pipelined step kernel's per-wave logic (csrc/kvr_trail.h), compiled for
one lane with g++ and replayed on the CPU in the orders its waves can take,
against the oracle."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import emul_kernel as E
import paper_2601_18999_amd as K
from oracle import oracle as O
from workload import generate, small_spec

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "emul")
CSRC = os.path.join(os.path.dirname(HERE), "..", "paper_2601_18999_amd", "csrc")


@pytest.fixture(scope="module")
def replay(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("ahead") / "libahead.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-ffp-contract=off", "-fPIC", "-shared",
                           "-Wno-unknown-pragmas", "-o", out, os.path.join(HERE, "kvr_emul_ahead.cpp")])
    lib = ctypes.CDLL(out)
    lib.emul_ahead.restype = ctypes.c_int
    lib.emul_ahead.argtypes = ([ctypes.POINTER(K.KvrConfig), ctypes.c_uint64] + [ctypes.c_void_p] * 8 +
                               [ctypes.c_uint32, ctypes.c_uint64, ctypes.c_void_p])
    return lib


UPDATE = {"nlms": 0, "rls": 1, "none": 2}


def check(lib, s, R, W, B, update, seed, ucap, order, **cfg):
    c = K.kvr_config_default(R, W, B, max(1, s.max_len), update=UPDATE[update], seed=seed, **cfg)
    arrays = [np.ascontiguousarray(s.tokens, np.int32), np.ascontiguousarray(s.offsets, np.uint64),
              np.ascontiguousarray(s.arrival_us, np.int64), np.ascontiguousarray(s.out_len, np.uint16)]
    route, hits = np.zeros((R, s.n), np.int32), np.zeros((R, s.n), np.int32)
    ah = np.zeros((R, s.n, W), np.int32)
    st = (K.KvrWorkerStats * (R * W))()
    counts = np.zeros(6, np.uint64)
    rc = lib.emul_ahead(ctypes.byref(c), s.n, *[a.ctypes.data for a in arrays], route.ctypes.data, hits.ctypes.data,
                        ah.ctypes.data, ctypes.cast(st, ctypes.c_void_p), ucap, order, counts.ctypes.data)
    assert rc == 0
    flat = K._stats_dicts(st, R * W)
    for r in range(R):
        o = O.run(s, W, B, replica=r, all_hits=True, update=update, seed=seed)
        np.testing.assert_array_equal(route[r], o["route"])
        np.testing.assert_array_equal(hits[r], o["hits"])
        np.testing.assert_array_equal(ah[r], o["all_hits"])
        for i in range(W):
            got, want = flat[r * W + i], o["workers"][i]
            assert {k: got[k] for k in want} == want, (r, i)
    return counts


@pytest.mark.parametrize("block", range(4))
def test_any_order_of_the_waves_matches_the_oracle(replay, block):
    """Random small instances (deep and shallow tries, tight and roomy caches,
    staged and unstaged candidates, an arena that the collector packs), each
    in a random order of the waves' work.  Every way in which a match on a
    worker under eviction can come out has to occur."""
    rng = np.random.default_rng(400 + block)
    total = np.zeros(6, np.uint64)
    for case in range(40):
        s = generate(small_spec(n=int(rng.integers(20, 200)), groups=int(rng.integers(1, 8)),
                                prefix_len=(1, int(rng.integers(2, 40))), suffix_len=(1, int(rng.integers(2, 24))),
                                vocab=int(rng.integers(2, 12)), seed=1000 * block + case))
        W = int(rng.integers(1, 6))
        B = int(max(s.max_len, rng.integers(2, 260)))
        tight = {"arena_words": 2 * (B + 2 * s.max_len + 64)} if case % 4 == 3 else {}
        total += check(replay, s, 2, W, B, ["nlms", "rls", "none"][case % 3], case, [8192, 4, 0][case % 3], case, **tight)
    assert (total > 0).all(), total


def test_shared_prefix_workload(replay):
    """The drifting-groups recipe with long edges (16-byte blocks in line and
    edges longer than a round of compares)."""
    s = generate(small_spec(n=300, groups=12, prefix_len=(128, 700), suffix_len=(32, 128), vocab=32000, seed=3))
    total = check(replay, s, 1, 3, 6000, "nlms", 1, 512, 9)
    assert total[1] > 0, total


@pytest.mark.parametrize("seed,words", [(14, 1.0), (362, 1.0), (880, 1.0), (13, 1.5), (921, 1.5), (666, 2), (703, 2)])
def test_arenas_that_the_live_data_just_fits(replay, seed, words):
    """Short edges in next to the smallest arena: a collection must not need more
    room than the words that are live, padding or not."""
    rng = np.random.default_rng(seed)
    s = generate(small_spec(n=int(rng.integers(50, 300)), groups=int(rng.integers(1, 8)),
                            prefix_len=(1, int(rng.integers(2, 6))), suffix_len=(1, int(rng.integers(2, 9))),
                            vocab=int(rng.integers(2, 12)), seed=seed))
    W = int(rng.integers(1, 4))
    B = int(max(s.max_len, rng.integers(2, 300)))
    arena = int((B + 2 * s.max_len + 64) * words)
    check(replay, s, 1, W, B, "nlms", seed, 8192, seed, arena_words=arena)
    e = E.run(s, 1, W, B, seed=seed, arena_words=arena)
    assert e["rc"] == 0 and sum(w["gc_runs"] for w in e["workers"][0]) > 0
    np.testing.assert_array_equal(e["all_hits"][0], O.run(s, W, B, replica=0, all_hits=True, seed=seed)["all_hits"])
