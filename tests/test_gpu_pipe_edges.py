"""The pipelined step kernel where its forms change, bit-exact against the
oracle on an MI355X: 12 or 16 waves (at 17 workers), two, three or four query
buffers (by the LDS that max_query_tokens leaves), a ring of draw words that
holds no whole insertion, the learned router's form or the baselines', and
batches checked by the step kernel itself or by kernels before it."""
import numpy as np
import pytest

import paper_2601_18999_amd as K
from gpu_helpers import assert_parity, gpu_run, note
from oracle import oracle as O
from streams import long_beside_short_stream, stream_of
from workload import generate, small_spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("router", ["lbgr", "cache_aware"])
@pytest.mark.parametrize("W,max_len", [
    (1, 4000),              # one worker: every query is routed to it
    (16, 900), (17, 900),   # 12 and 16 waves
    (23, 900), (24, 900),
    (4, 5848), (4, 5860),   # four and three query buffers
    (4, 7044), (4, 7056),   # three and two
    (64, 16384),            # two, and no room for draw words or candidates
])
def test_forms_of_the_pipelined_kernel(W, max_len, router):
    s = generate(small_spec(n=260, groups=5, prefix_len=(1, 500), suffix_len=(1, 300), vocab=9, seed=W + max_len))
    B = max(max_len, 1000)
    if max_len < 2000:
        B = max_len + 37  # evictions from the first queries on
    note(f"W={W} max_len={max_len} router={router}")
    R = {"lbgr": K.KVR_ROUTE_LBGR, "cache_aware": K.KVR_ROUTE_CACHE_AWARE}[router]
    res, stats = gpu_run(s, 2, W, B, batch=61, max_len=max_len, router=R)
    assert_parity(s, res, stats, W, B, range(2), router=router)


@pytest.mark.parametrize("batch", [31, 32, 33, 255, 256, 257])
@pytest.mark.parametrize("max_len", [31, 32, 256])
def test_batches_either_side_of_the_check_in_the_step_kernel(batch, max_len):
    """At most 256 queries and 8,192 tokens are checked by the step kernel."""
    s = generate(small_spec(n=520, groups=6, prefix_len=(1, 20), suffix_len=(1, 11), vocab=5, seed=batch))
    note(f"batch={batch} max_len={max_len}")
    res, stats = gpu_run(s, 3, 3, 300, batch=batch, max_len=max_len)
    assert_parity(s, res, stats, 3, 300, range(3))


@pytest.mark.parametrize("n", [5, 256, 257])
@pytest.mark.parametrize("fault", ["length", "arrival", "token"])
def test_an_invalid_batch_changes_nothing_on_either_path(n, fault):
    """The last query of the second batch is wrong: the batch is refused, with
    the same bits, and the first batch's results stay."""
    s = generate(small_spec(n=2 * n, groups=4, prefix_len=(2, 12), suffix_len=(2, 9), vocab=5, seed=n))
    if fault == "length":
        max_len = int(np.diff(s.offsets)[:-1].max())
        s.offsets = s.offsets.copy()
        extra = np.zeros(40, np.int32)
        s.tokens = np.concatenate([s.tokens, extra])
        s.offsets[-1] += 40
    else:
        max_len = s.max_len
        if fault == "arrival":
            s.arrival_us = s.arrival_us.copy()
            s.arrival_us[-1] = s.arrival_us[-2] - 1
        else:
            s.tokens = s.tokens.copy()
            s.tokens[-1] = -3
    sim = K.Simulator(2, 3, 200, max_len)
    try:
        sim.run(s, batch=n)
        st, bits = sim.check()
        stats = sim.stats(check=False)
    finally:
        sim.close()
    assert st != K.KVR_OK and bits == {"length": 1, "token": 2, "arrival": 4}[fault], (st, bits)
    assert all(sum(stats[r][i]["routed"] for i in range(3)) == n for r in range(2))


@pytest.mark.parametrize("B", [10600, 20000])
def test_an_insertion_that_outlasts_the_next_seven(B):
    """A prompt of 10,500 fresh tokens into a full cache, evicted while short
    prompts of other workers come and go, and then prefixes of earlier long
    prompts, matched beside those evictions."""
    s = long_beside_short_stream(np.random.default_rng(B), 10, 12, 10500, 24)
    note(f"B={B} max_len={s.max_len}")
    res, stats = gpu_run(s, 4, 12, B, batch=500, router=K.KVR_ROUTE_ROUND_ROBIN)
    assert sum(w["evictions"] for w in stats[0]) > 10500
    assert_parity(s, res, stats, 12, B, range(4), router="round_robin")


@pytest.mark.parametrize("batch", [2048, 2049, 5000])
def test_batches_launched_in_parts(batch):
    """The pipelined kernel takes at most 2,048 queries a launch: the parts
    follow one another as one batch, with its rows in the outputs."""
    s = generate(small_spec(n=5000, groups=9, prefix_len=(1, 20), suffix_len=(1, 9), vocab=5, seed=batch))
    note(f"batch={batch}")
    res, stats = gpu_run(s, 3, 3, 300, batch=batch)
    assert_parity(s, res, stats, 3, 300, range(3))


def test_a_replica_that_fails_stops_no_other_in_later_parts():
    """A completion ring one entry short of what the busiest replica needs: in one
    batch of several parts the others finish it."""
    s = generate(small_spec(n=5000, groups=9, prefix_len=(1, 20), suffix_len=(1, 9), vocab=5, seed=3))
    R, W, B = 8, 4, 300
    full = [O.run(s, W, B, replica=r, all_hits=True, router="random") for r in range(R)]
    caps = sorted(max(w["pending_max"] for w in o["workers"]) for o in full)
    assert caps[0] < caps[-1]
    res, _ = gpu_run(s, R, W, B, router=K.KVR_ROUTE_RANDOM, pending_capacity=caps[-1] - 1)
    assert res["status"] == K.KVR_ECAPACITY
    ok = 0
    for r in range(R):
        if max(w["pending_max"] for w in full[r]["workers"]) < caps[-1]:
            np.testing.assert_array_equal(res["route"][r], full[r]["route"])
            np.testing.assert_array_equal(res["all_hits"][r], full[r]["all_hits"])
            ok += 1
    assert 0 < ok < R


@pytest.mark.parametrize("W,max_len,B", [
    (4, 5848, 9000),     # 512 staged candidates: longer lists have a byte for each
    (3, 5848, 40000),    # lists of more than 8,192, which have none
    (64, 16384, 16384),  # some 30 staged candidates, bytes up to 480
])
def test_lists_longer_than_the_staging_area(W, max_len, B):
    """Thousands of short leaves and now and then a long prompt, whose evictions
    take whole blocks of draws."""
    rng = np.random.default_rng(W + B)
    n = {4: 6000, 3: 60000, 64: 4000}[W]
    paths = [rng.integers(0, 1 << 20, size=int(rng.integers(1, 8))) if j % 41 or j < n // 2 else
             rng.integers(0, 1 << 20, size=int(rng.integers(300, min(4000, max_len)))) for j in range(n)]
    if W == 64:
        paths = [p if j % 8 else rng.integers(0, 1 << 20, size=int(rng.integers(1, 400))) for j, p in enumerate(paths)]
        paths[::63] = [rng.integers(0, 1 << 20, size=int(rng.integers(4000, 16000))) for _ in paths[::63]]
    s = stream_of(rng, paths)
    res, stats = gpu_run(s, 1, W, B, batch=1500, max_len=max_len, router=K.KVR_ROUTE_ROUND_ROBIN)
    note(f"W={W} B={B} evictions={sum(w['evictions'] for w in stats[0])} nodes={max(w['nodes'] for w in stats[0])}")
    assert sum(w["evictions"] for w in stats[0]) > 20000
    assert_parity(s, res, stats, W, B, range(1), router="round_robin")


@pytest.mark.parametrize("evict", ["rlt", "lru"])
def test_edges_that_a_collection_has_packed(evict):
    """The smallest arena: the collector packs, and matches compare edges at any
    place within 16 bytes, of lengths around a round of compares (1,024)."""
    s = generate(small_spec(n=300, groups=8, prefix_len=(900, 1200), suffix_len=(1, 1100), vocab=3, seed=11))
    W, B = 3, 6000
    arena = B + 2 * s.max_len + 64
    res, stats = gpu_run(s, 2, W, B, batch=100, arena_words=arena, evict={"rlt": 0, "lru": 1}[evict])
    assert min(sum(w["gc_runs"] for w in st) for st in stats) > 10
    assert_parity(s, res, stats, W, B, range(2), evict=evict)


@pytest.mark.parametrize("R", [1024, 1025])
def test_batches_checked_for_many_replicas(R):
    """Up to 1,024 replicas the step kernel checks a small batch itself."""
    s = generate(small_spec(n=40, groups=3, prefix_len=(1, 9), suffix_len=(1, 6), vocab=5, seed=R))
    res, stats = gpu_run(s, R, 2, 60, batch=7)
    assert_parity(s, res, stats, 2, 60, [0, 511, R - 1])


@pytest.mark.parametrize("W,max_len,nbuf,words,staged", [
    (1, 4000, 4, 12000, 900), (24, 900, 4, 2700, 3000),
    (4, 5848, 4, 11696, 512), (4, 5860, 3, 17580, 512),
    (4, 7044, 3, 14088, 512), (4, 7056, 2, 21168, 512),
    (64, 16384, 2, 0, 20),
])
def test_the_form_is_the_one_that_the_rows_above_are_for(W, max_len, nbuf, words, staged):
    """Query buffers, at least so many draw words, and so many candidates."""
    import ctypes
    sim = K.Simulator(1, W, max(max_len, 1000), max_len)
    try:
        out = (ctypes.c_uint32 * 4)()
        f = K.load_library().kvr_internal_form
        f.argtypes, f.restype = [ctypes.c_void_p, ctypes.c_void_p], None
        f(sim.ctx, out)
    finally:
        sim.close()
    note(f"W={W} max_len={max_len}: {list(out)}")
    assert out[0] == 1 and out[1] == nbuf and out[2] >= words and out[3] >= staged
    if (W, max_len) == (64, 16384):
        assert out[2] == 0 and out[3] < 64
