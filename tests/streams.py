"""Small hand-built query streams shared by the CPU and GPU tests (input
plumbing only: no matching, scoring or eviction here)."""
from __future__ import annotations

import numpy as np

from workload.gen import Stream


def random_response_stream(rng: np.random.Generator, n: int, vocab: int, max_prompt: int, max_resp: int,
                           B: int) -> Stream:
    """Random complete paths q || a (prompt 1..max_prompt tokens, response
    0..max_resp tokens, |q| + |a| <= B) over a small vocabulary, so prompts
    are often cached whole and the responses after them partly cached too;
    Poisson-like arrivals up to 0.4 s apart."""
    lens, olen, toks = [], [], []
    for _ in range(n):
        L = int(rng.integers(1, max(1, min(max_prompt, B - max_resp)) + 1))
        o = int(rng.integers(0, max_resp + 1))
        toks.append(rng.integers(0, vocab, size=L + o).astype(np.int32))
        lens.append(L + o)
        olen.append(o)
    off = np.zeros(n + 1, dtype=np.uint64)
    off[1:] = np.cumsum(lens)
    return Stream(tokens=np.concatenate(toks), offsets=off,
                  arrival_us=np.cumsum(rng.integers(1, 400000, size=n)).astype(np.int64),
                  out_len=np.array(olen, dtype=np.uint16), spec={"kind": "random_responses", "n": n})


def stream_of(rng: np.random.Generator, paths) -> Stream:
    """The prompts of `paths`, in order, up to 0.1 s apart."""
    off = np.zeros(len(paths) + 1, dtype=np.uint64)
    off[1:] = np.cumsum([len(p) for p in paths])
    return Stream(tokens=np.concatenate(paths).astype(np.int32), offsets=off,
                  arrival_us=np.cumsum(rng.integers(1, 100000, size=len(paths))).astype(np.int64),
                  out_len=np.full(len(paths), 4, dtype=np.uint16), spec={"kind": "paths", "n": len(paths)})


def long_beside_short_stream(rng: np.random.Generator, cycles: int, W: int, long_len: int, short_len: int,
                             quiet: int = 8) -> Stream:
    """For W > quiet + 1 workers in round-robin order.  Each cycle brings the
    first worker one long fresh prompt, then `quiet` short ones that nothing
    caches, then prefixes of the cycle's and of the last cycle's long prompt,
    whose matches on the first worker end where its evictions may be under
    way."""
    paths, last = [], None
    for c in range(cycles):
        new = rng.integers(0, 1 << 20, size=long_len).astype(np.int32)
        new[0] = 2 * c
        paths.append(new)
        for _ in range(quiet):
            p = rng.integers(1 << 20, 1 << 30, size=int(rng.integers(1, short_len + 1))).astype(np.int32)
            paths.append(p)
        while len(paths) % W:
            old = last if last is not None and rng.integers(0, 4) else new
            paths.append(old[:int(rng.integers(1, long_len + 1))])
        last = new
    return stream_of(rng, paths)
