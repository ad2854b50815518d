"""The n = 4 walk kernel's launches: walks shared out among a block's wavefronts, backtracking states kept beside
them, against the oracle's walk of every walk on its own."""

import numpy as np
import pytest

import seeded_inputs
from oracle import walk as owalk
from oracle import zmat

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_1606_07413_amd import tcw
    assert torch.cuda.is_available()
    return tcw.Context(0)


# one walk, an odd number, one more pair than a block's 16 wavefronts, more than two rounds of them in a block
@pytest.mark.parametrize("walks,iters", [(1, 5), (3, 4), (34, 6), (2 * 16 * 256 * 2 + 35, 2)])
def test_walks_without_distinguished_points(ctx, walks, iters):
    """theta so small that no trail ends: a pair's two walks share 2 iters evaluations, a side-0 step first, two side-1
    steps together; a walk without a partner takes iters."""
    print("walks", walks, iters, flush=True)
    n, k, seed = 4, 4, 9
    tw = seeded_inputs.target_words(n, k, 31)
    u = zmat.target_from_words(n, tw.paulis, tw.clifford)
    spec = owalk.make_spec(u, n, k, 0, seed, delta=32)
    tgt = ctx.target_from_words(n, tw.paulis, tw.clifford)
    w = ctx.walk(tgt, k, 0, seed, 32, walks=walks, log2_table=12, cap=1 << 20)
    first = w.read_states(0, walks)
    w.run(iters)
    st = w.read_states(0, walks)
    assert w.stats().steps == walks * iters
    cache = {}

    def f(pt):
        if pt not in cache:
            cache[pt] = owalk.f(spec, pt)
        return cache[pt]

    pairs = (walks + 1) // 2
    for q in sorted({0, pairs // 2, pairs - 1, pairs - 2} - {-1}):
        both = 2 * q + 1 < walks
        cur = [int(first["cur"][2 * q]), int(first["cur"][2 * q + 1]) if both else None]
        done, left = [0, 0], 2 * iters if both else iters
        while left:
            s = [c >> 32 if c is not None else 1 for c in cur]
            if both and s == [1, 1] and left >= 2:
                who = (0, 1)
            else:
                who = (1,) if both and s[0] == 1 and s[1] == 0 else (0,)
            for i in who:
                cur[i] = f(cur[i])
                done[i] += 1
            left -= len(who)
        for i in range(2 if both else 1):
            assert int(st["cur"][2 * q + i]) == cur[i] and int(st["len"][2 * q + i]) == done[i], (q, i)
            assert int(st["start"][2 * q + i]) == int(first["start"][2 * q + i])
    w.end()
