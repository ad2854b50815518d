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


# small spaces, where many trails end in a cycle without a distinguished point: fewer trails than wavefronts,
# more (two at a time), one; caps below, at and above a trail's length
@pytest.mark.parametrize("n,k,delta,count,cap", [(4, 2, 3, 5000, 160), (4, 3, 5, 9000, 640), (4, 2, 4, 7, 3), (4, 2, 6, 1, 1280),
                                                 (4, 2, 2, 4500, 1), (3, 2, 4, 300, 320), (3, 4, 7, 700, 100), (2, 4, 5, 200, 640),
                                                 (1, 6, 4, 60, 7)])
def test_trails_and_cycles(ctx, n, k, delta, count, cap):
    import torch
    print("trails", n, k, delta, count, cap, flush=True)
    tw = seeded_inputs.target_words(n, max(k, 3), 77)
    tgt = ctx.target_from_words(n, tw.paulis, tw.clifford)
    chunk = tw.paulis[0] if k % 2 else 0
    u = zmat.target_from_words(n, tw.paulis, tw.clifford)
    spec = owalk.make_spec(u, n, k, chunk, 4, delta=delta)
    # f on the whole space by the step call, which the parity tests hold to the oracle; a few points here too
    pts = [x | (b << 32) for b in (0, 1) for x in range(spec.n_half)]
    pin = torch.tensor(pts, dtype=torch.int64, device="cuda:0")
    out = torch.empty_like(pin)
    ctx.step(tgt, k, chunk, 4, delta, pin, out)
    f = dict(zip(pts, out.cpu().tolist()))
    for pt in pts[:: max(1, len(pts) // 4)]:
        assert f[pt] == owalk.f(spec, pt)
    starts = [pts[seeded_inputs.uniform_below(6, i, len(pts))] for i in range(count)]
    dp = torch.empty(count, dtype=torch.int64, device="cuda:0")
    ln = torch.empty(count, dtype=torch.int32, device="cuda:0")
    ctx.trails(tgt, k, chunk, 4, delta, torch.tensor(starts, device="cuda:0"), cap, dp, ln)
    dp, ln = dp.cpu().tolist(), ln.cpu().tolist()
    want = {}
    for s in set(starts):
        pt, ans = s, (0, 0)
        for t in range(1, cap + 1):
            pt = f[pt]
            if owalk.distinguished(spec, pt):
                ans = (pt, t)
                break
        want[s] = ans
    assert [(d, l) for d, l in zip(dp, ln)] == [want[s] for s in starts]
    assert cap < 100 or delta < 3 or any(l == 0 for l in ln) or count == 1
