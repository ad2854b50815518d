"""Calls at the edges of their kernels' dispatch and of the context's memory."""

import numpy as np
import pytest

import seeded_inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_1606_07413_amd import tcw
    assert torch.cuda.is_available()
    return tcw.Context(0)


# every target of the first kind is found by its product of no rotation, at level 0, while the block's other
# wavefronts start the same level; the rest are found later, on targets in between
@pytest.mark.parametrize("n,count", [(1, 1), (1, 4500), (2, 3), (2, 4500)])
def test_labels_of_cliffords(ctx, n, count):
    import torch
    print("labels of Cliffords", n, count, flush=True)
    words = []
    for i in range(count):
        tw = seeded_inputs.target_words(n, 0 if i % 3 else 1, 500 + i % 50)
        words.append((tw.paulis, tw.clifford))
    feats = torch.empty((count, 16 ** n), dtype=torch.float32, device="cuda:0")
    labels = torch.empty(count, dtype=torch.int32, device="cuda:0")
    for h_max in (0, 2):
        ctx.label_batch(n, words, h_max, 3, feats, labels)
        # one rotation and a Clifford has T-count 1 (its channel representation has entries 1 / sqrt2)
        want = [0 if i % 3 else (1 if h_max else -1) for i in range(count)]
        assert labels.cpu().tolist() == want, h_max
    tgt = ctx.target_from_words(n, *words[-1])
    assert ctx.min_tcount(tgt, 0) == (0 if (count - 1) % 3 else -1)


@pytest.fixture
def full_memory():
    """Fills the GPU's memory to about the given number of bytes, in blocks, until the test ends."""
    import torch
    held = []

    def fill(leave):
        torch.cuda.synchronize()
        while True:
            room = torch.cuda.mem_get_info()[0] - leave
            if room < 1 << 26:
                return
            held.append(torch.empty(min(room, 16 << 30), dtype=torch.uint8, device="cuda:0"))
    yield fill
    held.clear()
    torch.cuda.empty_cache()


def test_allocations_take_the_pool_back(full_memory):
    """With the rest of the memory in use, a context's other allocations get what its idle pool holds (1 GiB of
    a label call's table): a walk session's table, a network; what does not fit at all is refused, and the
    refusal does not reach later calls."""
    import torch
    from paper_1606_07413_amd import tcw
    own = tcw.Context(0)
    tw = seeded_inputs.target_words(2, 4, 7)
    tgt = own.target_from_words(2, tw.paulis, tw.clifford)
    count = 16384
    words = [seeded_inputs.target_words(2, 1 + i % 8, 20 + i % 64) for i in range(count)]
    words = [(t.paulis, t.clifford) for t in words]
    feats = torch.empty((count, 256), dtype=torch.float32, device="cuda:0")
    labels = torch.empty(count, dtype=torch.int32, device="cuda:0")

    def fill_pool():
        own.label_batch(2, words, 4, 3, feats, labels)

    def walk(log2_table):
        w = own.walk(tgt, 4, 0, 3, 4, 64, log2_table, 1 << 10)
        w.run(4)
        assert w.stats().steps == 256
        w.end()

    before = torch.cuda.mem_get_info()[0]
    fill_pool()
    assert before - torch.cuda.mem_get_info()[0] >= 1 << 30
    full_memory(3 << 28)
    print("walk table beside an idle pool", flush=True)
    walk(26)
    assert torch.cuda.mem_get_info()[0] >= 1 << 30
    fill_pool()
    print("network beside an idle pool", flush=True)
    net = tcw.Network(own, 4096, 8192, 1, 11, seed=1)      # 4 x 128 MiB of FP32, 2 x 64 of BF16
    x = torch.zeros((2, 4096), dtype=torch.float32, device="cuda:0")
    probs = torch.empty((2, 11), dtype=torch.float32, device="cuda:0")
    net.forward(x, probs)
    assert torch.allclose(probs.sum(1), torch.ones(2, device="cuda:0"))
    net.free()
    print("more than there is", flush=True)
    with pytest.raises(tcw.TcwError) as err:
        walk(30)
    assert tcw.ERRORS[err.value.code] == "ENOMEM"
    walk(12)
    own.target_from_words(2, tw.paulis, tw.clifford)


def test_large_tables_are_not_kept():
    """A label call whose table takes 2 GiB (32,768 targets at n = 1 with T-count up to 20) gives the memory
    back when it returns."""
    import torch
    from paper_1606_07413_amd import tcw
    own = tcw.Context(0)
    count = 32768
    words = [seeded_inputs.target_words(1, i % 9, i % 50) for i in range(count)]
    feats = torch.empty((count, 16), dtype=torch.float32, device="cuda:0")
    labels = torch.empty(count, dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    own.label_batch(1, [(t.paulis, t.clifford) for t in words], 10, 3, feats, labels)
    after = torch.cuda.mem_get_info()[0]
    got = labels.cpu().tolist()
    assert all(0 <= g <= i % 9 for i, g in enumerate(got))
    assert before - after < 1 << 28


def test_batch_of_many_members(ctx):
    """More 4-qubit members than a grid's second dimension has blocks: their spaces are made together."""
    from paper_1606_07413_amd import tcw
    tw = seeded_inputs.target_words(4, 1, 5)
    tgt = ctx.target_from_words(4, tw.paulis, tw.clifford)
    p = ctx.default_params(4)
    p.k_max = p.depth_order_len = p.depth_order[0] = 1
    p.depth_order_kind = 2                       # depth 1 at its one chunk, first found
    p.chunk_first = p.chunk_last = tw.paulis[0]
    count = 65537
    print("batch of", count, flush=True)
    res, _ = ctx.search_batch([tgt] * count, [p] * count)
    assert all(r.status == 1 and r.t == 1 and r.paulis[0] == tw.paulis[0] for r in res)
    one = tcw.decomposition_of(ctx.search(tgt, p))
    for r in (res[0], res[-1]):
        dec = tcw.decomposition_of(r)
        assert (dec.paulis_desc, dec.perm, dec.sign) == (one.paulis_desc, one.perm, one.sign)


def enumerated(ctx, n, k, seed):
    """A target of k rotations and parameters that search depth k alone, exhaustively (the first hit ends it)."""
    tw = seeded_inputs.target_words(n, k, seed)
    p = ctx.default_params(n)
    p.k_max = p.depth_order[0] = k
    p.depth_order_kind, p.depth_order_len, p.enum_max, p.walks = 2, 1, 1 << 26, 1 << 18
    return ctx.target_from_words(n, tw.paulis, tw.clifford), p


def best_of(reps, fn):
    import time
    import torch
    out = []
    for _ in range(reps):
        t0 = time.perf_counter()
        fn()
        torch.cuda.synchronize()
        out.append(time.perf_counter() - t0)
    return min(out)


def test_enumerated_members_of_several_sizes(ctx):
    """Members with tables from 2^5 to 2^27 slots, some alike: as many candidates as a session's exhaustive walk
    of the same space has, and the single search's answer; and the one large table is read out by as many blocks as in a single search (the whole
    searches take about the same time, where 32 blocks took twice as long)."""
    specs = [(2, 12, 1), (1, 2, 2), (2, 4, 3), (3, 4, 4), (2, 4, 5), (1, 6, 6), (4, 2, 7)]
    members = [enumerated(ctx, *s) for s in specs]
    for _, p in members:
        p.iters_per_launch = 64
    res, _ = ctx.search_batch([t for t, _ in members], [p for _, p in members])
    for s, (t, p), r in zip(specs, members, res):
        n, k, _ = s
        points = 2 * (4 ** n - 1) ** (k // 2)
        w = ctx.walk(t, k, 0, p.seed, 0, min(points, p.walks), max(4, (4 * points - 1).bit_length()), 2, enumerate=True,
                     version=p.version)
        while w.stats().steps < points:
            w.run(64)
        claws = w.claws()[1]
        w.end()
        one = ctx.search(t, p)
        print("enumerated", s, r.status, r.t, r.stats.claws, claws, flush=True)
        assert (r.status, r.t, r.stats.steps) == (one.status, one.t, one.stats.steps) == (1, k, points)
        assert r.stats.claws == claws >= 1
    t, p = members[0]
    batch = best_of(4, lambda: ctx.search_batch([t], [p]))
    single = best_of(4, lambda: ctx.search(t, p))
    print("batch %.2f ms, single %.2f ms" % (batch * 1e3, single * 1e3), flush=True)
    assert batch < 1.5 * single


# (inputs, hidden width, layers, classes, batch) on both sides of each line: one row by K and by N for its K; a few
# rows by K (FP32, then in the hidden layers BF16) and N; the FP32 first product by N, by K and by its whole size;
# the output layer by K and rows
ROUTES = [(188, 96, 1, 11, 1), (192, 3072, 1, 11, 1), (192, 3073, 1, 11, 1), (40, 191, 2, 11, 1), (40, 192, 2, 11, 1),
          (252, 130, 1, 11, 2), (256, 130, 1, 11, 3), (1536, 2048, 1, 11, 8), (1536, 2049, 1, 11, 2), (1540, 64, 1, 11, 8),
          (40, 383, 2, 11, 5), (40, 384, 2, 11, 8), (40, 2048, 2, 11, 2), (40, 2052, 2, 11, 8),
          (4096, 2048, 1, 11, 513), (4096, 2049, 1, 11, 513), (4096, 2049, 1, 11, 512), (8196, 1025, 1, 11, 257),
          (6144, 1, 0, 11, 33), (6148, 1, 0, 11, 33), (8192, 1, 0, 11, 21), (8192, 1, 0, 11, 22), (8192, 1, 0, 5, 511),
          (8192, 1, 0, 5, 512), (8196, 1, 0, 5, 2047), (8196, 1, 0, 5, 2048)]


@pytest.mark.parametrize("inp,hidden,depth,classes,batch", ROUTES)
def test_network_routes(ctx, inp, hidden, depth, classes, batch):
    """Probabilities within the running error bound of the GPU's arithmetic (as in the gradient tests)."""
    import torch
    from oracle import mlp as omlp
    from paper_1606_07413_amd import tcw
    import test_gpu_mlp as base
    print("network", inp, hidden, depth, classes, batch, flush=True)
    params = seeded_inputs.mlp_init(inp, hidden, depth, classes, 7)
    x = (np.random.default_rng(batch).normal(size=(batch, inp)) * 0.5).astype(np.float32)
    net = tcw.Network(ctx, inp, hidden, depth, classes, init=tcw.flatten_params(params, depth))
    probs = torch.empty((batch, classes), dtype=torch.float32, device="cuda:0")
    net.forward(torch.tensor(x, device="cuda:0"), probs)
    pr = {k: (omlp.bf16_round(v) if k.startswith("W") else v) for k, v in params.items()}
    y = np.zeros(batch, dtype=np.int32)
    _, p_ref, p_bound = base.gradient_error_bounds(pr, omlp.bf16_round(x).astype(np.float64), y, depth)
    assert np.all(np.abs(probs.cpu().numpy().astype(np.float64) - p_ref) <= 2 * p_bound)


def forward_time(ctx, inp, hidden, depth, classes, batch, shift=0):
    import torch
    from paper_1606_07413_amd import tcw
    net = tcw.Network(ctx, inp, hidden, depth, classes, seed=1)
    x = torch.zeros(batch * inp + shift, dtype=torch.float32, device="cuda:0")[shift:].view(batch, inp)
    probs = torch.empty((batch, classes), dtype=torch.float32, device="cuda:0")

    def some():
        for _ in range(8):
            net.forward(x, probs)
    some()
    t = best_of(8, some) / 8 * 1e6
    net.free()
    print("forward", inp, hidden, depth, classes, batch, shift, "%.1f us" % t, flush=True)
    return t


# a pass takes no longer than one that does more: two rows and nine, 32 classes and 33, an aligned input and
# one that has to be converted first (78 and 41 us, 245 and 109, 834 and 751, with rules that looked at the rows or at
# the classes alone)
@pytest.mark.parametrize("less,more,most", [((16384, 2048, 1, 11, 2), (16384, 2048, 1, 11, 9), 1.3),
                                            ((65536, 1, 0, 32, 32), (65536, 1, 0, 33, 32), 1.3),
                                            ((16384, 4096, 1, 11, 4096), (16384, 4096, 1, 11, 4096, 1), 1.05)])
def test_less_work_takes_no_longer(ctx, less, more, most):
    assert forward_time(ctx, *less) < most * forward_time(ctx, *more)


# pairs of walks: fewer than blocks, one to a block, a whole run of 16 to a block, one pair less and more, an odd walk
@pytest.mark.parametrize("walks", [2, 511, 514, 8190, 8192, 8193, 16384 + 6])
def test_walks_over_blocks(ctx, walks):
    """n = 4, theta so small that no trail ends: every pair of walks makes its 2 x iters steps, once, and the walks of
    a session do what they do in a session of another size."""
    n, k, iters = 4, 7, 3
    tw = seeded_inputs.target_words(n, k, 31)
    tgt = ctx.target_from_words(n, tw.paulis, tw.clifford)
    print("walks", walks, flush=True)

    def session(count):
        w = ctx.walk(tgt, k, tw.paulis[0], 9, 32, count, 12, 1 << 20)
        w.run(iters)
        st, steps = w.read_states(0, count), w.stats().steps
        w.end()
        assert steps == count * iters
        pairs = st["len"][: count // 2 * 2].astype(np.int64).reshape(-1, 2).sum(1)
        assert np.all(pairs == 2 * iters) and (count % 2 == 0 or st["len"][-1] == iters)
        return st
    st, more = session(walks), session(walks // 2 * 2 + 34)
    assert np.array_equal(st[: walks // 2 * 2], more[: walks // 2 * 2])


def test_few_walks_spread_over_the_chip(ctx):
    """A launch of 64 walks takes less than two and a bit of one walk's: the pairs run beside each other, not on a
    few CUs (2.85 times while 16 pairs shared a block's wavefronts)."""
    n, k = 4, 7
    tw = seeded_inputs.target_words(n, k, 5)
    tgt = ctx.target_from_words(n, tw.paulis, tw.clifford)
    ms = {}
    for walks in (1, 64):
        w = ctx.walk(tgt, k, tw.paulis[0], 3, 12, walks, 16, 20 << 12)
        took = []
        for _ in range(8):
            w.run(64)
            took.append(w.last_ms())
        w.end()
        ms[walks] = min(took)
    print("one walk %.3f ms, 64 walks %.3f ms" % (ms[1], ms[64]), flush=True)
    assert ms[64] < 2.2 * ms[1]


@pytest.mark.parametrize("n,h_max", [(1, 1), (2, 2), (3, 1), (3, 3)])
def test_labels_within_their_range(ctx, n, h_max):
    """A label is -1 or at most 2 h_max, and a circuit of no more rotations than that is never -1."""
    import torch
    tws = [seeded_inputs.target_words(n, i % 11, 4000 + i) for i in range(66)]
    feats = torch.empty((66, 16 ** n), dtype=torch.float32, device="cuda:0")
    labels = torch.empty(66, dtype=torch.int32, device="cuda:0")
    ctx.label_batch(n, [(t.paulis, t.clifford) for t in tws], h_max, 3, feats, labels)
    for t, got in zip(tws, labels.cpu().tolist()):
        assert got == -1 or 0 <= got <= min(t.k, 2 * h_max)
        assert got >= 0 or t.k > 2 * h_max
