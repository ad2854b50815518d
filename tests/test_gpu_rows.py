"""Exact kernels that hold a matrix's rows in registers, against the CPU oracle: whole numbers, so equality."""

import numpy as np
import pytest

import seeded_inputs
from oracle import search as osearch
from oracle import walk as owalk
from oracle import zmat

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_1606_07413_amd import tcw
    assert torch.cuda.is_available()
    return tcw.Context(0)


def oracle_target(n, k, seed):
    tw = seeded_inputs.target_words(n, k, seed)
    return tw, zmat.target_from_words(n, tw.paulis, tw.clifford)


# (n, the target's rotations, the space's k): no rotation at all (k = 1), odd and even exponents, the deepest
# halves that 32-bit points allow (n = 1: 20 rotations, n = 2: 8, n = 3: 5, n = 4: 4)
@pytest.mark.parametrize("n,kt,k,count", [(1, 1, 1, 3), (1, 9, 9, 40), (1, 3, 41, 40), (2, 3, 3, 5), (2, 6, 6, 33),
                                          (2, 2, 17, 20), (3, 1, 1, 2), (3, 7, 7, 9), (3, 4, 11, 5), (4, 1, 1, 2),
                                          (4, 8, 8, 3)])
def test_claw_check_edges(ctx, n, kt, k, count):
    import torch
    print("claw rows", n, kt, k, count, flush=True)
    tw, u = oracle_target(n, kt, 60 + n + k)
    c = tw.paulis[0] if k % 2 else 0
    spec = owalk.make_spec(u, n, k, c, 1, delta=4)
    r = 4 ** n
    pts = [seeded_inputs.uniform_below(5, i, spec.n_half) for i in range(2 * count)]
    u0 = [owalk.pack(pts[2 * i], 0) for i in range(count)]
    u1 = [owalk.pack(pts[2 * i + 1], 1) for i in range(count)]
    if kt == k:
        xv, xw, _ = owalk.planted_points(n, k, tw.paulis)
        u0[-1], u1[-1] = owalk.pack(xw, 1), owalk.pack(xv, 0)     # a claw, the sides in either order
        u0[0], u1[0] = owalk.pack(xv, 0), owalk.pack(xw, 1)
    u1[1] = owalk.pack(pts[3], 0)                                 # two points of one side
    ok = torch.empty(count, dtype=torch.int32, device="cuda:0")
    perm = torch.empty((count, r), dtype=torch.int32, device="cuda:0")
    sign = torch.empty((count, r), dtype=torch.int8, device="cuda:0")
    ctx.claw_check(ctx.target_from_words(n, tw.paulis, tw.clifford), k, c, 1, torch.tensor(u0, device="cuda:0"),
                   torch.tensor(u1, device="cuda:0"), ok, perm, sign)
    ok, perm, sign = ok.cpu().numpy(), perm.cpu().numpy(), sign.cpu().numpy()
    for i in range(count):
        dec = osearch.claw_check(spec, u0[i], u1[i])
        assert ok[i] == (1 if dec is not None else 0), i
        assert np.array_equal(perm[i], dec.perm if dec else np.full(r, -1)), i
        assert np.array_equal(sign[i], dec.sign if dec else np.zeros(r)), i
    if kt == k:
        assert ok[0] == 1 and ok[-1] == 1


# labels and certificates whose halves take several levels: all on one side (h_max 0), one target and few
# (the products shared between wavefronts), more than one batch of targets, n = 1 and 2
@pytest.mark.parametrize("n,h_max,count", [(1, 3, 5), (1, 4, 300), (2, 2, 1), (2, 3, 40), (3, 0, 7), (3, 1, 1), (3, 1, 65),
                                           (3, 2, 3), (3, 2, 1100), (3, 3, 2)])
def test_labels_match_search(ctx, n, h_max, count):
    import torch
    print("labels", n, h_max, count, flush=True)
    tws = [seeded_inputs.target_words(n, i % (2 * h_max + 3), 9000 + i) for i in range(count)]
    feats = torch.empty((count, 16 ** n), dtype=torch.float32, device="cuda:0")
    labels = torch.empty(count, dtype=torch.int32, device="cuda:0")
    ctx.label_batch(n, [(t.paulis, t.clifford) for t in tws], h_max, 3, feats, labels)
    labels = labels.cpu().tolist()
    for i in list(range(min(count, 6))) + list(range(6, count, 97)):
        tgt = ctx.target_from_words(n, tws[i].paulis, tws[i].clifford)
        p = ctx.default_params(n)
        p.k_max, p.enum_max, p.chunk_parallel = min(2 * h_max, 5), 1 << 22, 0
        res = ctx.search(tgt, p)
        want = res.t if res.status == 1 else -1
        if want < 0 and 2 * h_max > 5:
            assert labels[i] in (-1, 6, 7, 8), i      # above the depths searched here
        else:
            assert labels[i] == want, i
        assert ctx.min_tcount(tgt, h_max, 17) == labels[i], i


@pytest.mark.parametrize("count", [4, 5])
def test_labels_by_own_and_stored_keys(ctx, count):
    """Up to four targets make the keys of their side themselves, more share stored ones, here in parts
    (three rotations on the targets' side): labels up to 6, and the certificate of each."""
    import torch
    print("labels", count, flush=True)
    tws = [seeded_inputs.target_words(3, 3 + i, 7700 + i) for i in range(count)]
    feats = torch.empty((count, 16 ** 3), dtype=torch.float32, device="cuda:0")
    labels = torch.empty(count, dtype=torch.int32, device="cuda:0")
    ctx.label_batch(3, [(t.paulis, t.clifford) for t in tws], 3, 5, feats, labels)
    for i, got in enumerate(labels.cpu().tolist()):
        assert got <= 3 + i and (got >= 0 or 3 + i > 6), i
        assert ctx.min_tcount(ctx.target_from_words(3, tws[i].paulis, tws[i].clifford), 3, 9) == got, i


def test_certificate_above_six(ctx):
    """h_max = 4: the target's products come in parts; the Toffoli's T-count is 7."""
    v = seeded_inputs.permutation_unitary(seeded_inputs.NAMED_GATES["toffoli"])
    tgt = ctx.target_from_unitary(3, v, 0)
    assert ctx.min_tcount(tgt, 4) == 7
    assert ctx.min_tcount(tgt, 3) == -1


def long_word(n, rotations, seed):
    """`rotations` seeded rotations and their inverses (R(P)^8 = I, so R(P)^7 = R(P)^T), then two more: an
    unreduced exponent far above the end's."""
    ps = seeded_inputs.target_words(n, rotations + 2, seed).paulis
    return [p for p in ps[:rotations]] + [p for p in reversed(ps[:rotations]) for _ in range(7)] + ps[rotations:]


# no rotation and no Clifford word, ragged Clifford words, words past the exponent at which rows are reduced
# on the way, more targets than blocks are started for one at a time
@pytest.mark.parametrize("n,count", [(1, 70), (2, 70), (3, 24)])
def test_batch_features(ctx, n, count):
    import torch
    from oracle import mlp as omlp
    print("batch features", n, count, flush=True)
    words = []
    for i in range(count):
        tw = seeded_inputs.target_words(n, i % 8, 300 + i, clifford_len=(0, 1, 5, 16 * n)[i % 4])
        words.append((tw.paulis, tw.clifford))
    words[5] = (long_word(n, 10, 7), words[5][1])
    words[6] = ([1] * 160, [])
    feats = torch.empty((count, 16 ** n), dtype=torch.float32, device="cuda:0")
    labels = torch.empty(count, dtype=torch.int32, device="cuda:0")
    ctx.label_batch(n, words, 1, 3, feats, labels)
    feats = feats.cpu().numpy()
    for i, (paulis, clifford) in enumerate(words):
        want = omlp.features(zmat.target_from_words(n, paulis, clifford))
        assert np.array_equal(feats[i].view(np.uint32), want.view(np.uint32)), i


def test_features_beyond_int8(ctx):
    """Entries beyond int8 (the general sort), and words too long for int8 refused by the batch."""
    import torch
    from oracle import mlp as omlp
    from paper_1606_07413_amd import tcw
    for n, k in ((1, 22), (2, 24), (3, 26)):
        print("features beyond int8", n, k, flush=True)
        tw = seeded_inputs.target_words(n, k, 12)
        if n == 1:
            tw.paulis = [1 + i % 3 for i in range(k)]     # no two neighbours alike: the exponent grows with each
        u = zmat.target_from_words(n, tw.paulis, tw.clifford)
        assert max(abs(int(v)) for row in u.A for v in row) > 127
        out = torch.empty(16 ** n, dtype=torch.float32, device="cuda:0")
        ctx.features(ctx.target_from_words(n, tw.paulis, tw.clifford), out)
        assert np.array_equal(out.cpu().numpy().view(np.uint32), omlp.features(u).view(np.uint32))
        with pytest.raises(tcw.TcwError):
            ctx.label_batch(n, [(tw.paulis, tw.clifford)], 1, 3, out, torch.empty(1, dtype=torch.int32, device="cuda:0"))


# no words at all; a Clifford word only, past one wavefront's worth of words; the most rotations that the
# rows take unreduced (56) and more; words that grow and come back (82 rotations)
@pytest.mark.parametrize("n,k,m", [(1, 0, 0), (2, 0, 0), (3, 0, 0), (4, 0, 0), (1, 9, 130), (2, 0, 65), (3, 3, 64),
                                   (3, 0, 200), (4, 9, 3), (1, 56, 2), (1, 57, 2), (2, 56, 5), (2, 57, 5), (3, 56, 1),
                                   (1, -1, 3), (2, -1, 3), (3, -1, 3)])
def test_target_words_edges(ctx, n, k, m):
    from paper_1606_07413_amd import tcw
    print("target words", n, k, m, flush=True)
    paulis = long_word(n, 10, 9) if k < 0 else seeded_inputs.target_words(n, k, 71).paulis
    clifford = seeded_inputs.random_clifford_word(n, 5, length=m)
    u = zmat.target_from_words(n, paulis, clifford)
    a, b, e = ctx.target_from_words(n, paulis, clifford).channel()
    assert e == u.e
    assert np.array_equal(a, np.array(u.A, dtype=np.int64)) and np.array_equal(b, np.array(u.B, dtype=np.int64))
    if k == 56 and n == 3:
        with pytest.raises(tcw.TcwError) as err:     # beyond int32 on the way
            ctx.target_from_words(n, seeded_inputs.target_words(n, 90, 71).paulis, clifford)
        assert err.value.code == tcw.TCW_EOVERFLOW


# a step's space made from the target: even and odd k, the smallest and the last chunk, a chunk that lowers the
# exponent and one that raises it; and the refusal of entries beyond int8 with nothing written
@pytest.mark.parametrize("n,k", [(1, 1), (1, 6), (2, 1), (2, 4), (2, 7), (3, 3), (3, 6), (3, 7), (4, 1), (4, 2), (4, 5)])
def test_spaces_of_chunks(ctx, n, k):
    import torch
    from paper_1606_07413_amd import tcw
    tw, u = oracle_target(n, k, 200 + n)
    tgt = ctx.target_from_words(n, tw.paulis, tw.clifford)
    for chunk in ([1, 4 ** n - 1, tw.paulis[0]] if k % 2 else [0]):
        print("space", n, k, chunk, flush=True)
        spec = owalk.make_spec(u, n, k, chunk, 5, delta=3)
        pts = seeded_inputs.random_points(spec.n_half, 5, 8) + [0, 1 << 32, spec.n_half - 1, (1 << 32) + spec.n_half - 1]
        pin = torch.tensor(pts, dtype=torch.int64, device="cuda:0")
        out, hh = torch.empty_like(pin), torch.empty_like(pin)
        ctx.step(tgt, k, chunk, 5, 3, pin, out, hh)
        want = [owalk.f_with_hash(spec, p) for p in pts]
        mask = (1 << 64) - 1
        assert [int(v) & mask for v in out.cpu().tolist()] == [w[0] for w in want]
        assert [int(v) & mask for v in hh.cpu().tolist()] == [w[1] for w in want]
    big = ctx.target_from_words(n, [1 + (5 * i) % 3 for i in range(20)], [])
    if n == 1:
        pin = torch.zeros(3, dtype=torch.int64, device="cuda:0")
        out = torch.full_like(pin, 77)
        with pytest.raises(tcw.TcwError) as err:
            ctx.step(big, 3, 1, 5, 3, pin, out)
        assert err.value.code == tcw.TCW_EOVERFLOW and out.cpu().tolist() == [77] * 3


def test_batch_opens_chunks_together(ctx):
    """Targets of every n in one batch (their spaces are made together per qubit count), exhaustively: the answers of
    the single searches."""
    from paper_1606_07413_amd import tcw
    tws = [seeded_inputs.target_words(n, k, 40 + n) for n, k in ((1, 3), (2, 3), (2, 4), (3, 3), (3, 4), (4, 2))]
    tgts = [ctx.target_from_words(t.n, t.paulis, t.clifford) for t in tws]
    ps = []
    for t in tws:
        p = ctx.default_params(t.n)
        p.k_max, p.enum_max = t.k, 1 << 20
        ps.append(p)
    res, _ = ctx.search_batch(tgts, ps)
    for t, tgt, p, r in zip(tws, tgts, ps, res):
        for par in (0, 1, 5):
            p.chunk_parallel = par
            one = ctx.search(tgt, p)
            print("batch", t.n, t.k, par, one.t, flush=True)
            assert (one.status, one.t, one.minimal) == (1, r.t, 1) and r.status == 1
            dec = tcw.decomposition_of(one)
            got = osearch.Decomposition(t=dec.t, paulis_desc=dec.paulis_desc, perm=dec.perm, sign=dec.sign)
            assert osearch.reconstruct(t.n, got).equals(zmat.target_from_words(t.n, t.paulis, t.clifford))
