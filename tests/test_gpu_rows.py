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
