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
