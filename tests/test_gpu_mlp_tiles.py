"""The depth-order network's products at the edges of their tiles: rows, columns and leading dimensions
that are odd, one short of a tile or one past it, each with the error bounds of the gradient test."""

import pytest

import test_gpu_mlp as base

pytestmark = pytest.mark.gpu

ctx = base.ctx

# (inputs, hidden width, batch) around the 64 x 128 tiles, the 32-row fragments and the pairs of columns
EDGES = [(16, 96, 1), (64, 33, 63), (256, 127, 64), (256, 129, 65), (264, 128, 131), (40, 1, 9)]


@pytest.mark.parametrize("inp,hidden,batch", EDGES)
def test_gradients_at_tile_edges(ctx, inp, hidden, batch):
    base.test_gradients_against_oracle(ctx, inp, hidden, batch)
