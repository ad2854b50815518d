"""The depth-order network's kernels at the edges of their tiles: rows, columns and leading dimensions that
are odd, one short of a tile or one past it, the output layer on both sides of its 32 classes, and the
Adam step with the BF16 weights that it leaves."""

import numpy as np
import pytest

import seeded_inputs
import test_gpu_mlp as base
from oracle import mlp as omlp

pytestmark = pytest.mark.gpu

ctx = base.ctx

# (inputs, hidden width, batch) around the 64 x 128 tiles, the 32-row fragments and the pairs of columns
EDGES = [(16, 96, 1), (64, 33, 63), (256, 127, 64), (256, 129, 65), (264, 128, 131), (40, 1, 9)]


@pytest.mark.parametrize("inp,hidden,batch", EDGES)
def test_gradients_at_tile_edges(ctx, inp, hidden, batch):
    base.test_gradients_against_oracle(ctx, inp, hidden, batch)


def small_net(ctx, inp, hidden, depth, classes, batch):
    import torch
    from paper_1606_07413_amd import tcw
    params = seeded_inputs.mlp_init(inp, hidden, depth, classes, 7)
    rng = np.random.default_rng(batch)
    x = rng.normal(size=(batch, inp)).astype(np.float32) * 0.5
    y = rng.integers(0, classes, batch).astype(np.int32)
    net = tcw.Network(ctx, inp, hidden, depth, classes, init=tcw.flatten_params(params, depth))
    return net, params, x, y, torch.tensor(x, device="cuda:0"), torch.tensor(y, device="cuda:0")


@pytest.mark.parametrize("inp,depth,classes,batch", [(64, 1, 2, 33), (1032, 0, 32, 31), (1032, 0, 33, 31),
                                                     (96, 2, 31, 32), (96, 1, 40, 65)])
def test_output_layer(ctx, inp, depth, classes, batch):
    """Probabilities, loss and every gradient within the running error bound of the GPU's arithmetic."""
    import torch
    print("output layer", inp, depth, classes, batch, flush=True)
    net, params, x, y, xd, yd = small_net(ctx, inp, 64, depth, classes, batch)
    g, loss = net.gradients(xd, yd)
    probs = torch.empty((batch, classes), dtype=torch.float32, device="cuda:0")
    net.forward(xd, probs)
    pr = {k: (omlp.bf16_round(v) if k.startswith("W") else v) for k, v in params.items()}
    xb = omlp.bf16_round(x).astype(np.float64)
    ref = omlp.gradients(pr, xb, y, depth)
    bounds, p_ref, p_bound = base.gradient_error_bounds(pr, xb, y, depth)
    assert abs(loss - omlp.loss(pr, xb, y, depth)) < 1e-2 * abs(loss)
    assert np.all(np.abs(probs.cpu().numpy().astype(np.float64) - p_ref) <= 2 * p_bound)
    off = 0
    for l in range(depth + 1):
        for name in (f"W{l}", f"b{l}"):
            size = params[name].size
            got = g[off:off + size].reshape(params[name].shape).astype(np.float64)
            off += size
            assert np.all(np.abs(got - ref[name]) <= 2 * bounds[name]), name


# the larger batches split the weight gradients' K: 2, 8 and 16 partial products
@pytest.mark.parametrize("inp,hidden,depth,classes,batch", [(33, 31, 2, 5, 21), (64, 32, 1, 32, 21), (7, 1, 0, 2, 21),
                                                            (33, 31, 1, 5, 519), (64, 40, 2, 11, 2056),
                                                            (40, 33, 1, 7, 8192)])
def test_adam_and_weight_copies(ctx, inp, hidden, depth, classes, batch):
    """The first Adam step from the gradients themselves (eight roundings of at most 2^-24 relative, and the
    subtraction's), and a forward pass on its BF16 weights: that of a new network with those parameters."""
    import torch
    from paper_1606_07413_amd import tcw
    print("adam", inp, hidden, depth, classes, batch, flush=True)
    net, params, _, _, xd, yd = small_net(ctx, inp, hidden, depth, classes, batch)
    p0 = net.params().astype(np.float64)
    g = net.gradients(xd, yd)[0].astype(np.float64)
    lr = 1e-3
    net.train_step(xd, yd, lr)
    p1 = net.params()
    step = lr * g / (np.abs(g) + 1e-8)
    tol = 2.0 ** -24 * np.abs(p0) + 16 * 2.0 ** -24 * np.abs(step)
    assert np.all(np.abs(p1 - (p0 - step)) <= tol)
    fresh = tcw.Network(ctx, inp, hidden, depth, classes, init=p1)
    a, b = (torch.empty((batch, classes), dtype=torch.float32, device="cuda:0") for _ in range(2))
    net.forward(xd, a)
    fresh.forward(xd, b)
    assert torch.equal(a, b)


@pytest.mark.parametrize("inp,hidden,batch,shift", [(36, 33, 1, 0), (36, 33, 8, 0), (38, 40, 3, 0), (516, 64, 2, 0),
                                                    (2052, 65, 9, 0), (2056, 129, 2049, 0), (1028, 65, 200, 0),
                                                    (64, 32, 4, 1), (64, 32, 70, 1)])
def test_forward_routes(ctx, inp, hidden, batch, shift):
    """Inference on few rows, on FP32 rows that the first product reads itself, and on rows that are not 16-byte
    aligned (shift floats past an aligned address): probabilities within the running error bound."""
    import torch
    print("forward", inp, hidden, batch, shift, flush=True)
    net, params, x, y, xd, _ = small_net(ctx, inp, hidden, 2, 11, batch)
    flat = torch.empty(batch * inp + shift, dtype=torch.float32, device="cuda:0")
    xs = flat[shift:].view(batch, inp)
    xs.copy_(xd)
    probs = torch.empty((batch, 11), dtype=torch.float32, device="cuda:0")
    net.forward(xs, probs)
    pr = {k: (omlp.bf16_round(v) if k.startswith("W") else v) for k, v in params.items()}
    xb = omlp.bf16_round(x).astype(np.float64)
    _, p_ref, p_bound = base.gradient_error_bounds(pr, xb, y, 2)
    assert np.all(np.abs(probs.cpu().numpy().astype(np.float64) - p_ref) <= 2 * p_bound)
