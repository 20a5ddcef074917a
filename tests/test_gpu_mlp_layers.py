"""The general kernels of the surrogate network, which take the networks the
whole-network kernels do not (more than 256 inputs, outputs or hidden units, or more
than four hidden layers): against the FP64 oracle, through both inference calls, and
bitwise against the whole-network kernels on networks that are the same but for
hidden units of zero weights."""
import numpy as np
import pytest

from oracle import mlp_oracle as M

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_07999_amd as g
    g.lib()
    return g


def _net(gl, shape, max_batch, params=None, seed=5, max_samples=8):
    g = np.random.default_rng(sum(shape))
    net = gl.MLP(*shape, max_batch=max_batch, max_samples=max_samples, seed=seed)
    if params is None:
        params = net.params()
        nb = shape[1] * shape[2] + shape[3]
        params[-nb:] = g.uniform(-0.2, 0.2, nb)
    net.params(set_to=params)
    net.set_scaling(-np.ones(shape[0]), np.full(shape[0], 2.0), np.full(shape[3], 0.25), np.full(shape[3], 0.5))
    return net, np.asarray(params, np.float32)


def _rows(shape, n, seed):
    g = np.random.default_rng(seed)
    return (g.uniform(-1, 2, (n, shape[0])).astype(np.float32), g.uniform(-1, 1, (n, shape[3])).astype(np.float32))


@pytest.mark.parametrize("shape,n", [((5, 257, 3, 2), 300), ((5, 64, 5, 2), 65), ((300, 64, 2, 2), 129), ((5, 33, 2, 300), 70),
                                     ((1, 300, 1, 1), 1)])
def test_forward_and_gradients_match_oracle(gl, shape, n):
    """Every element within 2^-8 (one BF16 rounding of an operand) of the sum of the
    magnitudes of its terms, as for the whole-network kernels."""
    net, p = _net(gl, shape, n + 3)
    X, Y = _rows(shape, n, n)
    Xs, Ys = M.scale_inputs(X, -1.0, 2.0), (Y - 0.25) / 0.5
    p = p.astype(np.float64)
    Zs, _ = M.forward(p, Xs, shape, bf16=True)
    rf = np.abs(net.infer(X).cpu().numpy() - (Zs[-1] * 0.5 + 0.25)) / (M.output_scales(p, Xs, shape, bf16=True) * 0.5 + 1e-30)
    gr, loss = net.grads(X, Y)
    lo, go = M.loss_and_grads(p, Xs, Ys, shape, bf16=True)
    rg = np.abs(gr - go) / (M.grad_scales(p, Xs, Ys, shape, bf16=True) + 1e-30)
    assert rf.max() < 2.0 ** -8 and rg.max() < 2.0 ** -8
    assert abs(loss - lo) < 2.0 ** -8 * lo


@pytest.mark.parametrize("shape", [(5, 257, 3, 2), (5, 64, 5, 2), (300, 64, 2, 3)])
def test_noalloc_equals_infer(gl, shape):
    """More rows than a pass of the scratch array (about 4000 at width 257) or of
    max_batch, then fewer, which must not see the first call's."""
    import torch
    net, _ = _net(gl, shape, 700)
    for n, seed in ((20011, 1), (37, 2), (1, 3)):
        X = torch.from_numpy(_rows(shape, n, seed)[0]).cuda()
        want = net.infer(X)
        assert torch.equal(net.infer_noalloc(X), want)
        assert bool(torch.isfinite(want).all())


def _widened(p, shape, width):
    """The same network with hidden layers of `width`: the added units have zero
    weights and biases, so their activations and gradients are zero."""
    Ws, bs = M.unpack(p, *shape)
    wide = (shape[0], width) + shape[2:]
    L, din, dout = M.dims(*wide)
    Wn, bn = [], []
    for l in range(L):
        w = np.zeros((dout[l], din[l]))
        w[:Ws[l].shape[0], :Ws[l].shape[1]] = Ws[l]
        b = np.zeros(dout[l])
        b[:len(bs[l])] = bs[l]
        Wn.append(w)
        bn.append(b)
    return wide, M.pack(Wn, bn).astype(np.float32)


def _narrowed(p, wide, shape):
    Ws, bs = M.unpack(p, *wide)
    L, din, dout = M.dims(*shape)
    return M.pack([Ws[l][:dout[l], :din[l]] for l in range(L)], [bs[l][:dout[l]] for l in range(L)]).astype(np.float32)


@pytest.mark.parametrize("shape", [(5, 256, 3, 2), (5, 256, 4, 17), (40, 100, 2, 3), (5, 60, 1, 2), (7, 17, 3, 1)])
def test_both_paths_are_bitwise_the_same(gl, shape):
    """Inference, gradients, loss and a short training run."""
    n, batch = 1000, 300
    a, p = _net(gl, shape, n, max_samples=n)
    wide, pw = _widened(p, shape, 257)
    b, _ = _net(gl, wide, n, params=pw, max_samples=n)
    for net in (a, b):
        net.set_output_power(0, np.full(shape[3], 2.0))
    import torch
    X, Y = _rows(shape, n, 3)
    X[:, 0] = np.abs(X[:, 0]) + 0.5
    assert torch.equal(a.infer(X), b.infer(X))
    (ga, la), (gb, lb) = a.grads(X[:777], Y[:777]), b.grads(X[:777], Y[:777])
    assert la == lb and np.array_equal(ga, _narrowed(gb, wide, shape))
    da, db = torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()
    ea, eb = (net.train(da, db, epochs=2, batch=batch, lr=1e-3, seed=4) for net in (a, b))
    assert np.array_equal(ea, eb)
    assert np.array_equal(a.params(), _narrowed(b.params(), wide, shape))
    assert torch.equal(a.infer(X), b.infer(X))
