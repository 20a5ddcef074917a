"""The surrogate's hand-written BF16 MFMA kernels against the FP64 network
oracle: forward outputs, gradients of one backward pass (the oracle rounds to
BF16 where the device stores BF16, so the remaining differences are FP32
accumulation order and rare one-ulp BF16 rounding differences), and a short
training run that must reduce the loss."""
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


SHAPE = (5, 256, 3, 2)
LO = np.array([1.0, 0.0, 0.0, 0.0, 0.0])
HI = np.array([3.0, 4.2, 10.0, 0.2, 1.0])
MU = np.array([0.5, -1.0])
SD = np.array([2.0, 3.0])


def _data(n, seed):
    g = np.random.default_rng(seed)
    X = g.uniform(LO, HI, size=(n, 5))
    Y = np.stack([np.sin(2 * X[:, 4]) * X[:, 0] + 0.1 * X[:, 2], np.cos(X[:, 1]) * X[:, 4]], axis=1)
    return X, Y


@pytest.mark.parametrize("n", [1, 70, 256, 1000])
def test_forward_matches_oracle(gl, n):
    net = gl.MLP(*SHAPE, max_batch=1024, max_samples=4096, seed=3)
    net.set_scaling(LO, HI, MU, SD)
    p = net.params().astype(np.float64)
    X, _ = _data(n, 5)
    got = net.infer(X.astype(np.float32)).cpu().numpy()
    Zs, _ = M.forward(p, M.scale_inputs(X.astype(np.float32), LO.astype(np.float32), HI.astype(np.float32)), SHAPE,
                      bf16=True)
    want = Zs[-1] * SD + MU
    assert np.abs(got - want).max() < 2e-2 * np.abs(want).max()
    assert np.corrcoef(got.ravel(), want.ravel())[0, 1] > 0.9999


def test_gradients_match_oracle(gl):
    net = gl.MLP(*SHAPE, max_batch=512, max_samples=4096, seed=4)
    net.set_scaling(LO, HI, MU, SD)
    p = net.params().astype(np.float64)
    X, Y = _data(384, 6)
    g, loss = net.grads(X.astype(np.float32), Y.astype(np.float32))
    Xs = M.scale_inputs(X.astype(np.float32), LO.astype(np.float32), HI.astype(np.float32))
    Ys = (Y.astype(np.float32) - MU) / SD
    lo_, go = M.loss_and_grads(p, Xs, Ys, SHAPE, bf16=True)
    assert abs(loss - lo_) < 1e-3 * lo_
    rel = np.linalg.norm(g - go) / np.linalg.norm(go)
    cos = g @ go / (np.linalg.norm(g) * np.linalg.norm(go))
    assert rel < 2e-2 and cos > 0.9998, (rel, cos)
    # per layer, including the tiny input and output layers
    L, din, dout = M.dims(*SHAPE)
    off = 0
    for l in range(L):
        k = din[l] * dout[l]
        a, b = g[off:off + k], go[off:off + k]
        assert np.linalg.norm(a - b) <= 3e-2 * np.linalg.norm(b) + 1e-12
        off += k


def test_training_reduces_loss_and_fits(gl):
    net = gl.MLP(*SHAPE, max_batch=1024, max_samples=65536, seed=7)
    X, Y = _data(32768, 8)
    net.set_scaling(LO, HI, Y.mean(0), Y.std(0))
    losses = net.train(X.astype(np.float32), Y.astype(np.float32), epochs=12, batch=512, lr=2e-3, seed=1)
    assert losses[-1] < 0.05 * losses[0], losses
    Xt, Yt = _data(4096, 9)
    pred = net.infer(Xt.astype(np.float32)).cpu().numpy()
    err = np.abs(pred - Yt).max(axis=0) / np.abs(Yt).max(axis=0)
    assert np.all(err < 0.1), err


def test_forward_and_gradients_match_oracle_elementwise(gl):
    """Every output and every gradient element within a bound derived from
    BF16 rounding: the device and the oracle round the same operands to BF16,
    but their FP32 and FP64 accumulations can land on the two sides of a BF16
    rounding boundary, which changes an operand by one BF16 ulp (2^-8
    relative).  An element then moves by at most 2^-8 times the sum of the
    magnitudes of its terms (oracle.grad_scales, oracle.output_scales), so
    |device - oracle| <= 2^-8 * scale per element, plus an FP32 floor."""
    n = 384
    net = gl.MLP(*SHAPE, max_batch=512, max_samples=4096, seed=11)
    net.set_scaling(LO, HI, MU, SD)
    p = net.params().astype(np.float64)
    X, Y = _data(n, 12)
    Xs = M.scale_inputs(X.astype(np.float32), LO.astype(np.float32), HI.astype(np.float32))
    # forward
    got = net.infer(X.astype(np.float32)).cpu().numpy()
    Zs, _ = M.forward(p, Xs, SHAPE, bf16=True)
    want = Zs[-1] * SD + MU
    scale = M.output_scales(p, Xs, SHAPE, bf16=True) * SD
    rf = np.abs(got - want) / (scale + 1e-30)
    # gradients
    g, loss = net.grads(X.astype(np.float32), Y.astype(np.float32))
    Ys = (Y.astype(np.float32) - MU) / SD
    _, go = M.loss_and_grads(p, Xs, Ys, SHAPE, bf16=True)
    A = M.grad_scales(p, Xs, Ys, SHAPE, bf16=True)
    rg = np.abs(g - go) / (A + 1e-30)
    L, din, dout = M.dims(*SHAPE)
    off, parts = 0, []
    for l in range(L):
        k = din[l] * dout[l]
        parts.append(("W%d" % (l + 1), rg[off:off + k]))
        off += k
    for l in range(L):
        parts.append(("b%d" % (l + 1), rg[off:off + dout[l]]))
        off += dout[l]
    print("forward: max |dev - orc| / scale = %.2e" % rf.max())
    for name, r in parts:
        print("%s: max |dev - orc| / scale = %.2e (median %.1e)" % (name, r.max(), np.median(r)))
    u = 2.0 ** -8
    assert rf.max() < u
    assert rg.max() < u


@pytest.mark.parametrize("shape,n", [((1, 1, 1, 1), 1), ((5, 16, 1, 2), 15), ((5, 17, 2, 16), 16), ((33, 48, 3, 17), 17),
                                     ((256, 255, 2, 40), 300), ((7, 256, 4, 256), 33), ((5, 256, 3, 2), 257)])
def test_whole_network_kernels_at_their_edges(gl, shape, n):
    """Networks up to 256 wide and four hidden layers run in whole-network
    kernels of 16-row tiles and 16-output blocks: widths, depths, inputs,
    outputs and rows around those sizes, every output and gradient element
    within the BF16 bound derived above."""
    g = np.random.default_rng(sum(shape) + n)
    net = gl.MLP(*shape, max_batch=n + 3, max_samples=8, seed=5)
    p = net.params()
    nb = shape[1] * shape[2] + shape[3]
    p[-nb:] = g.uniform(-0.2, 0.2, nb).astype(np.float32)     # biases too
    net.params(set_to=p)
    lo, hi = -np.ones(shape[0], np.float32), np.full(shape[0], 2.0, np.float32)
    net.set_scaling(lo, hi, np.full(shape[3], 0.25), np.full(shape[3], 0.5))
    X = g.uniform(-1, 2, (n, shape[0])).astype(np.float32)
    Y = g.uniform(-1, 1, (n, shape[3])).astype(np.float32)
    Xs, Ys = M.scale_inputs(X, lo, hi), (Y - 0.25) / 0.5
    p = p.astype(np.float64)
    got = net.infer(X).cpu().numpy()
    Zs, _ = M.forward(p, Xs, shape, bf16=True)
    rf = np.abs(got - (Zs[-1] * 0.5 + 0.25)) / (M.output_scales(p, Xs, shape, bf16=True) * 0.5 + 1e-30)
    gr, loss = net.grads(X, Y)
    lo_, go = M.loss_and_grads(p, Xs, Ys, shape, bf16=True)
    rg = np.abs(gr - go) / (M.grad_scales(p, Xs, Ys, shape, bf16=True) + 1e-30)
    print("shape %s n %d: forward %.1e, gradients %.1e of the scale" % (shape, n, rf.max(), rg.max()))
    assert rf.max() < 2.0 ** -8 and rg.max() < 2.0 ** -8
    assert abs(loss - lo_) < 2.0 ** -8 * lo_


def test_inference_does_not_depend_on_the_rows_of_a_call(gl):
    """The rows of a workgroup grow with the rows of a call (16, 32, 64): each
    row's outputs are bitwise the same in a call of its own size class."""
    import torch
    net = gl.MLP(*SHAPE, max_batch=64, max_samples=8, seed=6)
    net.set_scaling(LO, HI, MU, SD)
    net.set_output_power(0, [3.0, 2.0])
    X = torch.from_numpy(_data(33000, 7)[0].astype(np.float32)).cuda()
    small = torch.cat([net.infer(x.contiguous()) for x in X.split(3001)])
    for n in (33000, 32767, 4097, 4096):
        assert torch.equal(net.infer(X[:n].contiguous()), small[:n])


@pytest.mark.parametrize("shape", [(5, 256, 3, 2), (40, 33, 2, 70)])
@pytest.mark.parametrize("n", [4097, 16384, 16385, 24576, 24577])
def test_rows_a_workgroup(gl, shape, n):
    """16, 32, 48 or 64 rows a workgroup by the rows of the call: on either side of
    each line the outputs are those of calls of 16 rows a workgroup."""
    import torch
    net = gl.MLP(*shape, max_batch=64, max_samples=8, seed=7)
    net.set_scaling(np.zeros(shape[0]), np.ones(shape[0]), np.full(shape[3], 0.25), np.full(shape[3], 0.5))
    X = torch.from_numpy(np.random.default_rng(n).uniform(-1, 2, (n, shape[0])).astype(np.float32)).to("cuda")
    parts = [net.infer(X[k:k + 4096]).cpu().numpy() for k in range(0, n, 4096)]
    assert np.array_equal(net.infer(X).cpu().numpy(), np.concatenate(parts))


def test_half_a_billion_rows(gl):
    """More rows than the work items of one launch can take (2^29 rows of 64 a
    workgroup of 512 are 2^32): the call goes in passes, each row as in a call of
    its own.  The input repeats, so the outputs have to as well."""
    import torch
    net = gl.MLP(1, 40, 1, 1, max_batch=64, max_samples=8, seed=8)
    x = torch.rand(1 << 20, 1, generator=torch.Generator().manual_seed(3)).cuda()
    want = net.infer(x)
    X = x.repeat(513, 1)
    for got in (net.infer(X), net.infer_noalloc(X)):
        assert bool((got.view(513, 1 << 20) == want.view(1, 1 << 20)).all())
        del got


@pytest.mark.parametrize("shape", [(5, 256, 3, 2), (40, 33, 1, 40), (5, 257, 2, 2)])
@pytest.mark.parametrize("noalloc", [False, True])
def test_inference_in_place(gl, shape, noalloc):
    """Outputs written over the inputs (n_out <= n_in): those of separate
    arrays, over several passes.  The last shape runs layer by layer."""
    import ctypes
    import torch
    n, ni, no = 70001, shape[0], shape[3]
    net = gl.MLP(*shape, max_batch=2048, max_samples=8, seed=7)
    net.set_scaling(np.zeros(ni), np.ones(ni), np.full(no, 0.25), np.full(no, 0.5))
    X = torch.rand(n, ni, generator=torch.Generator().manual_seed(4)).cuda()
    want = net.infer(X)
    fn = gl.lib().gl_mlp_infer_noalloc if noalloc else gl.lib().gl_mlp_infer
    assert fn(net._h, ctypes.c_void_p(X.data_ptr()), ctypes.c_void_p(X.data_ptr()), n) == 0
    torch.cuda.synchronize()
    assert torch.equal(X.view(-1)[:n * no], want.view(-1))


@pytest.mark.parametrize("shape,groups", [((1, 3, 1, 1), 8), ((5, 8, 4, 2), 8), ((32, 32, 2, 32), 8), ((33, 31, 1, 2), 4),
                                          ((5, 33, 2, 2), 4), ((64, 64, 3, 64), 4), ((5, 65, 4, 2), 2), ((3, 9, 2, 80), 2),
                                          ((128, 128, 3, 128), 2), ((2, 129, 2, 1), 1)])
def test_narrow_networks(gl, shape, groups):
    """Networks up to 32, 64 and 128 wide (inputs and outputs too) run as 8, 4 and 2
    groups of rows a workgroup: outputs and gradients within the BF16 bound above, and
    on either side of each line of the rows' classes the outputs of small calls."""
    import torch
    g = np.random.default_rng(sum(shape))
    n, ni, no = 517, shape[0], shape[3]
    net = gl.MLP(*shape, max_batch=n, max_samples=8, seed=9)
    p = net.params()
    nb = shape[1] * shape[2] + no
    p[-nb:] = g.uniform(-0.2, 0.2, nb).astype(np.float32)
    net.params(set_to=p)
    lo, hi = -np.ones(ni, np.float32), np.full(ni, 2.0, np.float32)
    net.set_scaling(lo, hi, np.full(no, 0.25), np.full(no, 0.5))
    X = g.uniform(-1, 2, (n, ni)).astype(np.float32)
    Y = g.uniform(-1, 1, (n, no)).astype(np.float32)
    Xs, Ys = M.scale_inputs(X, lo, hi), (Y - 0.25) / 0.5
    p = p.astype(np.float64)
    Zs, _ = M.forward(p, Xs, shape, bf16=True)
    rf = np.abs(net.infer(X).cpu().numpy() - (Zs[-1] * 0.5 + 0.25)) / (M.output_scales(p, Xs, shape, bf16=True) * 0.5 + 1e-30)
    gr, _ = net.grads(X, Y)
    _, go = M.loss_and_grads(p, Xs, Ys, shape, bf16=True)
    rg = np.abs(gr - go) / (M.grad_scales(p, Xs, Ys, shape, bf16=True) + 1e-30)
    assert rf.max() < 2.0 ** -8 and rg.max() < 2.0 ** -8
    lines = [groups * r for r in (256 * 16, 512 * 32, 512 * 48)]
    big = torch.rand(lines[-1] + 1, ni, generator=torch.Generator().manual_seed(5)).cuda()
    want = torch.cat([net.infer(x.contiguous()) for x in big.split(4096)])
    for m in [k + d for k in lines for d in (0, 1)]:
        assert torch.equal(net.infer(big[:m].contiguous()), want[:m])
