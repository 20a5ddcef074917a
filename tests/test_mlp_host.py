"""Workspace of a network, sized on the host."""
import ctypes

import pytest

import paper_2307_07999_amd.glasma as G


def _bytes(shape, max_batch):
    L = G.lib()
    if not getattr(L, "_mlp_declared", False):
        G._mlp_declare(L)
        L._mlp_declared = True
    d, out = G.MLPDesc(*shape, max_batch), ctypes.c_size_t(0)
    assert L.gl_mlp_required_bytes(ctypes.byref(d), 8, ctypes.byref(out)) == 0
    return out.value


@pytest.mark.parametrize("shape", [(5, 8, 1, 2), (5, 8, 4, 2), (5, 16, 3, 2), (5, 33, 2, 2), (40, 64, 4, 17), (5, 256, 3, 2)])
def test_workspace_per_row_follows_the_network(shape):
    """A row of max_batch costs its own layers, padded to blocks of 16: BF16
    activations (inputs and hidden layers), BF16 and FP32 layer gradients (hidden layers
    and outputs), the deviations, and two FP32 scratch rows of the widest layer."""
    ni, w, depth, no = shape
    pad = lambda k: (k + 15) // 16 * 16
    row = 2 * (pad(ni) + depth * pad(w)) + 6 * (depth * pad(w) + pad(no)) + 4 * no + 8 * max(ni, w, no)
    n = 1 << 20
    assert abs(_bytes(shape, n + 16) - _bytes(shape, 16) - n * row) < 20 * 256
