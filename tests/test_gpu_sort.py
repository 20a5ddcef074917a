"""The particle sort by cell against numpy's stable sort.  Particles that are
never formed keep their cells, so after a sort the device order (which a
checkpoint stores with the particles' creation ids) is the stable order of the
cells they were set with.  Sizes around the one-workgroup sort (4096
particles), a sort tile (1024) and one, two and three digit passes; the batched
sort with lattices of different digits."""
import struct

import numpy as np
import pytest

from tests import seeded_inputs as si

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_07999_amd as g
    g.lib()
    return g


def _event(gl, N, n, seed):
    g = np.random.default_rng(seed)
    ev = gl.Event(N, 0.02 * N, 0.125, precision=32, max_steps=8, max_particles=n)
    one = np.zeros((2, 18, N * N))
    one[:, [0, 8, 16]] = 1.0
    ev.set_state(one, np.zeros((2, 8, N * N)), np.zeros((8, N * N)), np.zeros((8, N * N)), 1)
    # half of the particles crowd into a few cells, the last cell among them
    cell = g.integers(0, N, (2, n)).astype(np.int32)
    crowd = g.random(n) < 0.5
    cell[:, crowd] = np.where(g.random((1, crowd.sum())) < 0.3, N - 1, cell[:, crowd] // 8)
    ev.set_particles([(1.27, 1.0, gl.KIND_HEAVY_QUARK, 50.0)], cell, np.zeros((2, n)), np.zeros(n), np.zeros((3, n)),
                     np.ones((8, n)), np.zeros((3, n)), np.zeros(n, np.int32))
    return ev, cell[0].astype(np.int64) + N * cell[1]


def _ids(ev, n, tmp_path):
    """the creation ids in device order, from the event's checkpoint"""
    path = str(tmp_path / "order")
    ev.checkpoint(path)
    data = open(path, "rb").read()
    slots = (n + 255) // 256 * 256
    at = data.find(struct.pack("<QQ", 4, 4 * slots)) + 16
    assert at >= 16
    return np.frombuffer(data, np.int32, slots, at)


def _check(ev, key, tmp_path):
    n = len(key)
    ids = _ids(ev, n, tmp_path)
    assert np.array_equal(ids[:n], np.argsort(key, kind="stable"))
    assert np.all(ids[n:] == -1)


@pytest.mark.parametrize("N,n", [(2, 1), (3, 255), (16, 1025), (16, 4096), (22, 4097), (23, 12289), (243, 30001),
                                 (512, 5000), (513, 5000), (600, 4095), (1024, 70001)])
def test_device_order_is_the_stable_order_of_the_cells(gl, N, n, tmp_path):
    ev, key = _event(gl, N, n, N + n)
    ev.run(1)
    _check(ev, key, tmp_path)
    ev.set_sort_period(1)       # a sorted set again, its order applied by the next push or alone
    ev.run(3)
    _check(ev, key, tmp_path)


def test_batched_order(gl, tmp_path):
    sets = [_event(gl, N, n, N) for N, n in ((3, 300), (24, 5000), (162, 1), (600, 20000))]
    batch = gl.Batch([ev for ev, _ in sets])
    batch.config(shape=0, grid_mult=0, sort_every=2, graph_steps=4)
    batch.run(6)
    batch.close()
    for ev, key in sets:
        _check(ev, key, tmp_path)
