"""The site-field records: what the push reads of them, and the order a checkpoint
keeps them in, on lattices whose sites do not fill the groups of records."""
import struct

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_07999_amd as g
    g.lib()
    return g


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("N", [2, 3, 9, 27, 32])
def test_checkpoint_keeps_chunk_planes(gl, tmp_path, N, precision):
    """Chunk c of site x at c N^2 + x of the file, whatever the device's order;
    E_z, B_x, B_y and B_z are whole there (no half apart).  A restored event
    holds the same fields and makes the same step."""
    def event():
        ev = gl.Event(N, 0.02 * N, precision=precision, max_steps=8, max_particles=512)
        return ev
    a = event()
    a.init_glasma(1.0, 0.2, 2, 5)
    a.add_species(1.5, 0.5, gl.KIND_HEAVY_QUARK, 100, 3)
    a.evolve_fields(1)
    path = str(tmp_path / "c")
    a.checkpoint(path)
    F = a.site_fields().reshape(48, N * N)
    ts = precision // 8
    t = np.float64 if precision == 64 else np.float32
    nv, size = 16 // ts, 64 * N * N * ts
    raw = open(path, "rb").read()
    at = raw.index(struct.pack("<QQ", 2, size)) + 16
    file = np.frombuffer(raw, t, size // ts, at).reshape(64 // nv, N * N, nv)
    planes = file.transpose(0, 2, 1).reshape(64, N * N).astype(np.float64)
    assert np.array_equal(planes[16:48], F[16:48])
    b = event()
    b.restore(path)
    assert np.array_equal(b.site_fields(), a.site_fields())
    for ev in (a, b):
        ev.push_particles()
        ev.run(3)
    pa, pb = a.get_particles(), b.get_particles()
    for k in pa:
        assert np.array_equal(pa[k], pb[k]), k
    a.close()
    b.close()
