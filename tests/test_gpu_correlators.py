"""The field correlators where the accumulators, states and site fields overflow
the last-level cache: their arrays then take the streaming kernels."""
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


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("static,light", [(True, False), (False, True), (True, True)])
def test_streamed_correlators_of_a_tiled_lattice(gl, prec, static, light):
    """A 576^2 lattice (300 MB and more of arrays) tiled from one of 144^2 (a sixteenth of
    that): every site does what its image does, so the means agree to
    the rounding of sums of 3 10^5 FP64 terms in another order."""
    N, copies, steps = 144, 4, 20
    ev = [gl.Event(n, 0.02 * n, precision=prec, max_steps=steps, static_correlator=static, lightlike_correlator=light)
          for n in (N, N * copies)]
    ev[0].init_glasma(2.0, 0.2, 2, 5)
    s = ev[0].get_state()
    ev[1].set_state(*[np.tile(a.reshape(a.shape[:-1] + (N, N)), (1,) * (a.ndim - 1) + (copies, copies)).reshape(
        a.shape[:-1] + (N * N * copies * copies,)) for a in s[:4]], s[4])
    rows = []
    for e in ev:
        if static:
            e.static_start(0.0)
        if light:
            e.lightlike_start(0.005)
        e.evolve_fields(steps)
        rows.append((e.static_broadening() if static else None, e.lightlike_broadening() if light else None))
        e.close()
    for a, b in zip(*rows):
        if a is None:
            continue
        assert len(a) == len(b) > steps - 5 and np.array_equal(b[:, 4], a[:, 4] * copies ** 2)
        assert np.abs(b[:, 1:4] - a[:, 1:4]).max() < 1e-12 * np.abs(a[:, 1:4]).max()
