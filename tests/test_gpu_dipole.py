"""gl_dipole reads the stored Wilson line and nothing else: a workspace of ones,
whose Wilson lines have all real and imaginary parts 1, gives
D(r) = (1/3) sum over nine entries of 1 + 1 = 6 at every separation, whichever
way the sums are taken."""
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


def _event_of_ones(gl, N):
    import torch
    ev = gl.Event(N, 4.0)
    at = ev._ws_ptr - ev._ws.data_ptr()
    ev._ws[at:at + ev.nbytes // 8 * 8].view(torch.float64).fill_(1.0)
    return ev


@pytest.mark.parametrize("N", [5, 10, 50, 130, 250])
def test_every_lattice(gl, N):
    """Lattices that are not 2^a 3^b (no MV initialisation) included."""
    ev = _event_of_ones(gl, N)
    for rmax in sorted({1, max(1, N // 4), N // 2}):
        assert np.abs(ev.dipole(0, rmax) - 6.0).max() < 1e-12 * 6
    ev.close()
