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


@pytest.mark.parametrize("N", [5, 10, 50, 130, 250, 8, 64, 96, 243])
def test_every_lattice(gl, N):
    """Lattices that are not 2^a 3^b (no MV initialisation) included, and lattices
    whose line transforms nothing has prepared."""
    ev = _event_of_ones(gl, N)
    for rmax in sorted({1, max(1, N // 4), N // 2}):
        assert np.abs(ev.dipole(0, rmax) - 6.0).max() < 1e-12 * 6
    ev.close()


@pytest.mark.parametrize("N", [64, 72, 81, 256])
def test_few_separations_agree_with_the_whole_curve(gl, N):
    """Sums over sites (rmax <= 4, N <= 64) and spectra of the lines on either side of
    the line between them, on MV lines.  Both sum entries of magnitude <= 1, the
    spectra through transforms of some 10 eps a stage."""
    ev = gl.Event(N, 10.0 * N / 512)
    ev.init_glasma(2.767, 0.2, 5, 11)
    for nuc in (0, 1):
        D = ev.dipole(nuc, N // 2)
        assert abs(D[0] - 1.0) < 1e-13
        for rmax in (1, 4, 5, 6):
            assert np.abs(ev.dipole(nuc, rmax) - D[:rmax + 1]).max() < 1e-13
    ev.close()
