"""Small lattices run each field step and the push of the step before in one
launch (gl_run), with a third field state and a second site-field record.
The result is that of separate steps (gl_evolve_fields and
gl_push_particles, one kernel each) bit for bit: state, particles, series and
correlators, in calls of any length, across sorts, through a checkpoint and
into a batch."""
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


STEPS = (1, 2, 17, 16, 9)


def _event(gl, N, prec, n, corr=False):
    ev = gl.Event(N, 0.02 * N, 0.125, precision=prec, max_steps=64, max_particles=1024 + 2 * n,
                  static_correlator=corr, lightlike_correlator=corr)
    U, E, phi, pi = si.random_state(3, N, link_kind="near", eps=0.3)
    ev.set_state(np.transpose(U, (0, 2, 1)), np.transpose(E, (0, 2, 1)), phi.T, pi.T, 1)
    ev.add_species(1.27, 2.0, gl.KIND_HEAVY_QUARK, n, 4, tau_form_fm=0.01)
    ev.add_species(0.0, 10.0, gl.KIND_JET, n, 5, tau_form_fm=0.0)
    if corr:
        ev.static_start(0.01)
        ev.lightlike_start(0.0)
    return ev


def _separate(ev, steps):
    for _ in range(steps):
        ev.evolve_fields(1)
        ev.push_particles()


def _outputs(ev, corr=False):
    P = ev.get_particles()
    out = list(ev.get_state()) + [P[k] for k in sorted(P)] + [ev.series()]
    return out + ([ev.static_broadening(), ev.lightlike_broadening()] if corr else [])


def _same(a, b):
    return len(a) == len(b) and all(np.array_equal(x, y) for x, y in zip(a, b))


# lattices below, at and above one field tile and ragged, a large paired one;
# one particle, and blocks with padding
@pytest.mark.parametrize("N,prec,n,corr", [(4, 64, 1, False), (31, 64, 257, False), (40, 32, 1000, False),
                                           (33, 64, 300, True), (256, 64, 3000, False), (256, 32, 3000, False)])
def test_paired_run_equals_separate_steps(gl, N, prec, n, corr):
    a, b = _event(gl, N, prec, n, corr), _event(gl, N, prec, n, corr)
    for k in STEPS:
        a.run(k)
        _separate(b, k)
        assert _same(_outputs(a, corr), _outputs(b, corr)), k


def test_checkpoint_and_site_fields_after_a_paired_run(gl, tmp_path):
    a, b = _event(gl, 40, 64, 300), _event(gl, 40, 64, 300)
    a.run(8)
    a.evolve_fields(1)          # a particle step is due: site fields and the state at tau_n are read
    _separate(b, 8)
    b.evolve_fields(1)
    assert np.array_equal(a.site_fields(), b.site_fields())
    path = str(tmp_path / "c")
    a.checkpoint(path)
    c = _event(gl, 40, 64, 300)
    c.run(4)                    # its own buffers rotated otherwise
    c.restore(path)
    for ev in (a, c):
        ev.push_particles()
        ev.run(11)
    b.push_particles()
    _separate(b, 11)
    assert _same(_outputs(a), _outputs(b)) and _same(_outputs(c), _outputs(b))


def test_batch_after_paired_runs(gl):
    evs = [[_event(gl, N, 32, 300) for N in (24, 40)] for _ in range(2)]
    for ev in evs[0]:
        ev.run(6)
    for ev in evs[1]:
        _separate(ev, 6)
    for side in evs:
        batch = gl.Batch(side)
        batch.run(20)
        batch.close()
    for a, b in zip(*evs):
        a.run(5)
        _separate(b, 5)
        assert _same(_outputs(a), _outputs(b))


@pytest.mark.parametrize("prec,shape", [(64, 0), (32, 1), (32, 2)])
def test_paired_batch_equals_its_phases_apart(gl, prec, shape):
    """A batch of small lattices pairs its launches (grid_mult 0); a persistent
    walk runs the phases one after another.  Calls of every length modulo the
    three field states, with and without a graph, across sorts; one event fails
    and is masked from the same step on."""
    def batch(mult):
        evs = [_event(gl, N, prec, n) for N, n in ((31, 257), (40, 600), (4, 1), (64, 300))]
        d = evs[1].get_particles()
        d["p"][0, 123] = np.nan
        evs[1].set_particles([(1.27, 2.0, gl.KIND_HEAVY_QUARK, 0.01), (0.0, 10.0, gl.KIND_JET, 0.0)],
                             *[d[k] for k in ("cell", "off", "eta", "p", "Q", "p0", "species")])
        b = gl.Batch(evs)
        b.config(shape=shape, grid_mult=mult, sort_every=16, graph_steps=32)
        return evs, b
    (ea, a), (eb, b) = batch(0), batch(4)
    for k in (1, 2, 3, 33, 9, 1):
        for x in (a, b):
            try:
                x.run(k)
            except gl.GlasmaError as e:
                assert e.status == gl.GL_ENUMERIC
        assert np.array_equal(a.status(), b.status())
        for i, (x, y) in enumerate(zip(ea, eb)):
            if i != 1:
                assert _same(_outputs(x), _outputs(y)), (k, i)
                assert np.array_equal(x.site_fields(), y.site_fields())
    assert (a.status() > 0).tolist() == [False, True, False, False]     # once its particles have formed
    assert np.array_equal(ea[1].series(), eb[1].series(), equal_nan=True)
    a.close()
    b.close()


@pytest.mark.parametrize("prec,N,copies", [(64, 54, 2), (64, 27, 4), (32, 48, 4), (32, 144, 2)])
def test_fields_of_a_tiled_lattice(gl, prec, N, copies):
    """A periodic lattice tiled from a smaller one evolves as that one does, bit for
    bit: on one side of the line the field step's stores stay in the L2 caches, on
    the other they are written through them."""
    ev = gl.Event(N, 0.02 * N, precision=prec, max_steps=8)
    M = N * copies
    big = gl.Event(M, 0.02 * M, precision=prec, max_steps=8)
    ev.init_glasma(2.0, 0.2, 1, 5)
    tile = lambda a: np.tile(a.reshape(a.shape[:-1] + (N, N)), (1,) * (a.ndim - 1) + (copies, copies)).reshape(
        a.shape[:-1] + (M * M,))
    s = ev.get_state()
    big.set_state(*[tile(a) for a in s[:4]], s[4])
    for e in (ev, big):
        e.evolve_fields(5)
    for a, b in zip(ev.get_state()[:4], big.get_state()[:4]):
        assert np.array_equal(tile(a), b)
    ev.close()
    big.close()
