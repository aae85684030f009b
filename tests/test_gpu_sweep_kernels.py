"""Every kernel of a sweep that a lattice of its size can reach runs here, and
each test says which one it reached: printed Newton, a Neumann wall beside a
hot one, sweeps that store every level (the reverse mode), batches."""
import numpy as np
import pytest

import synth
from paper_2505_13097_amd import Stefan, StefanBatch, variant_names

pytestmark = pytest.mark.gpu

D, B, P, N = "dirichlet", "bounceback", "periodic", "neumann"


def _prob(nx, ny, q, storage, bc, at=8, **kw):
    x = np.arange(nx)[None, :]
    T0 = np.where(x < at, 1 - x / at, -0.5 * (1 - np.exp(-(x - at) / 16.0)))
    T0 = T0 + np.random.default_rng(2).uniform(-1e-3, 1e-3, (ny, nx))
    p = dict(tau=0.7, ste=0.2, delta=1.5 / (nx - 1), newton_mode="safeguarded")
    p.update(kw)
    return synth.Problem(dim=2, q=q, nx=nx, ny=ny, bc=bc,
                         wall_T=(1.0, -0.5, -0.4, -0.3), tol=1e-12, max_it=40,
                         storage=storage, scheme="irebm", T0=T0, **p)


def _against_single_steps(prob, steps, variants):
    names = variant_names(prob.q, prob.storage)
    out = []
    for v in [names.index("64x1/npt1")] + variants:
        g = Stefan(prob, variant=v)
        if v != names.index("64x1/npt1"):
            assert g.launches()[0] == "sweep_kernel", g.launches()
        for n in steps:
            g.step(n)
        out.append((g.state(), g.stats()))
        g.close()
    b, sb = out[0]
    for a, sa in out[1:]:
        assert np.array_equal(a, b)
        for k in ("steps", "max_newton_it", "nonconverged", "max_residual"):
            assert sa[k] == sb[k], k
        bar = 1e-12 * (abs(sb["energy"]) + sum(steps) * 9 * prob.nodes)
        for k in ("energy", "flux_in", "flux_out"):
            assert abs(sa[k] - sb[k]) <= bar, k


@pytest.mark.parametrize("q,storage,nx,ny", [
    (9, "f64", 811, 747), (5, "f64", 811, 747), (9, "f32", 1301, 1203),
    (5, "f32", 1301, 1203)])
@pytest.mark.parametrize("mode", ["plain", "safeguarded"])
def test_newton_modes_and_neumann_walls(q, storage, nx, ny, mode):
    two = variant_names(q, storage).index("128x4/t2/r32/nt")
    for at in (8, 60):
        prob = _prob(nx, ny, q, storage, (D, D, B, B), at, newton_mode=mode)
        _against_single_steps(prob, (7, 22), [-1, two])
        # (two-step variants of a lattice with a Neumann wall run single steps)
        for bc in ((D, N, D, N), (D, D, N, N)):
            _against_single_steps(
                _prob(nx, ny, q, storage, bc, at, newton_mode=mode),
                (7, 22), [-1])


# lattices on which a sweep never costs more than single steps (low ones have
# short segments): their forward tapes and recomputed states are swept
ALWAYS = [(9, "f64", 4700, 520), (5, "f64", 9000, 500), (9, "f32", 9100, 520),
          (5, "f32", 17500, 510)]


@pytest.mark.parametrize("q,storage,nx,ny", ALWAYS)
@pytest.mark.parametrize("mode", ["plain", "safeguarded"])
def test_reverse_mode_stores_every_level(q, storage, nx, ny, mode):
    """Tapes of 10 steps in segments of 7: launches of four, three and two
    steps and a single one left over, forward and recomputed.  Gradients equal
    those of single steps bit for bit."""
    prob = _prob(nx, ny, q, storage, (D, D, P, P), 8, newton_mode=mode,
                 wall_profile=(1.0 + 0.1 * np.sin(np.arange(ny) / 20.0), None,
                               None, None))
    one = variant_names(q, storage).index("64x1/npt1")
    g = np.linspace(0.5, 1.5, ny)
    for steps, interval in ((10, 7), (5, 5)):
        out = []
        for v in (-1, one):
            s = Stefan(prob, variant=v, flags=1)
            kernel, k, routed = s.launches()
            if v < 0:
                assert (kernel, routed) == ("sweep_kernel", False) and k >= 3
            tape = s.forward_tape(steps, interval)
            out.append((s.state(), s.backward_tape(g, tape)))
            s.close()
            del tape
        (sa, (wa, ga, da)), (sb, (wb, gb, db)) = out
        assert np.array_equal(sa, sb)
        assert ga == gb and da == db and np.array_equal(wa["x-"], wb["x-"])


@pytest.mark.parametrize("q,storage,nx,ny", ALWAYS)
def test_lattices_that_always_sweep(q, storage, nx, ny):
    """the front in the frame, in the short segments beside it, past them"""
    two = variant_names(q, storage).index("128x4/t2/r32/nt")
    for at in (8, 40, 200):
        prob = _prob(nx, ny, q, storage, (D, D, B, B), at)
        _against_single_steps(prob, (5, 12), [-1, two])


@pytest.mark.parametrize("mode", ["plain", "safeguarded"])
@pytest.mark.parametrize("q,storage", [(5, "f32"), (9, "f64"), (5, "f64"),
                                       (9, "f32")])
def test_batch_newton_modes(q, storage, mode):
    probs = [_prob(nx, ny, q, storage, bc, newton_mode=mode) for nx, ny, bc in
             [(300, 331, (D, D, B, B)), (120, 64, (D, D, P, P)),
              (40, 33, (D, D, B, B)), (700, 200, (D, D, P, P))]]
    names = variant_names(q, storage)
    a, ref = StefanBatch(probs), StefanBatch(probs)
    a.set_schedule(names.index("128x4/t2s/r32/nt"))
    assert a.launches() == ("batch_sweep_kernel", 4, True)
    ref.set_schedule(names.index("64x1/npt1"))
    assert ref.launches() == ("batch_step_kernel", 1, False)
    for n in (4, 9, 30):
        a.step(n)
        ref.step(n)
        for k in range(len(probs)):
            assert np.array_equal(a.temperature(k), ref.temperature(k)), (n, k)
    for sa, sb in zip(a.stats(), ref.stats()):
        for f in ("max_newton_it", "nonconverged", "max_residual"):
            assert sa[f] == sb[f], f
    a.close()
    ref.close()


def test_kernels_by_lattice():
    """what a handle says it launches, on either side of the lines of the
    rules that choose"""
    def of(nx, ny, q, storage, variant="", scheme="irebm"):
        p = _prob(nx, ny, q, storage, (D, D, B, B)).with_(scheme=scheme)
        v = variant_names(q, storage).index(variant) if variant else -1
        g = Stefan(p, variant=v)
        out = g.launches()
        g.close()
        return out
    assert of(201, 201, 9, "f64") == ("tile_kernel", 3, False)
    assert of(500, 500, 9, "f64") == ("step_kernel", 1, False)
    assert of(811, 739, 9, "f64") == ("step_kernel", 1, False)
    assert of(811, 740, 9, "f64") == ("sweep_kernel", 4, True)
    assert of(1300, 1153, 5, "f32") == ("step_kernel", 1, False)
    assert of(1300, 1154, 5, "f32") == ("sweep_kernel", 3, True)
    assert of(500, 500, 9, "f32", "128x4/t2/r32/nt") == ("step2_kernel", 2,
                                                         False)
    assert of(1300, 1300, 9, "f32", "128x4/t2/r32/nt") == ("sweep_kernel", 4,
                                                           True)
    assert of(300, 300, 9, "f32", scheme="eebm") == ("sweep_kernel", 4, False)
    assert of(300, 300, 9, "f32", "64x1/npt1") == ("step_kernel", 1, False)
