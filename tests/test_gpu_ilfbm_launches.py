"""ILFBM launches whose number of iterations follows the step before: few
iterations take few (not the time of a whole launch), and the states are the
same whatever the launches hold."""
import time

import numpy as np
import pytest
import torch

import synth
from paper_2505_13097_amd import Stefan

pytestmark = pytest.mark.gpu

D, N, P = "dirichlet", "neumann", "periodic"


def _prob(q, nx, ny, x, tol, max_it, storage="f64", ste=0.3):
    T0 = np.random.default_rng(nx + ny).uniform(-0.3, 0.3, (ny, nx))
    return synth.Problem(
        dim=1 if q == 3 else 2, q=q, nx=nx, ny=ny, tau=0.7, ste=ste,
        delta=0.05, bc=x + (P, P), wall_T=(0.6, -0.4, 0.0, 0.0), tol=tol,
        max_it=max_it, storage=storage, scheme="ilfbm", T0=T0)


def test_two_iterations_take_less_than_eight():
    """2 iterations a step against 8 on the same lattice, which a launch of
    always 8 does not tell apart: the tiles of 2 hold three times the nodes,
    so three quarters of the time leaves room for what does not shrink."""
    t = {}
    for cap in (2, 8):
        g = Stefan(_prob(9, 1601, 1601, (D, D), 1e-14, cap))
        g.step(2)
        best = 1e9
        for _ in range(4):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            g.step(6)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        assert g.stats()["max_newton_it"] == cap
        t[cap] = best / 6 * 1e6
        g.close()
    print(f"1601^2: {t[2]:.0f} us per step of 2 iterations, {t[8]:.0f} of 8",
          flush=True)
    assert t[2] < 0.75 * t[8], t


@pytest.mark.parametrize("q,nx,ny", [(9, 33, 40), (5, 100, 17), (9, 3, 3),
                                     (3, 700, 1)])
@pytest.mark.parametrize("x", [(D, D), (D, N), (P, P)])
def test_counts_that_change_from_step_to_step(q, nx, ny, x):
    """A lattice and its copy repeated along an axis (other tiles, the same
    arithmetic at every node): equal bits, iterations and residuals over steps
    that take one to a few dozen iterations each."""
    rep = (1, 2) if q == 3 else (2, 1)
    if q == 3:
        x = (P, P)
    for tol, max_it in ((1e-3, 60), (1e-6, 60), (1e-3, 1), (1e-12, 9)):
        prob = _prob(q, nx, ny, x, tol, max_it)
        two = prob.with_(nx=nx * rep[1], ny=ny * rep[0], dx=prob.dx,
                         T0=np.tile(prob.T0, rep))
        a, b = Stefan(prob), Stefan(two)
        counts = []
        for n in (1, 1, 1, 2, 3, 1, 8, 1):
            sa, sb = a.step(n, stats=True), b.step(n, stats=True)
            tag = (q, nx, ny, x, tol, n)
            assert np.array_equal(
                np.tile(a.state().reshape(q, ny, nx), (1,) + rep),
                b.state().reshape(q, two.ny, two.nx)), tag
            assert np.array_equal(
                np.tile(a.liquid().reshape(ny, nx), rep),
                b.liquid().reshape(two.ny, two.nx)), tag
            for k in ("max_newton_it", "nonconverged", "max_residual"):
                assert sa[k] == sb[k], (tag, k)
            counts.append(sa["max_newton_it"])
            a.reset_stats()
            b.reset_stats()
        print(q, nx, ny, x, tol, max_it, counts, flush=True)
        a.close()
        b.close()
