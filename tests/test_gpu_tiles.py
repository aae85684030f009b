"""Several steps per launch on tiles in LDS (the library default of small 2D
lattices) against one-step launches: the states bit for bit, the Newton
counters equal, energies and boundary fluxes to the rounding of their sums
(1e-12 of the sum of the magnitudes, a few thousand FP64 terms)."""
import numpy as np
import pytest
import torch

import synth
from paper_2505_13097_amd import Stefan, variant_names

pytestmark = pytest.mark.gpu

D, B, P, N = "dirichlet", "bounceback", "periodic", "neumann"
# the smallest lattice, one to three tiles a side, remainders, a tile's halo
# reaching round a periodic axis, and both ends of each tile size
SIZES = [(3, 3), (4, 3), (9, 8), (17, 3), (8, 25), (40, 33), (173, 173),
         (181, 174), (331, 331), (361, 360)]
WALLS = [(D, D, P, P), (D, D, B, B), (B, B, B, B), (P, P, P, P),
         (P, P, D, B), (D, N, D, N), (N, N, N, N)]


def _prob(nx, ny, q, bc, storage, scheme):
    rng = np.random.default_rng(nx * 1000 + ny)
    return synth.Problem(
        dim=2, q=q, nx=nx, ny=ny, tau=0.8, ste=0.2, delta=0.05, bc=bc,
        wall_T=(1.0, -0.5, 0.4, -0.2), tol=1e-12, max_it=40,
        storage=storage, scheme=scheme,
        T0=rng.uniform(-0.6, 0.6, (ny, nx)))


def _run(prob, steps, variant):
    g = Stefan(prob, variant=variant)
    for n in steps:
        g.step(n)
    st = g.stats()
    out = g.state(), st
    g.close()
    return out


@pytest.mark.parametrize("scheme", ["irebm", "eebm"])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: f"{s[0]}x{s[1]}")
def test_tiles_equal_single_steps(size, scheme):
    nx, ny = size
    big = nx * ny > 10000
    one = variant_names(5, "f64").index("64x1/npt1")
    for q, storage in ((5, "f64"), (9, "f32")) if big else (
            (5, "f64"), (5, "f32"), (9, "f64"), (9, "f32")):
        for bc in WALLS[:2] if big else WALLS:
            prob = _prob(nx, ny, q, bc, storage, scheme)
            # 2, 7 and 11: whole launches, uneven ones, a single step between
            steps = (2, 1, 7, 11)
            a, sa = _run(prob, steps, -1)
            b, sb = _run(prob, steps, one)
            tag = (nx, ny, q, storage, bc)
            assert np.array_equal(a, b), tag
            for k in ("steps", "max_newton_it", "nonconverged",
                      "max_residual"):
                assert sa[k] == sb[k], (tag, k)
            bar = 1e-12 * (abs(sb["energy"]) + 21 * 9 * nx * ny)
            for k in ("energy", "flux_in", "flux_out"):
                assert abs(sa[k] - sb[k]) <= bar, (tag, k)
    torch.cuda.synchronize()
    print(f"{nx}x{ny} {scheme}: equal", flush=True)


@pytest.mark.parametrize("n", [1100, 1500])
def test_large_tiles_equal_single_steps(n):
    """EEBM in FP64 keeps the tiles on lattices of millions of nodes (both
    of its large tile sizes)."""
    one = variant_names(9, "f64").index("64x1/npt1")
    prob = _prob(n, n + 37, 9, WALLS[1], "f64", "eebm")
    a, sa = _run(prob, (9,), -1)
    b, sb = _run(prob, (9,), one)
    assert np.array_equal(a, b)
    assert sa["steps"] == sb["steps"] == 9


def test_autotune_keeps_the_state_of_a_tiled_lattice():
    prob = _prob(60, 50, 5, WALLS[0], "f64", "eebm")
    g = Stefan(prob)
    g.step(5)
    before = g.state()
    v, ms = g.autotune(steps=6)
    assert 0 <= v < len(variant_names(5, "f64")) and ms > 0.0
    assert np.array_equal(before, g.state())
    g.step(8)
    after = g.state()
    g.close()
    assert np.array_equal(after, _run(prob, (13,), 0)[0])
