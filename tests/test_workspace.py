"""Workspace sizes of 3D lattices: two states and little else.  Statistics
slots are 32 bytes a block, and the smallest block that a large lattice
launches covers 256 nodes (64 x 4 nodes of one slice)."""
import pytest

import synth
from paper_2505_13097_amd.stefan import workspace_bytes


@pytest.mark.parametrize("n,q,storage", [(512, 19, "f32"), (512, 7, "f32"),
                                         (256, 7, "f64")])
def test_slots_of_large_3d_lattices(n, q, storage):
    prob = synth.cavity_3d(n=n, ny=n, nz=n, q=q, storage=storage)
    states = 2 * q * n ** 3 * (8 if storage == "f64" else 4)
    # the slots, the energy's and the fronts' sums, alignment
    rest = n ** 3 // 256 * 32 + n ** 3 // 2048 * 8 + 8 * n * n + (1 << 20)
    assert workspace_bytes(prob) <= states + rest


@pytest.mark.gpu
def test_one_wave_tilings_on_either_side_of_their_limit():
    """64x1/npt1/z1 and z2 by their names on lattices that run them and on
    ones that run the default instead: the default's states"""
    import numpy as np
    from paper_2505_13097_amd import Stefan, variant_names
    for n, ny, nz in ((40, 9, 7), (101, 63, 62), (101, 63, 63), (180, 180, 180)):
        for q in (7, 19):
            prob = synth.cavity_3d(n=n, ny=ny, nz=nz, q=q, storage="f64")
            names = variant_names(q, "f64")
            out = []
            for v in (-1, names.index("64x1/npt1/z1"),
                      names.index("64x1/npt1/z2")):
                g = Stefan(prob, variant=v)
                g.step(3)
                out.append((g.state(), g.stats()))
                g.close()
            for s, st in out[1:]:
                assert np.array_equal(s, out[0][0]), (n, q)
                assert st["max_newton_it"] == out[0][1]["max_newton_it"]
