"""The kernels that bench.py looks up in profiles exist in the library, and
its rates are of what a launch moves (no GPU)."""
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


def test_profiled_kernels_are_in_the_library():
    from paper_2505_13097_amd import _lib
    if not os.path.exists(_lib.LIB_PATH):
        from paper_2505_13097_amd import build
        build.build(verbose=False)
    with open(_lib.LIB_PATH, "rb") as f:
        lib = f.read()
    names = bench.DEFAULT_VARIANTS["batched"], "128x4/npt2/r16/nt"
    for vname in names:
        for mode in (0, 2):
            for k in bench.batch_roles(vname, mode).values():
                base = re.match(r"\w+", k).group(0).encode()
                assert base in lib, k
    assert bench.batch_roles(names[0], 2) == {
        "sweep": "batch_sweep_kernel<5, float, 2, 4>"}


def test_library_variants():
    for q, storage in ((3, "f64"), (5, "f32"), (9, "f32")):
        assert bench.library_variant(q, storage) >= 0


def test_summaries_name_current_files():
    """every kernel summary under profiles/ is of a kernel of the sources"""
    src = ""
    d = os.path.join(ROOT, "paper_2505_13097_amd", "csrc")
    for f in os.listdir(d):
        with open(os.path.join(d, f)) as h:
            src += h.read()
    for f in os.listdir(os.path.join(ROOT, "profiles")):
        with open(os.path.join(ROOT, "profiles", f)) as h:
            text = h.read()
        for k in set(re.findall(r"\b(\w+_kernel)<", text)):
            assert re.search(rf"\b{k}\b", src), (f, k)
