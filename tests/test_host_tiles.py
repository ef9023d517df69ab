"""The tile heights and z chunks that the launch rules choose for the shapes of
the bit-equality tests, so that a change of a rule cannot leave a kernel of the
fused schedules without a test (host side only, over the logging stand-in of the
HIP runtime: one block per CU of 256)."""
import re

import pytest

from tests import fake_hip
from tests import test_gpu_long_marches as long_marches
from tests import test_gpu_tile_heights as heights

SCRIPT = """
out = []
for which, lat in {lattices}.items():
    for precision in ("fp64", "fp32", "fp16dev", "bf16dev"):
        for walls in {walls}:
            for shape in {shapes}:
                for extra in ({{}}, dict(h_scheme=1)):
                    ctx = context(wl.base_params(shape=shape, bc=walls, **lat, **extra), precision, "fused")
                    B.gplbm_init_fields(ctx, 1 << 30, 1 << 31)
                    log()
                    B.gplbm_step(ctx, 1)
                    (kind, name, grid, block, zc), = log()
                    out.append([which, precision, walls, shape, name, grid[0], zc])
                    B.gplbm_destroy(ctx)
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


def _run(lib, lattices, walls, shapes):
    return fake_hip.run(lib, SCRIPT.format(lattices=lattices, walls=walls, shapes=shapes))


def test_long_marches_are_long(lib):
    rows = _run(lib, long_marches.LATTICES, long_marches.WALLS, long_marches.SHAPES)
    chunks = {}
    for which, precision, walls, shape, name, grid, zc in rows:
        chunks.setdefault(name, []).append((zc, shape[0]))
    assert len(chunks) == 48  # a basic and a general form, with walls and without
    for name, lengths in chunks.items():
        longest = max(zc for zc, nz in lengths)
        # five turns of a ring of four planes; all of 100 planes in the periodic
        # deviation march, which chooses the longest
        assert longest >= 20, name
        if "k_dev_fused3d" in name and name.endswith(("Lb0ELb0EEEvNS_3GeoENS_4CoefIfEENS_7DevStepEiiii",
                                                      "Lb1ELb0EEEvNS_3GeoENS_4CoefIfEENS_7DevStepEiiii")):
            assert longest == 100, name
        assert any(zc < nz and nz % zc for zc, nz in lengths), name  # a ragged last chunk


def _rows_and_store(name):
    """rows of a tile, and whether the next state is stored past the caches"""
    rows = int(re.search(r"fused2dILi64ELi(\d+)E", name).group(1))
    gen, walls, past = re.search(r"Lb([01])ELb([01])ELb([01])EE", name).groups()
    return rows, past == "1"


def test_every_height_is_reached(lib):
    want = {shape: rows for rows, shape in heights.HEIGHTS}
    rows = _run(lib, heights.LATTICES, heights.WALLS, [(1,) + shape for shape in want])
    for which, precision, walls, shape, name, grid, _ in rows:
        fp64, other = want[tuple(shape[1:])]
        assert _rows_and_store(name)[0] == (fp64 if precision == "fp64" else other), (shape, name)
    assert {r for pair in want.values() for r in pair} == {1, 4, 8, 13}


def test_both_stores_at_the_same_height(lib):
    for (kind, which), cases in heights.LARGE.items():
        for height, below, above in cases:
            rows = _run(lib, {which: heights.LATTICES[which]}, heights.WALLS[:2],
                        [(1, below, heights.NX), (1, above, heights.NX)])
            for _, precision, walls, shape, name, grid, _ in rows:
                if ("dev" if "dev" in precision else precision) == kind:
                    assert _rows_and_store(name) == (height, shape[1] == above), (shape, name)
