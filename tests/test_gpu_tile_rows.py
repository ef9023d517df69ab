"""The 2-D kernels choose the rows of a tile from the grid (1, 4, 8 or 13) and
load a whole tile before the first barrier.  Neither is part of the
arithmetic: the fused schedule must equal the split one bit for bit at every
height, on grids with ragged edges, single nodes along an axis, and walls."""
import numpy as np
import pytest

import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP device")]

# (ny, nx): one node, one row, one column, ragged columns and rows with 1, 4
# and 8 rows, a strip of 13-row tiles, and several passes over the chip
SHAPES = [(1, 1), (1, 200), (37, 2), (3, 63), (130, 129), (203, 257), (36, 5000), (529, 513)]


@pytest.mark.parametrize("walls", [(0, 0, 0), (1, 1, 0), (0, 1, 0)])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev", "bf16dev"])
@pytest.mark.parametrize("lattice,light", [(wl.D2Q9, 0), (wl.D2Q9, 1), (wl.D2Q5, 0)])
def test_fused_equals_split_at_every_tile_height(lattice, light, precision, walls):
    from paper_2111_05960_amd import Simulation
    for ny, nx in SHAPES:
        shape = (1, ny, nx)
        p = wl.base_params(lattice=lattice, shape=shape, bc=walls, h_lattice=light)
        rng = np.random.default_rng(7)
        phi0 = rng.uniform(0.0, 1.0, shape)
        c0 = rng.uniform(0.1, 1.0, shape)
        got = [Simulation(p, precision, s).init(phi0, c0).step(4).fields_device()
               for s in ("fused", "split")]
        for name, a, b in zip(("phi", "c", "mu"), *got):
            assert bool(torch.isfinite(a).all()), (shape, name)
            assert torch.equal(a, b), f"{name} differs at {shape}"
