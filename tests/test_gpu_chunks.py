"""The z chunk of the marching kernels follows the grid: from one plane per
block on small grids to the full length on large ones.  The chunk is not part
of the arithmetic, so the fused schedule must equal the split one bit for bit
at every length, with periodic planes and with walls."""
import numpy as np
import pytest

import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP device")]

# one-plane chunks (two planes and one), two- and three-plane chunks with a
# remainder, a chunk of about ten planes, and a long one on a wide grid
SHAPES = [(1, 9, 70), (2, 6, 65), (61, 64, 64), (70, 90, 100), (131, 52, 520)]


@pytest.mark.parametrize("walls", [(0, 0, 0), (1, 1, 1)])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev"])
@pytest.mark.parametrize("shape", SHAPES)
def test_fused_equals_split_at_every_chunk_length(shape, precision, walls):
    from paper_2111_05960_amd import Simulation
    p = wl.base_params(lattice=wl.D3Q19, shape=shape, bc=walls)
    rng = np.random.default_rng(5)
    phi0 = rng.uniform(0.0, 1.0, shape)
    c0 = rng.uniform(0.1, 1.0, shape)
    got = [Simulation(p, precision, s).init(phi0, c0).step(4).fields_device()
           for s in ("fused", "split")]
    for name, a, b in zip(("phi", "c", "mu"), *got):
        assert bool(torch.isfinite(a).all())
        assert torch.equal(a, b), f"{name} differs at {shape} {precision} walls {walls}"
