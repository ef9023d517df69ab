"""The per-node kernels deal the blocks of a plane out in bands, one per XCD,
from 32 blocks of 256 nodes on (deviation formats in 3-D, every format in
2-D).  Who computes a node is no part of the arithmetic: below, at and above
that size, with whole and with empty bands, and over more planes than a turn
of the bands, the node pair equals the fused kernels bit for bit."""
import numpy as np
import pytest

import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP device")]

# 31, 32, 33 and 57 blocks a plane; 57 leaves the last of 8 bands empty
SHAPES = [(5, 62, 128), (6, 64, 128), (9, 91, 92), (36, 113, 129), (1, 91, 92), (1, 113, 129)]


@pytest.mark.parametrize("walls", [(0, 0, 0), (1, 1, 1), (0, 1, 0)])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev", "bf16dev"])
@pytest.mark.parametrize("shape", SHAPES)
def test_bands_of_a_plane(shape, precision, walls):
    from paper_2111_05960_amd import Simulation
    flat = shape[0] == 1
    p = wl.base_params(lattice=wl.D2Q9 if flat else wl.D3Q19, shape=shape,
                       bc=walls[:2] + (0,) if flat else walls)
    rng = np.random.default_rng(23)
    phi0 = rng.uniform(0.0, 1.0, shape)
    c0 = rng.uniform(0.1, 1.0, shape)
    got = [Simulation(p, precision, s).init(phi0, c0).step(3).fields_device()
           for s in ("fused", "split")]
    for name, a, b in zip(("phi", "c", "mu"), *got):
        assert bool(torch.isfinite(a).all()), name
        assert torch.equal(a, b), name
