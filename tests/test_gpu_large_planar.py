"""2-D states beyond 300 MiB are stored past the caches (smaller ones through
them).  The way of a store is no part of the arithmetic: on both sides of that
size the fused schedule equals the split one bit for bit."""
import pytest

import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP device")]

# nodes at which the two states of a D2Q9 run pass 300 MiB, a little
# less and more; ragged in x and y
SIZES = {"fp64": 1_034_000, "fp32": 2_068_000, "fp16dev": 3_276_000, "bf16dev": 3_276_000}


@pytest.mark.parametrize("walls", [(0, 0, 0), (1, 1, 0)])
@pytest.mark.parametrize("precision", sorted(SIZES))
def test_stores_on_both_sides_of_the_cache(precision, walls):
    from paper_2111_05960_amd import Simulation
    for scale in (0.93, 1.07):
        nx = 1237
        shape = (1, int(scale * SIZES[precision]) // nx, nx)
        p = wl.base_params(lattice=wl.D2Q9, shape=shape, bc=walls)
        gen = torch.Generator(device="cuda").manual_seed(5)
        phi0 = torch.rand(shape, generator=gen, device="cuda", dtype=torch.float64)
        c0 = 0.1 + 0.9 * torch.rand(shape, generator=gen, device="cuda", dtype=torch.float64)
        got = [Simulation(p, precision, s).init(phi0, c0).step(3).fields_device()
               for s in ("fused", "split")]
        for name, a, b in zip(("phi", "c", "mu"), *got):
            assert bool(torch.isfinite(a).all()), (shape, name)
            assert torch.equal(a, b), f"{name} differs at {shape}"
