"""The 2-D kernels equal the node pair bit for bit at every tile height that the
launch rule chooses, on every lattice, format and scheme, and with the stores of
the next state through and past the caches at the same height.
tests/test_host_tiles.py holds the heights and stores that these shapes give."""
import pytest

import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP device")]

LATTICES = {"full": dict(lattice=wl.D2Q9), "h": dict(lattice=wl.D2Q9, h_lattice=1),
            "gh": dict(lattice=wl.D2Q5)}
PRECISIONS = ["fp64", "fp32", "fp16dev", "bf16dev"]
WALLS = [(0, 0, 0), (1, 1, 0), (0, 1, 0)]
SCHEMES = {"basic": {}, "alt+quad": dict(h_scheme=1, free_energy=1, eps_s=1.0, eps_l=1.5, m_s=1.0,
                                         m_l=0.1, df_min=0.0)}
# rows of a tile (FP64, other formats): (ny, nx), ragged in x and in y
HEIGHTS = [((1, 1), (129, 130)), ((4, 4), (203, 257)), ((8, 8), (307, 300)), ((8, 8), (509, 505)),
           ((13, 4), (36, 5000)), ((13, 8), (1003, 1000))]
# rows of a tile, and ny just below and above the size from which the next state
# is stored past the caches (nx = 1237)
NX = 1237
LARGE = {("fp64", "full"): [(8, 835, 838), (13, 831, 922)],
         ("fp64", "h"): [(8, 1023, 1159), (13, 1058, 1061)],
         ("fp64", "gh"): [(8, 1327, 1498), (13, 1444, 1446)], ("fp32", "full"): [(8, 1660, 1690)],
         ("fp32", "h"): [(8, 2100, 2140)], ("fp32", "gh"): [(8, 2870, 2910)],
         ("dev", "full"): [(8, 2630, 2670)], ("dev", "h"): [(8, 3160, 3200)],
         ("dev", "gh"): [(8, 3950, 3990)]}


def _compare(shape, which, precision, walls, scheme, steps):
    from paper_2111_05960_amd import Simulation
    gen = torch.Generator(device="cuda").manual_seed(29)
    phi0, c0 = torch.rand((2,) + shape, generator=gen, device="cuda", dtype=torch.float64)
    c0 = 0.1 + 0.9 * c0
    p = wl.base_params(shape=shape, bc=walls, **LATTICES[which], **SCHEMES[scheme])
    a, b = (Simulation(p, precision, s).init(phi0, c0).step(steps).fields_device()
            for s in ("fused", "split"))
    for name, x, y in zip(("phi", "c", "mu"), a, b):
        assert bool(torch.isfinite(x).all()), (shape, scheme, name)
        assert torch.equal(x, y), (shape, scheme, name)


@pytest.mark.parametrize("walls", WALLS)
@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("which", sorted(LATTICES))
def test_every_tile_height(which, precision, walls):
    for _, (ny, nx) in HEIGHTS:
        for scheme in SCHEMES:
            _compare((1, ny, nx), which, precision, walls, scheme, 4)


@pytest.mark.parametrize("walls", WALLS[:2])
@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("which", sorted(LATTICES))
def test_stores_through_and_past_the_caches(which, precision, walls):
    for rows, below, above in LARGE["dev" if "dev" in precision else precision, which]:
        for ny in (below, above):
            _compare((1, ny, NX), which, precision, walls, "basic", 3)
