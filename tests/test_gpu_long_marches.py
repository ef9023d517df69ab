"""Every form of the z-marching kernels (lattices, formats, schemes, with and
without walls) equals the node pair bit for bit over long chunks: the rings of
planes in the LDS turn many times, the last chunk is ragged, and a block goes on
to a second tile.  tests/test_host_tiles.py holds the chunk lengths that these
shapes give."""
import pytest

import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP device")]

LATTICES = {"full": dict(lattice=wl.D3Q19), "h": dict(lattice=wl.D3Q19, h_lattice=1),
            "gh": dict(lattice=wl.D3Q7)}
QUAD = dict(free_energy=1, eps_s=1.0, eps_l=1.5, m_s=1.0, m_l=0.1, df_min=0.0)
SCHEMES = {"basic": {}, "alt": dict(h_scheme=1), "quad": QUAD, "alt+quad": dict(h_scheme=1, **QUAD)}
WALLS = [(0, 0, 0), (1, 1, 1), (0, 0, 1), (1, 0, 0)]
# (nz, ny, nx): several columns of tiles; one column of very many
SHAPES = [(45, 300, 130), (131, 3000, 5), (100, 3250, 5)]


@pytest.mark.parametrize("walls", WALLS)
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev", "bf16dev"])
@pytest.mark.parametrize("which", sorted(LATTICES))
def test_long_march_equals_pair(which, precision, walls):
    from paper_2111_05960_amd import Simulation
    for shape in SHAPES:
        gen = torch.Generator(device="cuda").manual_seed(13)
        phi0, c0 = torch.rand((2,) + shape, generator=gen, device="cuda", dtype=torch.float64)
        c0 = 0.1 + 0.9 * c0
        for scheme in SCHEMES if precision != "bf16dev" else ("basic", "alt+quad"):
            p = wl.base_params(shape=shape, bc=walls, **LATTICES[which], **SCHEMES[scheme])
            a, b = (Simulation(p, precision, s).init(phi0, c0).step(3).fields_device()
                    for s in ("fused", "split"))
            for name, x, y in zip(("phi", "c", "mu"), a, b):
                assert bool(torch.isfinite(x).all()), (scheme, name)
                assert torch.equal(x, y), (shape, scheme, name)
