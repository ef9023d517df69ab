"""The per-node pair of kernels: addressed by 32-bit offsets inside a z plane,
threads over the nodes of a plane, bounced populations by a selected address.
AUTO steps with it on small 3-D grids (and in the deviation formats with
walls); it must give the bits of the fused kernels on any shape, and AUTO must
equal both."""
import numpy as np
import pytest

import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP device")]

LATTICES = {"full": dict(lattice=wl.D3Q19), "h": dict(lattice=wl.D3Q19, h_lattice=1),
            "gh": dict(lattice=wl.D3Q7)}
# one node along axes, planes shorter than a block, ragged blocks
SHAPES = [(1, 1, 1), (2, 1, 300), (5, 17, 15), (16, 16, 16), (33, 31, 65)]
QUAD = dict(free_energy=1, eps_s=1.0, eps_l=1.5, m_s=1.0, m_l=0.1, df_min=0.0)


def _fields(p, precision, schedule, steps=4):
    from paper_2111_05960_amd import Simulation
    rng = np.random.default_rng(11)
    phi0 = rng.uniform(0.0, 1.0, p["shape"])
    c0 = rng.uniform(0.1, 1.0, p["shape"])
    return Simulation(p, precision, schedule).init(phi0, c0).step(steps).fields_device()


@pytest.mark.parametrize("walls", [(0, 0, 0), (1, 1, 1), (1, 0, 0), (0, 0, 1)])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev", "bf16dev"])
@pytest.mark.parametrize("which", sorted(LATTICES))
def test_pair_equals_fused(which, precision, walls):
    for shape in SHAPES:
        p = wl.base_params(shape=shape, bc=walls, **LATTICES[which])
        ref = _fields(p, precision, "fused")
        for schedule in ("split", "auto"):
            for name, a, b in zip(("phi", "c", "mu"), ref, _fields(p, precision, schedule)):
                assert torch.equal(a, b), f"{name} differs at {shape}, {schedule}"


@pytest.mark.parametrize("variant", [dict(h_scheme=1), QUAD, dict(h_scheme=1, **QUAD),
                                     dict(counter_term=0), dict(anti_trapping=0)])
@pytest.mark.parametrize("walls", [(0, 0, 0), (1, 1, 1)])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev"])
def test_pair_equals_fused_variants(precision, walls, variant):
    p = wl.base_params(lattice=wl.D3Q19, shape=(20, 18, 70), bc=walls, **variant)
    for a, b in zip(_fields(p, precision, "fused"), _fields(p, precision, "auto")):
        assert torch.equal(a, b)
