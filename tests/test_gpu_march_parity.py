"""The z-marching kernels against the oracle, and against the node pair away
from the base parameter point: the 3-D cases of the parity tests with the fused
schedule asked for.  AUTO steps small 3-D grids by the node pair, so "auto" there
is the split schedule; the bars are those of the tests the cases come from."""
import numpy as np
import pytest

import workloads as wl
from tests import test_gpu_light_h as light
from tests import test_gpu_param_parity as params
from tests import test_gpu_parity as base
from tests import test_gpu_schemes as schemes

pytestmark = pytest.mark.gpu

gp = base.gp
FLAT = [c for c in params.SHAPES if c[0][0] > 1]


def _fp64(sim, res):
    assert sim.schedule == "fused"
    for n, (errs, ndiff) in res:
        print(f"  step {n}: errs={errs} differing={ndiff}", flush=True)
        assert max(errs.values()) <= 1e-11, (n, errs)


@pytest.mark.parametrize("case", base.CASES_3D)
def test_fp64_march(gp, oracle_mod, case):
    shape, bc, ct, at = case
    _fp64(*base._run_pair(gp, oracle_mod, wl.D3Q19, shape, bc, ct, at, "fp64", "fused", (0, 1, 7, 60),
                          seed=sum(shape)))
    for which in ("h", "gh"):
        _fp64(*light._run_pair(gp, oracle_mod, case, "fp64", "fused", (0, 1, 7, 60),
                               seed=sum(shape) + 1, which=which))


@pytest.mark.parametrize("variant", sorted(schemes.VARIANTS))
@pytest.mark.parametrize("case", base.CASES_3D)
def test_fp64_march_schemes(gp, oracle_mod, case, variant):
    _fp64(*schemes._run_pair(gp, oracle_mod, case, schemes.VARIANTS[variant], "fp64", "fused",
                             (0, 1, 7, 60), seed=sum(case[0])))


@pytest.mark.parametrize("extra", [{}, dict(h_lattice=1), dict(h_scheme=1)])
@pytest.mark.parametrize("case", FLAT)
@pytest.mark.parametrize("pset", sorted(params.PSETS))
def test_fp64_march_params(gp, oracle_mod, pset, case, extra):
    shape, bc, ct = case
    p = params._params(wl.D3Q19, shape, bc, ct, pset, **extra)
    _fp64(*params._run(gp, oracle_mod, p, "fp64", "fused", (0, 1, 7, 60), seed=sum(shape) + 3))


@pytest.mark.parametrize("case", base.CASES_3D[:2])
def test_fp32_march(gp, oracle_mod, case):
    shape, bc, ct, at = case
    _, res = base._run_pair(gp, oracle_mod, wl.D3Q19, shape, bc, ct, at, "fp32", "fused", (0, 200),
                            seed=7)
    for n, (errs, _) in res:
        assert max(errs.values()) <= 2e-5, (n, errs)


@pytest.mark.parametrize("case", FLAT)
@pytest.mark.parametrize("pset", sorted(params.PSETS))
def test_march_equals_pair_at_params(gp, pset, case):
    """FP32 and the deviation formats (whose h reference carries D_s and mu_eq)."""
    shape, bc, ct = case
    for precision in ("fp32", "fp16dev", "bf16dev"):
        for over in (dict(lattice=wl.D3Q19), dict(lattice=wl.D3Q19, h_lattice=1),
                     dict(lattice=wl.D3Q7)):
            p = params._params(over["lattice"], shape, bc, ct, pset,
                               h_lattice=over.get("h_lattice", 0))
            phi0, c0 = wl.random_state_fields(shape, seed=41)
            a, b = (gp.Simulation(p, precision, s).init(phi0, c0).step(20).fields()
                    for s in ("fused", "split"))
            for x, y in zip(a, b):
                assert np.isfinite(x).all() and np.array_equal(x, y), (precision, over)


@pytest.mark.parametrize("case", [((24, 20, 28), (0, 0, 0), 1), ((20, 18, 22), (1, 1, 1), 0)])
@pytest.mark.parametrize("pset", ["ds045_mu04_a", "sec42_precip"])
def test_dev_march_params_against_oracle(gp, oracle_mod, pset, case):
    shape, bc, ct = case
    p = params._params(wl.D3Q19, shape, bc, ct, pset)
    phi0, c0 = wl.random_state_fields(shape, seed=41)
    ref = oracle_mod.Oracle(p).init(phi0, c0).step(20).fields()
    for precision, scale in (("fp16dev", 1.0), ("bf16dev", 8.0)):
        got = gp.Simulation(p, precision, "fused").init(phi0, c0).step(20).fields()
        assert float(np.max(np.abs(got[0] - ref[0]))) <= 1e-4 * scale
        assert float(np.max(np.abs(got[1] - ref[1]))) <= 5e-4 * scale
