"""A segment of reverse steps hands the c that its steps share from one to the
next (periodic grids); single reverse steps pull it from the state.  Both give
the same bits, for any length of a segment and in any mixture."""
import numpy as np
import pytest

import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP device")]

CASES = [(wl.D2Q9, 0, (1, 23, 70)), (wl.D2Q9, 1, (1, 1, 5)), (wl.D2Q5, 0, (1, 40, 33)),
         (wl.D3Q19, 0, (9, 11, 67)), (wl.D3Q19, 1, (7, 8, 9)), (wl.D3Q7, 0, (10, 3, 20))]


def _aligned(nbytes):
    buf = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
    return buf, (buf.data_ptr() + 255) // 256 * 256


@pytest.mark.parametrize("walls", [(0, 0, 0), (1, 1, 1)])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev", "bf16dev"])
@pytest.mark.parametrize("lattice,light,shape", CASES)
def test_segment_equals_single_steps(lattice, light, shape, precision, walls):
    from paper_2111_05960_amd import Simulation, binding as B
    if shape[0] == 1:
        walls = walls[:2] + (0,)
    p = wl.base_params(lattice=lattice, shape=shape, bc=walls, h_lattice=light)
    rng = np.random.default_rng(17)
    phi0 = torch.as_tensor(rng.uniform(0.0, 1.0, shape), device="cuda").contiguous()
    c0 = torch.as_tensor(rng.uniform(0.1, 1.0, shape), device="cuda").contiguous()
    bars = [torch.as_tensor(rng.standard_normal(shape), device="cuda").contiguous() for _ in range(2)]
    sim = Simulation(p, precision).init(phi0, c0)
    stride = (B.gplbm_checkpoint_bytes(sim.params) + 255) // 256 * 256
    n = 5
    states, base = _aligned((n + 1) * stride)
    B.gplbm_save_state(sim.ctx, base)
    B.gplbm_step_chain(sim.ctx, base, stride, n)
    size = B.gplbm_adjoint_bytes(sim.params)
    work, wp = _aligned(size)

    def sweep(parts):
        """parts: lengths of segments from the top down, -1 for a single step"""
        B.gplbm_adjoint_begin(sim.ctx, wp, size, bars[0].data_ptr(), bars[1].data_ptr())
        top = n
        for m in parts:
            if m < 0:
                top -= 1
                B.gplbm_adjoint_step(sim.ctx, base + top * stride, base + (top + 1) * stride)
            else:
                top -= m
                B.gplbm_adjoint_segment(sim.ctx, base + top * stride, stride, m)
        assert top == 0
        g = [torch.empty_like(phi0), torch.empty_like(c0)]
        d = B.gplbm_adjoint_finish(sim.ctx, phi0.data_ptr(), c0.data_ptr(), g[0].data_ptr(),
                                   g[1].data_ptr())
        return g + [torch.tensor(list(d), dtype=torch.float64)]

    ref = sweep([-1] * n)
    for parts in ([5], [2, 3], [1, -1, 3], [4, -1], [0, 5]):
        for a, b in zip(ref, sweep(parts)):
            assert torch.equal(a, b), parts
