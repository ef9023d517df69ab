"""Every launch stays within what a launch can take (2^32 threads along x, 65535
blocks along y and z) on the grids that reach those limits: very many planes,
very long columns, very large planes.  Host side only, over the logging
stand-in of the HIP runtime: nothing of these sizes is allocated."""
import math

import pytest

from tests import fake_hip

SCRIPT = """
LATTICES = {{2: [dict(lattice=wl.D2Q9), dict(lattice=wl.D2Q9, h_lattice=1), dict(lattice=wl.D2Q5)],
            3: [dict(lattice=wl.D3Q19), dict(lattice=wl.D3Q19, h_lattice=1), dict(lattice=wl.D3Q7)]}}
shape = {shape}
dims = 2 if shape[0] == 1 else 3
out = []
for lat in LATTICES[dims]:
    for walls in ((0, 0, 0), (1, 1, dims - 2)):
        for precision in ("fp64", "fp32", "fp16dev", "bf16dev"):
            for schedule in ("auto", "split"):
                p = wl.base_params(shape=shape, bc=walls, **lat)
                q = B.make_params(p, precision, schedule)
                ctx = context(p, precision, schedule)
                log()
                B.gplbm_init_fields(ctx, 1 << 30, 1 << 31)
                B.gplbm_step(ctx, 1)
                B.gplbm_read_fields(ctx, 1 << 30, 1 << 31, 1 << 32)
                try:
                    B.gplbm_diagnostics(ctx, allow_nonfinite=True)
                except B.GplbmError:
                    pass  # the stand-in copies nothing back
                B.gplbm_adjoint_begin(ctx, 1 << 42, B.gplbm_adjoint_bytes(q), 0, 0)
                B.gplbm_adjoint_step(ctx, 1 << 38, 1 << 39)
                B.gplbm_adjoint_finish(ctx, 1 << 30, 1 << 31, 1 << 32, 1 << 33)
                out += [[precision, schedule] + v[1:4] for v in log() if v[0] == "launch"]
                B.gplbm_destroy(ctx)
"""

# (nz, ny, nx): planes beyond a launch's z blocks, and so many that the layers
# count too; a column beyond its y blocks at 4 rows each; a plane of 2^29 nodes,
# wide and narrow, and one of more than a run of blocks
SHAPES = [(65535, 2, 3), (65536, 2, 3), (70000, 3, 5), (200001, 1, 2), (1, 300000, 8),
          (1, 65544, 8192), (1, 1 << 27, 4), (3, 23171, 23171), (1, 33000, 33000)]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


@pytest.mark.parametrize("shape", SHAPES)
def test_launches_within_the_limits(lib, shape):
    nodes = shape[0] * shape[1] * shape[2]
    rows = fake_hip.run(lib, SCRIPT.format(shape=shape))
    assert rows
    per_node = ("k_init", "k_split", "k_dev_split", "k_fields", "k_dev_fields", "k_adj_seed",
                "k_adj_ra", "k_adj_rb", "k_adj_init", "k_dev_initI")
    for precision, schedule, name, grid, block in rows:
        what = (precision, schedule, name, grid, block)
        assert all(v >= 1 for v in grid + block), what
        assert grid[0] * block[0] < 1 << 32 and grid[1] <= 65535 and grid[2] <= 65535, what
        if any(k in name for k in per_node):
            assert math.prod(grid + block) >= nodes, what
