"""gplbm_schedule tells which schedule a context's steps run, also where AUTO
chose: the number of kernels a step launches follows from it (the library's
host side over the logging stand-in of the HIP runtime)."""
import pytest

from tests import fake_hip

SCRIPT = """
LATTICES = {"2d": dict(lattice=wl.D2Q9), "2d h": dict(lattice=wl.D2Q9, h_lattice=1),
            "2d gh": dict(lattice=wl.D2Q5), "3d": dict(lattice=wl.D3Q19),
            "3d h": dict(lattice=wl.D3Q19, h_lattice=1), "3d gh": dict(lattice=wl.D3Q7)}
out = []
for name, lat in LATTICES.items():
    shapes = [(1, 8, 512), (1, 700, 600)] if name[0] == "2" else [
        (1, 1, 1), (16, 20, 30), (100, 90, 70), (6, 500, 500), (128, 128, 128), (300, 300, 300)]
    for shape in shapes:
        for walls in ((0, 0, 0), (1, 1, 0)):
            for precision in ("fp64", "fp32", "fp16dev", "bf16dev"):
                for schedule in ("auto", "split", "fused"):
                    p = wl.base_params(shape=shape, bc=walls, **lat)
                    ctx = context(p, precision, schedule)
                    B.gplbm_init_fields(ctx, 1 << 30, 1 << 31)
                    log()
                    B.gplbm_step(ctx, 3)
                    kernels = [v[1] for v in log()]
                    out.append([name, shape, walls, precision, schedule, B.gplbm_schedule(ctx),
                                len(kernels), sum("split" in k for k in kernels)])
                    B.gplbm_destroy(ctx)
"""


@pytest.fixture(scope="module")
def rows(tmp_path_factory):
    return fake_hip.run(fake_hip.build(tmp_path_factory.mktemp("fake_hip")), SCRIPT)


def test_reported_schedule_is_the_one_that_runs(rows):
    split, fused = 1, 2
    for row in rows:
        asked, told, launches, of_pair = row[4:]
        assert told in (split, fused), row
        assert launches == (3 if told == fused else 6), row
        assert of_pair == (0 if told == fused else 6), row
        if asked != "auto":
            assert told == dict(split=split, fused=fused)[asked], row


def test_auto_takes_both(rows):
    told = {(r[0], r[5]) for r in rows if r[4] == "auto"}
    assert {("3d", 1), ("3d", 2), ("3d gh", 1), ("3d gh", 2)} <= told
    assert all(s == 2 for name, s in told if name[0] == "2")
