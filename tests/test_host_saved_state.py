"""Which way a saved state is copied, on the library's host side alone: by one
kernel only where the whole of it lies in one allocation of the context's own
device at an address that 16-byte vectors fit.  Anywhere else the runtime
copies, which refuses a size that reaches past an allocation: a kernel would
write there."""
import pytest

from tests import fake_hip

SCRIPT = """
p = wl.base_params(lattice=wl.{lattice}, shape={shape}, bc=(0, 0, 0))
ctx = context(p, "{precision}")
n = B.gplbm_checkpoint_bytes(B.make_params(p, "{precision}"))
B.gplbm_init_fields(ctx, 1 << 30, 1 << 31)
base = 1 << 36
alloc(base, n)                            # just large enough
alloc(2 * base, n - 1)                    # one byte short
alloc(3 * base, n + 4096)                 # room for a state behind its start
alloc(4 * base, n + 64, kind=1)           # pinned host memory
alloc(5 * base, n + 64, device=1)         # another device
alloc(6 * base, n + 64, kind=3)           # managed
places = dict(whole=base, short=2 * base, inside=3 * base + 4096, past=3 * base + 4096 + 16,
              odd=3 * base + 8, host=4 * base, peer=5 * base, managed=6 * base, unknown=7 * base)
out = {{}}
for name, at in places.items():
    for way in ("save", "load"):
        log()
        try:
            B.gplbm_save_state(ctx, at) if way == "save" else B.gplbm_load_state(ctx, at, 0)
            code = 0
        except B.GplbmError as e:
            code = e.code
        lines = log()
        out[name + " " + way] = [code, sum(v[0] == "launch" for v in lines),
                                 sum(v[1] for v in lines if v[0] == "copy"), n]
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


@pytest.mark.parametrize("precision,lattice,shape", [("fp64", "D3Q19", (5, 6, 7)),
                                                     ("fp16dev", "D2Q9", (1, 9, 11))])
def test_kernel_only_within_one_allocation(lib, precision, lattice, shape):
    got = fake_hip.run(lib, SCRIPT.format(lattice=lattice, shape=shape, precision=precision))
    for key, (code, launches, copied, n) in got.items():
        place = key.split()[0]
        if place in ("whole", "inside"):
            assert (code, launches, copied) == (0, 1, 0), key
        elif place in ("short", "past"):
            assert code == -3 and launches == 0 and copied < n, key
        else:
            assert (code, launches, copied) == (0, 0, n), key
