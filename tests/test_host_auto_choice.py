"""AUTO takes the schedule that was measured to be the faster, on boxes where the
two differ by more than 3% (us per step on MI355X, z-march and node pair; the
FP64 ones in the basic scheme).  Host side only, over the logging stand-in of the HIP runtime (one block
per CU of 256)."""
import pytest

from tests import fake_hip

# lattice of g and h, walls on every face, (nz, ny, nx), z-march, node pair
MEASURED = [
    ("full", 0, (24, 285, 285), 328.5, 357.7), ("full", 0, (125, 125, 125), 328.3, 355.5),
    ("full", 0, (1218, 40, 40), 387.4, 339.9), ("full", 0, (6, 570, 570), 388.6, 362.6),
    ("full", 0, (64, 64, 64), 54.3, 39.0), ("full", 0, (24, 218, 218), 231.4, 209.4),
    ("full", 1, (24, 285, 285), 409.9, 356.3), ("full", 1, (158, 158, 158), 754.9, 679.6),
    ("h", 0, (24, 285, 285), 237.6, 252.9), ("h", 0, (125, 125, 125), 212.6, 249.2),
    ("h", 0, (64, 16, 1904), 190.7, 231.2), ("h", 0, (79, 79, 79), 77.7, 57.5),
    ("h", 0, (6, 288, 288), 65.7, 59.0), ("h", 1, (24, 285, 285), 289.2, 251.8),
    ("gh", 0, (6, 570, 570), 116.9, 136.7), ("gh", 0, (24, 285, 285), 112.5, 133.1),
    ("gh", 0, (125, 125, 125), 117.1, 129.8), ("gh", 0, (6, 437, 437), 88.1, 76.7),
    ("gh", 0, (64, 64, 64), 21.7, 16.5), ("gh", 1, (24, 405, 405), 230.4, 269.2),
    ("gh", 1, (6, 570, 570), 125.5, 135.8), ("gh", 1, (6, 811, 811), 259.1, 277.1),
    ("gh", 1, (105, 105, 105), 88.6, 72.3), ("gh", 1, (1218, 40, 40), 182.0, 124.4),
]
# precision, alternative h scheme, walls, (nz, ny, nx), on D3Q19
MEASURED_NARROW = [
    ("fp16dev", 0, 0, (256, 256, 256), 901, 964), ("fp16dev", 0, 0, (512, 512, 512), 6772, 7996),
    ("fp16dev", 0, 0, (301, 301, 301), 2034, 1827), ("fp16dev", 0, 0, (26, 1109, 1109), 2721, 2210),
    ("fp16dev", 0, 0, (26, 1088, 1088), 1819, 1876), ("bf16dev", 0, 0, (511, 512, 510), 12234, 8276),
    ("fp16dev", 1, 0, (384, 384, 384), 3696, 3368), ("fp16dev", 1, 0, (512, 512, 512), 8339, 8010),
    ("bf16dev", 0, 0, (26, 1109, 1109), 2790, 2191), ("fp16dev", 0, 1, (256, 256, 256), 1253, 939),
    ("fp32", 0, 0, (60, 731, 731), 2944, 3235), ("fp32", 1, 1, (511, 512, 510), 16363, 12798),
    ("fp32", 1, 1, (128, 500, 500), 3128, 2847), ("fp32", 1, 1, (384, 384, 384), 4742, 5040),
    ("fp32", 1, 0, (60, 731, 731), 2947, 3272), ("fp32", 0, 0, (64, 64, 64), 37, 22),
]
SCRIPT = """
LATTICES = {{"full": dict(lattice=wl.D3Q19), "h": dict(lattice=wl.D3Q19, h_lattice=1),
            "gh": dict(lattice=wl.D3Q7)}}
out = [B.gplbm_schedule(context(wl.base_params(shape=shape, bc=(w, w, w), **LATTICES[which])))
       for which, w, shape, march, pair in {measured}]
out += [B.gplbm_schedule(context(wl.base_params(lattice=wl.D3Q19, shape=shape, bc=(w, w, w),
                                                h_scheme=alt), precision))
        for precision, alt, w, shape, march, pair in {narrow}]
"""


def test_auto_takes_the_faster(tmp_path):
    told = fake_hip.run(fake_hip.build(tmp_path),
                        SCRIPT.format(measured=MEASURED, narrow=MEASURED_NARROW))
    wrong = [(m, t) for m, t in zip(MEASURED + MEASURED_NARROW, told)
             if t != (2 if m[-2] < m[-1] else 1)]
    assert not wrong
