"""GPU parity of the matrix-unit kernel for fully-connected layers: ragged channel counts, every count of eight-image groups,
reduction lengths that are no multiple of a step, one step and less, bit for bit on small integers and within the storage
type's tolerance on random data."""
import pytest

from paper_1611_06945_amd import workloads as wl
from paper_1611_06945_amd.workloads import ConvShape

from gpu_util import TOL
from test_gpu_parity import assert_bit_exact, int_case, random_case

pytestmark = pytest.mark.gpu

SHAPES = [
    ConvShape(9, 8, 1, 1, 1, 1, 1, 1, 0),       # one vector per row, one output channel
    ConvShape(16, 24, 1, 1, 17, 1, 1, 1, 0),    # a row past a tile, part of a step
    ConvShape(17, 40, 3, 5, 64, 3, 5, 1, 0),    # 600 elements: a step and a piece for some waves only
    ConvShape(33, 64, 2, 4, 100, 2, 4, 1, 0),   # 512 elements: exactly one step per wave in 16 bits
    ConvShape(64, 136, 6, 6, 40, 6, 6, 1, 0),   # 4896 elements: more steps than in flight
    ConvShape(20, 256, 7, 7, 33, 7, 7, 1, 0),
    ConvShape(3, 194, 7, 7, 50, 7, 7, 1, 0),    # 9506 elements: rows on 4-byte boundaries only, split and whole
    ConvShape(18, 3, 6, 5, 20, 6, 5, 1, 0),     # 90 elements: one cut vector per row
    # every other count of eight-image groups (each is an instantiation with its own loads in flight; an odd one leaves half of
    # its last LDS block unwritten), whole rows ...
    ConvShape(25, 136, 6, 6, 33, 6, 6, 1, 0),
    ConvShape(32, 72, 4, 4, 17, 4, 4, 1, 0),
    ConvShape(41, 136, 6, 6, 20, 6, 6, 1, 0),
    ConvShape(56, 264, 4, 4, 40, 4, 4, 1, 0),
    # ... and rows whose end is cut, most of them long enough for the four-way split
    ConvShape(16, 194, 7, 7, 20, 7, 7, 1, 0),
    ConvShape(48, 7, 3, 6, 17, 3, 6, 1, 0),
    ConvShape(32, 194, 7, 7, 18, 7, 7, 1, 0),
    ConvShape(40, 2, 5, 9, 33, 5, 9, 1, 0),
    ConvShape(49, 338, 7, 7, 19, 7, 7, 1, 0),
    ConvShape(64, 194, 7, 7, 16, 7, 7, 1, 0),
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.F16, wl.BF16])
@pytest.mark.parametrize("si", range(len(SHAPES)))
def test_shapes(si, dtype):
    shape = SHAPES[si]
    icase = int_case(shape, dtype, 4500 + si)
    rcase = random_case(shape, dtype, 4550 + si, relu=bool(si % 2))
    mine = [(i, n) for i, n in enumerate(icase.variant_names()) if "_mfma_rows16_" in n]
    assert mine, shape
    for vi, name in mine:
        print(name, shape, flush=True)
        assert_bit_exact(icase, icase.run(variant=vi), name)
        err = rcase.error(rcase.run(variant=vi))
        assert err <= TOL[dtype], "%s: %.3g" % (name, err)
