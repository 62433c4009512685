"""GPU parity of the many-pixel window kernel (fp16/bf16) where its tiles, slabs and stores have their edges: against the
CPU oracle, bit for bit on small-integer data (every partial sum is exact, so any order of additions gives the same
bits) and within the storage type's tolerance on random data.  Plain formats run behind the kernel's conversion launch;
channel-innermost tensors with packed filters run it directly, with either output format."""
import numpy as np
import pytest

import oracle
from paper_1611_06945_amd import binding as B
from paper_1611_06945_amd import workloads as wl
from paper_1611_06945_amd.workloads import ConvShape

from gpu_util import TOL, DeviceCase, to_host_f64
from test_gpu_packed import PackedCase

pytestmark = pytest.mark.gpu

SHAPES = [
    ConvShape(1, 8, 16, 16, 32, 3, 3, 1, 1),     # one image, one tile exactly (256 pixels), half a channel group
    ConvShape(3, 17, 13, 17, 33, 3, 3, 1, 1),    # one channel over a group, one row over a block, odd image size
    ConvShape(5, 100, 15, 9, 130, 3, 3, 1, 1),   # ragged channels on both sides, tiles over several images
    ConvShape(2, 48, 16, 24, 64, 3, 3, 1, 0),    # no border; 308 pixels: stores by element, last tile mostly empty
    ConvShape(2, 32, 14, 20, 96, 3, 3, 1, 2),    # border as wide as the window's reach; 16 x 22 outputs: 16-byte stores
    ConvShape(1, 16, 5, 224, 72, 3, 3, 1, 1),    # the longest rows
    ConvShape(9, 16, 8, 8, 64, 3, 3, 1, 1),      # whole images per tile, 16-byte stores
    ConvShape(3, 40, 13, 12, 96, 5, 5, 1, 2),    # 5x5
    ConvShape(2, 16, 27, 27, 160, 5, 5, 1, 1),   # 5x5, border narrower than half the window
]


def data_of(shape, dtype, seed, ints):
    if ints:
        return wl.small_int_case(shape, dtype, seed)
    return {"in": wl.to_storage(wl.draw(("halfnormal", 1.0), shape.in_shape(), seed), dtype),
            "filt": wl.to_storage(wl.draw(("normal", wl.he_sigma(shape)), shape.filt_shape(), seed + 1), dtype),
            "bias": wl.draw(("uniform", -0.1, 0.1), (shape.K,), seed + 2)}


@pytest.mark.parametrize("ints", [True, False])
@pytest.mark.parametrize("dtype", [wl.F16, wl.BF16])
@pytest.mark.parametrize("si", range(len(SHAPES)))
def test_plain_formats(si, dtype, ints):
    shape = SHAPES[si]
    case = DeviceCase(shape, dtype, data_of(shape, dtype, 4100 + si, ints), relu=bool(si % 2))
    mine = [(i, n) for i, n in enumerate(case.variant_names()) if n.startswith("bwin_")]
    assert mine, shape
    for i, name in mine:
        print(name, shape, dtype, flush=True)
        out = case.run(variant=i)
        if ints:
            want = wl.storage_to_f64(wl.to_storage(case.ref().astype(np.float32), dtype), dtype)
            assert np.array_equal(to_host_f64(out, dtype), want), name
        else:
            assert case.error(out) <= TOL[dtype], name


# layers whose input is read as it is (4 MiB and more, rows of whole 8-byte pieces, more than one group of 16 channels)
UNCOPIED = [
    ConvShape(150, 36, 20, 20, 100, 3, 3, 1, 1),  # half a group of 8 channels at the end, tiles over several images
    ConvShape(36, 100, 18, 36, 34, 3, 3, 1, 0),   # no border, ragged channels on both sides
    ConvShape(4, 33, 132, 124, 40, 3, 3, 1, 1),   # rows too long for most tiles; one channel over two groups
    ConvShape(171, 96, 16, 8, 64, 3, 3, 1, 2),    # border as wide as the window's reach, stores of 16 bytes
    ConvShape(820, 40, 8, 8, 33, 3, 3, 1, 1),     # whole images per tile
    ConvShape(1, 17, 1030, 120, 64, 3, 3, 1, 1),  # one image
    ConvShape(40, 100, 28, 20, 97, 5, 5, 1, 2),   # 5x5
    ConvShape(70, 36, 37, 24, 128, 5, 5, 1, 1),   # 5x5, border narrower than half the window
]


@pytest.mark.parametrize("ints", [True, False])
@pytest.mark.parametrize("dtype", [wl.F16, wl.BF16])
@pytest.mark.parametrize("si", range(len(UNCOPIED)))
def test_input_read_as_it_is(si, dtype, ints):
    shape = UNCOPIED[si]
    case = DeviceCase(shape, dtype, data_of(shape, dtype, 4300 + si, ints), relu=bool(si % 2))
    mine = [(i, n) for i, n in enumerate(case.variant_names()) if n.startswith("bwin_") and n.endswith("_p")]
    assert mine, shape
    for i, name in mine:
        print(name, shape, dtype, flush=True)
        out = case.run(variant=i)
        if ints:
            want = wl.storage_to_f64(wl.to_storage(case.ref().astype(np.float32), dtype), dtype)
            assert np.array_equal(to_host_f64(out, dtype), want), name
        else:
            assert case.error(out) <= TOL[dtype], name


def test_input_read_as_it_is_keeps_images_apart():
    """The channels behind a group's last one are the next image's, and the rows beside a border are another image's."""
    shape = UNCOPIED[0]
    data = data_of(shape, wl.BF16, 4400, True)
    plain = DeviceCase(shape, wl.BF16, data)
    data = dict(data, **{"in": data["in"].copy()})
    data["in"][1::2] = 0x7F80  # +infinity
    case = DeviceCase(shape, wl.BF16, data)
    for i, name in enumerate(case.variant_names()):
        if name.startswith("bwin_") and name.endswith("_p"):
            got, want = (to_host_f64(c.run(variant=i), wl.BF16) for c in (case, plain))
            assert np.array_equal(got[::2], want[::2]), name


@pytest.mark.parametrize("out_nhwc", [False, True])
@pytest.mark.parametrize("dtype", [wl.F16, wl.BF16])
@pytest.mark.parametrize("si", [i for i, s in enumerate(SHAPES) if s.C % 16 == 0])
def test_packed_filters(si, dtype, out_nhwc):
    shape = SHAPES[si]
    if out_nhwc and shape.K % 8:
        pytest.skip("channel-innermost output needs K % 8 == 0")
    for ints in (True, False):
        case = PackedCase(shape, dtype, data_of(shape, dtype, 4200 + si, ints), out_nhwc, relu=not ints)
        mine = [(i, n) for i, n in enumerate(case.names()) if n.startswith("pwin_big_")]
        assert mine, shape
        for i, name in mine:
            print(name, shape, dtype, flush=True)
            got = case.run(variant=i)
            if ints:
                want = wl.storage_to_f64(wl.to_storage(case.ref.astype(np.float32), dtype), dtype)
                assert np.array_equal(got, want), name
            else:
                assert oracle.max_normalised_error(got, case.ref) <= TOL[dtype], name
