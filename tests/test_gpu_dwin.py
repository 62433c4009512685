"""GPU parity of the one-launch window kernel (fp16/bf16, any stride, plain and channel-innermost formats) where its tiles, slabs, filter
rows and chunks have their edges: bit for bit on small-integer data (every partial sum is exact, so any order of additions gives
the same bits), within the storage type's tolerance on random data, and with infinite filters beside a ragged last chunk."""
import numpy as np
import pytest

import oracle
from paper_1611_06945_amd import binding as B
from paper_1611_06945_amd import workloads as wl
from paper_1611_06945_amd.workloads import ConvShape

from gpu_util import TOL, DeviceCase, empty_out, to_device, to_host_f64
from test_gpu_bwin import data_of

pytestmark = pytest.mark.gpu

SHAPES = [
    ConvShape(1, 256, 13, 13, 48, 3, 3, 1, 1),    # whole chunks of every size; tiles that end inside a row
    ConvShape(3, 17, 13, 17, 34, 3, 3, 1, 1),     # odd channels: filter rows on odd elements; one channel over a group
    ConvShape(2, 8, 4, 4, 2, 3, 3, 1, 0),         # narrowest rows, two filters, one group of channels
    ConvShape(5, 100, 15, 9, 130, 3, 3, 1, 1),    # half a 16-byte piece behind the last channel, tiles over several images
    ConvShape(2, 40, 16, 24, 72, 3, 3, 1, 2),     # border as wide as the window's reach, 16-byte stores
    ConvShape(3, 33, 21, 30, 32, 3, 3, 2, 1),     # stride 2, rows whose last four pixels overlap the four before
    ConvShape(2, 64, 20, 42, 128, 3, 3, 2, 0),    # stride 2 without a border, columns that no window reaches
    ConvShape(4, 24, 19, 16, 16, 3, 3, 3, 2),     # stride as wide as the window
    ConvShape(3, 40, 13, 12, 96, 5, 5, 1, 2),     # 5x5
    ConvShape(3, 21, 14, 14, 6, 5, 5, 1, 2),      # 5x5, odd channels
    ConvShape(1, 136, 9, 11, 8, 5, 5, 1, 1),      # 5x5, a group over a whole chunk of channels
]


@pytest.mark.parametrize("ints", [True, False])
@pytest.mark.parametrize("dtype", [wl.F16, wl.BF16])
@pytest.mark.parametrize("si", range(len(SHAPES)))
def test_plain_formats(si, dtype, ints):
    shape = SHAPES[si]
    case = DeviceCase(shape, dtype, data_of(shape, dtype, 5100 + si, ints), relu=bool(si % 2))
    mine = [(i, n) for i, n in enumerate(case.variant_names()) if n.startswith("dwin_")]
    assert mine and all(B.conv_variant_workspace(case.desc, i) == 0 for i, _ in mine), shape
    for i, name in mine:
        print(name, shape, dtype, flush=True)
        out = case.run(variant=i, with_ws=False)
        if ints:
            want = wl.storage_to_f64(wl.to_storage(case.ref().astype(np.float32), dtype), dtype)
            assert np.array_equal(to_host_f64(out, dtype), want), name
        else:
            assert case.error(out) <= TOL[dtype], name


@pytest.mark.parametrize("ints", [True, False])
@pytest.mark.parametrize("dtype", [wl.F16, wl.BF16])
@pytest.mark.parametrize("si", [i for i, s in enumerate(SHAPES) if s.C % 8 == 0 and s.K % 8 == 0 and s.stride < 3])
def test_channel_innermost(si, dtype, ints):
    import torch

    shape = SHAPES[si]
    data = data_of(shape, dtype, 5200 + si, ints)
    d = B.desc_of(shape, dtype, relu=bool(si % 2), in_nhwc=True, out_nhwc=True, filt_krsc=True)
    x, f = (to_device(data[k], dtype).permute(0, 2, 3, 1).contiguous() for k in ("in", "filt"))
    b = to_device(data["bias"], wl.F32)
    ref = oracle.conv_fwd(wl.storage_to_f64(data["in"], dtype), wl.storage_to_f64(data["filt"], dtype), data["bias"].astype(np.float64),
                          stride=shape.stride, pad=shape.pad, relu=bool(si % 2))
    n, k, oh, ow = shape.out_shape()
    mine = [(i, m) for i, m in enumerate(B.conv_variant_name(d, i) for i in range(B.conv_variant_count(d))) if m.startswith("nhwc_dwin_")]
    assert mine, shape
    for i, name in mine:
        print(name, shape, dtype, flush=True)
        out = empty_out((n, oh, ow, k), dtype)
        B.conv_force_variant(d, i)
        try:
            B.conv_fwd(d, x, f, b, out)
            torch.cuda.synchronize()
        finally:
            B.conv_force_variant(d, -1)
        got = to_host_f64(out, dtype).transpose(0, 3, 1, 2)
        if ints:
            assert np.array_equal(got, wl.storage_to_f64(wl.to_storage(ref.astype(np.float32), dtype), dtype)), name
        else:
            assert oracle.max_normalised_error(got, ref) <= TOL[dtype], name


@pytest.mark.parametrize("C", [17, 20, 24, 100])
def test_infinite_filters_stay_in_their_own_row(C):
    """The last chunk of a filter row is followed by the next row, the last channel of an image by the next image: infinities there reach
    only the outputs that they belong to."""
    shape = ConvShape(2, C, 12, 14, 34, 3, 3, 1, 1)
    data = data_of(shape, wl.F16, 5300 + C, False)
    data["filt"][1] = np.inf   # behind filter 0
    data["in"][1, 0] = np.inf  # behind the last channel of image 0
    case = DeviceCase(shape, wl.F16, data, relu=False)
    names = case.variant_names()
    for i, name in enumerate(names):
        if not name.startswith("dwin_"):
            continue
        got = to_host_f64(case.run(variant=i, with_ws=False), wl.F16)
        keep = [k for k in range(shape.K) if k != 1]
        assert np.all(np.isfinite(got[0, keep])), name
        assert np.max(np.abs(got[0, keep] - case.ref()[0, keep])) <= TOL[wl.F16] * np.max(np.abs(case.ref()[0, keep])), name
