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

from gpu_util import TOL, DeviceCase, empty_out, to_host_f64, torch_mod
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
    mine = [(i, n) for i, n in enumerate(case.variant_names()) if n.startswith("bwin_") and n.endswith("_p")]
    assert mine, shape
    for i, name in mine:
        got, want = (to_host_f64(c.run(variant=i), wl.BF16) for c in (case, plain))
        assert np.array_equal(got[::2], want[::2]), name


@pytest.mark.parametrize("where", ["filters", "inputs"])
def test_input_read_as_it_is_with_values_that_are_not_finite(where):
    """The products and their order are those of the form that copies the input: the same bits, not finite in the same places."""
    shape = UNCOPIED[0]
    data = data_of(shape, wl.F16, 4410, False)
    x, f = data["in"].copy(), data["filt"].copy()
    if where == "filters":
        f[5, 35, 0, 0], f[70, 0, 2, 1], f[99, 17, 1, 1] = np.inf, np.nan, -np.inf
    else:
        x[0, 35, 0, 0], x[75, 16, 19, 19], x[149, 0, 7, 0] = np.inf, np.nan, -np.inf
    case = DeviceCase(shape, wl.F16, dict(data, **{"in": x, "filt": f}), relu=False)
    index = {n: i for i, n in enumerate(case.variant_names())}
    mine = [n for n in index if n.startswith("bwin_") and n.endswith("_p")]
    assert mine, shape
    for name in mine:
        got, want = (to_host_f64(case.run(variant=index[n]), wl.F16) for n in (name, name[:-2]))
        assert np.isfinite(want).any() and not np.isfinite(want).all(), name
        assert np.array_equal(got, want, equal_nan=True), name


# packed filters above 2 MiB: channel tiles in turn instead of side by side.  Inputs just below the kernel's limit of 2 GiB, look-ahead
# included: many images with ragged channels, one image whose channels lie 3.9 MB apart
FAR = [
    ConvShape(9, 520, 24, 24, 250, 3, 3, 1, 1),
    ConvShape(1100, 300, 55, 56, 40, 3, 3, 1, 1),
    ConvShape(1, 520, 17850, 112, 64, 3, 3, 1, 1),
]


@pytest.mark.parametrize("si", range(len(FAR)))
def test_input_read_as_it_is_far_apart(si):
    """Bit for bit on small integers, at windows spread over the outputs, the first and the last ones among them."""
    torch = torch_mod()
    shape, (N, C, H, W) = FAR[si], FAR[si].in_shape()
    packed = (shape.K + 31) // 32 * ((C + 15) // 16) * 1024 * shape.R * shape.S
    assert packed > 2 << 20 if si == 0 else 2 * N * (C + 16) * H * W > 0.99 * 2**31
    g = torch.Generator(device="cuda")
    g.manual_seed(4420 + si)
    x = torch.empty(shape.in_shape(), dtype=torch.float16, device="cuda")
    for n in range(N):
        x[n] = torch.randint(-2, 3, (C, H, W), generator=g, device="cuda")
    f = torch.randint(-2, 3, shape.filt_shape(), generator=g, device="cuda").half()
    at = torch.cat([torch.zeros(1, dtype=torch.int64), torch.randint(0, N * shape.OH * shape.OW, (400,), generator=torch.Generator().manual_seed(si)),
                    torch.tensor([N * shape.OH * shape.OW - 1])]).cuda()
    n, oy, ox = at // (shape.OH * shape.OW), at // shape.OW % shape.OH, at % shape.OW
    want = torch.zeros(len(at), shape.K, dtype=torch.float64, device="cuda")
    for r in range(3):
        for s in range(3):
            y, xx = oy + r - shape.pad, ox + s - shape.pad
            ok = (y >= 0) & (y < H) & (xx >= 0) & (xx < W)
            v = x[n, :, y.clamp(0, H - 1), xx.clamp(0, W - 1)].double() * ok[:, None]
            want += v @ f[:, :, r, s].double().t().contiguous()
    desc = B.desc_of(shape, wl.F16, relu=False)
    mine = [(i, nm) for i, nm in enumerate(B.conv_variant_name(desc, i) for i in range(B.conv_variant_count(desc))) if nm.startswith("bwin_") and nm.endswith("_p")]
    assert mine, shape
    ws = torch.empty(max(B.conv_variant_workspace(desc, i) for i, _ in mine), dtype=torch.uint8, device="cuda")
    for i, name in mine:
        print(name, shape, flush=True)
        out = empty_out(shape.out_shape(), wl.F16)
        B.conv_force_variant(desc, i)
        try:
            B.conv_fwd_ws(desc, x, f, None, out, ws, ws.numel())
            torch.cuda.synchronize()
        finally:
            B.conv_force_variant(desc, -1)
        assert not bool(torch.isnan(out).any()), name
        assert bool((out[n, :, oy, ox].double() == want.half().double()).all()), name


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
