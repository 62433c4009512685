"""GPU parity of the first-layer kernel on split products (fp32, 3 channels) where its tiles, staged rows and reduction steps have their
edges, no further from 64 bits than the gather kernels, and with values that its bf16 parts cannot carry."""
import numpy as np
import pytest

import oracle
from paper_1611_06945_amd import binding as B
from paper_1611_06945_amd import workloads as wl
from paper_1611_06945_amd.workloads import ConvShape

from gpu_util import TOL, DeviceCase, to_host_f64, torch_mod

pytestmark = pytest.mark.gpu

SHAPES = [
    ConvShape(1, 3, 11, 11, 5, 11, 11, 4, 0),     # one pixel, five filters
    ConvShape(2, 3, 71, 75, 96, 11, 11, 4, 0),    # 16 x 17 pixels: a full tile and a ragged one per image
    ConvShape(1, 3, 40, 300, 33, 11, 11, 4, 3),   # rows longer than 256 columns, a filter over a block, columns of zeros
    ConvShape(1, 3, 23, 14, 64, 11, 11, 4, 10),   # border as wide as it may be
    ConvShape(2, 3, 20, 9, 40, 7, 7, 2, 3),       # the last piece of a row overlaps the one before
    ConvShape(1, 3, 33, 131, 64, 7, 7, 2, 0),
    ConvShape(3, 3, 7, 8, 1, 7, 7, 2, 2),
]


def variants_of(case):
    mine = [(i, n) for i, n in enumerate(case.variant_names()) if n.startswith("swins_")]
    assert mine, case.shape
    return mine


def data_of(shape, seed):
    return {"in": wl.draw(("uniform", -128.0, 128.0), shape.in_shape(), seed), "filt": wl.draw(("normal", wl.he_sigma(shape)), shape.filt_shape(), seed + 1),
            "bias": wl.draw(("uniform", -0.1, 0.1), (shape.K,), seed + 2)}


@pytest.mark.parametrize("ints", [True, False])
@pytest.mark.parametrize("si", range(len(SHAPES)))
def test_parity(si, ints):
    shape = SHAPES[si]
    case = DeviceCase(shape, wl.F32, wl.small_int_case(shape, wl.F32, 6100 + si) if ints else data_of(shape, 6100 + si), relu=bool(si % 2))
    for i, name in variants_of(case):
        print(name, shape, flush=True)
        out = case.run(variant=i)
        if ints:
            assert np.array_equal(to_host_f64(out, wl.F32), case.ref()), name
        else:
            assert case.error(out) <= TOL[wl.F32], name


def test_no_further_from_64_bits_than_the_gather_kernels():
    case = DeviceCase(ConvShape(2, 3, 99, 99, 96, 11, 11, 4, 0), wl.F32, data_of(ConvShape(2, 3, 99, 99, 96, 11, 11, 4, 0), 6200), relu=False)
    ref = case.ref()
    err = {n: np.linalg.norm(to_host_f64(case.run(variant=i), wl.F32) - ref) / np.linalg.norm(ref)
           for i, n in enumerate(case.variant_names()) if n.startswith(("swins_", "ug_")) and "_sk" not in n}
    gather = min(e for n, e in err.items() if n.startswith("ug_"))
    for n, e in err.items():
        if n.startswith("swins_"):
            assert e <= gather, (n, e, gather)


@pytest.mark.parametrize("R,stride,pad", [(11, 4, 0), (7, 2, 3)])
def test_values_beyond_the_parts(R, stride, pad):
    """Infinities, NaN and numbers whose scaled parts overflow give what the definition gives, and reach no other output; the smallest
    numbers lose nothing."""
    shape = ConvShape(2, 3, 47, 45, 34, R, R, stride, pad)
    data = data_of(shape, 6300)
    data["in"][0, 1, 20, 21] = np.inf
    data["in"][1, 2, 30, 11] = np.nan
    data["filt"][3] = 3e38
    data["filt"][5] *= np.float32(2.0 ** -120)
    case = DeviceCase(shape, wl.F32, data, relu=False)
    with np.errstate(over="ignore", invalid="ignore"):
        ref = case.ref().astype(np.float32).astype(np.float64)
    for i, name in variants_of(case):
        got = to_host_f64(case.run(variant=i), wl.F32)
        # (a sum of 3e38 x pixels overflows in fp32 in one order and not in another: that filter is only checked not to leak)
        ks = [k for k in range(shape.K) if k != 3]
        assert np.array_equal(np.isfinite(got[:, ks]), np.isfinite(ref[:, ks])), name
        for k in ks:
            m = np.isfinite(ref[:, k])
            assert np.max(np.abs(got[:, k][m] - ref[:, k][m])) <= TOL[wl.F32] * np.max(np.abs(ref[:, k][m])), (name, k)


def test_output_close_to_the_size_limit():
    """1828 images, the most that the 96-channel tile accepts: 95 of the last tile's channels do not exist, and their stores aim past
    2 GiB.  Small integers: bit for bit what a gather kernel gives, and nothing written behind the output."""
    torch = torch_mod()
    shape = ConvShape(1828, 3, 227, 227, 97, 11, 11, 4, 0)
    g = torch.Generator(device="cuda")
    g.manual_seed(6400)

    def ints(dims, r):
        return torch.randint(-r, r + 1, dims, generator=g, device="cuda", dtype=torch.int32).float()

    x, f, b = ints(shape.in_shape(), 3), ints(shape.filt_shape(), 2), ints((shape.K,), 4)
    desc = B.desc_of(shape, wl.F32, relu=True)
    names = [B.conv_variant_name(desc, i) for i in range(B.conv_variant_count(desc))]
    gather = [n for n in names if not n.startswith("swins_") and "_sk" not in n][-1]
    mine = [n for n in names if n.startswith("swins_")]
    assert any(n.endswith("_M96N256") for n in mine)
    n_out, spare = shape.N * shape.K * shape.OH * shape.OW, 1 << 20
    want = None
    for name in [gather] + mine:
        print(name, shape, flush=True)
        buf = torch.full((n_out + spare,), float("nan"), device="cuda")
        i = names.index(name)
        ws = torch.empty(max(256, B.conv_variant_workspace(desc, i)), dtype=torch.uint8, device="cuda")
        B.conv_force_variant(desc, i)
        try:
            B.conv_fwd_ws(desc, x, f, b, buf[:n_out], ws, ws.numel())
            torch.cuda.synchronize()
        finally:
            B.conv_force_variant(desc, -1)
        assert bool(torch.isnan(buf[n_out:]).all()), name
        want = buf[:n_out] if want is None else want
        assert torch.equal(buf[:n_out], want), name


def test_7x7_no_further_from_64_bits_than_the_gather_kernels():
    shape = ConvShape(2, 3, 75, 71, 64, 7, 7, 2, 3)
    case = DeviceCase(shape, wl.F32, data_of(shape, 6210), relu=False)
    ref = case.ref()
    err = {n: np.linalg.norm(to_host_f64(case.run(variant=i), wl.F32) - ref) / np.linalg.norm(ref)
           for i, n in enumerate(case.variant_names()) if n.startswith(("swins_", "ug_")) and "_sk" not in n}
    gather = min(e for n, e in err.items() if n.startswith("ug_"))
    mine = [n for n in err if n.startswith("swins_")]
    assert mine
    for n in mine:
        assert err[n] <= gather, (n, err[n], gather)


def absolute_sums(case):
    """Sum of |in * filt| + |bias| of every output: what the rounding errors of a sum are measured against."""
    s = case.shape
    return oracle.conv_fwd(np.abs(case.data["in"]).astype(np.float64), np.abs(case.data["filt"]).astype(np.float64),
                           np.abs(case.data["bias"]).astype(np.float64), stride=s.stride, pad=s.pad, relu=False)


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("R,stride,pad", [(11, 4, 0), (7, 2, 3)])
def test_finite_results_beyond_the_scaled_range(R, stride, pad, relu):
    """Operands that overflow once scaled by 2^24 (above about 2^103) and sums that overflow once scaled by 2^48 (above 2^79), in a call whose
    results are all finite: every one is what the definition gives, the ordinary ones beside them too.  Ragged tiles: 100 pixels
    of 256 and 528 of 768, 34 and 97 filters."""
    for K in (34, 97):
        shape = ConvShape(2, 3, 47, 47 - 4 * (R == 7), K, R, R, stride, pad)
        data = data_of(shape, 6500 + K)
        x, f = data["in"], data["filt"]
        f[3] = 0.0
        f[3, 1, R // 2, 2] = np.float32(2.0 ** 110)   # one tap: its products are finite, its parts are not
        f[K - 1] = 0.0
        f[K - 1, 2, 0, R - 1] = -np.float32(2.0 ** 104)
        f[5] = np.abs(f[5]) * np.float32(2.0 ** 80)   # sums of about 2^86 from parts that are all finite
        x[1, :, 20:24, :] = 0.0
        x[1, 0, 9, 9] = np.float32(1.5 * 2.0 ** 105)  # a pixel beyond it, beside ordinary filters: results of about 2^103
        f[5, 0] = f[3, 0] = f[K - 1, 0] = 0.0         # (times the large filters it would be beyond fp32)
        case = DeviceCase(shape, wl.F32, data, relu=relu)
        ref, size = case.ref(), absolute_sums(case)
        assert np.abs(ref).max() < 2.0 ** 126 and np.abs(ref[:, 5]).max() > 2.0 ** 82 and np.abs(ref[0, 3]).max() > 2.0 ** 110
        for i, name in variants_of(case):
            print(name, shape, relu, flush=True)
            got = to_host_f64(case.run(variant=i), wl.F32)
            assert np.all(np.isfinite(got)), name
            # (a sum of n terms in fp32, whatever the order: n + 1 roundings of 2^-24 of the terms' sizes)
            bound = (3 * R * R + 1) * 2.0 ** -24 * size
            assert np.all(np.abs(got - ref) <= bound), (name, np.max(np.abs(got - ref) / bound))


@pytest.mark.parametrize("R,stride,pad", [(11, 4, 0), (7, 2, 3)])
def test_infinities_keep_their_sign_and_nan_stays_nan(R, stride, pad):
    shape = ConvShape(2, 3, 47, 45, 34, R, R, stride, pad)
    data = data_of(shape, 6600)
    data["in"][0, 1, 20, 21] = np.inf
    data["in"][0, 2, 40, 40] = -np.inf
    data["in"][1, 2, 30, 11] = np.nan
    data["filt"][4] = np.abs(data["filt"][4])
    data["filt"][4, 0, 0, 0] = -np.inf
    case = DeviceCase(shape, wl.F32, data, relu=False)
    with np.errstate(invalid="ignore"):
        ref = case.ref()
    assert np.isnan(ref).any() and (ref == np.inf).any() and (ref == -np.inf).any()
    for i, name in variants_of(case):
        got = to_host_f64(case.run(variant=i), wl.F32)
        assert np.array_equal(np.isnan(got), np.isnan(ref)), name
        assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)]), name
        finite = np.isfinite(ref)
        assert np.max(np.abs(got[finite] - ref[finite])) <= TOL[wl.F32] * np.max(np.abs(ref[finite])), name
