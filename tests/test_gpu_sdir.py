"""GPU parity of the direct window kernel on split products (fp32) where its tiles, slabs and channel steps have their edges: bit
for bit on small integers (the splits and every sum are exact), within a bound that shows a lost partial product on random data, and
on operands that the parts cannot carry, where the sums are taken again from the definition."""
import numpy as np
import pytest

import oracle
from paper_1611_06945_amd import binding as B
from paper_1611_06945_amd import workloads as wl
from paper_1611_06945_amd.workloads import ConvShape

from gpu_util import TOL, DeviceCase, empty_out, to_host_f64, torch_mod
from test_gpu_parity import assert_bit_exact, int_case, random_case

pytestmark = pytest.mark.gpu

SHAPES = [
    ConvShape(1, 8, 5, 5, 17, 5, 5, 1, 2),      # half a channel step, one tile, rows shorter than a half wave
    ConvShape(3, 17, 13, 13, 33, 5, 5, 1, 2),   # one channel over a step, one filter over a block, tiles across images
    ConvShape(9, 40, 4, 3, 70, 3, 3, 1, 1),     # several images a tile, three steps
    ConvShape(2, 130, 19, 23, 64, 3, 3, 2, 1),  # nine steps: waves with one more than others
    ConvShape(2, 16, 30, 20, 40, 3, 3, 3, 0),   # windows side by side
    ConvShape(2, 24, 33, 21, 100, 5, 5, 2, 1),  # a border smaller than the window needs to keep its size
    ConvShape(1, 64, 57, 55, 48, 3, 3, 1, 1),   # wide rows
    ConvShape(1, 20, 9, 8, 32, 5, 5, 4, 4),     # the largest stride and border, fewer rows than a tile spans
    ConvShape(2, 137, 9, 7, 70, 5, 5, 1, 2),    # every form: two rounds of channels or more, in the last one some of the waves without any
    ConvShape(2, 137, 9, 7, 70, 3, 3, 1, 1),
    ConvShape(3, 273, 7, 7, 33, 5, 5, 1, 2),    # three rounds of eight waves
    ConvShape(3, 273, 9, 11, 65, 3, 3, 2, 1),
]


def variants_of(case):
    return [(i, n) for i, n in enumerate(case.variant_names()) if n.startswith("sdir_")]


@pytest.mark.parametrize("si", range(len(SHAPES)))
def test_shapes(si):
    shape = SHAPES[si]
    icase = int_case(shape, wl.F32, 4600 + si, relu=bool(si % 2), use_bias=si != 1)
    rcase = random_case(shape, wl.F32, 4650 + si, relu=not si % 2)
    mine = variants_of(icase)
    assert mine, shape
    for vi, name in mine:
        print(name, shape, flush=True)
        assert_bit_exact(icase, icase.run(variant=vi), name)
        err = rcase.error(rcase.run(variant=vi))
        assert err <= 1e-6, "%s: %.3g" % (name, err)  # (any partial product left out: 3e-6 and more)


@pytest.mark.parametrize("kind", ["corners", "filter", "huge", "tiny", "infinities"])
@pytest.mark.parametrize("si", [1, 2, 3, 5])
def test_sums_again_and_small_operands(si, kind):
    shape = SHAPES[si]
    x = wl.draw(("halfnormal", 1.0), shape.in_shape(), 4694).astype(np.float32)
    f = wl.draw(("normal", wl.he_sigma(shape)), shape.filt_shape(), 4695).astype(np.float32)
    if kind == "corners":
        x[0, 0, 0, 0], x[-1, -1, -1, -1], x[-1, 3, 0, -1], x[0, 5, -1, 0] = np.nan, np.inf, -np.inf, np.nan
    elif kind == "filter":
        f[shape.K // 2, 1, 2, 0], f[-1, -1, 0, 1] = np.nan, -np.inf
    elif kind == "huge":  # finite, every sum beyond what the scaled products can hold
        x *= np.float32(1e26)
    elif kind == "tiny":  # the third parts would be below bf16's normal numbers without the scale
        x, f = (x.astype(np.float64) * 2.0**-120).astype(np.float32), (f.astype(np.float64) * 2.0**80).astype(np.float32)
    else:
        x[:] = np.inf
    bias = np.full(shape.K, 0.0 if kind == "tiny" else 0.25, dtype=np.float32)
    case = DeviceCase(shape, wl.F32, {"in": x, "filt": f, "bias": bias}, relu=False)
    with np.errstate(all="ignore"):
        ref = case.ref()
    finite = np.isfinite(ref)
    for vi, name in variants_of(case):
        print(name, shape, kind, flush=True)
        got = to_host_f64(case.run(variant=vi), wl.F32)
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)]), name
        if kind == "tiny":
            assert np.abs(got - ref).max() <= 1e-6 * np.abs(ref).max(), name
        elif finite.any():
            assert oracle.max_normalised_error(got[finite], ref[finite]) <= TOL[wl.F32], name


@pytest.mark.parametrize("relu", [False, True])
def test_biases_that_are_not_finite(relu):
    """A NaN bias is the result of its channel where no activation drops it, and so is an infinite one."""
    shape = SHAPES[3]
    data = {"in": wl.draw(("halfnormal", 1.0), shape.in_shape(), 4696).astype(np.float32),
            "filt": wl.draw(("normal", wl.he_sigma(shape)), shape.filt_shape(), 4697).astype(np.float32), "bias": np.full(shape.K, 0.25, dtype=np.float32)}
    data["bias"][[0, 5, 31, 40]] = np.nan, np.inf, -np.inf, np.nan
    case = DeviceCase(shape, wl.F32, data, relu=relu)
    ref = case.ref()
    assert np.isnan(ref).any() != relu
    for vi, name in variants_of(case):
        got = to_host_f64(case.run(variant=vi), wl.F32)
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)]), name
        finite = np.isfinite(ref)
        assert oracle.max_normalised_error(got[finite], ref[finite]) <= TOL[wl.F32], name


@pytest.mark.parametrize("shape", [ConvShape(3, 220, 16, 16, 160, 5, 5, 1, 2), ConvShape(2, 176, 40, 40, 16, 5, 5, 1, 2), ConvShape(2, 416, 33, 33, 64, 5, 5, 1, 2), ConvShape(2, 256, 13, 13, 64, 3, 3, 2, 1)])
def test_no_less_precise_than_the_split_gemm_it_replaces(shape):
    """Error against 64 bits (2-norm) of every tile beside that of the implicit GEMM that splits the reduction over eight workgroups, the most
    precise of the kernels these layers ran on.  One chain of roundings over all channels and taps: 1.03 of it in the second layer."""
    data = {"in": wl.draw(("halfnormal", 1.0), shape.in_shape(), 4698).astype(np.float32),
            "filt": wl.draw(("normal", wl.he_sigma(shape)), shape.filt_shape(), 4699).astype(np.float32), "bias": np.zeros(shape.K, np.float32)}
    case = DeviceCase(shape, wl.F32, data, relu=False)

    def error(vi):
        return np.linalg.norm(to_host_f64(case.run(variant=vi), wl.F32) - case.ref()) / np.linalg.norm(case.ref())

    split = min(error(i) for i, n in enumerate(case.variant_names()) if n.startswith("ug_") and n.endswith("_sk8"))
    for vi, name in variants_of(case):
        err = error(vi)
        print(name, "%.3g %.3g" % (err, split), flush=True)
        assert err <= split, name


@pytest.mark.parametrize("shape", [ConvShape(20, 256, 13, 13, 96, 3, 3, 1, 1), ConvShape(6, 256, 15, 15, 48, 3, 3, 1, 1)])
def test_no_less_precise_than_the_split_window_kernel_it_replaces(shape):
    """... and at 3x3 beside the fp32 window kernel that splits the reduction over four workgroups: 2.2e-7 in the first layer, one chain over all
    channels and taps 2.8e-7."""
    data = {"in": wl.draw(("halfnormal", 1.0), shape.in_shape(), 4688).astype(np.float32),
            "filt": wl.draw(("normal", wl.he_sigma(shape)), shape.filt_shape(), 4689).astype(np.float32), "bias": np.zeros(shape.K, np.float32)}
    case = DeviceCase(shape, wl.F32, data, relu=False)

    def error(vi):
        return np.linalg.norm(to_host_f64(case.run(variant=vi), wl.F32) - case.ref()) / np.linalg.norm(case.ref())

    split = min(error(i) for i, n in enumerate(case.variant_names()) if n.startswith("wconv_") and n.endswith("_sk4"))
    for vi, name in variants_of(case):
        err = error(vi)
        print(name, "%.3g %.3g" % (err, split), flush=True)
        assert err <= split, name


@pytest.mark.parametrize("kind", ["corners", "filter", "infinities"])
@pytest.mark.parametrize("si", [1, 2, 3, 5, 9])
def test_sums_again_under_the_activation(si, kind):
    """A sum that is a NaN or -infinity is dropped by the activation, +infinity is not; channels and pixels past the last ones are not stored."""
    shape = SHAPES[si]
    x = wl.draw(("normal", 1.0), shape.in_shape(), 4692).astype(np.float32)
    f = wl.draw(("normal", wl.he_sigma(shape)), shape.filt_shape(), 4693).astype(np.float32)
    if kind == "corners":
        x[0, 0, 0, 0], x[-1, -1, -1, -1], x[-1, 3, 0, -1], x[0, 5, -1, 0] = np.nan, np.inf, -np.inf, np.nan
    elif kind == "filter":
        f[shape.K // 2, 1, 2, 0], f[-1, -1, 0, 1] = np.nan, -np.inf
    else:
        x[0] = np.inf
    case = DeviceCase(shape, wl.F32, {"in": x, "filt": f, "bias": wl.draw(("normal", 0.1), (shape.K,), 4691).astype(np.float32)}, relu=True)
    with np.errstate(all="ignore"):
        ref = case.ref()
    finite = np.isfinite(ref)
    for vi, name in variants_of(case):
        got = to_host_f64(case.run(variant=vi), wl.F32)
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)]), name
        assert oracle.max_normalised_error(got[finite], ref[finite]) <= TOL[wl.F32], name


# The largest time allowed, in calls on ordinary data; measured with a wave for each output and with pixels that share a wave
@pytest.mark.parametrize("kind,limit", [("one infinity", 20), ("NaN everywhere", 5), ("beyond the range", 60)])  # 43, 6; 410, 0.9; 400, 18
def test_data_that_is_not_finite_takes_a_few_calls_time(kind, limit):
    torch = torch_mod()
    shape = ConvShape(50, 424, 14, 14, 96, 5, 5, 1, 2)
    g = torch.Generator(device="cuda")
    g.manual_seed(4690)
    x = torch.randn(shape.in_shape(), generator=g, device="cuda").abs_()
    f = torch.randn(shape.filt_shape(), generator=g, device="cuda").mul_(wl.he_sigma(shape))
    desc = B.desc_of(shape, wl.F32, relu=True)
    assert B.conv_variant_name(desc, -1).startswith("sdir_")
    out, ws = empty_out(shape.out_shape(), wl.F32), torch.empty(B.conv_workspace_bytes(desc), dtype=torch.uint8, device="cuda")

    def us():
        return min(B.conv_time_us(desc, x, f, None, out, ws, ws.numel(), launches=3) for _ in range(3))

    plain = us()
    if kind == "one infinity":
        x[7, 100, 6, 6] = float("inf")
    elif kind == "NaN everywhere":
        x.fill_(float("nan"))
    else:
        x.mul_(1e26)  # finite, every sum beyond what the scaled products can hold
    special = us()
    print("%s: %.0f us, %.0f on ordinary data" % (kind, special, plain), flush=True)
    assert special <= limit * plain
