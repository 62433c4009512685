"""GPU parity of the many-pixel pointwise kernel (fp16/bf16, plain formats): channel counts of half a group, ragged filter
counts, tiles that end inside an image and past the last pixel, fewer and more groups than are in flight; bit for bit on
small integers and within the storage type's tolerance on random data."""
import numpy as np
import pytest

import oracle
from paper_1611_06945_amd import workloads as wl
from paper_1611_06945_amd.workloads import ConvShape

from gpu_util import TOL, DeviceCase, to_host_f64
from test_gpu_parity import assert_bit_exact, int_case, random_case

pytestmark = pytest.mark.gpu

SHAPES = [
    ConvShape(1, 8, 2, 1, 1, 1, 1, 1, 0),        # one pixel pair, half a group, one filter
    ConvShape(3, 24, 6, 7, 33, 1, 1, 1, 0),      # 42 pixels an image: pairs only
    ConvShape(5, 136, 14, 14, 130, 1, 1, 1, 0),  # ragged filters, an odd group count, tiles across images
    ConvShape(2, 272, 16, 18, 72, 1, 1, 1, 0),   # 17 groups: more than two rounds of the ring
    ConvShape(1, 520, 8, 8, 128, 1, 1, 1, 0),    # the largest filter tile that fits
    ConvShape(4, 16, 32, 16, 256, 1, 1, 1, 0),   # whole tiles
]


@pytest.mark.parametrize("dtype", [wl.F16, wl.BF16])
@pytest.mark.parametrize("si", range(len(SHAPES)))
def test_shapes(si, dtype):
    shape = SHAPES[si]
    icase = int_case(shape, dtype, 4600 + si)
    rcase = random_case(shape, dtype, 4650 + si, relu=bool(si % 2))
    mine = [(i, n) for i, n in enumerate(icase.variant_names()) if n.startswith("pwb_")]
    assert mine, shape
    for vi, name in mine:
        print(name, shape, flush=True)
        assert_bit_exact(icase, icase.run(variant=vi, with_ws=False), name)
        err = rcase.error(rcase.run(variant=vi, with_ws=False))
        assert err <= TOL[dtype], "%s: %.3g" % (name, err)


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("dtype", [wl.F16, wl.BF16])
@pytest.mark.parametrize("C", [72, 144])  # five groups (the last one half) and nine: no multiple of any ring
def test_infinite_filter_values(C, dtype, relu):
    """An infinite weight makes its own output channel infinite (inputs are positive) and touches no other."""
    shape = ConvShape(3, C, 6, 8, 40, 1, 1, 1, 0)
    x = wl.to_storage(wl.draw(("halfnormal", 1.0), shape.in_shape(), 4690) + 0.5, dtype)
    f = wl.draw(("normal", wl.he_sigma(shape)), shape.filt_shape(), 4691)
    f[5, 0], f[17, 15], f[33, C - 1] = np.inf, np.inf, np.inf
    case = DeviceCase(shape, dtype, {"in": x, "filt": wl.to_storage(f, dtype), "bias": np.zeros(shape.K, np.float32)}, relu=relu)
    ref = case.ref()
    hit = np.zeros(ref.shape, dtype=bool)
    hit[:, [5, 17, 33]] = True
    assert np.array_equal(np.isposinf(ref), hit) and np.isfinite(ref[~hit]).all()
    mine = [(i, n) for i, n in enumerate(case.variant_names()) if n.startswith("pwb_")]
    assert mine
    for vi, name in mine:
        got = to_host_f64(case.run(variant=vi, with_ws=False), dtype)
        assert np.array_equal(np.isposinf(got), hit), name
        assert oracle.max_normalised_error(got[~hit], ref[~hit]) <= TOL[dtype], name
