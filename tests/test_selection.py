"""The library's own selection (no measurement at hand) against measured times: layers for which the kernel named first took
clearly longer than one the selection had before or has now.  CPU only: the cost model is host code."""
import pytest

from paper_1611_06945_amd import binding as B
from paper_1611_06945_amd import workloads as wl
from paper_1611_06945_amd.workloads import ConvShape


def picks(shape, dtype, fmt="nchw"):
    nh = fmt != "nchw"
    d = B.desc_of(shape, dtype, relu=True, in_nhwc=nh, out_nhwc=nh, filt_packed=fmt == "packed")
    return B.conv_variant_name(d, -1), B.conv_variant_name(d, -2)


# rows too short for 16 waves to share: us of the matrix-unit kernel, of the tiles
@pytest.mark.parametrize("N,C,K,dtype", [
    (62, 48, 50, wl.BF16),    # 7.5, 3.7
    (49, 17, 2048, wl.F32),   # 9.2, 3.5
    (32, 28, 1000, wl.F16),   # 7.7, 3.3
    (50, 64, 200, wl.F32),    # 8.8, 5.5
    (18, 101, 20, wl.F32),    # 7.3, 4.9
])
def test_short_fully_connected_rows_go_to_the_tiles(N, C, K, dtype):
    for name in picks(ConvShape(N, C, 1, 1, K, 1, 1, 1, 0), dtype):
        assert "_mfma_rows16_" not in name, name


# ... and longer ones do not, split where their workgroups are few: us split, whole, of the tiles
@pytest.mark.parametrize("shape,dtype,split", [
    (ConvShape(64, 194, 7, 7, 40, 7, 7, 1, 0), wl.F32, True),     # 23, 52, 40
    (ConvShape(64, 512, 7, 7, 10, 7, 7, 1, 0), wl.F16, True),     # 19, 43, 111
    (ConvShape(20, 2048, 1, 1, 10, 1, 1, 1, 0), wl.F16, False),   # too short to split, 6, 24
    (ConvShape(40, 2048, 1, 1, 1000, 1, 1, 1, 0), wl.F32, False),  # too short to split, 11, 38
    (ConvShape(20, 256, 6, 6, 4096, 6, 6, 1, 0), wl.F16, False),  # 25, 16, 32
])
def test_long_fully_connected_rows_go_to_the_matrix_unit_kernel(shape, dtype, split):
    name, nows = picks(shape, dtype)
    assert "_mfma_rows16_" in name and name.endswith("_sk4") == split, name
    assert "_mfma_rows16_" in nows and not nows.endswith("_sk4"), nows
