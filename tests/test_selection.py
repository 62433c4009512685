"""The library's own selection (no measurement at hand) against measured times: layers for which the kernel named first took
clearly longer than one the selection had before or has now.  CPU only: the cost model is host code."""
import dataclasses

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


# 16-bit pointwise layers: what was taken, its us, what may be taken, its us
@pytest.mark.parametrize("shape,dtype,slow,slow_us,fast_us", [
    (ConvShape(2, 128, 125, 125, 64, 1, 1, 1, 0), wl.F16, ("pwk_f16_M64N32_w8", "pwk_f16_M32N32"), 20.8, 12.1),
    (ConvShape(14, 128, 30, 28, 112, 1, 1, 1, 0), wl.F16, ("pwk_f16_M64N32_w8", "pwk_f16_M32N32"), 16.2, 9.7),
    (ConvShape(12, 208, 15, 15, 320, 1, 1, 1, 0), wl.BF16, ("pwk_bf16_M64N32_w8", "pwk_bf16_M32"), 11.5, 7.4),
    (ConvShape(48, 1024, 40, 38, 8, 1, 1, 1, 0), wl.F16, ("ug_", "igemm_"), 59.0, 39.0),
    (ConvShape(21, 880, 58, 58, 10, 1, 1, 1, 0), wl.F16, ("ug_", "igemm_"), 52.0, 35.6),
    (ConvShape(14, 448, 47, 47, 16, 1, 1, 1, 0), wl.BF16, ("ug_", "igemm_"), 14.7, 12.4),
])
def test_pointwise_layers_keep_the_faster_kernel(shape, dtype, slow, slow_us, fast_us):
    for name in picks(shape, dtype):
        assert not name.startswith(slow), (name, slow_us, fast_us)


def test_many_pixels_of_a_pointwise_layer_go_to_the_streaming_kernel():
    for name in picks(ConvShape(64, 256, 28, 28, 128, 1, 1, 1, 0), wl.F16):  # us: 12.4, of the wave-split kernel 33
        assert name.startswith("pwb_f16_M64N512"), name


# window layers of few pixels: the many-pixel kernel's us, the packed-filter kernel's us
@pytest.mark.parametrize("shape,dtype,fmt", [
    (ConvShape(13, 384, 5, 4, 80, 5, 5, 1, 2), wl.F16, "packed"),     # 31.7, 10.6
    (ConvShape(15, 416, 15, 15, 48, 3, 3, 1, 1), wl.BF16, "packed"),  # 18.3, 6.5
    (ConvShape(53, 352, 8, 6, 112, 3, 3, 1, 0), wl.F16, "packed"),    # 17.3, 6.2
    (ConvShape(17, 416, 9, 9, 208, 3, 3, 1, 1), wl.F16, "packed"),    # 18.6, 8.5
    (ConvShape(7, 448, 8, 8, 800, 3, 3, 1, 1), wl.F16, "nchw"),       # 24.6, 15.3
    (ConvShape(57, 608, 15, 15, 27, 5, 5, 1, 2), wl.F16, "nchw"),     # 68.2, 46.7
])
def test_window_layers_of_few_pixels_keep_the_packed_filter_kernel(shape, dtype, fmt):
    name = picks(shape, dtype, fmt)[0]
    assert name.startswith("pwin_") and "_big_" not in name, name


@pytest.mark.parametrize("fmt,prefix", [("nchw", "bwin_bf16_3x3_M64N512"), ("packed", "pwin_big_bf16_3x3_M64N512")])
def test_window_layers_of_many_pixels_go_to_the_many_pixel_kernel(fmt, prefix):
    name = picks(ConvShape(64, 64, 56, 56, 192, 3, 3, 1, 1), wl.BF16, fmt)[0]  # us: 51 (47), of the packed-filter kernel 105 (84)
    assert name.startswith(prefix), name


# many-pixel layers on the plain formats, input copied or read as it is: us copied, as it is
@pytest.mark.parametrize("shape,dtype,uncopied", [
    (ConvShape(1012, 32, 16, 16, 64, 3, 3, 1, 1), wl.BF16, True),   # 24.0, 18.6
    (ConvShape(475, 32, 28, 28, 64, 3, 3, 1, 1), wl.BF16, True),    # 30.6, 25.8
    (ConvShape(33, 256, 24, 24, 192, 3, 3, 1, 1), wl.F16, True),    # 27.9, 24.7
    (ConvShape(25, 128, 40, 40, 64, 5, 5, 1, 2), wl.BF16, True),    # 28.2, 25.7
    (ConvShape(66, 16, 56, 56, 256, 3, 3, 1, 1), wl.F16, False),    # 33.2, 36.3: one chunk of channels
    (ConvShape(40, 16, 40, 40, 256, 3, 3, 1, 1), wl.BF16, False),   # 14.5, 15.3
    (ConvShape(47, 18, 49, 49, 336, 3, 3, 1, 1), wl.BF16, False),   # 43, 50: rows of 98 bytes
])
def test_many_pixel_layers_are_copied_where_that_is_faster(shape, dtype, uncopied):
    name = picks(shape, dtype)[0]
    assert name.startswith("bwin_") and name.endswith("_p") == uncopied, name


# layers on either side of 32 MiB of input, which nothing in these kernels depends on: us of the one-launch kernel with one image more, of
# the window kernel that was taken there while the other was held back behind that line
@pytest.mark.parametrize("shape", [
    ConvShape(40, 256, 40, 40, 64, 3, 3, 1, 1),   # 44, 64
    ConvShape(83, 256, 28, 28, 256, 3, 3, 1, 1),  # 124, 214
])
def test_picks_without_a_workspace_do_not_flip_with_one_image_more(shape):
    more = dataclasses.replace(shape, N=shape.N + 1)
    names = [picks(s, wl.F16)[1] for s in (shape, more)]
    assert names[0] == names[1] and names[0].startswith("dwin_"), names


# ... and with one: us of the form that reads the input as it is, of the best one behind a copy, with one image more (and with twice as many)
@pytest.mark.parametrize("shape", [
    ConvShape(83, 64, 56, 56, 192, 3, 3, 1, 1),   # 67, 70 (111, 130)
    ConvShape(83, 256, 28, 28, 256, 3, 3, 1, 1),  # 79, 81 (127, 141)
    ConvShape(167, 128, 28, 28, 128, 3, 3, 1, 1),  # 45, 51 (70, 87)
    ConvShape(668, 32, 28, 28, 64, 3, 3, 1, 1),   # 33, 38 (56, 72)
    ConvShape(113, 256, 24, 24, 192, 3, 3, 1, 1),  # 61, 66 (97, 112)
    ConvShape(81, 128, 40, 40, 64, 5, 5, 1, 2),   # 64, 65 (91, 105)
])
def test_picks_with_a_workspace_do_not_flip_with_one_image_more(shape):
    for N in (shape.N, shape.N + 1, 2 * shape.N):
        name = picks(dataclasses.replace(shape, N=N), wl.BF16)[0]
        assert name.startswith("bwin_") and name.endswith("_p"), (N, name)


def test_large_layers_read_as_they_are_fit_the_static_scratch():
    d = B.desc_of(ConvShape(96, 64, 56, 56, 192, 3, 3, 1, 1), wl.BF16, relu=True)
    names = [B.conv_variant_name(d, i) for i in range(B.conv_variant_count(d))]
    assert B.conv_variant_workspace(d, names.index(B.conv_variant_name(d, -1))) <= 1 << 20 < B.CONV_STATIC_SCRATCH_BYTES


# us of the one-launch kernel, of the kernels behind a conversion launch
@pytest.mark.parametrize("shape", [
    ConvShape(40, 128, 64, 56, 32, 3, 3, 1, 1),  # 25, 31
    ConvShape(39, 944, 28, 26, 10, 3, 3, 1, 1),  # 44, 57
])
def test_layers_with_large_inputs_go_to_the_one_launch_kernel_where_it_is_faster(shape):
    assert all(name.startswith("dwin_") for name in picks(shape, wl.BF16)), picks(shape, wl.BF16)


# 5x5 layers of many pixels: us of the kernel behind a conversion launch, of the one-launch kernel
@pytest.mark.parametrize("shape,dtype", [
    (ConvShape(97, 600, 30, 30, 16, 5, 5, 1, 2), wl.BF16),   # 131, 155
    (ConvShape(83, 160, 45, 43, 16, 5, 5, 1, 2), wl.F16),    # 62, 73
    (ConvShape(156, 192, 32, 30, 16, 5, 5, 1, 2), wl.F16),   # 70, 82
])
def test_5x5_layers_of_many_pixels_keep_the_many_pixel_kernel(shape, dtype):
    assert picks(shape, dtype)[0].startswith("bwin_"), picks(shape, dtype)


# ... unless their filters' channels fill no groups of 16
@pytest.mark.parametrize("shape", [
    ConvShape(6, 61, 19, 22, 448, 5, 5, 1, 2),   # 20, 15
    ConvShape(29, 68, 17, 17, 112, 5, 5, 1, 2),  # 21, 16
])
def test_5x5_layers_of_ragged_channels_go_to_the_one_launch_kernel(shape):
    assert picks(shape, wl.F16)[0].startswith("dwin_"), picks(shape, wl.F16)


def test_a_last_round_is_rated_by_its_fullest_cu():
    # 560 workgroups of 64 x 128 outputs, three to a CU on 48 of 256 CUs: 20.4 us; tiles of 32 x 128 16.6
    name = picks(ConvShape(63, 64, 32, 35, 56, 3, 3, 1, 1), wl.F16)[0]
    assert name.startswith("dwin_f16_3x3_M32N128"), name


# channel-innermost layers, with (-1) or without (-2) a workspace: us of the gathering kernel, of the one-launch window kernel (or of the
# tile of it) that was taken
@pytest.mark.parametrize("shape,dtype,which,slow", [
    (ConvShape(29, 480, 20, 23, 48, 3, 3, 2, 1), wl.BF16, -1, "nhwc_dwin_"),                # 14.1, 19.6
    (ConvShape(3, 256, 16, 19, 248, 3, 3, 2, 1), wl.BF16, -1, "nhwc_dwin_bf16_3x3_M64N64"),  # 9.1, 11.2
    (ConvShape(56, 16, 37, 37, 48, 3, 3, 1, 1), wl.F16, -2, "nhwc_dwin_f16_3x3_M32N"),      # 10.1, 11.7
    (ConvShape(1, 104, 56, 59, 352, 3, 3, 2, 1), wl.BF16, -2, "nhwc_dwin_bf16_3x3_M128"),   # 8.4, 11.6
])
def test_channel_innermost_layers_keep_the_faster_kernel(shape, dtype, which, slow):
    d = B.desc_of(shape, dtype, relu=True, in_nhwc=True, out_nhwc=True, filt_krsc=True)
    assert not B.conv_variant_name(d, which).startswith(slow), B.conv_variant_name(d, which)


# fp32 first layers: us of the gather kernels' best, of the kernel on split products
@pytest.mark.parametrize("N,R,split", [
    (1, 11, False),  # 11.3, 17.4
    (2, 11, False),  # 14.8, 17.8
    (5, 11, True),   # 19.3, 18.3
    (12, 11, True),  # 38.7, 27.2
    (1, 7, False),   # 9.6, 11.7
    (4, 7, True),    # 19.0, 15.1
    (8, 7, True),    # 30.7, 23.3
])
def test_first_layers_go_to_split_products_where_they_are_faster(N, R, split):
    shape = ConvShape(N, 3, 227, 227, 96, 11, 11, 4, 0) if R == 11 else ConvShape(N, 3, 224, 224, 64, 7, 7, 2, 3)
    name, nows = picks(shape, wl.F32)
    assert name.startswith("swins_") == split, name
    assert not nows.startswith("swins_"), nows


# fp32 3x3 layers with a workspace: us of the fp32 Winograd kernels' best (of the fastest kernel without a transform, where that one was taken), of
# Winograd on split products
@pytest.mark.parametrize("shape,split", [
    (ConvShape(64, 64, 56, 56, 64, 3, 3, 1, 1), True),     # 127, 72
    (ConvShape(64, 64, 56, 56, 128, 3, 3, 1, 1), True),    # 232, 127
    (ConvShape(64, 64, 56, 56, 192, 3, 3, 1, 1), True),    # 337, 166
    (ConvShape(16, 128, 28, 28, 256, 3, 3, 1, 1), True),   # 58, 40
    (ConvShape(8, 96, 40, 40, 100, 3, 3, 1, 1), True),     # 26, 21
    (ConvShape(20, 256, 13, 13, 384, 3, 3, 1, 1), True),   # 45, 35
    (ConvShape(79, 64, 17, 12, 384, 3, 3, 1, 1), True),    # 88 (no transform), 41
    (ConvShape(16, 24, 55, 50, 24, 3, 3, 1, 1), False),    # 12.9, 20.7
    (ConvShape(4, 24, 21, 21, 384, 3, 3, 1, 1), False),    # 8.4, 14.1
    (ConvShape(42, 16, 22, 22, 17, 3, 3, 1, 1), False),    # 7.1, 11.7
])
def test_3x3_layers_go_to_split_products_where_they_are_faster(shape, split):
    name, nows = picks(shape, wl.F32)
    assert name.startswith("winos_" if split else "wino_"), name
    assert not nows.startswith("winos_"), nows


# fp32 5x5 and strided 3x3 layers with a workspace: us of the fastest other kernel (or of the one that was taken), of the direct kernel on split products
@pytest.mark.parametrize("shape,direct", [
    (ConvShape(43, 160, 6, 9, 32, 5, 5, 1, 2), True),      # 31.1, 18.8: taken with a start above zero for this form
    (ConvShape(17, 160, 9, 7, 32, 5, 5, 1, 2), True),      # 31.3, 18.7: ... and this
    (ConvShape(1, 160, 17, 20, 49, 5, 5, 1, 2), True),     # 31.2, 21.1: ... and this
    (ConvShape(50, 424, 14, 14, 96, 5, 5, 1, 2), True),    # 234, 115
    (ConvShape(36, 32, 41, 39, 49, 5, 5, 1, 2), True),     # 63, 35
    (ConvShape(4, 496, 7, 10, 104, 5, 5, 1, 2), True),     # 55, 41
    (ConvShape(13, 112, 35, 33, 352, 3, 3, 2, 1), True),   # 41, 37
    (ConvShape(16, 19, 10, 13, 32, 3, 3, 2, 1), False),    # 7.0, 8.7
    (ConvShape(5, 440, 18, 18, 112, 3, 3, 2, 1), False),   # 21.7, 32.7
    (ConvShape(2, 432, 41, 41, 48, 3, 3, 2, 1), False),    # 21.3, 41.2
    (ConvShape(1, 432, 64, 62, 48, 5, 5, 1, 2), False),    # 69, 125
    (ConvShape(1, 16, 23, 23, 352, 5, 5, 1, 2), False),    # 6.1, 10.6
])
def test_5x5_and_strided_layers_go_to_the_direct_kernel_where_it_is_faster(shape, direct):
    name, nows = picks(shape, wl.F32)
    assert name.startswith("sdir_") == direct, name
    assert not nows.startswith(("sdir_", "winos_")), nows


# split Winograd by 64 channels x 64 tiles, a row of planes per wave, or by fewer: us of the best of either
@pytest.mark.parametrize("shape,wide", [
    (ConvShape(64, 64, 56, 56, 192, 3, 3, 1, 1), True),    # 160, 182
    (ConvShape(16, 128, 28, 28, 256, 3, 3, 1, 1), True),   # 34.4, 40.6
    (ConvShape(23, 128, 28, 28, 128, 3, 3, 1, 1), True),   # 30.0, 38.8
    (ConvShape(27, 128, 28, 28, 64, 3, 3, 1, 1), True),    # 20.7, 23.2: 83 halved tiles
    (ConvShape(8, 64, 56, 56, 64, 3, 3, 1, 1), True),      # 16.0, 17.6
    (ConvShape(19, 128, 28, 28, 128, 3, 3, 1, 1), True),   # 23.3, 25.6
    (ConvShape(4, 64, 33, 33, 304, 3, 3, 1, 1), True),     # 18.2, 20.5
    (ConvShape(17, 256, 13, 13, 384, 3, 3, 1, 1), False),  # 37.0, 34.1
    (ConvShape(20, 256, 13, 13, 384, 3, 3, 1, 1), False),  # 36.6, 35.1
    (ConvShape(13, 128, 14, 14, 384, 3, 3, 1, 1), False),  # 25.0, 19.7
])
def test_many_tiles_of_split_winograd_go_to_the_row_of_planes_kernel(shape, wide):
    name, nows = picks(shape, wl.F32)
    assert name.startswith("winos_") and name.startswith("winos_f32_M64T64_") == wide, name
    assert not nows.startswith(("sdir_", "winos_")), nows
