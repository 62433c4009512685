"""Host side of the fp32 window kernels on split products (CPU only): which layers they accept at the upper end of the library's range."""
import pytest

from paper_1611_06945_amd import binding as B
from paper_1611_06945_amd import workloads as wl
from paper_1611_06945_amd.workloads import ConvShape

def names_of(shape):
    d = B.desc_of(shape, wl.F32, relu=True)
    return [B.conv_variant_name(d, i) for i in range(B.conv_variant_count(d))]


def forms(shape, prefix):
    return {n for n in names_of(shape) if n.startswith(prefix)}


def test_launches_of_four_thousand_million_threads_are_refused():
    """One filter, a border much larger than the image: 2^23 tiles of 32 pixels and more, of 512 threads each."""
    def shape(N):
        return ConvShape(N, 8, 1, 1, 1, 5, 5, 1, 4)
    most = ((1 << 23) - 1) * 32 // 25  # images whose 25 outputs each fill fewer than 2^23 tiles
    eight = "sdir_f32_5x5_M32N32_w1k8_s192"
    assert eight in names_of(shape(most))
    assert eight not in names_of(shape(most + 2)) and forms(shape(most + 2), "sdir_") and len(names_of(shape(most + 2))) > 14


# input and 16 (64) spare channels, output and a tile's spare channels below 2 GiB
@pytest.mark.parametrize("prefix,spare", [("sdir_f32_3x3_M32N128", 16), ("winos_f32_M64T64", 64)])
def test_inputs_stay_below_2_gib_with_their_spare_channels(prefix, spare):
    C, H = 64, 56
    most = (((1 << 31) - 1) // (4 * H * H) - spare) // C
    assert forms(ConvShape(most, C, H, H, 40, 3, 3, 1, 1), prefix)
    assert not forms(ConvShape(most + 1, C, H, H, 40, 3, 3, 1, 1), prefix) and names_of(ConvShape(most + 1, C, H, H, 40, 3, 3, 1, 1))


@pytest.mark.parametrize("prefix,spare", [("sdir_f32_3x3_M64N128", 64), ("sdir_f32_5x5_M32N64", 32), ("winos_f32_M64T64", 0)])
def test_outputs_stay_below_2_gib_with_the_spare_channels_of_a_tile(prefix, spare):
    R, K, H = (5 if "5x5" in prefix else 3), 130, 24
    most = (((1 << 31) - 1) // (4 * H * H) - spare) // K
    assert forms(ConvShape(most, 8, H, H, K, R, R, 1, R // 2), prefix)
    assert not forms(ConvShape(most + 1, 8, H, H, K, R, R, 1, R // 2), prefix) and names_of(ConvShape(most + 1, 8, H, H, K, R, R, 1, R // 2))
