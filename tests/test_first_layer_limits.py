"""Which fp32 first layers the kernels on split products accept at the upper end of the library's range (CPU only: the checks are host
code).  Their addresses are 32-bit sums; a layer past what those hold stays with the other kernels."""
import pytest

from paper_1611_06945_amd import binding as B
from paper_1611_06945_amd import workloads as wl
from paper_1611_06945_amd.workloads import ConvShape


def split_variants(shape):
    """Workspace of each kernel on split products that takes the layer, by its tile."""
    d = B.desc_of(shape, wl.F32, relu=True)
    names = [B.conv_variant_name(d, i) for i in range(B.conv_variant_count(d))]
    assert any(not n.startswith("swins_") for n in names), shape  # whoever refuses it, somebody serves it
    mine = {n.split("_")[-1]: B.conv_variant_workspace(d, i) for i, n in enumerate(names) if n.startswith("swins_")}
    assert mine or not B.conv_variant_name(d, -1).startswith("swins_")
    return mine


# past 4 GiB of split filters a 32-bit size is a small number again
@pytest.mark.parametrize("shape", [ConvShape(1, 3, 71, 71, 1740000, 11, 11, 4, 0), ConvShape(1, 3, 13, 13, 4100000, 7, 7, 2, 0)])
def test_split_filters_past_4_gib_are_refused(shape):
    assert not split_variants(shape)


# 3 KB per 32 filters and step (26 steps at 11x11, 11 at 7x7), and a tile's spare blocks behind the last one, stay below 2 GiB
@pytest.mark.parametrize("H,R,stride,steps,tm", [(71, 11, 4, 26, 96), (71, 11, 4, 26, 32), (13, 7, 2, 11, 64), (13, 7, 2, 11, 32)])
def test_split_filters_stay_within_32_bit_offsets(H, R, stride, steps, tm):
    blocks = ((1 << 31) - 1) // (steps * 3072) - tm // 32  # the most that fit
    name = "M%dN256" % tm
    assert split_variants(ConvShape(1, 3, H, H, blocks * 32, R, R, stride, 0))[name] == blocks * steps * 3072
    assert name not in split_variants(ConvShape(1, 3, H, H, blocks * 32 + 1, R, R, stride, 0))


# a store of a channel that does not exist has to miss the output: 2 GiB plus the offset of its row must not pass 4 GiB
@pytest.mark.parametrize("N,H,K,R,stride,pad,tm", [
    (1828, 227, 97, 11, 4, 0, 96),  # one channel of the last tile exists, 95 do not
    (613, 227, 289, 11, 4, 0, 32),
    (657, 224, 65, 7, 2, 3, 64),
    (1295, 224, 33, 7, 2, 3, 32),
])
def test_spare_channels_of_the_last_tile_stay_out_of_range(N, H, K, R, stride, pad, tm):
    inside, beyond = ConvShape(N, 3, H, H, K, R, R, stride, pad), ConvShape(N + 1, 3, H, H, K, R, R, stride, pad)
    plane, lim = 4 * inside.OH * inside.OW, 1 << 31
    assert (N * K + tm) * plane < lim <= ((N + 1) * K + tm) * plane and (N + 1) * K * plane < lim
    assert "M%dN256" % tm in split_variants(inside)
    assert "M%dN256" % tm not in split_variants(beyond)
