"""Host side of the fp32 window kernels on split products (CPU only): how the row-of-planes Winograd kernel deals its tiles, which layers
either kernel accepts at the upper end of the library's range, which of the direct kernel's forms the GPU tests reach, and what the benchmark
rates kernels on split products by."""
import re
import subprocess

import pytest

from paper_1611_06945_amd import binding as B
from paper_1611_06945_amd import build
from paper_1611_06945_amd import workloads as wl
from paper_1611_06945_amd.workloads import ConvShape

DEAL = r"""
#include <cstdio>
#include <vector>
#include "winow_deal.h"
using namespace convfwd;

// longest chain of a workgroup in halves of a tile, every tile done once (a whole, or its two halves); -1 where that does not hold
static int chain(int tiles)
{
    const int grid = winow_grid(tiles);
    std::vector<int> done(2 * tiles, 0);
    int longest = 0;
    if (grid < 1 || grid > 256) return -1;
    for (int b = 0; b < grid; ++b) {
        const WinowShare s = winow_share(tiles, grid, b & 7);
        int q = b >> 3, mine = 0;
        const int whole = s.halved ? s.full : s.count;
        for (; q < whole; q += s.wgs, mine += 2) ++done[2 * (s.first + q)], ++done[2 * (s.first + q) + 1];
        if (q < s.units) ++done[2 * s.first + s.full + q], ++mine;
        if (mine > longest) longest = mine;
    }
    for (int n : done) if (n != 1) return -1;
    return longest;
}

int main()
{
    for (int t = 1; t <= 4100; ++t) printf("%d\n", chain(t));
}
"""


def test_few_tiles_are_halved_on_every_xcd(tmp_path):
    """A last round of at most 128 tiles is of halves, whatever their number, as the ratings have it; ahead of it 256 a round."""
    src, exe = tmp_path / "deal.cpp", tmp_path / "deal"
    src.write_text(DEAL)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", build.CSRC, "-o", str(exe), str(src)])
    chains = [int(x) for x in subprocess.check_output([str(exe)], text=True).split()]
    for tiles, halves in enumerate(chains, 1):
        rest = tiles % 256
        assert halves == 2 * (tiles // 256) + (0 if rest == 0 else 1 if rest <= 128 else 2), (tiles, halves)


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


def test_parity_shapes_reach_every_form_of_the_direct_kernel():
    """Each form runs a layer of two rounds of channels and more, and one whose last round leaves some of its waves without channels."""
    from test_gpu_sdir import SHAPES

    rounds, ragged = {}, set()
    for s in SHAPES:
        for n in forms(s, "sdir_"):
            split, chunks = int(re.search(r"k(\d+)_s", n).group(1)), -(-s.C // 16)
            rounds[n] = max(rounds.get(n, 0), -(-chunks // split))
            if chunks > split and chunks % split:
                ragged.add(n)
    assert len(rounds) == 14 and min(rounds.values()) >= 2, rounds
    assert ragged == {n for n in rounds if "k1_" not in n}, set(rounds) - ragged


@pytest.mark.parametrize("variant,shape,executed", [
    ("sdir_f32_5x5_M32N64_w2k2_s384", ConvShape(50, 424, 14, 14, 96, 5, 5, 1, 2), 12.0 * 96 * 9856 * 432 * 25),
    ("sdir_f32_3x3_M64N128_w4k1_s768", ConvShape(13, 112, 35, 33, 352, 3, 3, 2, 1), 12.0 * 384 * 4096 * 112 * 9),
    ("swins_f32_11x11s4_c3_M96N256", ConvShape(20, 3, 227, 227, 96, 11, 11, 4, 0), 12.0 * 96 * 20 * 3072 * 416),
    ("swins_f32_7x7s2_c3_M64N256", ConvShape(20, 3, 224, 224, 64, 7, 7, 2, 3), 12.0 * 64 * 20 * 12544 * 176),
    ("winos_f32_M64T64_p768", ConvShape(64, 64, 56, 56, 192, 3, 3, 1, 1), 12.0 * 16 * 192 * 50176 * 64),
])
def test_bench_rates_split_products_as_six_bf16_products(variant, shape, executed):
    import bench

    assert variant in names_of(shape)
    assert bench.executed_mfma_flops(variant, shape) == executed and bench.mfma_dtype(variant, "f32") == "bf16"
