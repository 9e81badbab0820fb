"""Which 3x3 convolutions the resident-row kernel takes: the dispatch rule, compiled for the host and asked (no GPU).

The shapes are ones timed in both kernels (us alone, gathering kernel and resident rows); the rule must send each to the faster
one.  Results do not depend on it: both kernels add in the same order.
"""
import os
import subprocess

import pytest

import workloads as wl
from paper_2111_10672_amd.build import hipcc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "conv3_impl.h"
using namespace spb;
int main() {
  int n, image, cin, cout, transposed;
  while (std::scanf("%d %d %d %d %d", &n, &image, &cin, &cout, &transposed) == 5) {
    GemmProblem g;   // cin, cout: of the product; an input gradient gathers the output's gradient
    g.dtype = DType::BF16; g.a_layout = Layout::RowK; g.a_gather = Gather::ConvRows;
    g.b_layout = transposed ? Layout::KRow : Layout::RowK; g.b_gather = transposed ? Gather::ConvWeightT : Gather::None;
    ConvGeom& c = g.conv;
    c.n = n; c.sh = c.sw = c.rh = c.rw = image; c.sc = cin; c.r = c.s = 3; c.stride = 1; c.pad = c.pad_w = 1; c.transposed = transposed;
    c.w_cin = cout; c.w_cout = cin;
    g.M = n * image * image; g.N = cout; g.K = 9 * cin; g.lda = g.K; g.ldb = transposed ? cout : g.K; g.ldc = cout;
    const auto t = gemm_dma_detail::conv3_tile(g);
    std::printf("%d:%dx%d\n", (int)gemm_dma_detail::conv3_accepts(g), t.bm, t.bn);
  }
}
"""

# (images, size, channels in, channels out, input gradient), us in the gathering kernel, us in the resident-row kernel
TIMED = [
    ((31, 14, 256, 256, 0), 30, 18), ((64, 14, 256, 256, 1), 43, 26), ((320, 8, 256, 256, 0), 49, 45), ((128, 14, 256, 256, 0), 50, 57),
    ((255, 14, 256, 256, 1), 88, 130), ((63, 32, 256, 256, 0), 80, 114), ((256, 32, 256, 256, 1), 349, 526), ((144, 16, 256, 256, 0), 78, 71),
    ((64, 7, 512, 512, 0), 51, 33), ((128, 7, 512, 512, 1), 76, 56), ((256, 7, 512, 512, 0), 87, 106), ((32, 16, 512, 512, 0), 66, 102),
    ((64, 16, 512, 512, 0), 88, 217), ((256, 16, 512, 512, 1), 290, 635), ((82, 16, 192, 192, 0), 39, 28), ((254, 16, 192, 192, 0), 55, 71),
    ((150, 16, 192, 192, 1), 74, 58), ((122, 14, 384, 384, 0), 83, 119), ((31, 14, 384, 384, 0), 46, 42), ((510, 28, 128, 128, 0), 174, 149),
    ((32, 28, 128, 128, 1), 28, 19), ((128, 56, 128, 128, 0), 185, 234), ((32, 100, 128, 128, 0), 149, 203), ((255, 56, 64, 64, 0), 154, 94),
    ((32, 200, 64, 64, 0), 254, 215), ((2, 200, 64, 64, 0), 25, 30), ((1, 100, 128, 128, 0), 19, 21), ((1000, 16, 256, 64, 0), 137, 123),
    ((512, 8, 128, 512, 1), 53, 57), ((1024, 8, 512, 128, 0), 98, 112), ((32, 16, 64, 256, 1), 13, 11), ((20, 16, 512, 512, 0), 63, 74),
    ((20, 16, 512, 512, 1), 72, 64),
]


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("conv3_rule")
    src, exe = d / "rule.hip", d / "rule"
    src.write_text(PROGRAM)
    subprocess.run([hipcc(), "-std=c++17", "--offload-host-only", "-I" + os.path.join(ROOT, "paper_2111_10672_amd", "csrc"),
                    "-I" + os.path.join(ROOT, "include"), str(src), "-o", str(exe)], check=True, capture_output=True, text=True)

    def run(shapes):
        out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, s)) for s in shapes), check=True, capture_output=True, text=True).stdout
        return [line.split(":") for line in out.split()]
    return run


@pytest.fixture(scope="module")
def accepts(ask):
    return lambda shapes: [taken == "1" for taken, _ in ask(shapes)]


def test_each_timed_shape_goes_to_the_faster_kernel(accepts):
    got = accepts([s for s, _, _ in TIMED])
    wrong = [(s, g, r) for (s, g, r), resident in zip(TIMED, got) if resident != (r < g)]
    assert len(got) == len(TIMED) and not wrong, wrong


def test_what_the_kernel_does_not_hold_stays_refused(accepts):
    # channels that are not whole 64-groups; a row too wide for the patch of the smallest tile
    assert accepts([(8, 14, 96, 96, 0), (8, 14, 32, 64, 1), (1, 255, 512, 512, 0), (2, 40, 512, 512, 1)]) == [False] * 4


# The configurations that run each large tile with a part-filled last one.
@pytest.mark.parametrize("name,block,tile", [
    ("odd_tiles_128x64_resnet_basic_bf16", 0, "128x64"), ("odd_tiles_stride2_resnet_basic_bf16", 0, "128x64"),
    ("odd_tiles_stride2_resnet_basic_bf16", 1, "128x64"), ("odd_tiles_256x64_resnet_basic_bf16", 0, "256x64"),
    ("odd_tiles_128x128_resnet_basic_bf16", 0, "128x128"), ("odd_tiles_64x128_resnet_basic_bf16", 0, "64x128"),
])
def test_configurations_of_part_filled_tiles(ask, name, block, tile):
    cfg = wl.get_config(name)
    b = wl.resnet_layout(cfg)["blocks"][block]
    shape, width = b["out_hw"][0], b["cout"]
    assert cfg["batch"] * shape * shape % int(tile.split("x")[0])
    assert ask([(cfg["batch"], shape, width, width, t) for t in (0, 1)]) == [["1", tile]] * 2
