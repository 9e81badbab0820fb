"""Which small products take 32 x 64 tiles and which 64 x 64: the rule, compiled for the host and asked (no GPU).

The shapes are ones timed in both (us, alone); the rule must give each the faster tile.  Results do not depend on it: both sum the
same quarters of k in the same order.
"""
import os
import subprocess

import pytest

from paper_2111_10672_amd.build import hipcc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "gemm_dma_impl.h"
using namespace spb;
int main() {
  int kind, beside;
  GemmProblem g;
  g.dtype = DType::BF16;
  while (std::scanf("%d %d %d %d %d", &kind, &g.M, &g.N, &g.K, &beside) == 5) {
    g.a_layout = kind ? Layout::KRow : Layout::RowK;   // weight gradient or forward
    g.b_layout = g.a_layout;
    g.beside = beside;
    std::printf("%d\n", gemm_dma_detail::small_product_fits(g) && gemm_dma_detail::small_product_tile64(g) && gemm_dma_detail::small_product_rows32(g));
  }
}
"""

# (weight gradient, rows, columns, k), us in 32 x 64 tiles, us in 64 x 64
TIMED = [
    ((0, 504, 768, 768), 6.1, 7.1), ((0, 1000, 333, 3128), 15.3, 19.1), ((0, 2804, 127, 3128), 15.5, 20.6), ((0, 333, 768, 2048), 8.9, 10.2),
    ((0, 504, 1000, 4096), 12.9, 15.6), ((0, 333, 768, 3128), 16.0, 13.1), ((0, 343, 1280, 3240), 16.9, 13.4), ((0, 324, 752, 3568), 16.6, 13.7),
    ((0, 341, 1232, 3512), 18.2, 15.1), ((0, 473, 865, 2032), 13.7, 10.8),
    ((1, 127, 3128, 504), 5.7, 6.6), ((1, 127, 3128, 768), 8.4, 7.4), ((1, 127, 3128, 2804), 22.1, 16.1), ((1, 100, 3128, 8192), 56.8, 41.8),
    ((1, 122, 3624, 7358), 57.1, 34.8), ((1, 128, 4008, 4503), 39.9, 26.1), ((1, 97, 3464, 7841), 60.3, 41.8), ((1, 100, 4096, 2804), 11.9, 13.8),
    ((1, 333, 1336, 8192), 37.9, 43.0), ((1, 500, 768, 4096), 16.6, 20.0), ((1, 1000, 512, 2804), 13.9, 16.6), ((1, 200, 1336, 1500), 10.7, 11.7),
]


@pytest.fixture(scope="module")
def takes32(tmp_path_factory):
    d = tmp_path_factory.mktemp("small_tile_rule")
    src, exe = d / "rule.hip", d / "rule"
    src.write_text(PROGRAM)
    subprocess.run([hipcc(), "-std=c++17", "--offload-host-only", "-I" + os.path.join(ROOT, "paper_2111_10672_amd", "csrc"),
                    "-I" + os.path.join(ROOT, "include"), str(src), "-o", str(exe)], check=True, capture_output=True, text=True)

    def ask(shapes, beside):
        out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, s)) + f" {beside}" for s in shapes), check=True, capture_output=True, text=True).stdout
        return [line == "1" for line in out.split()]
    return ask


def test_each_timed_shape_gets_the_faster_tile(takes32):
    got = takes32([s for s, _, _ in TIMED], 0)
    wrong = [(s, a, b) for (s, a, b), rows32 in zip(TIMED, got) if rows32 != (a < b)]
    assert len(got) == len(TIMED) and not wrong, wrong


# The encoder's weight gradients share the chip with its input-gradient chain, and more workgroups are worse for the step.
def test_products_beside_another_chain_keep_the_fewer_workgroups(takes32):
    assert not any(takes32([(1, 896, 448, 1600), (1, 320, 1280, 3080), (1, 768, 512, 2048)], 1))
