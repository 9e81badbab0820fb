"""Which products touch their weights ahead: the rules, compiled for the host and asked (no GPU).

Touching makes the first tile wait for a whole panel of weights.  It pays where those come from HBM and costs where they are
in cache, as a perceptron's are: it took 3 to 7 % of a step of 2048 to 8192 rows of 768 to 2048 features.
"""
import os
import subprocess

import pytest

from paper_2111_10672_amd.build import hipcc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "conv3_impl.h"
using namespace spb;
int main() {
  GemmProblem g;   // a forward product as the models describe it
  g.dtype = DType::BF16; g.a_layout = g.b_layout = Layout::RowK;
  int in_hbm, bm, bn, lone;
  while (std::scanf("%d %d %d %d %d %d %d", &g.M, &g.N, &g.K, &in_hbm, &bm, &bn, &lone) == 7) {
    g.b_in_hbm = in_hbm;
    std::printf("%d\n", gemm_detail::make_params(g, bm, bn).touch_blocks > 0 && gemm_dma_detail::touching_pays(g, bm, bn, lone));
  }
  std::printf("%d %d %d %d\n", weights_driven_out(37000000, 257000000), weights_driven_out(76000000, 257000000), weights_driven_out(96000000, 290000000),
              weights_driven_out(264000000, 1800000000));
}
"""

# (rows, columns, k, weights in HBM, tile, alone on its CU), whether it touches
ASKED = [
    ((8192, 1024, 1024, 0, 128, 128, 0), 0), ((2048, 2048, 2048, 0, 128, 128, 1), 0), ((4096, 2048, 2048, 0, 256, 192, 0), 0), ((8192, 2048, 2048, 0, 256, 256, 1), 0),
    ((8192, 1024, 1024, 1, 128, 128, 0), 1), ((4096, 768, 3072, 1, 128, 128, 1), 1), ((4096, 1024, 1024, 1, 128, 128, 1), 0), ((4096, 1024, 4096, 1, 128, 128, 1), 0),
    ((5160, 896, 896, 1, 128, 128, 0), 0), ((7320, 768, 768, 1, 128, 128, 0), 1),
    ((8192, 512, 512, 1, 128, 128, 1), 1), ((12544, 256, 1024, 1, 128, 128, 1), 1), ((4096, 2304, 768, 1, 256, 192, 0), 1), ((3720, 2304, 768, 1, 256, 192, 0), 0), ((8192, 4096, 1024, 1, 256, 256, 1), 1),
]


@pytest.fixture(scope="module")
def answers(tmp_path_factory):
    d = tmp_path_factory.mktemp("touch_rule")
    src, exe = d / "rule.hip", d / "rule"
    src.write_text(PROGRAM)
    subprocess.run([hipcc(), "-std=c++17", "--offload-host-only", "-I" + os.path.join(ROOT, "paper_2111_10672_amd", "csrc"),
                    "-I" + os.path.join(ROOT, "include"), str(src), "-o", str(exe)], check=True, capture_output=True, text=True)
    return subprocess.run([str(exe)], input="\n".join(" ".join(map(str, a)) for a, _ in ASKED), check=True, capture_output=True, text=True).stdout.split()


def test_only_products_whose_weights_lie_in_hbm_touch_them(answers):
    assert answers[:len(ASKED)] == [str(want) for _, want in ASKED]


def test_steps_that_fit_the_cache_leave_the_weights_there(answers):
    # encoders: 1 and 3 layers of 896 features and 48 x 128 tokens, 3 layers of 1024, 12 of 768 and 32 x 128 with their backward pass
    assert answers[len(ASKED):] == ["0", "0", "1", "1"]
