"""Lanes of one wave that exchange values through LDS come together between the parts of the exchange (no GPU).

LDS operations of a wave complete in order, so these exchanges need no wait; but without a convergent operation between
writing and reading the compiler may run lanes that take no part in a later store ahead of the others or behind them, which gave
wrong rows once.  Results show that only where it happens, so this asks the compiled code of every such kernel: between
the last write of a part and the first read of the next it has a wave barrier (a mark, not an instruction).
"""
import os
import re
import subprocess

import pytest

from paper_2111_10672_amd.build import FLAGS, hipcc

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2111_10672_amd", "csrc")

# one 32-row piece per wave: a tile of a convolution over resident rows, one of the gathering kernels
TILES = r"""
#include "conv3_impl.h"
namespace spb { namespace gemm_dma_detail {
template __global__ void conv3_kernel<64, 64, 4, 2, 2, 3, Layout::RowK>(GemmParams, int);
template __global__ void gemm_bf16_dma_kernel<128, 64, 3, 4, 1, Layout::RowK, Layout::RowK, Gather::None, Gather::None>(GemmParams);
} }
"""

# source (None: the tiles above), kernel, wave barriers at least: what its exchanges have, once each
KERNELS = [
    (None, "conv3_kernel", 2), (None, "gemm_bf16_dma_kernel", 2),
    ("attention.hip", "attention_fwd_kernel", 3), ("attention.hip", "attention_bwd_kernel", 9),
    ("attention_rows.hip", "attention_rows_fwd_kernel", 4), ("attention_rows.hip", "attention_rows_bwd_kernel", 4),
    ("conv3_wgrad.hip", "conv3_wgrad_kernel", 10),
]


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    d = tmp_path_factory.mktemp("wave_exchange")
    (d / "tiles.hip").write_text(TILES)
    runs = {}
    for source in sorted({s or "" for s, _, _ in KERNELS}):
        path = os.path.join(CSRC, source) if source else str(d / "tiles.hip")
        out = d / ((source or "tiles") + ".s")
        runs[source] = (out, subprocess.Popen([hipcc(), *FLAGS, "-I" + CSRC, "-S", "--offload-device-only", path, "-o", str(out)],
                                              stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL))
    text = {}
    for source, (out, run) in runs.items():
        assert run.wait() == 0, source
        text[source] = out.read_text()
    return text


def _functions(text, kernel):
    """The bodies of the kernels of that name (every instance of a template)."""
    return [body for name, body in re.findall(r"^(_Z[\w]*):[^\n]*\n(.*?)^\.Lfunc_end", text, re.S | re.M) if kernel in name]


@pytest.mark.parametrize("source,kernel,least", KERNELS)
def test_lanes_come_together_between_the_parts_of_an_exchange(assembly, source, kernel, least):
    bodies = _functions(assembly[source or ""], kernel)
    assert bodies
    for body in bodies:
        assert body.count("wave barrier") >= least
