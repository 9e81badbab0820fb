"""A product that is asked for the row sums of A goes to a kernel that forms them, or is refused: libspb.so's dispatch on the
stand-in for the HIP runtime (fake_hip.cpp), no GPU."""
import os
import subprocess

import pytest

import paper_2111_10672_amd
from paper_2111_10672_amd.build import hipcc

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PACKAGE = os.path.dirname(os.path.abspath(paper_2111_10672_amd.__file__))

PROGRAM = r"""
#include <cstdio>
#include "kernels.h"
using namespace spb;
extern "C" { const char* fake_log(); void fake_clear(); }
int main() {
  char kind[16];
  int sums;
  while (std::scanf("%15s %d", kind, &sums) == 2) {
    void* const at = reinterpret_cast<void*>(4096);   // (an address that nothing reads)
    GemmProblem g;
    g.dtype = kind[0] == 'f' ? DType::F32 : DType::BF16;
    g.epilogue = Epilogue::StoreF32;
    g.A = g.B = g.C = at;
    if (sums) g.a_row_sum = static_cast<float*>(at);
    if (kind[1] == 'c') {         // weight gradient of a convolution, 5x5 over 16 x 16 pixels
      ConvGeom& c = g.conv;
      c.n = 2; c.sh = c.sw = c.rh = c.rw = 16; c.sc = 8; c.r = c.s = 5; c.stride = 1; c.pad = c.pad_w = 2;
      g.a_layout = g.b_layout = Layout::KRow; g.b_gather = Gather::ConvPatchT;
      g.M = 64; g.N = 200; g.K = 512; g.lda = 64; g.ldb = 200; g.ldc = 200;
    } else if (kind[1] == 'k') {  // weight gradient of a dense layer
      g.a_layout = g.b_layout = Layout::KRow;
      g.M = 64; g.N = 256; g.K = 784; g.lda = 64; g.ldb = 256; g.ldc = 256;
    } else {                      // forward
      g.a_layout = g.b_layout = Layout::RowK;
      g.M = 64; g.N = 256; g.K = 784; g.lda = g.ldb = 784; g.ldc = 256;
    }
    fake_clear();
    const int e = (int)launch_gemm(g, nullptr);
    std::printf("%d %s\n", e, e ? "-" : fake_log());
  }
}
"""


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    d = tmp_path_factory.mktemp("row_sum_routes")
    runtime, src, exe = d / "libamdhip64.so.7", d / "ask.hip", d / "ask"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-Wl,-soname,libamdhip64.so.7", os.path.join(HERE, "fake_hip.cpp"), "-o", str(runtime)],
                   check=True)
    subprocess.run([hipcc(), "-std=c++17", "--offload-host-only", "-I" + os.path.join(PACKAGE, "csrc"), "-I" + os.path.join(ROOT, "include"), str(src),
                    "-Wl," + os.path.join(PACKAGE, "libspb.so"), "-Wl," + str(runtime), "-Wl,-rpath," + PACKAGE, "-Wl,--allow-shlib-undefined",
                    "-o", str(exe)], check=True, capture_output=True, text=True)

    def ask(kind, sums):
        env = dict(os.environ, LD_LIBRARY_PATH=str(d))
        return subprocess.run([str(exe)], input=f"{kind} {sums}", env=env, check=True, capture_output=True, text=True).stdout.split(None, 1)
    return ask


@pytest.mark.parametrize("kind,plain,with_sums", [
    ("ff", "gemm_f32_tiny_kernel", "gemm_f32_small_kernel"), ("fk", "gemm_f32_small_kernel", "gemm_f32_small_kernel"),
    ("bf", "gemm_bf16_", "gemm_kernel"), ("bk", "gemm_bf16_", "gemm_bf16_"), ("bc", "gemm_bf16_", None)])
def test_row_sums_are_formed_or_refused(route, kind, plain, with_sums):
    error, kernel = route(kind, 0)
    assert error == "0" and plain in kernel, kernel
    error, kernel = route(kind, 1)
    assert error == "1" if with_sums is None else error == "0" and with_sums in kernel, (error, kernel)
