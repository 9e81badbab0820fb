// Input gradient of a convolution of stride 2 (or its 1 x 1 projection) without the taps that meet no output.
//
// Output pixel (p, q) is read by input pixel (a, b) through tap (r, s) where 2 p = a + pad - r and 2 q = b + pad - s: only taps of the
// pixel's own parity contribute, a quarter of them all told (3 x 3: 4, 2, 2 or 1 of 9).  The gathering product over all taps multiplies
// zeros for the others.  Here the input pixels are taken class by class, the four (a mod 2, b mod 2), each class a product of its own
// over its own taps (stride 1 inside the class), all four in one launch, the one with most taps first; the rows of a
// class lie two apart in the result, so the epilogue takes them from a table.  What is left out are zeros: same bits.
// 128 channels from 28 x 28 to 56 x 56 pixels, batch 64, in the step: 129 -> 61 us; what is left is the epilogue's traffic (three tensors
// read, one written) more than the taps.  Steps: 32-pixel basic CNN 1410 -> 1291 us, 224-pixel bottleneck CNN 5290 -> 5029.
#include <algorithm>

#include "gemm_dma_impl.h"

namespace spb {
namespace gemm_dma_detail {

struct Stride2Class {
  ConvGeom conv;             // rows: the class's pixels; gathered: the output gradient; r x s: the class's taps
  int M, tiles_m;
  int first_block;           // of the launch
  int first_row;             // tile rows of the classes before it
  int tap_r, tap_s;          // the class's first tap in the whole kernel; the next ones are two further
  int at_r, at_s;            // parity of its pixels
};
struct Stride2Classes {
  Stride2Class c[4];
  int height, width;         // of the input
  int taps, taps_w;          // of the whole kernel
};

template <int BM, int BN, int STAGES, int WAVES_M, int WAVES_N>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void conv_stride2_dgrad_kernel(GemmParams p, Stride2Classes k) {
  constexpr int NW = WAVES_M * WAVES_N;
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N, TM = WM / 32, TN = WN / 32;
  constexpr int kStageBytes = (BM + BN) * kRowBytes;
  constexpr int kLoadsPerTile = (BM + BN) / (8 * NW);
  constexpr int kBatch = (TM + TN) <= 2 ? 4 : ((TM + TN) <= 4 ? 2 : 1);
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  int* rows = reinterpret_cast<int*>(lds + STAGES * kStageBytes);

  int which = 0;
#pragma unroll
  for (int c = 1; c < 4; ++c)
    if ((int)blockIdx.x >= k.c[c].first_block) which = c;
  const Stride2Class cls = k.c[which];
  int tile_m, tile_n;
  xcd_tile_grouped(blockIdx.x - cls.first_block, cls.tiles_m, p.tiles_n, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave % WAVES_M, wn = wave / WAVES_M;

  const int groups = cls.conv.sc / kTileK, n_tiles = cls.conv.r * cls.conv.s * groups;
  TileSource<BM, Layout::RowK, Gather::ConvRows, NW> src_a;
  TileSource<BN, Layout::KRow, Gather::None, NW> src_b;
  src_a.init(static_cast<const bf16_t*>(p.A), 0, m0, cls.M, wave, lane, 0, cls.conv);
  src_b.init(static_cast<const bf16_t*>(p.B), k.taps * p.ldb, n0, p.N, wave, lane, 0, cls.conv);   // weights [co][tap][ci]: a k-row every `taps`
  int group = 0, tap_r = cls.tap_r, tap_s = cls.tap_s;
  auto issue = [&](int t) {
    char* stage = lds + (t % STAGES) * kStageBytes;
    src_a.issue(t, 0, stage, wave, 0, cls.conv);
    src_b.issue_at(src_b.panel + ((size_t)group * kTileK * k.taps + tap_r * k.taps_w + tap_s) * p.ldb * 2, stage + BM * kRowBytes, wave);
    if (++group == groups) {
      group = 0;
      tap_s += 2;
      if (tap_s >= k.taps_w) { tap_s = cls.tap_s; tap_r += 2; }
    }
  };
#pragma unroll
  for (int t = 0; t < STAGES - 1; ++t)
    if (t < n_tiles) issue(t);

  if ((int)threadIdx.x < BM) {   // which pixel a row is
    const int m = m0 + (int)threadIdx.x, per_image = cls.conv.rh * cls.conv.rw;
    const int n = m / per_image, in_image = m - n * per_image, a = in_image / cls.conv.rw, b = in_image - a * cls.conv.rw;
    rows[threadIdx.x] = m < cls.M ? (n * k.height + 2 * a + cls.at_r) * k.width + 2 * b + cls.at_s : -1;
  }

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  for (int t = 0; t < n_tiles; ++t) {
    if (t + STAGES - 2 < n_tiles) wait_loads_and_barrier<(STAGES - 2) * kLoadsPerTile>();
    else wait_loads_and_barrier<0>();
    if (t + STAGES - 1 < n_tiles) issue(t + STAGES - 1);
    const char* as = lds + (t % STAGES) * kStageBytes;
    const char* bs = as + BM * kRowBytes;
#pragma unroll
    for (int kb = 0; kb < 4; kb += kBatch) {
      u32x4 a[kBatch * TM], b[kBatch * TN];
#pragma unroll
      for (int g = 0; g < kBatch; ++g) {
#pragma unroll
        for (int i = 0; i < TM; ++i) a[g * TM + i] = read_fragment_asm<BM, Layout::RowK>(as, wm * WM + i * 32, kb + g, lane);
#pragma unroll
        for (int j = 0; j < TN; ++j) b[g * TN + j] = read_fragment<BN, Layout::KRow>(bs, wn * WN + j * 32, kb + g, lane);
      }
      fragments_ready(a, b);
#pragma unroll
      for (int g = 0; g < kBatch; ++g)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, b[g * TN + j]),
                                                                __builtin_bit_cast(bf16x8, a[g * TM + i]), acc[i][j], 0, 0, 0);
    }
  }
  wait_loads_and_barrier<0>();   // every wave is done with the ring, and the table of rows is there
  float* stage = reinterpret_cast<float*>(lds) + wave * (32 * (WN + 4));
  store_wave_tile<WM, WN, WAVES_M, true>(p, acc, stage, m0 + wm * WM, n0 + wn * WN, lane, 0, wm, cls.first_row + tile_m, rows + wm * WM);
}

namespace {

// The four classes, most taps first, in tiles of bm rows; returns the tile rows of all.
int stride2_classes(const GemmProblem& q, int bm, int tiles_n, Stride2Classes* out, int* blocks) {
  const ConvGeom& c = q.conv;
  out->height = c.rh; out->width = c.rw;
  out->taps = c.r * c.s; out->taps_w = c.s;
  Stride2Class all[4];
  for (int i = 0; i < 4; ++i) {
    Stride2Class& x = all[i];
    x.at_r = i >> 1; x.at_s = i & 1;
    x.tap_r = (x.at_r + c.pad) & 1; x.tap_s = (x.at_s + c.pad_w) & 1;
    x.conv = c;
    x.conv.stride = 1;
    x.conv.rh = (c.rh - x.at_r + 1) / 2; x.conv.rw = (c.rw - x.at_s + 1) / 2;
    x.conv.r = (c.r - x.tap_r + 1) / 2; x.conv.s = (c.s - x.tap_s + 1) / 2;
    x.conv.pad = (x.at_r + c.pad - x.tap_r) / 2; x.conv.pad_w = (x.at_s + c.pad_w - x.tap_s) / 2;
    x.M = c.n * x.conv.rh * x.conv.rw;
    x.tiles_m = (x.M + bm - 1) / bm;
  }
  std::stable_sort(all, all + 4, [](const Stride2Class& a, const Stride2Class& b) { return a.conv.r * a.conv.s > b.conv.r * b.conv.s; });
  int rows = 0;
  *blocks = 0;
  for (int i = 0; i < 4; ++i) {
    all[i].first_block = *blocks; all[i].first_row = rows;
    *blocks += all[i].tiles_m * tiles_n;
    rows += all[i].tiles_m;
    out->c[i] = all[i];
  }
  return rows;
}

template <int BM, int BN, int STAGES, int WAVES_M, int WAVES_N>
hipError_t launch_stride2(const GemmProblem& q, hipStream_t stream) {
  GemmParams p = make_params(q, BM, BN);
  Stride2Classes k;
  int blocks;
  const int tile_rows = stride2_classes(q, BM, p.tiles_n, &k, &blocks);
  if (q.col_partial_rows) *q.col_partial_rows = tile_rows;
  constexpr size_t lds_bytes = (size_t)STAGES * (BM + BN) * kRowBytes + BM * sizeof(int);
  static_assert((size_t)WAVES_M * WAVES_N * 32 * (BN / WAVES_N + 4) * 4 <= (size_t)STAGES * (BM + BN) * kRowBytes, "epilogue staging fits in the tile ring");
  auto kernel = conv_stride2_dgrad_kernel<BM, BN, STAGES, WAVES_M, WAVES_N>;
  if (lds_bytes > 64 * 1024)
    if (hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kernel), lds_bytes); e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, dim3(blocks), dim3(64 * WAVES_M * WAVES_N), lds_bytes, stream, p, k);
  return hipGetLastError();
}

}  // namespace
}  // namespace gemm_dma_detail

// Whole 64-channel groups of the gradient (a tile of k lies on one tap) and whole 16-byte pieces of columns; column sums need room for
// the classes' own last tiles.
bool conv_stride2_dgrad_accepts(const GemmProblem& q) {
  const ConvGeom& c = q.conv;
  return q.a_gather == Gather::ConvRows && q.b_gather == Gather::ConvWeightT && c.transposed && c.stride == 2 && c.sc % gemm_dma_detail::kTileK == 0 &&
         c.w_cout == c.sc && c.w_cin == q.N && q.ldb == q.N && q.N % 8 == 0 && q.M == c.n * c.rh * c.rw && q.k_splits == 1 && q.batch == 1 &&
         (q.epilogue == Epilogue::BiasAct || (q.epilogue == Epilogue::AffineBwdStore && q.col_partial_spare >= 3));
}

// As for the other gathering products: 64-wide tiles for 64 columns; 128 x 128 while that fills the chip; else 64 x 64.
hipError_t launch_conv_stride2_dgrad(const GemmProblem& q, hipStream_t stream) {
  using namespace gemm_dma_detail;
  if (q.N <= 64 && tile_count(q, 128, 64) >= 256) return launch_stride2<128, 64, 3, 4, 1>(q, stream);
  if (q.N > 64 && tile_count(q, 128, 128) >= 256) return launch_stride2<128, 128, 2, 2, 2>(q, stream);
  return launch_stride2<64, 64, 4, 2, 2>(q, stream);
}

}  // namespace spb
