// 3 x 3 convolutions of stride 1 over whole 64-channel groups, forward and input gradient, as implicit products
//   C[pixel, n] = sum over (tap, channel) of x[pixel + tap][channel] * w(n, tap, channel)
// with the rows of x resident in LDS.
//
// The gathering kernels of gemm_dma_impl.h fetch a tile of x once per tap: nine times the bytes through a CU's vector-memory
// path, with a bounds check and a 64-bit address per 16 bytes, and ring slots for both operands.  But the pixels a tile of BM
// consecutive output pixels reads, over all nine taps, are one stretch of BM + 2 W + 2 pixels of the tensor (image after
// image, row after row).  Here a workgroup fetches that stretch once, whole, and a tap is an offset into it; the lanes whose
// pixel lies outside the image read zeros instead.  What the loop still loads is the weights.
//
// What bounds it (cycles per 64 of k, workgroup alone on its CU): 128 x 128 tiles with eight waves 830, of which 512 are matrix
// work (counted over whole launches, in networks of 32-pixel images, the matrix cores are busy 13 to 16 %); the LDS reads add 190 and the
// weights' loads 110.  64 x 64: 460, of 128.  Around the loop, 4500 cycles until the patch is
// in and 2000 to 4000 for the epilogue.  Measured and dropped: the loads of a tile spread over its k-groups (+20 % a tile: the
// scalar work of four pieces), weights with padded rows (level: no channel conflict), a fourth ring stage where it costs no
// occupancy (level or slower).
//
// The order of k, (tap, channel) ascending in groups of 16, is that of the gathering kernels: same bits.
#pragma once
#include <algorithm>
#include "gemm_dma_impl.h"

namespace spb {
namespace gemm_dma_detail {

// Where 16-byte chunk `chunk` of a patch row lies in its 128 bytes: a tap reads 32 consecutive rows from any first row.
__device__ __forceinline__ int patch_offset(int row, int chunk) { return row * kRowBytes + (((chunk ^ (row ^ (row >> 3 & 1))) & 7) << 4); }

// Rows of the patch (whole 8-row instructions) and the LDS of a workgroup.  256 bytes of zeros follow each group's rows: a lane
// whose pixel lies outside the image reads them at its own place modulo 256, which keeps it in the banks it had.  (One common
// zero row cost 20 % of the LDS cycles in conflicts.)
constexpr int kZeroBytes = 256;
inline int patch_rows(int bm, int width) { return (bm + 2 * width + 2 + 7) / 8 * 8; }
inline size_t conv3_lds(int bm, int bn, int stages, int width, int channels) {
  return (size_t)(channels / kTileK) * ((size_t)patch_rows(bm, width) * kRowBytes + kZeroBytes) + (size_t)stages * bn * kRowBytes + kTouchBytes;
}

// The loop runs k-group by k-group (16 of k: TM x TN matrix instructions a wave).  An LDS read takes longer than a k-group's
// matrix work, so the fragments of the k-group AHEAD steps on are requested while this one is multiplied, in AHEAD + 1 sets
// of registers, and a wave waits until all but the younger AHEAD - 1 k-groups' reads are in (LDS reads return in order).
template <int BM, int BN, int STAGES, int WAVES_M, int WAVES_N, int AHEAD, Layout LB>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void conv3_kernel(GemmParams p, int rows) {
  constexpr int NW = WAVES_M * WAVES_N;
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  constexpr int TM = WM / 32, TN = WN / 32;
  static_assert((NW == 4 || NW == 8) && TM >= 1 && TN >= 1 && WM % 32 == 0 && WN % 32 == 0, "whole 32 x 32 blocks");
  static_assert(AHEAD == 3 || AHEAD == 7, "the sets of registers are those of one tile or two");
  constexpr int kSets = AHEAD + 1, kTiles = kSets / 4;      // tiles per round of the sets
  constexpr int kReads = TM + (LB == Layout::RowK ? TN : 2 * TN);   // LDS instructions per k-group
  static_assert((AHEAD - 1) * kReads <= 15, "the reads in flight are counted in four bits");
  static_assert(STAGES >= 2 + kTiles, "ring depth");
  using SourceB = TileSource<BN, LB, Gather::None, NW>;

  extern __shared__ __attribute__((aligned(1024))) char lds[];
  int tile_m, tile_n;
  xcd_tile_grouped(blockIdx.x, p.tiles_m, p.tiles_n, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave % WAVES_M, wn = wave / WAVES_M;
  const int channels = p.conv.sc, width = p.conv.rw, height = p.conv.rh, groups = channels / kTileK;
  const int group_bytes = rows * kRowBytes + kZeroBytes;
  char* ring = lds + groups * group_bytes;

  if constexpr (LB == Layout::RowK) touch_panel<BN, NW>(p, tile_m, n0, STAGES - 1, ring + STAGES * BN * kRowBytes, wave, lane);
  // ---- the zeros, then the patch: row j is pixel m0 - W - 1 + j (clamped into the tensor: what lies outside is masked)
  for (int g = wave; g < groups; g += NW)
    if (lane < kZeroBytes / 16) *reinterpret_cast<u32x4*>(lds + g * group_bytes + rows * kRowBytes + lane * 16) = u32x4{0u, 0u, 0u, 0u};
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  {
    const int r8 = lane >> 3, pc = lane & 7;
    for (int j = wave * 8; j < rows; j += NW * 8) {
      const int row = j + r8, pixel = min(max(m0 - width - 1 + row, 0), p.M - 1);
      const char* src = static_cast<const char*>(p.A) + ((size_t)pixel * channels + (((pc ^ (row ^ (row >> 3 & 1))) & 7) << 3)) * 2;
      for (int g = 0; g < groups; ++g)
        __builtin_amdgcn_global_load_lds((global_ptr_t)(src + g * (kTileK * 2)), (lds_ptr_t)(lds + g * group_bytes + j * kRowBytes), 16, 0, 0);
    }
  }

  // ---- weights: tile t = (tap, group); tiles are issued in order
  SourceB src_b;
  const int ldw = LB == Layout::RowK ? p.ldb : 9 * p.ldb;   // KRow: [channel][tap][n], a k-row every nine
  src_b.init(static_cast<const bf16_t*>(p.B), ldw, n0, p.N, wave, lane, 0, p.conv);
  const int n_tiles = 9 * groups;
  const char* issue_at = src_b.panel;
  const size_t group_step = LB == Layout::RowK ? (size_t)kTileK * 2 : (size_t)kTileK * 9 * p.ldb * 2;
  const ptrdiff_t tap_step = LB == Layout::RowK ? (ptrdiff_t)group_step : (ptrdiff_t)p.ldb * 2 - (ptrdiff_t)(groups - 1) * (ptrdiff_t)group_step;
  int issue_left = n_tiles, issue_g = groups;
  char* issue_slot = ring;
  auto issue = [&]() {
    if (issue_left == 0) return;
    --issue_left;
    src_b.issue_at(issue_at, issue_slot, wave);
    if (--issue_g == 0) { issue_g = groups; issue_at += tap_step; }
    else issue_at += group_step;
    issue_slot += BN * kRowBytes;
    if (issue_slot == ring + STAGES * BN * kRowBytes) issue_slot = ring;
  };
#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s) issue();

  // ---- this lane's rows of the patch
  uint32_t inside[TM];     // bit tap: the pixel that tap reads lies in the image
  int row0[TM];            // patch row of the lane's pixel itself
  const int sign = p.conv.transposed ? -1 : 1;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int r = wm * WM + 32 * i + (lane & 31), m = m0 + r;
    const int in_image = m % (height * width), a = in_image / width, b = in_image - a * width;
    row0[i] = r + width + 1;
    inside[i] = 0;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int dr = sign * (tap / 3 - 1), dc = sign * (tap % 3 - 1);
      if ((unsigned)(a + dr) < (unsigned)height && (unsigned)(b + dc) < (unsigned)width) inside[i] |= 1u << tap;
    }
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)lds;
  const uint32_t ring0 = (uint32_t)(uintptr_t)(lds_ptr_t)ring;
  // LDS address of a fragment's chunk for k-group 0 of a tap's first channel group; k-group kg is at address ^ (kg << 5)
  auto tap_address = [&](int tap, uint32_t (&out)[TM]) {
    const int r = (tap * 21846) >> 16, c = tap - 3 * r;              // tap = 3 r + c
    const int shift = sign * ((r - 1) * width + (c - 1));
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int at = patch_offset(row0[i] + shift, half);
      out[i] = lds0 + (uint32_t)((inside[i] >> tap) & 1 ? at : rows * kRowBytes + (at & (kZeroBytes - 1)));
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  auto pin = [] { __builtin_amdgcn_sched_barrier(0); };
  u32x4 fa[kSets][TM], fb[kSets][TN];
  using ReaderB = FragmentReader<BN, LB, TN>;
  ReaderB reader_b;
  reader_b.init(wn * WN, lane);
  uint32_t at_a[TM], at_b[ReaderB::kN];   // the tile being read
  auto fetch = [&](auto set, auto kg, auto f) {   // fragment f of a k-group: A's, then B's
    constexpr int S = decltype(set)::value, KG = decltype(kg)::value, F = decltype(f)::value;
    if constexpr (F < TM) asm volatile("ds_read_b128 %0, %1" : "=v"(fa[S][F]) : "v"(at_a[F] ^ (uint32_t)(KG << 5)));
    else if constexpr (F < TM + TN) fb[S][F - TM] = ReaderB::template read<F - TM, KG>(at_b);
  };
  int tap = 0, g = 0, slot = 0;   // of the tile being read
  auto next_tile = [&]() {        // (behind the last tile: some tile's addresses, whose fragments are read and not used)
    if (++slot == STAGES) slot = 0;
    if (++g == groups) {
      g = 0;
      tap = tap == 8 ? 0 : tap + 1;
      tap_address(tap, at_a);
    } else {
#pragma unroll
      for (int i = 0; i < TM; ++i) at_a[i] += (uint32_t)group_bytes;
    }
    reader_b.at(ring0 + slot * (BN * kRowBytes), at_b);
  };

  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  pin();
  __builtin_amdgcn_s_barrier();
  pin();
  tap_address(0, at_a);
  reader_b.at(ring0, at_b);
  static_for<AHEAD>([&](auto q) {
    constexpr int Q = decltype(q)::value;
    if constexpr (Q == 4) next_tile();
    static_for<TM + TN>([&](auto f) { fetch(q, std::integral_constant<int, Q % 4>{}, f); });
  });

  // K-group q of the round that starts at tile t.  Its last fragments to be requested are those of k-group q + AHEAD: k-group 3 of the
  // tile being read, then - behind the barrier that finds the next tile whole - the next tile's 0, 1, 2.
  auto step = [&](int t, auto q) {
    constexpr int Q = decltype(q)::value, kg = Q % 4, to = (Q + AHEAD) % kSets;
    asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"((AHEAD - 1) * kReads) : "memory");
#pragma unroll
    for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(fa[Q][i]));
#pragma unroll
    for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(fb[Q][j]));
    pin();
    static_for<TM * TN>([&](auto idx_c) {
      constexpr int idx = decltype(idx_c)::value, i = idx / TN, j = idx % TN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fb[Q][j]),   // operands exchanged:
                                                          __builtin_bit_cast(bf16x8, fa[Q][i]), acc[i][j], 0, 0, 0);  // see store_wave_tile
      constexpr int kSlot = (TM + TN + TM * TN - 1) / (TM * TN);
      static_for<kSlot>([&](auto s) { fetch(std::integral_constant<int, to>{}, std::integral_constant<int, (kg + 3) % 4>{}, std::integral_constant<int, idx * kSlot + decltype(s)::value>{}); });
      pin();
    });
    if constexpr (kg == 0) {
      // Every read of tile r - 1 has returned, in every wave once all are here, so its ring slot is free.  The tile to be read next,
      // r + kTiles, has landed once each wave has seen its own loads in, but for those of the tiles behind it.
      const int r = t + Q / 4;
      if (r + STAGES - 2 < n_tiles) __builtin_amdgcn_s_waitcnt(waitcnt_imm((STAGES - 2 - kTiles) * SourceB::kInstr, 15));
      else __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 15));
      pin();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      issue();
      next_tile();
      pin();
    }
  };
  for (int t = 0; t < n_tiles; t += kTiles) {
    static_for<4>([&](auto q) { step(t, q); });
    if constexpr (kTiles == 2)
      if (t + 1 < n_tiles) static_for<4>([&](auto q) { step(t, std::integral_constant<int, decltype(q)::value + 4>{}); });
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  // the reads behind the last tile have come in too: until here their registers belong to nobody else
#pragma unroll
  for (int q = 0; q < kSets; ++q) {
#pragma unroll
    for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(fa[q][i]));
#pragma unroll
    for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(fb[q][j]));
  }
  __syncthreads();   // every wave has its last fragments in registers: patch and ring are dead
  float* stage = reinterpret_cast<float*>(lds) + wave * (32 * (WN + 4));
  store_wave_tile<WM, WN, WAVES_M>(p, acc, stage, m0 + wm * WM, n0 + wn * WN, lane, 0, wm, tile_m);
}

template <int BM, int BN, int STAGES, int WAVES_M, int WAVES_N, int AHEAD, Layout LB>
hipError_t launch_conv3_tile(const GemmProblem& q, hipStream_t stream) {
  GemmParams p = make_params(q, BM, BN);
  const size_t staging = (size_t)WAVES_M * WAVES_N * 32 * (BN / WAVES_N + 4) * 4;
  const size_t lds_bytes = std::max(conv3_lds(BM, BN, STAGES, q.conv.rw, q.conv.sc), staging);
  auto kernel = conv3_kernel<BM, BN, STAGES, WAVES_M, WAVES_N, AHEAD, LB>;
  if (hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kernel), 160 * 1024); e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, dim3(p.tiles_m * p.tiles_n), dim3(64 * WAVES_M * WAVES_N), lds_bytes, stream, p, patch_rows(BM, q.conv.rw));
  return hipGetLastError();
}

// Tile choice, from every tile timed on the shapes of 32- and 224-pixel networks (us, forward; the gathering kernel's time in
// front):  one nearly full round of 128 x 128 (12544 x 256 x 2304: 34 -> 19, 128 x 64 26), with eight waves, since a workgroup is alone
// on its CU (four waves of 64 x 64: 20);  for 64 columns 256 x 64, two workgroups a CU (131072 x 64 x 576: 26 -> 16, 128 x 64 18);
// 128 x 64 while that fills the chip (8192 x 256 x 2304: 25 -> 14, 64 x 64 15);  64 x 128 where the patch of 128 pixels does not
// fit (3136 x 512 x 4608: 46 -> 24, 64 x 64 36);  else 64 x 64 (4096 x 256 x 2304: 21 -> 12, 2048 x 512 x 4608: 37 -> 18).
// A ring of three 64-k tiles of weights does where it leaves room for another workgroup; lone small tiles take four.
struct Conv3Tile { int bm, bn, stages; };
inline Conv3Tile conv3_tile(const GemmProblem& q) {
  auto tiles = [&](int tm, int tn) { return tile_count(q, tm, tn); };
  auto fits = [&](int bm, int bn, int stages) { return conv3_lds(bm, bn, stages, q.conv.rw, q.conv.sc) <= 160 * 1024; };
  if (q.N > 64 && tiles(128, 128) >= 160 && tiles(128, 128) <= 256 && fits(128, 128, 3)) return {128, 128, 3};
  if (q.N <= 64 && tiles(256, 64) >= 448 && fits(256, 64, 3)) return {256, 64, 3};
  if (tiles(128, 64) >= 160 && fits(128, 64, 3)) return {128, 64, 3};
  if (q.N > 64 && tiles(64, 128) >= 160 && fits(64, 128, 4)) return {64, 128, 4};
  return {64, 64, 4};
}

// Whether that is faster than the gathering kernels.  The resident rows leave a CU to one workgroup from 192 channels on (128 where
// the image is wide), and from the third round of such workgroups on the gathering kernels' larger tiles catch up: alone, forward,
// gathering kernel against resident rows, 12032 x 256 x 2304 (one round) 37 and 24 us, 20480 x 256 x 2304 (three) 49 and 45, 25088 (four) 50 and
// 57, 65024 (eight, where 256 x 256 tiles make one) 79 and 112; 16384 x 512 x 4608 in 64 x 64 tiles (eight) 88 and 217.  Two workgroups a CU cover
// each other: 399840 x 128 x 1152 174 and 149, 524288 x 64 x 576 96 and 60.  So: where a round or two is all there is, where two share a
// CU, and for up to 64 columns, which the gathering kernels take in narrow tiles (256000 x 64 x 2304: 137 and 123); but not where the patch is
// more than four times the tile (10000 x 128 x 1152, 100 pixels a row: 19 and 21; 80000 x 64 x 576, 200 a row: 25 and 30).  For the rest by the time
// both should take, from lines through 180 timed shapes: per round a fixed part and one per 64 of k, for the tile that launch_layouts
// would choose; wrong by at most 6 % on those shapes.
inline bool conv3_pays(const GemmProblem& q) {
  const Conv3Tile t = conv3_tile(q);
  const int width = q.conv.rw, channels = q.conv.sc;
  const bool lone = 2 * conv3_lds(t.bm, t.bn, t.stages, width, channels) > 160 * 1024;
  auto rounds = [&](int tm, int tn, int at_once) { return (double)((tile_count(q, tm, tn) + at_once - 1) / at_once); };
  const double own_rounds = rounds(t.bm, t.bn, lone ? 256 : 512);
  if (own_rounds <= 1) return true;
  if (lone && patch_rows(t.bm, width) > 4 * t.bm) return false;
  if (own_rounds <= 2 || q.N <= 64 || (!lone && (q.N <= 128 || channels <= 64))) return true;
  const double k = q.K / (double)kTileK;
  const double own = own_rounds * ((lone ? 1.8 + 0.38 * k : 0.75 * k) + 0.02 * std::max(patch_rows(t.bm, width) - 160, 0));
  const long t192 = tile_count(q, 256, 192), t256 = tile_count(q, 256, 256), t128 = tile_count(q, 128, 128);
  if (q.M >= 256 && t192 >= 176 && t192 <= 256 && (long)((q.N + 191) / 192) * 192 * 20 <= (long)q.N * 21) return own <= 25 + 1.07 * k;
  if (q.M >= 256 && q.N >= 256 && t256 >= 176 && (t256 <= 256 || t256 >= 448)) return own <= rounds(256, 256, 256) * (25 + 1.45 * k);
  if (t128 > 256) return own <= (rounds(128, 128, 512) + 0.15) * (12 + 0.83 * k);
  if (t128 >= 192) return own <= 12 + 0.74 * k;
  return own_rounds <= (q.b_gather == Gather::ConvWeightT ? 3 : 2);   // 64 x 64 gathered: 5120 x 512 x 4608 forward 63 and 74, input gradient 72 and 64
}

// Whether a product is such a convolution, with a patch that leaves room for the smallest tile's ring.
inline bool conv3_accepts(const GemmProblem& q) {
  const ConvGeom& c = q.conv;
  return q.a_gather == Gather::ConvRows && c.r == 3 && c.s == 3 && c.stride == 1 && c.pad == 1 && c.pad_w == 1 && c.sh == c.rh && c.sw == c.rw && c.sc % kTileK == 0 &&
         q.K == 9 * c.sc && q.k_splits == 1 && q.batch == 1 && q.M == c.n * c.rh * c.rw &&
         (q.b_gather == Gather::ConvWeightT ? c.w_cout == c.sc && c.w_cin == q.N && q.ldb == q.N : q.b_layout == Layout::RowK && q.b_gather == Gather::None) &&
         conv3_lds(64, 64, 4, c.rw, c.sc) <= 160 * 1024 && conv3_pays(q);
}

template <Layout LB>
hipError_t launch_conv3(const GemmProblem& q, hipStream_t stream) {
  const Conv3Tile t = conv3_tile(q);
  if (t.bm == 256) return launch_conv3_tile<256, 64, 3, 8, 1, 3, LB>(q, stream);
  if (t.bm == 128 && t.bn == 128) return launch_conv3_tile<128, 128, 3, 4, 2, 3, LB>(q, stream);
  if (t.bm == 128) return launch_conv3_tile<128, 64, 3, 4, 1, 3, LB>(q, stream);
  if (t.bn == 128) return launch_conv3_tile<64, 128, 4, 2, 2, 3, LB>(q, stream);
  return launch_conv3_tile<64, 64, 4, 2, 2, LB == Layout::RowK ? 7 : 3, LB>(q, stream);
}

}  // namespace gemm_dma_detail
}  // namespace spb
