// Weight gradient of a 3 x 3 convolution of stride 1 over whole 64-channel groups:
//   dw[co][tap][ci] = sum over pixels of dy[pixel][co] * x[pixel + tap][ci]
// with all nine taps of a 64 x 64 block of channels in one workgroup.
//
// The gathering product fetches x once per tap and multiplies 64 x 64 or 128 x 128 blocks of (tap, ci) columns with a fragment read
// per matrix instruction.  Here the pixels are numbered with one column of zeros behind every image row and one row of
// zeros behind every image, so that a tap is the same shift everywhere; a step takes 64 of them, the rows of dy and the stretch of
// 64 + 2 W + 4 rows of x that their taps reach, and a wave multiplies its 32 x 32 block of channels for all nine taps: nine matrix
// instructions on ten transposing fragment reads.  The zeros cost (1 + 1/W) (1 + 1/H), the shared x saves nine tenths of the loads.
//
// Eight waves: four blocks of channels, and two waves on each that take half of a step's pixels and exchange their sums at the end.
// Alone, 128 workgroups (us): 131072 pixels of 64 channels 25, 32768 of 128 25, 8192 of 256 27, 2048 of 512 30; 2100 to 2300 cycles a step, of
// which 1152 are matrix work: 160 KB of transposing reads and 25 KB of loads at the 88 bytes a clock that the LDS gives.  With four
// waves 2400 cycles.  In the step of the 32-pixel basic CNN the gathering products took 50, 32, 29 and 33 us on 200 to 350 workgroups
// each; the step went from 1257 to 1177 us, that of the 224-pixel bottleneck CNN from 4950 to 4876.
//
// Which pixel a row is comes from a table in LDS, worked out for up to 48 steps at a time (a longer slice drains the ring and starts again
// behind them); -1 stands for the zeros.  The slices of the pixel range go to
// float32 partial results that the unit's reduction adds up in order.
#include <algorithm>

#include "gemm_dma_impl.h"

namespace spb {
namespace gemm_dma_detail {

constexpr int kWgradStages = 4, kWgradAhead = 6;
constexpr int kWgradTable = 48;           // steps whose pixels the table holds at a time
constexpr int kWgradLoads = 6;            // a wave's loads of a step at most: 48 instructions of 8 rows
// Workgroups of a launch, beside the input-gradient chain of the other stream: 96, 128, 160, 224 gave steps of 1201, 1181, 1187, 1204 us on
// the 32-pixel basic CNN and 4943, 4900, 4875, 4871 on the 224-pixel bottleneck CNN.  Where that makes more than kWgradTable steps a slice,
// a unit's chain is long enough for more: 128, 160, 192, 256 gave 1893, 1850, 1820, 1790 us for three blocks of 256 x 64 x 64 x 64, 3522, 3348, 3250,
// 3255 for 256 x 32 x 32 x 256, 6279, 6089, 5949, 6354 for 256 x 48 x 48 x 192, 4931, 4738, 4728, 4812 for the 224-pixel basic CNN at batch 250.
// (As many as keep a slice within one table, 353 for the first: 1848 us and 52 MB of partial results a buffer instead of 28.)
constexpr int kWgradBlocks = 128, kWgradBlocksLong = 192;
// Fewer steps a slice than this do not pay for the start and the exchange: five steps 14.7 us for 4056 pixels of 128 channels and 16.0 for 8112, where
// the gathering product takes 12.1 and 14.2.  46 CNNs with their two streams: from 6 steps on 0.990 of the time with every size here, from
// 10 0.982, from 13 0.977, from 17 0.978, from 26 0.979, never 0.981 (48 images of 49 x 49, 35 units: 3513 -> 3414 us, 3397 before this kernel).
constexpr int kWgradLeastSteps = 13;
constexpr size_t kExchangeBytes = 4 * 4 * 4096;
inline int wgrad_x_rows(int width) { return (kTileK + 2 * width + 4 + 7) / 8 * 8; }
inline int wgrad_tiles(const ConvGeom& c) { return (int)(((long long)c.n * (c.rh + 1) * (c.rw + 1) + kTileK - 1) / kTileK); }
inline size_t wgrad_lds(const ConvGeom& c, int tiles_per_slice) {
  const size_t table = (size_t)(std::min(tiles_per_slice, kWgradTable) - 1) * kTileK + wgrad_x_rows(c.rw);
  const size_t loop = (size_t)kWgradStages * (kTileK + wgrad_x_rows(c.rw)) * kRowBytes + table * sizeof(int);
  return std::max(loop, kExchangeBytes);
}

// LDS reads a wave has issued behind those of step s when it waits for them: two per fragment, the next k-group's A ahead of its first tap
constexpr int reads_behind(int s) {
  int n = 0;
  for (int u = s + 1; u < s + kWgradAhead; ++u) n += 2 + (u % 9 == 0 ? 2 : 0);
  return n;
}

__global__ __launch_bounds__(512) void conv3_wgrad_kernel(GemmParams p, int x_rows) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave & 1, wn = (wave >> 1) & 1, pixels = wave >> 2;   // its block of channels; which half of a step's pixels
  const int co0 = blockIdx.x % p.tiles_m * 64, ci0 = blockIdx.x / p.tiles_m * 64;
  const int width = p.conv.rw, height = p.conv.rh, channels = p.conv.sc, pitch = width + 1;
  const int slot_bytes = (kTileK + x_rows) * kRowBytes;      // 64 rows of dy, then the rows of x
  const int all = p.conv.n * (height + 1) * pitch;
  const int t_end = min((all + kTileK - 1) / kTileK, ((int)blockIdx.y + 1) * p.k_tiles_per_split);
  int t_first = blockIdx.y * p.k_tiles_per_split;            // of the steps the table holds
  int n_tiles = max(min(t_end - t_first, kWgradTable), 0);   // them
  int* table = reinterpret_cast<int*>(lds + kWgradStages * slot_bytes);

  // ---- row e of the table: number first * 64 - (W + 2) + e
  auto fill_table = [&]() {
    for (int e = threadIdx.x; e < (n_tiles - 1) * kTileK + x_rows; e += 512) {
      const int q = t_first * kTileK - (width + 2) + e;
      const int row = q / pitch, b = q - row * pitch, n = row / (height + 1), a = row - n * (height + 1);
      table[e] = q >= 0 && q < all && b < width && a < height ? (n * height + a) * width + b : -1;
    }
    __syncthreads();
  };

  // ---- loads: instruction u = 8 i + wave of a tile is rows 8 u .. of its slot.  A lane's chunk: rows k and k + 2 lie half a row apart (krow_rot).
  const int n_loads = ((kTileK + x_rows) / 8 - wave + 7) / 8;   // this wave's
  const int r8 = lane >> 3, chunk = (lane & 7) ^ (((r8 >> 1) & 1) << 2);
  const char* dy = static_cast<const char*>(p.A) + (size_t)(co0 + chunk * 8) * 2;
  const char* x = static_cast<const char*>(p.B) + (size_t)(ci0 + chunk * 8) * 2;
  auto load = [&](auto i_c, int pixel, int slot) {
    constexpr int i = decltype(i_c)::value;
    const char* src = i == 0 ? dy + (size_t)pixel * p.lda * 2 : x + (size_t)pixel * channels * 2;
    if (pixel < 0) src = reinterpret_cast<const char*>(kZeroChunk);
    const uint32_t dst = (uint32_t)(uintptr_t)(lds_ptr_t)(lds + slot * slot_bytes + (i * 8 + wave) * 8 * kRowBytes);
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "s"(dst) : "m0");
  };
  int pixel[kWgradLoads];   // the rows of the tile to be loaded next (valid after an s_waitcnt lgkmcnt and a pin)
  auto look_up = [&](int t) {
#pragma unroll
    for (int i = 0; i < kWgradLoads; ++i) {
      const int e = min(t, n_tiles - 1) * kTileK + (i == 0 ? wave * 8 + width + 2 : ((min(i, n_loads - 1) - 1) * 8 + wave) * 8) + r8;
      const uint32_t at = (uint32_t)(uintptr_t)(lds_ptr_t)(table + e);
      asm volatile("ds_read_b32 %0, %1" : "=v"(pixel[i]) : "v"(at));
    }
  };
  auto looked_up = [&]() {
#pragma unroll
    for (int i = 0; i < kWgradLoads; ++i) asm volatile("" : "+v"(pixel[i]));
  };

  // ---- fragments
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)lds;
  FragmentReader<64, Layout::KRow, 1> reader_a;
  reader_a.init(wm * 32, lane);
  reader_a.off[0] += (uint32_t)(pixels * 32 * kRowBytes);   // (rotations repeat every four rows)
  uint32_t off_b[9], at_a[1], at_b[9];
  {
    const int j = lane & 15, g = lane >> 4, ci = wn * 32 + 16 * (g & 1) + 4 * (j & 3);
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int row = pixels * 32 + 8 * (g >> 1) + (j >> 2) + width + 2 + (tap / 3 - 1) * pitch + tap % 3 - 1;
      off_b[tap] = (uint32_t)((kTileK + row) * kRowBytes + ((((ci >> 3) + krow_rot<64>(row)) & 7) << 4) + (ci & 7) * 2);
    }
  }
  auto at_slot = [&](int slot) {
    const uint32_t base = lds0 + (uint32_t)(slot * slot_bytes);
    reader_a.at(base, at_a);
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) at_b[tap] = off_b[tap] + base;
  };
  u32x4 fa[2], fb[9];
  auto fetch = [&](auto step) {   // the fragments of step 9 kg + tap of the tile at hand: kg of this wave's two k-groups
    constexpr int S = decltype(step)::value, kg = S / 9, tap = S % 9;
    if constexpr (tap == 0) fa[kg & 1] = FragmentReader<64, Layout::KRow, 1>::template read<0, kg>(at_a);
    uint2 lo, hi;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(at_b[tap]), "n"(16 * kg * kRowBytes));
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(at_b[tap]), "n"((16 * kg + 4) * kRowBytes));
    fb[tap] = u32x4{lo.x, lo.y, hi.x, hi.y};
  };
  f32x16 acc[9];
#pragma unroll
  for (int tap = 0; tap < 9; ++tap)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[tap][r] = 0.f;

  auto pin = [] { __builtin_amdgcn_sched_barrier(0); };
  auto wait_loads = [&](bool younger) {   // all but the tile behind the next
    if (!younger) { __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 15)); return; }
    switch (n_loads) {
      case 2: __builtin_amdgcn_s_waitcnt(waitcnt_imm(2, 15)); break;
      case 3: __builtin_amdgcn_s_waitcnt(waitcnt_imm(3, 15)); break;
      case 4: __builtin_amdgcn_s_waitcnt(waitcnt_imm(4, 15)); break;
      case 5: __builtin_amdgcn_s_waitcnt(waitcnt_imm(5, 15)); break;
      case 6: __builtin_amdgcn_s_waitcnt(waitcnt_imm(6, 15)); break;
      default: __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 15));
    }
  };
  while (n_tiles > 0) {
    fill_table();
    for (int t = 0; t < min(2, n_tiles); ++t) {
      look_up(t);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      looked_up();
      static_for<kWgradLoads>([&](auto i) { if (decltype(i)::value < n_loads) load(i, pixel[decltype(i)::value], t); });
    }
    wait_loads(n_tiles > 1);
    pin();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    look_up(2);
    at_slot(0);
    static_for<kWgradAhead>([&](auto s) { fetch(s); });
    constexpr int kSteps = 18;
    int slot = 0;
    for (int t = 0; t < n_tiles; ++t) {
      // Tile t + 2 goes where tile t - 2 was: every wave had all of that in registers when it came to the barrier of tile t - 1.
      const int next_slot = (slot + 1) % kWgradStages, load_slot = (slot + 2) % kWgradStages;
      static_for<kSteps>([&](auto s_c) {
        constexpr int s = decltype(s_c)::value, kg = s / 9, tap = s % 9;
        if constexpr (s == kSteps - kWgradAhead) {
          // All of this tile has been requested: on to tile t + 1, which has landed once every wave has seen its own loads in.
          wait_loads(t + 2 < n_tiles);
          pin();
          asm volatile("" ::: "memory");
          __builtin_amdgcn_s_barrier();
          asm volatile("" ::: "memory");
          look_up(t + 3);
          at_slot(next_slot);
        }
        asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(reads_behind(s)) : "memory");
        asm volatile("" : "+v"(fb[tap]));
        if constexpr (tap == 0) asm volatile("" : "+v"(fa[kg & 1]));
        if constexpr (s == 0) looked_up();
        pin();
        acc[tap] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fb[tap]), __builtin_bit_cast(bf16x8, fa[kg & 1]), acc[tap], 0, 0, 0);
        fetch(std::integral_constant<int, (s + kWgradAhead) % kSteps>{});
        if constexpr (s % 2 == 1 && s / 2 < kWgradLoads)   // one load every other step: the memory path takes one per 16 to 22 cycles
          if (s / 2 < n_loads && t + 2 < n_tiles) load(std::integral_constant<int, s / 2>{}, pixel[s / 2], load_slot);
        pin();
      });
      slot = next_slot;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    // what was read behind the last tile has come in too: until here its registers belong to nobody else
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) asm volatile("" : "+v"(fb[tap]));
    looked_up();
    asm volatile("" : "+v"(fa[0]), "+v"(fa[1]));
    __syncthreads();   // every wave is done with the ring and the table
    t_first += n_tiles;
    n_tiles = min(t_end - t_first, kWgradTable);
  }

  // ---- the two halves of the pixels: one wave of a pair finishes taps 0 to 4, the other 5 to 8, two of each at a time
  auto exchange = [&](int of, int which) { return reinterpret_cast<f32x4*>(lds + ((of * 4 + (wave & 3)) * 2 + which) * 4096 + lane * 16); };   // of: whose sums
  static_for<3>([&](auto round_c) {
    constexpr int round = decltype(round_c)::value;
    auto give = [&](auto tap_c, int which) {
      constexpr int tap = decltype(tap_c)::value;
#pragma unroll
      for (int g = 0; g < 4; ++g) exchange(pixels, which)[g * 64] = f32x4{acc[tap][4 * g], acc[tap][4 * g + 1], acc[tap][4 * g + 2], acc[tap][4 * g + 3]};
    };
    auto take = [&](auto tap_c, int which) {   // in the order of the pixels, whichever wave adds them
      constexpr int tap = decltype(tap_c)::value;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 v = exchange(pixels ^ 1, which)[g * 64];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[tap][4 * g + e] = acc[tap][4 * g + e] + v[e];
      }
    };
    if (round > 0) __syncthreads();
    static_for<2>([&](auto w) {
      constexpr int low = 2 * round + decltype(w)::value, high = 5 + low;
      if constexpr (low < 5) { if (pixels == 1) give(std::integral_constant<int, low>{}, decltype(w)::value); }
      if constexpr (high < 9) { if (pixels == 0) give(std::integral_constant<int, high>{}, decltype(w)::value); }
    });
    __syncthreads();
    static_for<2>([&](auto w) {
      constexpr int low = 2 * round + decltype(w)::value, high = 5 + low;
      if constexpr (low < 5) { if (pixels == 0) take(std::integral_constant<int, low>{}, decltype(w)::value); }
      if constexpr (high < 9) { if (pixels == 1) take(std::integral_constant<int, high>{}, decltype(w)::value); }
    });
  });
  __syncthreads();

  // ---- partial results: 32 x 32 floats per tap, parked so that whole 128-byte row pieces leave
  constexpr int kPitch = 36;
  float* stage = reinterpret_cast<float*>(lds) + wave * (32 * kPitch);
  float* out = static_cast<float*>(p.C) + (size_t)blockIdx.y * p.M * p.ldc + (size_t)(co0 + wm * 32) * p.ldc + ci0 + wn * 32;
  static_for<9>([&](auto tap_c) {
    constexpr int tap = decltype(tap_c)::value;
    if (pixels != (tap < 5 ? 0 : 1)) return;
    lanes_together();
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<f32x4*>(stage + (lane & 31) * kPitch + 8 * g + 4 * half) = f32x4{acc[tap][4 * g], acc[tap][4 * g + 1], acc[tap][4 * g + 2], acc[tap][4 * g + 3]};
    lanes_together();
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int row = it * 8 + (lane >> 3), c = (lane & 7) * 4;
      *reinterpret_cast<f32x4*>(out + (size_t)row * p.ldc + tap * channels + c) = *reinterpret_cast<const f32x4*>(stage + row * kPitch + c);
    }
  });
}

}  // namespace gemm_dma_detail

using namespace gemm_dma_detail;

// Slices of the pixel range for about kWgradBlocks workgroups (beside the input-gradient chain of the other stream), at least 256 pixels each
// (the zeros not counted: no more slices than the gathering product takes of a model small enough for the library's own workspace); for about
// kWgradBlocksLong where the slices would be long.  0: not this kernel's convolution, or one of too few steps.
int conv3_wgrad_splits(const ConvGeom& c, int c_out) {
  if (c.r != 3 || c.s != 3 || c.stride != 1 || c.pad != 1 || c.pad_w != 1 || c.transposed || c.sh != c.rh || c.sw != c.rw || c.sc % 64 || c_out % 64) return 0;
  if ((long long)c.n * (c.rh + 1) * (c.rw + 1) > 0x7FFFFFFFLL - 4096 || kTileK + wgrad_x_rows(c.rw) > 64 * kWgradLoads || wgrad_lds(c, kWgradTable) > 160 * 1024) return 0;
  const int blocks = c.sc / 64 * (c_out / 64);
  const int pixel_tiles = (int)(((long long)c.n * c.rh * c.rw + kTileK - 1) / kTileK);
  const int s = std::min((kWgradBlocks + blocks - 1) / blocks, std::max(pixel_tiles / 4, 1));
  const int steps = (wgrad_tiles(c) + s - 1) / s;
  if (steps < kWgradLeastSteps) return 0;
  return steps <= kWgradTable ? s : (kWgradBlocksLong + blocks - 1) / blocks;
}

bool conv3_wgrad_accepts(const GemmProblem& q) {
  return q.b_gather == Gather::ConvPatchT && q.a_gather == Gather::None && q.a_layout == Layout::KRow && q.epilogue == Epilogue::StoreF32 && !q.bias &&
         !q.a_row_sum && q.alpha == 1.f && q.batch == 1 && q.N == 9 * q.conv.sc && q.ldc == q.N && q.K == q.conv.n * q.conv.rh * q.conv.rw &&
         conv3_wgrad_splits(q.conv, q.M) > 0;
}

hipError_t launch_conv3_wgrad(const GemmProblem& q, hipStream_t stream) {
  GemmParams p = make_params(q, 64, 64);
  p.k_tiles_per_split = (wgrad_tiles(q.conv) + q.k_splits - 1) / q.k_splits;
  const size_t lds_bytes = wgrad_lds(q.conv, p.k_tiles_per_split);
  if (hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(conv3_wgrad_kernel), 160 * 1024); e != hipSuccess) return e;
  hipLaunchKernelGGL(conv3_wgrad_kernel, dim3(p.tiles_m * (q.conv.sc / 64), q.k_splits), dim3(512), lds_bytes, stream, p, wgrad_x_rows(q.conv.rw));
  return hipGetLastError();
}

}  // namespace spb
