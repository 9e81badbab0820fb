// Attention of sequences of any length, heads of 64 features: ctx = softmax(Q K^T / sqrt(d)) V and its backward, without
// the [seq, seq] matrices in memory.  A workgroup owns 128 rows (queries, or in attention_long_dkv_kernel keys) of one
// (batch entry, head), 32 per wave, and walks the other side in tiles of 64 rows: the next pair of tiles is on its way
// into LDS (direct-to-LDS loads, two buffers) while one is used.  The forward pass keeps a running maximum and sum per
// query and stores, above the cut, only their combination L = log2(sum of exp2(scores)); the backward pass forms
// P = exp2(scores - L) again.
//
// Every product runs with the MFMA operands arranged so that the wave's own 32 rows are the columns of the result: a
// lane holds, of own row lane % 32, the other side's rows 8 (r / 4) + 4 (lane / 32) + r % 4 in register r.  Row-wise
// statistics then are in-lane work plus one exchange, and eight consecutive registers, rounded to bfloat16, are an
// operand of the next product (P for ctx and dV, dS for dQ and dK never pass through LDS).  That operand's order of k
// differs between the half-waves, so its partner is read in the same order (TransposedReader).
//
// Bound: one head's four (six with the recomputation) products are few flops per score, so the vector work per score -
// one exponential at quarter rate and a handful of full-rate instructions - is as long as the matrix work; memory
// traffic is a few passes over qkv.  Measured inside the encoder step (8 x 512 tokens, 12 heads): forward 16 us, dQ 29,
// dK and dV 43, where separate products with softmax passes over float32 scores took 82 and 180; the step 7.08 -> 4.69 ms.
// Sequences of at most 128 run the kernels of attention.hip, which keep P: level at 128 in the step (32 x 128 tokens).
#include <algorithm>

#include "gemm_dma_impl.h"

namespace spb {
namespace {
using namespace gemm_dma_detail;

constexpr int kHeadDim = 64, kOwnRows = 128, kTileRows = 64;
constexpr int kTileBytes = kTileRows * kRowBytes;   // 8 KB: 64 rows of 64 features, chunks permuted as lds_offset says

// The two direct-to-LDS instructions with which a wave brings its share of a 64-row tile.  Rows beyond the sequence
// read its last row again: their scores are masked, or meet P = 0, or end in rows nobody stores.
struct RowTile {
  uint32_t row[2], chunk[2];
  __device__ __forceinline__ void init(int wave, int lane) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int slot = (i * 4 + wave) * 64 + lane, r = slot >> 3;
      row[i] = r;
      chunk[i] = (((slot & 7) ^ r ^ ((r >> 3) & 3)) & 7) * 16;    // the inverse of lds_offset
    }
  }
  // base and ld are the same for the whole wave
  __device__ __forceinline__ void issue(const bf16_t* base, int ld, int row0, int seq, char* tile, int wave) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t off = (uint32_t)min(row0 + (int)row[i], seq - 1) * (uint32_t)(ld * 2) + chunk[i];
      const uint32_t dst = (uint32_t)(uintptr_t)(lds_ptr_t)(tile + (i * 4 + wave) * 1024);
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base), "s"(dst) : "m0");
    }
  }
};
// 64 floats of a per-row array (row0 a multiple of 64, the array padded to whole own-row blocks), by one wave
__device__ __forceinline__ void issue_row_values(const float* base, int row0, char* dst_lds, int lane) {
  const uint32_t off = (uint32_t)(row0 + lane) * 4u;
  const uint32_t dst = (uint32_t)(uintptr_t)(lds_ptr_t)dst_lds;
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" : : "v"(off), "s"(base), "s"(dst) : "m0");
}

// Operand fragments of 32 tile rows x 16 features, feature group g: reads as in read_fragment, addresses worked out once.
struct RowReader {
  uint32_t off[4];
  __device__ __forceinline__ void init(int lane) {
#pragma unroll
    for (int g = 0; g < 4; ++g) off[g] = (uint32_t)lds_offset(lane & 31, 2 * g + (lane >> 5));
  }
  __device__ __forceinline__ u32x4 read(const char* tile, int block, int g) const {
    return *reinterpret_cast<const u32x4*>(tile + off[g] + block * (32 * kRowBytes));
  }
};

// Operand fragments of 32 features (block n) x 16 tile rows (k-group kg), transposed on the way out of LDS, in the order
// of k that accumulators have: half-wave hh receives rows 16 kg + 4 hh + (0..3) and 16 kg + 8 + 4 hh + (0..3).
// The four rows a 16-lane group touches lie in both 128-byte halves of the banks and, within a half, in chunks that
// differ by the row permutation, so the tile that RowReader reads serves here as it lies.
// Valid after an s_waitcnt lgkmcnt and a pin (ready()).
struct TransposedReader {
  uint32_t off[2][4];   // [feature block][(rows / 8) % 4]
  __device__ __forceinline__ void init(int lane) {
    const int j = lane & 15, g = lane >> 4;
    const int r0 = 4 * (g >> 1) + (j >> 2);
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        off[n][c] = (uint32_t)(r0 * kRowBytes + (((4 * n + 2 * (g & 1) + ((j & 3) >> 1)) ^ r0 ^ c) & 7) * 16 + (j & 1) * 8);
  }
  // KG counts k-groups from the tile's start
  template <int KG>
  __device__ __forceinline__ u32x4 read(uint32_t tile, int n) const {
    uint2 lo, hi;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(off[n][(2 * KG) & 3] + tile), "n"(16 * KG * kRowBytes));
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(off[n][(2 * KG + 1) & 3] + tile), "n"((16 * KG + 8) * kRowBytes));
    return u32x4{lo.x, lo.y, hi.x, hi.y};
  }
};
template <int A, int B>
__device__ __forceinline__ void ready(u32x4 (&f)[A][B]) {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
  for (int a = 0; a < A; ++a)
#pragma unroll
    for (int b = 0; b < B; ++b) asm volatile("" : "+v"(f[a][b]));
}

__device__ __forceinline__ f32x16 mfma(const u32x4& rows, const u32x4& cols, const f32x16& acc) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, rows), __builtin_bit_cast(bf16x8, cols), acc, 0, 0, 0);
}
__device__ __forceinline__ void clear(f32x16& a) {
#pragma unroll
  for (int r = 0; r < 16; ++r) a[r] = 0.f;
}
// registers 8 h .. 8 h + 7 of an accumulator as the bfloat16 operand of k-group h of its 32 rows
__device__ __forceinline__ u32x4 as_operand(const f32x16& a, int h) {
  return u32x4{pack_bf16(a[8 * h], a[8 * h + 1]), pack_bf16(a[8 * h + 2], a[8 * h + 3]), pack_bf16(a[8 * h + 4], a[8 * h + 5]), pack_bf16(a[8 * h + 6], a[8 * h + 7])};
}
// This lane's row (own row lane % 32) of an operand: 4 fragments of 16 features
__device__ __forceinline__ void load_row(const bf16_t* row, int hh, u32x4 (&f)[4]) {
#pragma unroll
  for (int g = 0; g < 4; ++g) f[g] = *reinterpret_cast<const u32x4*>(row + 16 * g + 8 * hh);
}
// [64 features x 32 own rows] accumulators times `mul` to one bfloat16 row per lane pair: the half-waves exchange halves
// of chunks (8 features), so each lane writes whole 16-byte chunks.
__device__ __forceinline__ void store_row(bf16_t* row, const f32x16 (&o)[2], float mul, int hh, bool inside) {
#pragma unroll
  for (int n = 0; n < 2; ++n)
#pragma unroll
    for (int g = 0; g < 4; g += 2) {
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = pack_bf16(o[n][4 * g + 2 * e] * mul, o[n][4 * g + 2 * e + 1] * mul);
      const auto x = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
      const auto y = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
      if (inside) *reinterpret_cast<u32x4*>(row + 32 * n + 8 * (g + hh)) = u32x4{x[0], y[0], x[1], y[1]};
    }
}

// Workgroups of one (batch entry, head) share its K and V (or Q and dctx): their ids are a multiple of `heads_total`
// apart, so with a multiple of 8 of those they run on one XCD, behind one L2.
struct Place {
  int z, own0, lane, wave, qi, hh;
  __device__ __forceinline__ Place(int heads_total) {
    z = blockIdx.x % heads_total;
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    own0 = (int)(blockIdx.x / heads_total) * kOwnRows + 32 * wave;
    qi = lane & 31; hh = lane >> 5;
  }
};

__global__ __launch_bounds__(256, 2) void attention_long_fwd_kernel(const bf16_t* __restrict__ qkv, int ld_qkv, float* __restrict__ lse,
                                                                    bf16_t* __restrict__ ctx, int ld_ctx, int heads, int heads_total, int seq,
                                                                    int seq_padded, float scale_log2) {
  __shared__ __attribute__((aligned(1024))) char lds[2][2][kTileBytes];   // [buffer][K, V]
  const Place at(heads_total);
  const int b = at.z / heads, h = at.z - b * heads, hidden = heads * kHeadDim;
  const bf16_t* base = qkv + (size_t)b * seq * ld_qkv + h * kHeadDim;
  const int own = at.own0 + at.qi;
  RowTile tile; tile.init(at.wave, at.lane);
  RowReader rows; rows.init(at.lane);
  TransposedReader cols; cols.init(at.lane);
  auto issue = [&](int t) {
    tile.issue(base + hidden, ld_qkv, t * kTileRows, seq, lds[t & 1][0], at.wave);
    tile.issue(base + 2 * hidden, ld_qkv, t * kTileRows, seq, lds[t & 1][1], at.wave);
  };
  issue(0);
  u32x4 q[4];
  load_row(base + (size_t)min(own, seq - 1) * ld_qkv, at.hh, q);
  f32x16 o[2];
  clear(o[0]); clear(o[1]);
  float m = -INFINITY, sum = 0.f;
  const int tiles = (seq + kTileRows - 1) / kTileRows;
  const bool idle = at.own0 >= seq;      // whole wave beyond the sequence: it only brings its share of the tiles
  for (int t = 0; t < tiles; ++t) {
    wait_loads_and_barrier<0>();
    if (t + 1 < tiles) issue(t + 1);
    if (idle) continue;
    const char* k_tile = lds[t & 1][0];
    const uint32_t v_tile = (uint32_t)(uintptr_t)(lds_ptr_t)lds[t & 1][1];
    f32x16 s[2];
    clear(s[0]); clear(s[1]);
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int j = 0; j < 2; ++j) s[j] = mfma(rows.read(k_tile, j, g), q[g], s[j]);
    u32x4 v[4][2];
    static_for<4>([&](auto kg) {
#pragma unroll
      for (int n = 0; n < 2; ++n) v[kg.value][n] = cols.read<kg.value>(v_tile, n);
    });
    if ((t + 1) * kTileRows > seq) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (t * kTileRows + 32 * j + 8 * (r >> 2) + 4 * at.hh + (r & 3) >= seq) s[j][r] = -INFINITY;
    }
    float top = s[0][0];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) top = fmaxf(top, s[j][r]);
    top = fmaxf(top, __shfl_xor(top, 32, 64)) * scale_log2;
    if (__any(top > m)) {                 // (the first tile always: m is -infinity, and every tile has a key inside)
      const float m_new = fmaxf(m, top), keep = __builtin_amdgcn_exp2f(m - m_new);
      m = m_new;
      sum *= keep;
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[n][r] *= keep;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) { s[j][r] = __builtin_amdgcn_exp2f(fmaf(s[j][r], scale_log2, -m)); sum += s[j][r]; }
    ready(v);
#pragma unroll
    for (int kg = 0; kg < 4; ++kg) {
      const u32x4 p = as_operand(s[kg >> 1], kg & 1);
#pragma unroll
      for (int n = 0; n < 2; ++n) o[n] = mfma(v[kg][n], p, o[n]);
    }
  }
  sum += __shfl_xor(sum, 32, 64);
  if (lse && at.hh == 0) lse[(size_t)at.z * seq_padded + own] = own < seq ? m + __builtin_amdgcn_logf(sum) : INFINITY;   // beyond the sequence P = exp2(-inf) = 0
  store_row(ctx + ((size_t)b * seq + own) * ld_ctx + h * kHeadDim, o, 1.f / sum, at.hh, own < seq);
}

// dQ = dS K with dS = P (dP - D) / sqrt(d), dP = dctx V^T, D = row sum of dctx * ctx (= row sum of dP * P).  Also writes
// D for attention_long_dkv_kernel.
__global__ __launch_bounds__(256, 2) void attention_long_dq_kernel(const bf16_t* __restrict__ qkv, int ld_qkv, const float* __restrict__ lse,
                                                                   const bf16_t* __restrict__ ctx, const bf16_t* __restrict__ dctx, int ld_ctx,
                                                                   bf16_t* __restrict__ dqkv, float* __restrict__ dsum, int heads, int heads_total,
                                                                   int seq, int seq_padded, float scale_log2, float scale) {
  __shared__ __attribute__((aligned(1024))) char lds[2][2][kTileBytes];   // [buffer][K, V]
  const Place at(heads_total);
  const int b = at.z / heads, h = at.z - b * heads, hidden = heads * kHeadDim;
  const bf16_t* base = qkv + (size_t)b * seq * ld_qkv + h * kHeadDim;
  const int own = at.own0 + at.qi, row = min(own, seq - 1);
  RowTile tile; tile.init(at.wave, at.lane);
  RowReader rows; rows.init(at.lane);
  TransposedReader cols; cols.init(at.lane);
  auto issue = [&](int t) {
    tile.issue(base + hidden, ld_qkv, t * kTileRows, seq, lds[t & 1][0], at.wave);
    tile.issue(base + 2 * hidden, ld_qkv, t * kTileRows, seq, lds[t & 1][1], at.wave);
  };
  issue(0);
  u32x4 q[4], dc[4];
  load_row(base + (size_t)row * ld_qkv, at.hh, q);
  load_row(dctx + ((size_t)b * seq + row) * ld_ctx + h * kHeadDim, at.hh, dc);
  float d = 0.f;
  {
    u32x4 c[4];
    load_row(ctx + ((size_t)b * seq + row) * ld_ctx + h * kHeadDim, at.hh, c);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      float x[8], y[8];
      unpack_bf16x8(c[g], x);
      unpack_bf16x8(dc[g], y);
#pragma unroll
      for (int e = 0; e < 8; ++e) d = fmaf(x[e], y[e], d);
    }
    d += __shfl_xor(d, 32, 64);
    if (at.hh == 0) dsum[(size_t)at.z * seq_padded + own] = own < seq ? d : 0.f;
  }
  const float l = lse[(size_t)at.z * seq_padded + row];
  f32x16 o[2];
  clear(o[0]); clear(o[1]);
  const int tiles = (seq + kTileRows - 1) / kTileRows;
  const bool idle = at.own0 >= seq;
  for (int t = 0; t < tiles; ++t) {
    wait_loads_and_barrier<0>();
    if (t + 1 < tiles) issue(t + 1);
    if (idle) continue;
    const char* k_tile = lds[t & 1][0];
    const char* v_tile = lds[t & 1][1];
    f32x16 s[2], dp[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) { clear(s[j]); clear(dp[j]); }
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        s[j] = mfma(rows.read(k_tile, j, g), q[g], s[j]);
        dp[j] = mfma(rows.read(v_tile, j, g), dc[g], dp[j]);
      }
    u32x4 k[4][2];
    static_for<4>([&](auto kg) {
#pragma unroll
      for (int n = 0; n < 2; ++n) k[kg.value][n] = cols.read<kg.value>((uint32_t)(uintptr_t)(lds_ptr_t)k_tile, n);
    });
    if ((t + 1) * kTileRows > seq) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (t * kTileRows + 32 * j + 8 * (r >> 2) + 4 * at.hh + (r & 3) >= seq) s[j][r] = -INFINITY;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) dp[j][r] = __builtin_amdgcn_exp2f(fmaf(s[j][r], scale_log2, -l)) * (dp[j][r] - d);
    ready(k);
#pragma unroll
    for (int kg = 0; kg < 4; ++kg) {
      const u32x4 ds = as_operand(dp[kg >> 1], kg & 1);
#pragma unroll
      for (int n = 0; n < 2; ++n) o[n] = mfma(k[kg][n], ds, o[n]);
    }
  }
  store_row(dqkv + ((size_t)b * seq + own) * ld_qkv + h * kHeadDim, o, scale, at.hh, own < seq);
}

// dK = dS^T Q and dV = P^T dctx: own rows are keys, the tiles hold queries and their dctx, L and D.
__global__ __launch_bounds__(256, 2) void attention_long_dkv_kernel(const bf16_t* __restrict__ qkv, int ld_qkv, const float* __restrict__ lse,
                                                                    const float* __restrict__ dsum, const bf16_t* __restrict__ dctx, int ld_ctx,
                                                                    bf16_t* __restrict__ dqkv, int heads, int heads_total, int seq, int seq_padded,
                                                                    float scale_log2, float scale) {
  __shared__ __attribute__((aligned(1024))) char lds[2][2][kTileBytes];   // [buffer][Q, dctx]
  __shared__ __attribute__((aligned(256))) float stats[2][2][kTileRows];  // [buffer][L, D]
  const Place at(heads_total);
  const int b = at.z / heads, h = at.z - b * heads, hidden = heads * kHeadDim;
  const bf16_t* base = qkv + (size_t)b * seq * ld_qkv + h * kHeadDim;
  const bf16_t* dc_base = dctx + (size_t)b * seq * ld_ctx + h * kHeadDim;
  const int own = at.own0 + at.qi, row = min(own, seq - 1);
  RowTile tile; tile.init(at.wave, at.lane);
  RowReader rows; rows.init(at.lane);
  TransposedReader cols; cols.init(at.lane);
  auto issue = [&](int t) {
    tile.issue(base, ld_qkv, t * kTileRows, seq, lds[t & 1][0], at.wave);
    tile.issue(dc_base, ld_ctx, t * kTileRows, seq, lds[t & 1][1], at.wave);
    if (at.wave < 2) issue_row_values((at.wave ? dsum : lse) + (size_t)at.z * seq_padded, t * kTileRows, reinterpret_cast<char*>(stats[t & 1][at.wave]), at.lane);
  };
  issue(0);
  u32x4 k[4], v[4];
  load_row(base + hidden + (size_t)row * ld_qkv, at.hh, k);
  load_row(base + 2 * hidden + (size_t)row * ld_qkv, at.hh, v);
  f32x16 dk[2], dv[2];
#pragma unroll
  for (int n = 0; n < 2; ++n) { clear(dk[n]); clear(dv[n]); }
  const int tiles = (seq + kTileRows - 1) / kTileRows;
  const bool idle = at.own0 >= seq;
  for (int t = 0; t < tiles; ++t) {
    wait_loads_and_barrier<0>();
    if (t + 1 < tiles) issue(t + 1);
    if (idle) continue;
    const char* q_tile = lds[t & 1][0];
    const char* c_tile = lds[t & 1][1];
    static_for<2>([&](auto block) {          // 32 queries at a time
      constexpr int j = block.value;
      f32x16 s, dp;
      clear(s); clear(dp);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        s = mfma(rows.read(q_tile, j, g), k[g], s);
        dp = mfma(rows.read(c_tile, j, g), v[g], dp);
      }
      u32x4 ct[2][2], qt[2][2];
      static_for<2>([&](auto half) {
        constexpr int kg = 2 * j + half.value;
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          ct[half.value][n] = cols.read<kg>((uint32_t)(uintptr_t)(lds_ptr_t)c_tile, n);
          qt[half.value][n] = cols.read<kg>((uint32_t)(uintptr_t)(lds_ptr_t)q_tile, n);
        }
      });
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 l = *reinterpret_cast<const f32x4*>(&stats[t & 1][0][32 * j + 8 * g + 4 * at.hh]);
        const f32x4 d = *reinterpret_cast<const f32x4*>(&stats[t & 1][1][32 * j + 8 * g + 4 * at.hh]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = 4 * g + e;
          s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], scale_log2, -l[e]));
          dp[r] = s[r] * (dp[r] - d[e]);
        }
      }
      ready(ct);
      ready(qt);
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const u32x4 p = as_operand(s, half), ds = as_operand(dp, half);
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          dv[n] = mfma(ct[half][n], p, dv[n]);
          dk[n] = mfma(qt[half][n], ds, dk[n]);
        }
      }
    });
  }
  bf16_t* out = dqkv + ((size_t)b * seq + own) * ld_qkv + h * kHeadDim;
  store_row(out + hidden, dk, scale, at.hh, own < seq);
  store_row(out + 2 * hidden, dv, 1.f, at.hh, own < seq);
}

constexpr float kLog2e = 1.4426950408889634f;

int padded(int seq) { return (seq + kOwnRows - 1) / kOwnRows * kOwnRows; }
bool aligned16(const void* a, const void* b, const void* c = nullptr, const void* d = nullptr) {
  return !((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b) | reinterpret_cast<uintptr_t>(c) | reinterpret_cast<uintptr_t>(d)) & 15);
}

}  // namespace

bool attention_long_accepts(int seq, int head_dim, int ld_qkv, int ld_ctx) {
  // (a lane's offset inside one batch entry is 32 bits)
  return head_dim == kHeadDim && seq >= 1 && ld_qkv % 8 == 0 && ld_ctx % 8 == 0 && (long long)seq * std::max(ld_qkv, ld_ctx) < (1ll << 30);
}

size_t attention_long_row_floats(int heads_total, int seq) { return (size_t)heads_total * padded(seq); }

hipError_t launch_attention_long_fwd(const void* qkv, int ld_qkv, float* lse, void* ctx, int ld_ctx, int batch, int heads, int seq, int head_dim,
                                     float scale, hipStream_t stream) {
  if (!qkv || !ctx || batch <= 0 || heads <= 0 || !attention_long_accepts(seq, head_dim, ld_qkv, ld_ctx) || !aligned16(qkv, ctx)) return hipErrorInvalidValue;
  const int z = batch * heads;
  hipLaunchKernelGGL(attention_long_fwd_kernel, dim3(z * (padded(seq) / kOwnRows)), dim3(256), 0, stream, static_cast<const bf16_t*>(qkv), ld_qkv, lse,
                     static_cast<bf16_t*>(ctx), ld_ctx, heads, z, seq, padded(seq), scale * kLog2e);
  return hipGetLastError();
}

hipError_t launch_attention_long_bwd(const void* qkv, int ld_qkv, const float* lse, const void* ctx, const void* dctx, int ld_ctx, void* dqkv, float* dsum,
                                     int batch, int heads, int seq, int head_dim, float scale, hipStream_t stream) {
  if (!qkv || !lse || !ctx || !dctx || !dqkv || !dsum || batch <= 0 || heads <= 0 || !attention_long_accepts(seq, head_dim, ld_qkv, ld_ctx) ||
      !aligned16(qkv, ctx, dctx, dqkv))
    return hipErrorInvalidValue;
  const int z = batch * heads;
  const dim3 grid(z * (padded(seq) / kOwnRows));
  hipLaunchKernelGGL(attention_long_dq_kernel, grid, dim3(256), 0, stream, static_cast<const bf16_t*>(qkv), ld_qkv, lse, static_cast<const bf16_t*>(ctx),
                     static_cast<const bf16_t*>(dctx), ld_ctx, static_cast<bf16_t*>(dqkv), dsum, heads, z, seq, padded(seq), scale * kLog2e, scale);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  hipLaunchKernelGGL(attention_long_dkv_kernel, grid, dim3(256), 0, stream, static_cast<const bf16_t*>(qkv), ld_qkv, lse, dsum,
                     static_cast<const bf16_t*>(dctx), ld_ctx, static_cast<bf16_t*>(dqkv), heads, z, seq, padded(seq), scale * kLog2e, scale);
  return hipGetLastError();
}

}  // namespace spb
