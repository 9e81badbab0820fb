// Attention over 129 to 512 positions, heads of 64 features: one workgroup per (batch entry, head) and 32 queries.
//   forward:   S = Q K^T / sqrt(d),  P = softmax(S),  ctx = P V            (P goes to memory only where it is kept)
//   backward:  dP = dctx V^T,  dS = P (dP - sum(dP P)) / sqrt(d),  dQ = dS K;  dS goes to memory, for dK = dS^T Q
// As batched products and softmax passes the float32 scores went to memory and back twice per pass and layer: 83 and
// 126 us of kernels per layer of 8 x 512 tokens and 12 heads in the step, where these take 39 and 55 (7017 -> 5812 us for
// the step of twelve layers).
//
// The four waves share a row of 32 queries and divide the keys: a wave's scores are 32 queries x at most 128 keys, 64
// registers a lane, so a row of 512 is held whole and its exponentials are worked out once.  That - some 10 vector
// instructions an element at 4 cycles, 16 for the exponential itself - is what bounds the forward kernel (8 x 512 tokens, 12 heads: the vector
// ALUs are at work half of a CU's cycles, the matrix cores 5 %); 80 KB of LDS
// let two workgroups share a CU and cover each other's exchanges.
//
// Every sum is added in the order of the passes these kernels replace (and which other head sizes and longer rows still
// take), so a model gives the same bits either way: twelve layers amplify one changed rounding to the size of bfloat16's
// error.  That is: the exponentials of a row (and dP P) per column modulo 64, in the order of the columns, then pairwise
// over column distances 32, 16, ... 1; P V and dS K over a quarter of the keys per partial sum where the batched product
// would have run in the small-product kernel, else over all keys in one chain.
#include "gemm_dma_impl.h"

namespace spb {
namespace {
using namespace gemm_dma_detail;
#pragma clang fp contract(off)   // every product is rounded where the passes stored it

constexpr int kHeadDim = 64, kQueries = 32;
constexpr int kTileBytes = kHeadDim * kRowBytes;            // 64 keys x 64 features
constexpr int kStageWave = kQueries * kRowBytes;            // 32 rows x 64 keys of P or dS on their way out, per wave
constexpr int kStageBytes = 4 * kStageWave;                 // also: the chain of partial row sums, maxima, totals
constexpr int kMaxAt = 8192, kTotalAt = kMaxAt + 4 * kQueries * 4;
constexpr size_t rows_lds(int tpw) { return (size_t)4 * tpw * kTileBytes + kStageBytes; }
static_assert(2 * rows_lds(2) <= 160 * 1024, "two workgroups share a CU");

typedef float row_regs[2][16];   // one 64-key tile of scores: [32-key block j][r]: key 32 j + 8 (r / 4) + 4 (lane / 32) + r % 4 of query lane % 32

// Column sums modulo 64, one per register and half-wave, added over column distances 32, 16, 8, 4 (the other half-wave), 2, 1.
__device__ __forceinline__ float butterfly(const row_regs& z) {
  float a[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) a[r] = z[0][r] + z[1][r];
#pragma unroll
  for (int r = 0; r < 8; ++r) a[r] = a[r] + a[r + 8];
#pragma unroll
  for (int r = 0; r < 4; ++r) a[r] = a[r] + a[r + 4];
#pragma unroll
  for (int r = 0; r < 4; ++r) a[r] = a[r] + __shfl_xor(a[r], 32, 64);
  return (a[0] + a[2]) + (a[1] + a[3]);
}

// One row-wise total per query, added up tile by tile along the keys: wave w continues the column sums wave w - 1 left
// in LDS.  add(t, z) adds tile t's registers to z.  All waves return the total of their lane's query.
template <int TPW, class Add>
__device__ __forceinline__ float chained_total(char* stage, int wave, int last_wave, int n_tiles, int lane, Add&& add) {
  float* total = reinterpret_cast<float*>(stage + kTotalAt);
  for (int w = 0; w <= last_wave; ++w) {
    if (wave == w) {
      row_regs z;
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          f32x4 v = {0.f, 0.f, 0.f, 0.f};
          if (w > 0) v = *reinterpret_cast<const f32x4*>(stage + (4 * j + g) * 1024 + lane * 16);
#pragma unroll
          for (int e = 0; e < 4; ++e) z[j][4 * g + e] = v[e];
        }
#pragma unroll
      for (int t = 0; t < TPW; ++t)
        if (t < n_tiles) add(t, z);
      if (w < last_wave) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int g = 0; g < 4; ++g)
            *reinterpret_cast<f32x4*>(stage + (4 * j + g) * 1024 + lane * 16) = f32x4{z[j][4 * g], z[j][4 * g + 1], z[j][4 * g + 2], z[j][4 * g + 3]};
      } else {
        const float t = butterfly(z);
        if (lane < kQueries) total[lane] = t;
      }
    }
    __syncthreads();
  }
  return total[lane & 31];
}

// 64 keys of one query row block in bfloat16 as MFMA operands, from registers packed two keys to a word (word 2 g + e of
// block j: keys 32 j + 8 g + 4 hh + 2 e, + 1): the two half-waves exchange halves so that each holds 8 consecutive keys,
// fragment kg = keys 16 kg + 8 hh + (0..7) - the order of k of a product that reads its operand from memory.
__device__ __forceinline__ void to_fragments(const uint32_t (&pp)[2][8], u32x4 (&frag)[4]) {
#pragma unroll
  for (int kg = 0; kg < 4; ++kg) {
    const int j = kg >> 1, g = 2 * (kg & 1);
    const auto x = __builtin_amdgcn_permlane32_swap(pp[j][2 * g], pp[j][2 * g + 2], false, false);
    const auto y = __builtin_amdgcn_permlane32_swap(pp[j][2 * g + 1], pp[j][2 * g + 3], false, false);
    frag[kg] = u32x4{x[0], y[0], x[1], y[1]};
  }
}

// The same 64 keys to memory as whole 128-byte row pieces, through the wave's staging rows.  LDS operations of one wave
// complete in order.  out: row q0, first key of the tile; keys: how many of its keys exist.
__device__ __forceinline__ void store_rows(const u32x4 (&frag)[4], char* mine, bf16_t* out, int ld, int rows, int keys, int lane) {
  lanes_together();
#pragma unroll
  for (int kg = 0; kg < 4; ++kg) *reinterpret_cast<u32x4*>(mine + lds_offset(lane & 31, 2 * kg + (lane >> 5))) = frag[kg];
  lanes_together();
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int row = it * 8 + (lane >> 3), chunk = lane & 7;
    if (row < rows && chunk * 8 < keys)
      *reinterpret_cast<u32x4*>(out + (size_t)row * ld + chunk * 8) = *reinterpret_cast<const u32x4*>(mine + lds_offset(row, chunk));
  }
  lanes_together();
}

// out[32 queries, 64 features] = sum over keys of frag x tile, by all four waves; tiles are KRow tiles in the wave's own
// part of LDS, which the partial results take over.  in_quarters: a wave's sum starts at zero and the waves' sums are added
// in wave order; otherwise wave w starts from wave w - 1's.
template <int TPW>
__device__ __forceinline__ void keys_product(const u32x4 (&frag)[TPW][4], char* tiles, int wave, int last_wave, int n_tiles, bool in_quarters,
                                             bf16_t* out, int ld, int rows, int lane) {
  const int qi = lane & 31, hh = lane >> 5;
  f32x16 o[2];
#pragma unroll
  for (int n = 0; n < 2; ++n)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[n][r] = 0.f;
  char* mine = tiles + wave * (TPW * kTileBytes);
  // 32 rows x 64 floats, the 16 chunks of a row permuted by the row so that neither the writes (32 rows at once) nor
  // the row-wise reads meet on a bank
  auto parked = [&](int w, int row, int chunk) { return reinterpret_cast<f32x4*>(tiles + w * (TPW * kTileBytes) + row * (kHeadDim * 4) + ((chunk ^ (row & 15)) << 4)); };
  auto multiply = [&]() {
#pragma unroll
    for (int t = 0; t < TPW; ++t)
      if (t < n_tiles) {
#pragma unroll
        for (int kg = 0; kg < 4; ++kg) {
          u32x4 a[1] = {frag[t][kg]}, b[2];
          b[0] = read_fragment<kHeadDim, Layout::KRow>(mine + t * kTileBytes, 0, kg, lane);
          b[1] = read_fragment<kHeadDim, Layout::KRow>(mine + t * kTileBytes, 32, kg, lane);
          fragments_ready(a, b);
#pragma unroll
          for (int n = 0; n < 2; ++n)
            o[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, b[n]), __builtin_bit_cast(bf16x8, a[0]), o[n], 0, 0, 0);
        }
      }
    lanes_together();
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int g = 0; g < 4; ++g) *parked(wave, qi, 8 * n + 2 * g + hh) = f32x4{o[n][4 * g], o[n][4 * g + 1], o[n][4 * g + 2], o[n][4 * g + 3]};
  };
  if (in_quarters) {
    if (wave <= last_wave) multiply();
  } else {
    for (int w = 0; w <= last_wave; ++w) {
      if (wave == w) {
        if (w > 0) {
#pragma unroll
          for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              const f32x4 v = *parked(w - 1, qi, 8 * n + 2 * g + hh);
#pragma unroll
              for (int e = 0; e < 4; ++e) o[n][4 * g + e] = v[e];
            }
        }
        multiply();
      }
      if (w < last_wave) __syncthreads();
    }
  }
  __syncthreads();
  // wave w finishes rows 8 w ..: one 16-byte piece per lane
  const int row = 8 * wave + (lane >> 3), c = (lane & 7) * 2;
  if (row >= rows) return;
  const int from = in_quarters ? 0 : last_wave;
  f32x4 v0 = *parked(from, row, c), v1 = *parked(from, row, c + 1);
  for (int w = from + 1; w <= last_wave; ++w) {
    v0 += *parked(w, row, c);
    v1 += *parked(w, row, c + 1);
  }
  const float v[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
  *reinterpret_cast<u32x4*>(out + (size_t)row * ld + c * 4) = pack_bf16x8(v);
}

struct RowBlock { int z, b, h, q0; };
// All query blocks of one (batch entry, head) on one XCD: they read the same keys and values.
__device__ __forceinline__ RowBlock row_block(int block, int n_blocks, int q_blocks, int heads) {
  const int run = xcd_tile(block, n_blocks);
  RowBlock rb;
  rb.z = run / q_blocks;
  rb.q0 = (run - rb.z * q_blocks) * kQueries;
  rb.b = rb.z / heads;
  rb.h = rb.z - rb.b * heads;
  return rb;
}

// Products of 32 rows at `a` (row q) with the 64-row tiles of keys at `b`, operands exchanged: s[t] as row_regs.  Rows beyond the
// sequence are clamped to its last one.
template <int TPW>
__device__ __forceinline__ void row_products(const bf16_t* a, int lda, const bf16_t* b, int ldb, int q, int key0, int seq, int n_tiles, int lane, f32x16 (&s)[TPW][2]) {
  const int half = (lane >> 5) * 8;
  u32x4 fa[4], fb[TPW][2][4];
  const bf16_t* arow = a + (size_t)min(q, seq - 1) * lda + half;
#pragma unroll
  for (int kg = 0; kg < 4; ++kg) fa[kg] = *reinterpret_cast<const u32x4*>(arow + 16 * kg);
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const bf16_t* brow = b + (size_t)min(key0 + 64 * t + 32 * j + (lane & 31), seq - 1) * ldb + half;
#pragma unroll
      for (int kg = 0; kg < 4; ++kg) fb[t][j][kg] = *reinterpret_cast<const u32x4*>(brow + 16 * kg);
    }
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[t][j][r] = 0.f;
#pragma unroll
      for (int kg = 0; kg < 4; ++kg)
        s[t][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fb[t][j][kg]), __builtin_bit_cast(bf16x8, fa[kg]), s[t][j], 0, 0, 0);
    }
}

// The wave's 64-row tiles of a [seq, 64] operand into its part of LDS, as KRow tiles; rows beyond the sequence are zeros.
template <int TPW>
__device__ __forceinline__ void issue_tiles(const bf16_t* base, int ld, int seq, int first, int n_tiles, char* tiles, int wave, int lane) {
  TileSource<kHeadDim, Layout::KRow, Gather::None, 1> src;
  ConvGeom none{};
  src.init(base, ld, 0, kHeadDim, 0, lane, first, none);
#pragma unroll
  for (int t = 0; t < TPW; ++t)
    if (t < n_tiles) src.issue(first + t, seq, tiles + (wave * TPW + t) * kTileBytes, 0, ld, none);
}

template <int TPW>
__global__ __launch_bounds__(256, 2) void attention_rows_fwd_kernel(const bf16_t* __restrict__ qkv, int ld_qkv, bf16_t* __restrict__ prob,
                                                                    bf16_t* __restrict__ ctx, int ld_ctx, int heads, int seq, int q_blocks,
                                                                    float scale, int in_quarters) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  char* tiles = lds;
  char* stage = lds + 4 * TPW * kTileBytes;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const RowBlock rb = row_block(blockIdx.x, gridDim.x, q_blocks, heads);
  const int hidden = heads * kHeadDim;
  const bf16_t* base = qkv + (size_t)rb.b * seq * ld_qkv + rb.h * kHeadDim;
  const int all_tiles = (seq + 63) >> 6, last_wave = (all_tiles - 1) / TPW;
  const int first = wave * TPW, n_tiles = min(max(all_tiles - first, 0), TPW);   // this wave's 64-key tiles
  const int key0 = first * 64;

  f32x16 s[TPW][2];
  row_products<TPW>(base, ld_qkv, base + hidden, ld_qkv, rb.q0 + (lane & 31), key0, seq, n_tiles, lane, s);
  issue_tiles<TPW>(base + 2 * hidden, ld_qkv, seq, first, n_tiles, tiles, wave, lane);   // V, while the softmax is worked out

  float m = -INFINITY;
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        // (the sequence is a multiple of 8: eight keys exist or do not together)
        s[t][j][r] = key0 + 64 * t + 32 * j + 8 * (r >> 2) < seq ? s[t][j][r] * scale : -INFINITY;
        m = fmaxf(m, s[t][j][r]);
      }
  m = fmaxf(m, __shfl_xor(m, 32, 64));
  float* maxima = reinterpret_cast<float*>(stage + kMaxAt);
  if (lane < kQueries) maxima[wave * kQueries + lane] = m;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 4; ++w) m = fmaxf(m, maxima[w * kQueries + (lane & 31)]);
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        s[t][j][r] = key0 + 64 * t + 32 * j + 8 * (r >> 2) < seq ? expf(s[t][j][r] - m) : 0.f;
  const float sum = chained_total<TPW>(stage, wave, last_wave, n_tiles, lane, [&](int t, row_regs& z) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) z[j][r] = z[j][r] + s[t][j][r];
  });
  const float inv = 1.f / sum;
  __syncthreads();   // the staging rows take over the chain's place
  u32x4 frag[TPW][4];
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    uint32_t pp[2][8];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 8; ++e) pp[j][e] = pack_bf16(s[t][j][2 * e] * inv, s[t][j][2 * e + 1] * inv);
    to_fragments(pp, frag[t]);
  }
  wait_own_loads<0>();   // V
  const int rows = seq - rb.q0;
  if (prob) {
#pragma unroll
    for (int t = 0; t < TPW; ++t)
      if (t < n_tiles)
        store_rows(frag[t], stage + wave * kStageWave, prob + ((size_t)rb.z * seq + rb.q0) * seq + key0 + 64 * t, seq, rows, seq - key0 - 64 * t, lane);
  }
  keys_product<TPW>(frag, tiles, wave, last_wave, n_tiles, in_quarters != 0, ctx + ((size_t)rb.b * seq + rb.q0) * ld_ctx + rb.h * kHeadDim, ld_ctx, rows, lane);
}

template <int TPW>
__global__ __launch_bounds__(256, 2) void attention_rows_bwd_kernel(const bf16_t* __restrict__ qkv, int ld_qkv, const bf16_t* __restrict__ prob,
                                                                    const bf16_t* __restrict__ dctx, int ld_ctx, bf16_t* __restrict__ dscore,
                                                                    bf16_t* __restrict__ dqkv, int heads, int seq, int q_blocks, float scale,
                                                                    int in_quarters) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  char* tiles = lds;
  char* stage = lds + 4 * TPW * kTileBytes;
  const int lane = threadIdx.x & 63, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const RowBlock rb = row_block(blockIdx.x, gridDim.x, q_blocks, heads);
  const int hidden = heads * kHeadDim;
  const bf16_t* base = qkv + (size_t)rb.b * seq * ld_qkv + rb.h * kHeadDim;
  const int all_tiles = (seq + 63) >> 6, last_wave = (all_tiles - 1) / TPW;
  const int first = wave * TPW, n_tiles = min(max(all_tiles - first, 0), TPW);
  const int key0 = first * 64, q = rb.q0 + (lane & 31);

  // P of this wave's keys as 16-byte pieces (keys 8 c .. 8 c + 7), the lower half-wave the even c and the upper the odd
  // ones; two v_permlane32_swap per pair of pieces hand each lane its half of both
  const bf16_t* prow = prob + ((size_t)rb.z * seq + min(q, seq - 1)) * seq;
  u32x4 praw[TPW][4];
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int key = key0 + 64 * t + 8 * (2 * c + hh);
      praw[t][c] = key < seq ? *reinterpret_cast<const u32x4*>(prow + key) : u32x4{0u, 0u, 0u, 0u};
    }
  f32x16 d[TPW][2];
  row_products<TPW>(dctx + (size_t)rb.b * seq * ld_ctx + rb.h * kHeadDim, ld_ctx, base + 2 * hidden, ld_qkv, q, key0, seq, n_tiles, lane, d);
  uint32_t pw[TPW][2][8];   // two keys to a word: word 2 g + e of block j holds keys 32 j + 8 g + 4 hh + 2 e, + 1
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const auto x = __builtin_amdgcn_permlane32_swap(praw[t][c][0], praw[t][c][2], false, false);
      const auto y = __builtin_amdgcn_permlane32_swap(praw[t][c][1], praw[t][c][3], false, false);
      const int g = 2 * (c & 1);
      pw[t][c >> 1][2 * g] = x[0]; pw[t][c >> 1][2 * g + 1] = y[0];
      pw[t][c >> 1][2 * g + 2] = x[1]; pw[t][c >> 1][2 * g + 3] = y[1];
    }
  auto p_of = [&](int t, int j, int r) { return __uint_as_float(r & 1 ? pw[t][j][r >> 1] & 0xFFFF0000u : pw[t][j][r >> 1] << 16); };
  issue_tiles<TPW>(base + hidden, ld_qkv, seq, first, n_tiles, tiles, wave, lane);   // K, while dS is worked out
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (key0 + 64 * t + 32 * j + 8 * (r >> 2) >= seq) d[t][j][r] = 0.f;
  const float dot = chained_total<TPW>(stage, wave, last_wave, n_tiles, lane, [&](int t, row_regs& z) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) z[j][r] = __builtin_fmaf(d[t][j][r], p_of(t, j, r), z[j][r]);
  });
  __syncthreads();   // the staging rows take over the chain's place
  u32x4 frag[TPW][4];
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    uint32_t ds[2][8];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 8; ++e)
        ds[j][e] = pack_bf16(p_of(t, j, 2 * e) * (d[t][j][2 * e] - dot) * scale, p_of(t, j, 2 * e + 1) * (d[t][j][2 * e + 1] - dot) * scale);
    to_fragments(ds, frag[t]);
  }
  wait_own_loads<0>();   // K
  const int rows = seq - rb.q0;
#pragma unroll
  for (int t = 0; t < TPW; ++t)
    if (t < n_tiles)
      store_rows(frag[t], stage + wave * kStageWave, dscore + ((size_t)rb.z * seq + rb.q0) * seq + key0 + 64 * t, seq, rows, seq - key0 - 64 * t, lane);
  keys_product<TPW>(frag, tiles, wave, last_wave, n_tiles, in_quarters != 0, dqkv + ((size_t)rb.b * seq + rb.q0) * ld_qkv + rb.h * kHeadDim, ld_qkv, rows, lane);
}

// dV = P^T dctx and dK = dS^T Q where their sums run in quarters: the tiles of the small-product kernel for all heads and both
// products in one launch.  On their own these were two launches of 768 workgroups (8 x 512 tokens, 12 heads) whose rings, 128 KB,
// leave a CU to one of them, and the tiles of a head lay on eight XCDs: 36 us each in the step.  A ring of one tile per wave lets two share a
// CU, and a head's tiles, which read the same P or dS columns and the same Q or dctx, lie on one XCD: 49 us for both (the step
// 5812 -> 5609 us).
__global__ __launch_bounds__(256) void attention_rows_keys_kernel(GemmParams dv, GemmParams dk) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const int tiles = dv.tiles_m * dv.tiles_n;
  const int run = xcd_tile(blockIdx.x, gridDim.x);
  const int z2 = run / tiles, tile = run - z2 * tiles;
  if (z2 & 1) small_product<64, 64, 1, Layout::KRow, Layout::KRow>(dk, tile, z2 >> 1, lds);
  else small_product<64, 64, 1, Layout::KRow, Layout::KRow>(dv, tile, z2 >> 1, lds);
}

bool aligned16(const void* a, const void* b, const void* c, const void* d = nullptr, const void* e = nullptr) {
  return ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b) | reinterpret_cast<uintptr_t>(c) | reinterpret_cast<uintptr_t>(d) |
           reinterpret_cast<uintptr_t>(e)) & 15) == 0;
}

// Whether the batched product [seq, 64] = [seq, seq] x [seq, 64] would run in the small-product kernel, whose four waves
// sum a quarter of k each.
int sums_in_quarters(int batch_heads, int seq) {
  GemmProblem g;
  g.M = seq; g.N = kHeadDim; g.K = seq; g.batch = batch_heads;
  return small_product_fits(g) ? 1 : 0;
}

template <class Kernel>
hipError_t prepare_rows(Kernel kernel, size_t lds_bytes) {
  return lds_bytes > 64 * 1024 ? raise_lds_limit(reinterpret_cast<const void*>(kernel), lds_bytes) : hipSuccess;
}

}  // namespace

// Rows of up to 128 keys are held whole by one wave each (attention.hip); more than 512 would not fit the registers.
bool attention_rows_accepts(int seq, int head_dim, int ld_qkv, int ld_ctx) {
  return head_dim == kHeadDim && seq > 128 && seq <= 512 && seq % 8 == 0 && ld_qkv % 8 == 0 && ld_ctx % 8 == 0;
}

hipError_t launch_attention_rows_fwd(const void* qkv, int ld_qkv, void* prob, void* ctx, int ld_ctx, int batch, int heads, int seq,
                                     int head_dim, float scale, hipStream_t stream) {
  if (!qkv || !ctx || batch <= 0 || heads <= 0 || !attention_rows_accepts(seq, head_dim, ld_qkv, ld_ctx) || !aligned16(qkv, ctx, prob)) return hipErrorInvalidValue;
  const int q_blocks = (seq + kQueries - 1) / kQueries, quarters = sums_in_quarters(batch * heads, seq);
  auto go = [&](auto kernel, size_t lds_bytes) -> hipError_t {
    if (hipError_t e = prepare_rows(kernel, lds_bytes); e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(batch * heads * q_blocks), dim3(256), lds_bytes, stream, static_cast<const bf16_t*>(qkv), ld_qkv,
                       static_cast<bf16_t*>(prob), static_cast<bf16_t*>(ctx), ld_ctx, heads, seq, q_blocks, scale, quarters);
    return hipGetLastError();
  };
  return seq <= 256 ? go(attention_rows_fwd_kernel<1>, rows_lds(1)) : go(attention_rows_fwd_kernel<2>, rows_lds(2));
}

hipError_t launch_attention_rows_bwd(const void* qkv, int ld_qkv, const void* prob, const void* dctx, int ld_ctx, void* dscore, void* dqkv,
                                     int batch, int heads, int seq, int head_dim, float scale, hipStream_t stream) {
  if (!qkv || !prob || !dctx || !dscore || !dqkv || batch <= 0 || heads <= 0 || !attention_rows_accepts(seq, head_dim, ld_qkv, ld_ctx) ||
      !aligned16(qkv, prob, dctx, dscore, dqkv))
    return hipErrorInvalidValue;
  const int q_blocks = (seq + kQueries - 1) / kQueries, quarters = sums_in_quarters(batch * heads, seq);
  auto go = [&](auto kernel, size_t lds_bytes) -> hipError_t {
    if (hipError_t e = prepare_rows(kernel, lds_bytes); e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(batch * heads * q_blocks), dim3(256), lds_bytes, stream, static_cast<const bf16_t*>(qkv), ld_qkv,
                       static_cast<const bf16_t*>(prob), static_cast<const bf16_t*>(dctx), ld_ctx, static_cast<bf16_t*>(dscore),
                       static_cast<bf16_t*>(dqkv), heads, seq, q_blocks, scale, quarters);
    return hipGetLastError();
  };
  return seq <= 256 ? go(attention_rows_bwd_kernel<1>, rows_lds(1)) : go(attention_rows_bwd_kernel<2>, rows_lds(2));
}

bool attention_rows_keys_accepts(const GemmProblem& dv, const GemmProblem& dk) {
  return small_product_fits(dv) && small_product_fits(dk) && gemm_dma_accepts(dv) && gemm_dma_accepts(dk) && dv.M == dk.M && dv.N == kHeadDim &&
         dk.N == kHeadDim && dv.batch == dk.batch && dv.batch <= 65535 && (long long)2 * dv.batch * ((dv.M + 63) / 64) <= 0x7FFFFFFF;
}

hipError_t launch_attention_rows_keys(const GemmProblem& dv, const GemmProblem& dk, hipStream_t stream) {
  if (!attention_rows_keys_accepts(dv, dk)) return hipErrorInvalidValue;
  const GemmParams pv = make_params(dv, 64, 64), pk = make_params(dk, 64, 64);
  constexpr size_t lds_bytes = small_product_lds(64, 64, 1);
  if (hipError_t e = prepare_rows(attention_rows_keys_kernel, lds_bytes); e != hipSuccess) return e;
  hipLaunchKernelGGL(attention_rows_keys_kernel, dim3(2 * dv.batch * pv.tiles_m * pv.tiles_n), dim3(256), lds_bytes, stream, pv, pk);
  return hipGetLastError();
}

}  // namespace spb
