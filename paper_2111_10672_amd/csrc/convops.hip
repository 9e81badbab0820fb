// Memory-bound kernels of the residual-CNN units (activations NHWC bfloat16, channel counts multiples of 8):
// the backward of "per-channel affine -> ReLU" with its per-channel reductions, the pools, channel padding of
// the 3-channel input, and the fixed-order sum of split-k partial products.  Each moves every tensor through
// HBM once, in 16-byte pieces along the channel index.
#include <algorithm>
#include <type_traits>

#include "kernels.h"

namespace spb {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void unpack8(const u32x4& w, float (&f)[8]) {
#pragma unroll
  for (int d = 0; d < 4; ++d) { f[2 * d] = __uint_as_float(w[d] << 16); f[2 * d + 1] = __uint_as_float(w[d] & 0xFFFF0000u); }
}
__device__ __forceinline__ uint32_t pack2(float lo, float hi) { return bf16_pack2(lo, hi); }
__device__ __forceinline__ u32x4 pack8(const float (&f)[8]) {
  u32x4 o;
#pragma unroll
  for (int d = 0; d < 4; ++d) o[d] = pack2(f[2 * d], f[2 * d + 1]);
  return o;
}
__device__ __forceinline__ float bf(uint16_t v) { return __uint_as_float(((uint32_t)v) << 16); }
__device__ __forceinline__ uint16_t to_bf16(float v) { return bf16_round(v); }

// Backward of z = scale * y + shift followed by an optional ReLU whose output is `act`:
//   dz = dout * [act > 0]   (dz = dout without act);   dy = scale * dz;   dsum = dz (optional)
//   partial[block][0][c] = sum over the block's rows of dz * y;   partial[block][1][c] = sum of dz
// Without y the latter alone, partial[block][c]; without partial neither.
// A workgroup takes a range of rows (blockIdx.x) of a slab of at most 256 channels (blockIdx.y), so that wide
// tensors still give many workgroups while the partial sums stay small next to the tensor.  Thread t owns chunk
// t % slab_chunks of the slab, rows (t / slab_chunks), (t / slab_chunks) + rows_per_pass, ...
constexpr int kAffineSlabChunks = 32;
__global__ __launch_bounds__(256) void affine_relu_bwd_kernel(const uint16_t* __restrict__ dout, const uint16_t* __restrict__ act,
                                                              const uint16_t* __restrict__ y, const uint16_t* __restrict__ scale,
                                                              uint16_t* __restrict__ dy, uint16_t* __restrict__ dsum,
                                                              float* __restrict__ partial, long long rows, int channels, int rows_per_block) {
  extern __shared__ float sh[];  // [rows_per_pass][slab_chunks][16]
  const int chunks = channels >> 3;
  const int slab_chunks = min(chunks, kAffineSlabChunks);
  const int rows_per_pass = 256 / slab_chunks;
  const int local_chunk = threadIdx.x % slab_chunks, lane_row = threadIdx.x / slab_chunks;
  const int chunk = blockIdx.y * slab_chunks + local_chunk;
  const bool active = lane_row < rows_per_pass && chunk < chunks;
  float s1[8], s0[8], sc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) { s1[e] = 0.f; s0[e] = 0.f; sc[e] = 0.f; }
  if (active) unpack8(*reinterpret_cast<const u32x4*>(scale + chunk * 8), sc);
  const long long first = (long long)blockIdx.x * rows_per_block;
  const long long last = min(rows, first + rows_per_block);
  if (active) {
    // four rows per trip, all their loads requested before the first is used
    auto finish = [&](size_t off, const u32x4& dw, const u32x4& yw, const u32x4& aw) {
      float d[8], o[8];
      unpack8(dw, d);
      if (act) {
        float a[8];
        unpack8(aw, a);
#pragma unroll
        for (int e = 0; e < 8; ++e) if (!(a[e] > 0.f)) d[e] = 0.f;
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) { s0[e] += d[e]; o[e] = sc[e] * d[e]; }
      if (y) {
        float yv[8];
        unpack8(yw, yv);
#pragma unroll
        for (int e = 0; e < 8; ++e) s1[e] += d[e] * yv[e];
      }
      *reinterpret_cast<u32x4*>(dy + off) = pack8(o);
      if (dsum) *reinterpret_cast<u32x4*>(dsum + off) = pack8(d);
    };
    // The three inputs are read here for the last time in the step (the gradient, the kept pre-affine output, the
    // kept activation): streaming loads, so they do not push the freshly written dy, which the next product reads,
    // out of the caches.  Four rows per trip, all their loads requested before the first is used.
    const u32x4 zero = {0u, 0u, 0u, 0u};
    auto fetch = [&](const uint16_t* base, size_t off) { return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + off)); };
    long long r = first + lane_row;
    const size_t pass = (size_t)rows_per_pass * channels;
    for (; r + 3 * rows_per_pass < last; r += 4 * rows_per_pass) {
      const size_t off0 = (size_t)r * channels + chunk * 8;
      u32x4 d[4], yv[4], a[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        d[u] = fetch(dout, off0 + u * pass);
        yv[u] = y ? fetch(y, off0 + u * pass) : zero;
        a[u] = act ? fetch(act, off0 + u * pass) : zero;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) finish(off0 + u * pass, d[u], yv[u], a[u]);
    }
    for (; r < last; r += rows_per_pass) {
      const size_t off = (size_t)r * channels + chunk * 8;
      finish(off, fetch(dout, off), y ? fetch(y, off) : zero, act ? fetch(act, off) : zero);
    }
  }
  if (!partial) return;
  if (lane_row < rows_per_pass) {  // lanes past the tensor's last chunk park zeros
    float* mine = sh + ((size_t)lane_row * slab_chunks + local_chunk) * 16;
#pragma unroll
    for (int e = 0; e < 8; ++e) { mine[e] = s1[e]; mine[8 + e] = s0[e]; }
  }
  __syncthreads();
  // column sums over the block's row lanes, in lane order
  const int slab_cols = slab_chunks * 8;
  for (int col = threadIdx.x; col < 2 * slab_cols; col += 256) {
    const int which = col / slab_cols, c = col % slab_cols;
    const int channel = blockIdx.y * slab_cols + c;
    if (channel >= channels) continue;
    float acc = 0.f;
    for (int l = 0; l < rows_per_pass; ++l) acc += sh[((size_t)l * slab_chunks + (c >> 3)) * 16 + which * 8 + (c & 7)];
    if (y) partial[((size_t)blockIdx.x * 2 + which) * channels + channel] = acc;
    else if (which) partial[(size_t)blockIdx.x * channels + channel] = acc;
  }
}

// ---- small fixed-order reductions, many per launch (see ReduceTask) ----
typedef float f32x4 __attribute__((ext_vector_type(4)));
// (512: a row of the longest reductions, a 3x3 convolution of 64 channels in 128 slices, is one workgroup's: see reduce_rows_block)
constexpr int kReduceThreads = 512;

// p[0] + p[stride] + ... (every step-th of count slices from `from` on, in order): eight requested at a time, and what is left over four, two and
// one at a time.  (An unrolled loop leaves up to seven to a loop that waits for each.)
template <typename V>
__device__ __forceinline__ V sum_slices(const V* __restrict__ p, size_t stride, int from, int count, int step) {
  V s = {};
  const V* at = p + (size_t)from * stride;
  const size_t hop = (size_t)step * stride;
  int left = from < count ? (count - from + step - 1) / step : 0;
  auto take = [&](auto n) {
    constexpr int N = decltype(n)::value;
    V v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = at[i * hop];
#pragma unroll
    for (int i = 0; i < N; ++i) s += v[i];
    at += N * hop;
    left -= N;
  };
  while (left >= 8) take(std::integral_constant<int, 8>{});
  if (left >= 4) take(std::integral_constant<int, 4>{});
  if (left >= 2) take(std::integral_constant<int, 2>{});
  if (left >= 1) take(std::integral_constant<int, 1>{});
  return s;
}

// Column sums of partial [count][columns].  A workgroup takes 16 neighbouring columns: thread (g, c) adds rows g, g + kGroups, ... of
// column c in order - the 16 threads of a group read 64 contiguous bytes, where one wavefront per column touched a cache line
// per lane - and the group sums of a column are added in group order: the same bits on every run.
template <int kGroups>
__device__ __forceinline__ void reduce_columns_block(unsigned block, const ReduceTask& k) {
  __shared__ float sh[kGroups][17];
  const bool pairs = k.kind == ReduceTask::kPairs;
  const int columns = pairs ? 2 * k.width : k.width;
  const int c = threadIdx.x & 15, g = threadIdx.x >> 4;
  const int col = block * 16 + c;
  sh[g][c] = col < columns ? sum_slices(k.partial + col, columns, g, k.count, kGroups) : 0.f;
  __syncthreads();
  if (threadIdx.x < 16 && col < columns) {
    float t = 0.f;
#pragma unroll
    for (int q = 0; q < kGroups; ++q) t += sh[q][c];
    if (col < k.width) k.out[col] = t;
    if (pairs && col >= k.width) k.out_b[col - k.width] = t;
    if (!pairs && k.out_b) k.out_b[col] = t;
  }
}

// out[j] = sum over slices of partial[slice][map(j)], slices added in index order; map drops padded input channels.
__device__ __forceinline__ void splitk_reduce_block(unsigned block, const float* __restrict__ partial, int slices, long long slice_stride,
                                                    float* __restrict__ out, long long numel, int cin, int cin_padded) {
  const long long j = (long long)block * kReduceThreads + threadIdx.x;
  if (j >= numel) return;
  const long long src = cin == cin_padded ? j : (j / cin) * cin_padded + (j % cin);
  out[j] = sum_slices(partial + src, slice_stride, 0, slices, 1);
}

// The same for tensors without channel padding, four neighbouring elements per thread.
__device__ __forceinline__ void splitk_reduce4_block(unsigned block, const f32x4* __restrict__ partial, int slices, long long slice_stride4,
                                                     f32x4* __restrict__ out, long long numel4) {
  const long long j = (long long)block * kReduceThreads + threadIdx.x;
  if (j < numel4) out[j] = sum_slices(partial + j, slice_stride4, 0, slices, 1);
}
// Many slices: 32 groups of four elements per workgroup and sixteen threads on each, which take every sixteenth slice; their sums are
// added in order.  (One thread a group: 9216 threads with 39 slices each, 18 to 27 us beside the input-gradient chain.)
constexpr int kWideSlices = 16;
__device__ __forceinline__ void splitk_reduce4_wide_block(unsigned block, const f32x4* __restrict__ partial, int slices, long long slice_stride4,
                                                          f32x4* __restrict__ out, long long numel4, f32x4* sh) {
  constexpr int kPhases = kReduceThreads / 32;
  const int c = threadIdx.x & 31, phase = threadIdx.x >> 5;
  const long long j = (long long)block * 32 + c;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  if (j < numel4) s = sum_slices(partial + j, slice_stride4, phase, slices, kPhases);
  sh[threadIdx.x] = s;
  __syncthreads();
  if (phase == 0 && j < numel4) {
#pragma unroll
    for (int q = 1; q < kPhases; ++q) s += sh[q * 32 + c];
    out[j] = s;
  }
}

// Output channels of a convolution's weight gradient (see make_conv_weight_task): S[k] = sum over the slices, dW[k] = scale * S[k],
// dscale = sum_k w[k] * S[k], k in groups of four.  k.threads threads (a power of two, 64 to 512) have a channel's whole row, so the dot product
// needs no second pass.  Rows of fewer groups than that share the slices out among threads / row of them per group, whose sums are added
// in order.  As few threads as leave each six loads or fewer, which sum_slices has in flight together (alone, 1024 rows of 64 groups in 12 slices and the
// unit's other sums: 11.4 us with a workgroup per row, 10.0 so).
__device__ __forceinline__ void reduce_rows_block(unsigned block, const ReduceTask& k, f32x4* sh) {
  __shared__ float dots[kReduceThreads / 64];
  const int n = k.width, t = threadIdx.x & (k.threads - 1), first = threadIdx.x - t;   // place in the row's threads, and theirs in the workgroup
  const int row = block * (kReduceThreads / k.threads) + first / k.threads;
  const bool exists = row < k.rows;
  const f32x4* partial = reinterpret_cast<const f32x4*>(k.partial) + (size_t)row * n;
  const uint2* w = static_cast<const uint2*>(k.weight) + (size_t)row * n;
  f32x4* out = reinterpret_cast<f32x4*>(k.out) + (size_t)row * n;
  const float sc = exists ? bf(static_cast<const uint16_t*>(k.scale)[row]) : 0.f;
  float dot = 0.f;
  auto finish = [&](int c, const f32x4& s) {
    const uint2 b = w[c];
    out[c] = s * sc;
    dot += __uint_as_float(b.x << 16) * s[0] + __uint_as_float(b.x & 0xFFFF0000u) * s[1] + __uint_as_float(b.y << 16) * s[2] +
           __uint_as_float(b.y & 0xFFFF0000u) * s[3];
  };
  auto sum = [&](int c, int from, int step) { return sum_slices(partial + c, k.stride, from, k.count, step); };
  const int phases = k.threads / n;
  if (phases <= 1) {
    if (exists)
      for (int c = t; c < n; c += k.threads) finish(c, sum(c, 0, 1));
  } else {
    const int phase = t / n, c = t - phase * n;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    if (exists && phase < phases) s = sum(c, phase, phases);
    sh[threadIdx.x] = s;
    __syncthreads();
    if (exists && t < n) {
      for (int q = 1; q < min(phases, k.count); ++q) s += sh[first + q * n + t];
      finish(t, s);
    }
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) dot += __shfl_xor(dot, d);
  if ((threadIdx.x & 63) == 0) dots[threadIdx.x >> 6] = dot;
  __syncthreads();
  if (exists && t == 0) {
    float v = dots[first / 64];
    for (int q = 1; q < k.threads / 64; ++q) v += dots[first / 64 + q];
    k.out_b[row] = v;
  }
}

// Several of the reductions above in one launch: the column sums of a unit's affine backward passes and the k-slice
// sums of its weight gradients are a handful of tiny kernels each bound by its launch; a table in the kernel
// arguments says which range of workgroups does which.
__device__ __forceinline__ int task_of(const ReduceTable& t, unsigned& block) {
  int i = 0;
  while (i + 1 < t.n && block >= t.end_block[i]) ++i;
  if (i) block -= t.end_block[i - 1];
  return i;
}
__global__ __launch_bounds__(kReduceThreads) void unit_reduce_kernel(ReduceTable t) {
  __shared__ f32x4 sh[kReduceThreads];
  unsigned block = blockIdx.x;
  const ReduceTask& k = t.task[task_of(t, block)];
  if (k.kind == ReduceTask::kPairs || k.kind == ReduceTask::kColumns) reduce_columns_block<kReduceThreads / 16>(block, k);
  else if (k.kind == ReduceTask::kRows4) reduce_rows_block(block, k, sh);
  else if (k.kind == ReduceTask::kSlices4Wide)
    splitk_reduce4_wide_block(block, reinterpret_cast<const f32x4*>(k.partial), k.count, k.stride, reinterpret_cast<f32x4*>(k.out), k.numel, sh);
  else if (k.kind == ReduceTask::kSlices4)
    splitk_reduce4_block(block, reinterpret_cast<const f32x4*>(k.partial), k.count, k.stride, reinterpret_cast<f32x4*>(k.out), k.numel);
  else splitk_reduce_block(block, k.partial, k.count, k.stride, k.out, k.numel, k.cin, k.cin_padded);
}
// A table of column sums only, at a pass's end with nothing beside it (the layer norms' of an encoder): bound by the start of its 2400
// workgroups where there are few rows to add and by HBM where there are many, so workgroups of half as many threads and no more LDS than these
// sums need (24 pairs of 768 columns: over 32 rows 8.0 us in the kernel above, 4.1 so; over 256 rows 20.1 and 15.0).
constexpr int kColumnThreads = 256;
__global__ __launch_bounds__(kColumnThreads) void column_sums_kernel(ReduceTable t) {
  unsigned block = blockIdx.x;
  const int i = task_of(t, block);
  reduce_columns_block<kColumnThreads / 16>(block, t.task[i]);
}

// The same with a bfloat16 result (the input gradient of a product whose k range was cut into slices, with the ReLU below it where there is one):
// eight neighbouring elements per thread, slices added in index order, one rounding at the end.
__global__ __launch_bounds__(256) void splitk_reduce_bf16_kernel(const f32x4* __restrict__ partial, int slices, long long slice_stride4,
                                                                 const u32x4* __restrict__ mask, u32x4* __restrict__ out, long long numel8) {
  const long long j = (long long)blockIdx.x * 256 + threadIdx.x;
  if (j >= numel8) return;
  const u32x4 m = mask ? mask[j] : u32x4{};
  const f32x4 lo = sum_slices(partial + 2 * j, slice_stride4, 0, slices, 1), hi = sum_slices(partial + 2 * j + 1, slice_stride4, 0, slices, 1);
  float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  if (mask) {
    float a[8];
    unpack8(m, a);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = a[e] > 0.f ? v[e] : 0.f;
  }
  out[j] = pack8(v);
}

// 3x3 window, stride 2, padding 1 (acting as -inf); the first maximum in row-major window order wins.
// which[n, oh, ow, c] (optional) = index 0..8 of the winning window position.
__global__ __launch_bounds__(256) void maxpool_fwd_kernel(const uint16_t* __restrict__ x, uint16_t* __restrict__ out, uint8_t* __restrict__ which,
                                                          int n, int h, int w, int c, int oh, int ow) {
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long long)n * oh * ow * c) return;
  const int ch = idx % c;
  long long t = idx / c;
  const int j = t % ow; t /= ow;
  const int i = t % oh;
  const int b = t / oh;
  float best = -INFINITY;
  int arg = 0;
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const int hi = 2 * i + r - 1, wi = 2 * j + s - 1;
      if ((unsigned)hi < (unsigned)h && (unsigned)wi < (unsigned)w) {
        const float v = bf(x[((size_t)(b * h + hi) * w + wi) * c + ch]);
        if (v > best) { best = v; arg = r * 3 + s; }
      }
    }
  out[idx] = to_bf16(best);
  if (which) which[idx] = (uint8_t)arg;
}

// The same, eight channels (16 bytes) per thread, for channel counts that are multiples of 8.
__global__ __launch_bounds__(256) void maxpool_fwd8_kernel(const uint16_t* __restrict__ x, uint16_t* __restrict__ out, uint8_t* __restrict__ which,
                                                           int n, int h, int w, int c, int oh, int ow) {
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  const int c8 = c >> 3;
  if (idx >= (long long)n * oh * ow * c8) return;
  const int chunk = idx % c8;
  long long t = idx / c8;
  const int j = t % ow; t /= ow;
  const int i = t % oh;
  const int b = t / oh;
  float best[8];
  int arg[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) { best[e] = -INFINITY; arg[e] = 0; }
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const int hi = 2 * i + r - 1, wi = 2 * j + s - 1;
      if ((unsigned)hi < (unsigned)h && (unsigned)wi < (unsigned)w) {
        float v[8];
        unpack8(*reinterpret_cast<const u32x4*>(x + ((size_t)(b * h + hi) * w + wi) * c + chunk * 8), v);
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (v[e] > best[e]) { best[e] = v[e]; arg[e] = r * 3 + s; }
      }
    }
  const size_t o = (size_t)idx * 8;
  *reinterpret_cast<u32x4*>(out + o) = pack8(best);
  if (which) {
    uint2 wbits;
    wbits.x = arg[0] | (arg[1] << 8) | (arg[2] << 16) | (arg[3] << 24);
    wbits.y = arg[4] | (arg[5] << 8) | (arg[6] << 16) | (arg[7] << 24);
    *reinterpret_cast<uint2*>(which + o) = wbits;
  }
}

// da[n, h, w, c] = sum of dout over the (at most 4) windows whose maximum sat at (h, w).
__global__ __launch_bounds__(256) void maxpool_bwd_kernel(const uint16_t* __restrict__ dout, const uint8_t* __restrict__ which,
                                                          uint16_t* __restrict__ da, int n, int h, int w, int c, int oh, int ow) {
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long long)n * h * w * c) return;
  const int ch = idx % c;
  long long t = idx / c;
  const int wi = t % w; t /= w;
  const int hi = t % h;
  const int b = t / h;
  float acc = 0.f;
  for (int i = (hi + 1) / 2 - (hi & 1); i <= (hi + 1) / 2; ++i) {     // windows with 2i-1 <= hi <= 2i+1: one for even hi, two for odd
    if (i < 0 || i >= oh) continue;
    for (int j = (wi + 1) / 2 - (wi & 1); j <= (wi + 1) / 2; ++j) {
      if (j < 0 || j >= ow) continue;
      const size_t o = ((size_t)(b * oh + i) * ow + j) * c + ch;
      if (which[o] == (hi - 2 * i + 1) * 3 + (wi - 2 * j + 1)) acc += bf(dout[o]);
    }
  }
  da[idx] = to_bf16(acc);
}

// pooled[n, c] = mean over the hw pixels of x[n, :, c]
__global__ __launch_bounds__(256) void avgpool_fwd_kernel(const uint16_t* __restrict__ x, uint16_t* __restrict__ pooled, int n, int hw, int c) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= n * c) return;
  const int b = idx / c, ch = idx % c;
  float acc = 0.f;
  for (int p = 0; p < hw; ++p) acc += bf(x[((size_t)b * hw + p) * c + ch]);
  pooled[idx] = to_bf16(acc / (float)hw);
}

// dx[n, p, c] = dpooled[n, c] / hw
__global__ __launch_bounds__(256) void avgpool_bwd_kernel(const uint16_t* __restrict__ dpooled, uint16_t* __restrict__ dx, int n, int hw, int c) {
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long long)n * hw * c) return;
  const int ch = idx % c;
  const int b = idx / ((long long)hw * c);
  dx[idx] = to_bf16(bf(dpooled[b * c + ch]) / (float)hw);
}

// out[row, 0..c_out) = in[row, 0..c_in) followed by zeros; a thread writes 8 channels of a row with one store (a store of 2 bytes per
// thread: 64 images of 224 x 224 x 3 53 us, 18 so)
__global__ __launch_bounds__(256) void pad_channels_kernel(const uint16_t* __restrict__ in, uint16_t* __restrict__ out, long long rows, int c_in, int c_out) {
  const int chunks = c_out >> 3;
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  const long long row = idx / chunks;
  if (row >= rows) return;
  const int first = (int)(idx - row * chunks) * 8;
  uint16_t v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = first + e < c_in ? in[row * c_in + first + e] : (uint16_t)0;
  u32x4 o;
#pragma unroll
  for (int d = 0; d < 4; ++d) o[d] = v[2 * d] | ((uint32_t)v[2 * d + 1] << 16);
  *reinterpret_cast<u32x4*>(out + idx * 8) = o;
}

unsigned blocks_for(long long n) { return (unsigned)((n + 255) / 256); }

}  // namespace

// rows handled by one workgroup of the affine backward kernel, and the size of its partial buffer
static int affine_slab_chunks(int channels) { return std::min(channels >> 3, kAffineSlabChunks); }
static int affine_slabs(int channels) { return ((channels >> 3) + affine_slab_chunks(channels) - 1) / affine_slab_chunks(channels); }
static int affine_rows_per_block(long long rows, int channels) {
  const int per_pass = 256 / affine_slab_chunks(channels);
  const long long row_blocks = std::max(1, 1024 / affine_slabs(channels));  // about a thousand workgroups in all
  long long want = (rows + row_blocks - 1) / row_blocks;
  want = (want + per_pass - 1) / per_pass * per_pass;
  return (int)std::max<long long>(want, 4LL * per_pass);
}
size_t affine_partial_floats(long long rows, int channels) {
  const int rpb = affine_rows_per_block(rows, channels);
  return (size_t)((rows + rpb - 1) / rpb) * 2 * channels;
}

hipError_t launch_affine_relu_bwd(const void* dout, const void* act, const void* y, const void* scale, void* dy, void* dsum,
                                  float* partial, float* dscale, float* dshift, long long rows, int channels, hipStream_t s, ReduceTask* deferred) {
  if (!dout || !scale || !dy || rows <= 0 || channels <= 0 || channels % 8 || channels > 2048) return hipErrorInvalidValue;
  if (partial ? !dshift || !deferred || (y && !dscale) : y != nullptr) return hipErrorInvalidValue;
  const int rpb = affine_rows_per_block(rows, channels);
  const int blocks = (int)((rows + rpb - 1) / rpb);
  const int slab_chunks = affine_slab_chunks(channels);
  const size_t lds = (size_t)(256 / slab_chunks) * slab_chunks * 16 * sizeof(float);
  hipLaunchKernelGGL(affine_relu_bwd_kernel, dim3(blocks, affine_slabs(channels)), dim3(256), lds, s, (const uint16_t*)dout, (const uint16_t*)act,
                     (const uint16_t*)y, (const uint16_t*)scale, (uint16_t*)dy, (uint16_t*)dsum, partial, rows, channels, rpb);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  if (partial && y) {   // the caller adds the column sums up later (launch_unit_reduce)
    deferred->kind = ReduceTask::kPairs; deferred->partial = partial; deferred->count = blocks; deferred->width = channels;
    deferred->out = dscale; deferred->out_b = dshift; deferred->blocks = reduce_pairs_blocks(channels);
  } else if (partial) {
    *deferred = make_columns_task(partial, blocks, channels, dshift, nullptr);
  }
  return hipSuccess;
}

ReduceTask make_columns_task(const float* partial, int count, int width, float* out, float* out_copy) {
  ReduceTask t;
  t.kind = ReduceTask::kColumns; t.partial = partial; t.count = count; t.width = width; t.out = out; t.out_b = out_copy;
  t.blocks = (unsigned)((width + 15) / 16);
  return t;
}

bool make_conv_weight_task(const float* partial, int slices, int channels, int row, const void* weight, const void* scale, float* dw, float* dscale,
                           ReduceTask* task) {
  if (!partial || !weight || !scale || !dw || !dscale || !task || slices < 1 || channels <= 0 || row <= 0 || row % 4 ||
      ((reinterpret_cast<uintptr_t>(partial) | reinterpret_cast<uintptr_t>(weight) | reinterpret_cast<uintptr_t>(dw)) & 15))
    return false;
  task->kind = ReduceTask::kRows4;
  task->partial = partial; task->count = slices; task->width = row / 4; task->stride = (long long)channels * (row / 4);
  task->weight = weight; task->scale = scale; task->out = dw; task->out_b = dscale;
  task->rows = channels;
  task->threads = 64;
  while (task->threads < kReduceThreads && (long long)task->width * slices > 6LL * task->threads) task->threads *= 2;
  task->blocks = (unsigned)((channels + kReduceThreads / task->threads - 1) / (kReduceThreads / task->threads));
  return true;
}

bool make_splitk_reduce_task(const float* partial, int slices, long long slice_stride, float* out, long long numel, int cin, int cin_padded,
                             ReduceTask* task) {
  if (!partial || !out || !task || slices < 1 || numel <= 0 || cin <= 0 || cin_padded < cin) return false;
  task->partial = partial; task->count = slices; task->out = out; task->out_b = nullptr; task->width = 0;
  task->cin = cin; task->cin_padded = cin_padded;
  if (cin == cin_padded && numel % 4 == 0 && slice_stride % 4 == 0 && (reinterpret_cast<uintptr_t>(partial) & 15) == 0 &&
      (reinterpret_cast<uintptr_t>(out) & 15) == 0) {
    task->kind = slices >= kWideSlices ? ReduceTask::kSlices4Wide : ReduceTask::kSlices4;
    task->stride = slice_stride / 4; task->numel = numel / 4;
  } else {
    task->kind = ReduceTask::kSlices; task->stride = slice_stride; task->numel = numel;
  }
  task->blocks = task->kind == ReduceTask::kSlices4Wide ? (unsigned)((task->numel + 31) / 32) : (unsigned)((task->numel + kReduceThreads - 1) / kReduceThreads);
  return true;
}

hipError_t launch_unit_reduce(const ReduceTask* tasks, int n, hipStream_t s) {
  if (!tasks || n < 1) return hipErrorInvalidValue;
  for (int first = 0; first < n; first += ReduceTable::kMax) {   // more than a table holds: several launches
    ReduceTable t;
    t.n = std::min(n - first, (int)ReduceTable::kMax);
    unsigned end = 0;
    bool columns_only = true;
    for (int i = 0; i < t.n; ++i) {
      t.task[i] = tasks[first + i];
      if (t.task[i].blocks == 0) return hipErrorInvalidValue;
      columns_only = columns_only && (t.task[i].kind == ReduceTask::kPairs || t.task[i].kind == ReduceTask::kColumns);
      end += t.task[i].blocks;
      t.end_block[i] = end;
    }
    if (columns_only) hipLaunchKernelGGL(column_sums_kernel, dim3(end), dim3(kColumnThreads), 0, s, t);
    else hipLaunchKernelGGL(unit_reduce_kernel, dim3(end), dim3(kReduceThreads), 0, s, t);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_splitk_reduce_bf16(const float* partial, int slices, long long slice_stride, const void* mask, void* out, long long numel, hipStream_t s) {
  if (!partial || !out || slices < 1 || numel <= 0 || numel % 8 || slice_stride % 4 || slice_stride < numel ||
      ((reinterpret_cast<uintptr_t>(partial) | reinterpret_cast<uintptr_t>(mask) | reinterpret_cast<uintptr_t>(out)) & 15))
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(splitk_reduce_bf16_kernel, dim3(blocks_for(numel / 8)), dim3(256), 0, s, reinterpret_cast<const f32x4*>(partial), slices,
                     slice_stride / 4, static_cast<const u32x4*>(mask), static_cast<u32x4*>(out), numel / 8);
  return hipGetLastError();
}

hipError_t launch_maxpool_fwd(const void* x, void* out, uint8_t* which, int n, int h, int w, int c, hipStream_t s) {
  if (!x || !out || n <= 0 || h <= 0 || w <= 0 || c <= 0) return hipErrorInvalidValue;
  const int oh = (h - 1) / 2 + 1, ow = (w - 1) / 2 + 1;
  const bool aligned = ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(out)) & 15) == 0 && (reinterpret_cast<uintptr_t>(which) & 7) == 0;
  if (c % 8 == 0 && aligned) {
    hipLaunchKernelGGL(maxpool_fwd8_kernel, dim3(blocks_for((long long)n * oh * ow * (c / 8))), dim3(256), 0, s, (const uint16_t*)x, (uint16_t*)out, which, n, h, w, c, oh, ow);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(maxpool_fwd_kernel, dim3(blocks_for((long long)n * oh * ow * c)), dim3(256), 0, s, (const uint16_t*)x, (uint16_t*)out, which, n, h, w, c, oh, ow);
  return hipGetLastError();
}

hipError_t launch_maxpool_bwd(const void* dout, const uint8_t* which, void* da, int n, int h, int w, int c, hipStream_t s) {
  if (!dout || !which || !da || n <= 0 || h <= 0 || w <= 0 || c <= 0) return hipErrorInvalidValue;
  const int oh = (h - 1) / 2 + 1, ow = (w - 1) / 2 + 1;
  hipLaunchKernelGGL(maxpool_bwd_kernel, dim3(blocks_for((long long)n * h * w * c)), dim3(256), 0, s, (const uint16_t*)dout, which, (uint16_t*)da, n, h, w, c, oh, ow);
  return hipGetLastError();
}

hipError_t launch_avgpool_fwd(const void* x, void* pooled, int n, int hw, int c, hipStream_t s) {
  if (!x || !pooled || n <= 0 || hw <= 0 || c <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(avgpool_fwd_kernel, dim3(blocks_for((long long)n * c)), dim3(256), 0, s, (const uint16_t*)x, (uint16_t*)pooled, n, hw, c);
  return hipGetLastError();
}

hipError_t launch_avgpool_bwd(const void* dpooled, void* dx, int n, int hw, int c, hipStream_t s) {
  if (!dpooled || !dx || n <= 0 || hw <= 0 || c <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(avgpool_bwd_kernel, dim3(blocks_for((long long)n * hw * c)), dim3(256), 0, s, (const uint16_t*)dpooled, (uint16_t*)dx, n, hw, c);
  return hipGetLastError();
}

hipError_t launch_pad_channels(const void* in, void* out, long long rows, int c_in, int c_out, hipStream_t s) {
  if (!in || !out || rows <= 0 || c_in <= 0 || c_out < c_in || c_out % 8 || (reinterpret_cast<uintptr_t>(out) & 15)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(pad_channels_kernel, dim3(blocks_for(rows * (c_out / 8))), dim3(256), 0, s, (const uint16_t*)in, (uint16_t*)out, rows, c_in, c_out);
  return hipGetLastError();
}

}  // namespace spb
