// Softmax cross-entropy, forward and gradient in one pass over the logits (the loss that ends the
// forward pass and starts the backward pass, Sec. 1-2 of the paper).  Memory-bound: every logit is
// read from HBM once (the row stays in registers or L2 for the second sweep) and every gradient
// entry is written once.
#include "kernels.h"

namespace spb {
namespace {

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ void store_dz(float* p, float v) { *p = v; }
__device__ __forceinline__ void store_dz(uint16_t* p, float v) { *p = bf16_round(v); }

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// 65 to 2048 classes: one row per wave, the row in registers as VALS floats per lane (column = lane + 64 i), read once
// with every load in flight.  A lane adds its exponentials in the order of i, the lanes are added as a tree, and the
// gradient is exp(z - lse): the bits do not depend on VALS, and another order of the sum shows in where a bfloat16
// gradient rounds.  Bound by latency for few rows (256 x 100 on 64 workgroups: 3.2 us, 3.8 us with three sweeps) and by HBM
// for many (8192 x 2048 with mean_kernel and the events around them: 37 us, 53 us with three sweeps; rows in 16-byte
// pieces as below: 30 us, other bits).
template <typename DZ, int VALS>
__global__ __launch_bounds__(256) void softmax_xent_wave_kernel(const float* __restrict__ logits, int ldz, const int32_t* __restrict__ labels,
                                                                int rows, int classes, DZ* __restrict__ dz, int lddz,
                                                                float* __restrict__ row_loss) {
  const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + ((int)threadIdx.x >> 6);
  if (row >= rows) return;                           // whole waves, no barrier follows
  const float* z = logits + (size_t)row * ldz;
  const int y = labels[row];
  float v[VALS], m = -INFINITY, s = 0.f;
#pragma unroll
  for (int i = 0; i < VALS; ++i) {
    v[i] = -INFINITY;
    if (lane + 64 * i < classes) v[i] = z[lane + 64 * i];
  }
#pragma unroll
  for (int i = 0; i < VALS; ++i) m = fmaxf(m, v[i]);
  m = wave_max(m);
#pragma unroll
  for (int i = 0; i < VALS; ++i)
    if (lane + 64 * i < classes) s += expf(v[i] - m);
  s = wave_sum(s);
  const float lse = m + logf(s), inv_rows = 1.f / (float)rows;
  DZ* out = dz + (size_t)row * lddz;
#pragma unroll
  for (int i = 0; i < VALS; ++i) {
    const int c = lane + 64 * i;
    if (c < classes) store_dz(out + c, (expf(v[i] - lse) - (c == y ? 1.f : 0.f)) * inv_rows);
  }
  for (int c = classes + lane; c < lddz; c += 64) store_dz(out + c, 0.f);  // keep the pitch padding zero
  // a label outside [0, classes) contributes no target term instead of reading out of bounds
  if (lane == 0) row_loss[row] = lse - ((unsigned)y < (unsigned)classes ? z[y] : 0.f);
}

// Longer rows: one workgroup of 512 threads per row, the whole row in registers as VECS 16-byte vectors per thread: the
// logits are read from memory exactly once, with every load of the row in flight together; the exponentials are kept and
// only scaled for the gradient.  Columns between `classes` and the pitch count as minus infinity on the way in and come
// out as zero.  Bound by HBM (6 bytes per logit with a bfloat16 gradient) for large rows x classes, by latency below.
// VECS is the smallest that holds the row, because every vector costs its exponentials whether it holds columns or not
// (1000 rows of 4999 classes: 27.5 us with room for 32768 columns, 10.2 us with room for 8192; same bits).
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kXentThreads = 512;
__device__ __forceinline__ void store_dz4(float* p, const f32x4& v) { *reinterpret_cast<f32x4*>(p) = v; }
__device__ __forceinline__ void store_dz4(uint16_t* p, const f32x4& v) {
  *reinterpret_cast<uint2*>(p) = make_uint2(bf16_pack2(v[0], v[1]), bf16_pack2(v[2], v[3]));
}
template <typename DZ, int VECS>
__global__ __launch_bounds__(kXentThreads) void softmax_xent_kernel(const float* __restrict__ logits, int ldz, const int32_t* __restrict__ labels,
                                                                   int rows, int classes, DZ* __restrict__ dz, int lddz,
                                                                   float* __restrict__ row_loss) {
  __shared__ float red[kXentThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = blockIdx.x;
  const float* z = logits + (size_t)row * ldz;
  const int y = labels[row];
  f32x4 v[VECS];
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < VECS; ++i) {
    const int c = 4 * ((int)threadIdx.x + kXentThreads * i);
    v[i] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    if (c + 4 <= ldz) v[i] = *reinterpret_cast<const f32x4*>(z + c);
  }
#pragma unroll
  for (int i = 0; i < VECS; ++i) {
    const int c = 4 * ((int)threadIdx.x + kXentThreads * i);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (c + e >= classes) v[i][e] = -INFINITY;
      m = fmaxf(m, v[i][e]);
    }
  }
  m = wave_max(m);
  if (lane == 0) red[wave] = m;
  __syncthreads();
  m = red[0];
#pragma unroll
  for (int w = 1; w < kXentThreads / 64; ++w) m = fmaxf(m, red[w]);
  __syncthreads();
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < VECS; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) { v[i][e] = expf(v[i][e] - m); s += v[i][e]; }
  s = wave_sum(s);
  if (lane == 0) red[wave] = s;
  __syncthreads();
  s = red[0];
#pragma unroll
  for (int w = 1; w < kXentThreads / 64; ++w) s += red[w];
  const float scale = 1.f / (s * (float)rows), inv_rows = 1.f / (float)rows;
  DZ* out = dz + (size_t)row * lddz;
#pragma unroll
  for (int i = 0; i < VECS; ++i) {
    const int c = 4 * ((int)threadIdx.x + kXentThreads * i);
    if (c + 4 <= lddz) {
      f32x4 g = v[i] * scale;
      // a label outside [0, classes) contributes no target term
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (c + e == y && y < classes) g[e] -= inv_rows;
      store_dz4(out + c, g);
    }
  }
  if (threadIdx.x == 0) row_loss[row] = m + logf(s) - ((unsigned)y < (unsigned)classes ? z[y] : 0.f);
}

// Rows longer than any of those (or pitches and pointers that are not whole 16-byte pieces): one workgroup per row,
// three sweeps over it.
template <typename DZ>
__global__ __launch_bounds__(256) void softmax_xent_any_kernel(const float* __restrict__ logits, int ldz, const int32_t* __restrict__ labels,
                                                               int rows, int classes, DZ* __restrict__ dz, int lddz, float* __restrict__ row_loss) {
  __shared__ float red[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = blockIdx.x;
  const float* z = logits + (size_t)row * ldz;
  float m = -INFINITY;
  for (int c = threadIdx.x; c < classes; c += 256) m = fmaxf(m, z[c]);
  m = wave_max(m);
  if (lane == 0) red[wave] = m;
  __syncthreads();
  m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  __syncthreads();
  float s = 0.f;
  for (int c = threadIdx.x; c < classes; c += 256) s += expf(z[c] - m);
  s = wave_sum(s);
  if (lane == 0) red[wave] = s;
  __syncthreads();
  s = (red[0] + red[1]) + (red[2] + red[3]);
  const float lse = m + logf(s), inv_rows = 1.f / (float)rows;
  const int y = labels[row];
  DZ* out = dz + (size_t)row * lddz;
  for (int c = threadIdx.x; c < classes; c += 256) store_dz(out + c, (expf(z[c] - lse) - (c == y ? 1.f : 0.f)) * inv_rows);
  for (int c = classes + threadIdx.x; c < lddz; c += 256) store_dz(out + c, 0.f);  // keep the pitch padding zero
  if (threadIdx.x == 0) row_loss[row] = lse - ((unsigned)y < (unsigned)classes ? z[y] : 0.f);
}

// Adds the per-row losses in a fixed order (same result on every run) and stores the mean: thread t rows t, t + 256, ..., eight loads in flight at
// a time (one at a time: 4096 rows 5.5 us, 4.6 so; 1000 rows level).
__global__ __launch_bounds__(256) void mean_kernel(const float* __restrict__ row_loss, int rows, float* __restrict__ out) {
  __shared__ float red[4];
  float s = (int)threadIdx.x < rows ? row_loss[threadIdx.x] : 0.f;
  for (int base = threadIdx.x + 256; base < rows; base += 8 * 256) {
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = base + i * 256 < rows ? row_loss[base + i * 256] : 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) s += v[i];
  }
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) out[0] = ((red[0] + red[1]) + (red[2] + red[3])) / (float)rows;
}

// Few classes (a perceptron's 10-way head): a row takes lpr lanes (the power of two that holds its classes), so a
// wave works on 64 / lpr rows.  ONE_BLOCK: a single workgroup of 1024 threads takes all rows and adds up the mean as
// well (each wave's rows in order, then the waves in order), which saves the second launch; otherwise a workgroup
// takes 256 / lpr rows.
template <typename DZ, bool ONE_BLOCK>
__global__ __launch_bounds__(ONE_BLOCK ? 1024 : 256) void softmax_xent_few_kernel(const float* __restrict__ logits, int ldz,
                                                                                 const int32_t* __restrict__ labels, int rows, int classes, int lpr,
                                                                                 DZ* __restrict__ dz, int lddz, float* __restrict__ row_loss,
                                                                                 float* __restrict__ loss_out) {
  constexpr int kThreads = ONE_BLOCK ? 1024 : 256;
  __shared__ float red[kThreads / 64];
  const int sub = threadIdx.x % lpr, per_pass = kThreads / lpr;
  const float inv_rows = 1.f / (float)rows;
  float acc = 0.f;
  for (int base = blockIdx.x * per_pass; base < rows; base += gridDim.x * per_pass) {
    const int row = base + (int)threadIdx.x / lpr;
    const bool live = row < rows, mine = live && sub < classes;
    const float z = mine ? logits[(size_t)row * ldz + sub] : -INFINITY;
    const int y = live ? labels[row] : 0;
    float m = z;
    for (int o = lpr >> 1; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    float s = mine ? expf(z - m) : 0.f;
    for (int o = lpr >> 1; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (!live) continue;                       // no shuffles below
    const float lse = m + logf(s);
    DZ* out = dz + (size_t)row * lddz;
    if (mine) store_dz(out + sub, (expf(z - lse) - (sub == y ? 1.f : 0.f)) * inv_rows);
    for (int c = classes + sub; c < lddz; c += lpr) store_dz(out + c, 0.f);  // keep the pitch padding zero
    // a label outside [0, classes) contributes no target term
    const bool labelled = (unsigned)y < (unsigned)classes;
    if (labelled ? sub == y : sub == 0) {
      const float l = labelled ? lse - z : lse;
      if constexpr (ONE_BLOCK) acc += l;
      else row_loss[row] = l;
    }
  }
  if constexpr (ONE_BLOCK) {
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      float t = red[0];
#pragma unroll
      for (int w = 1; w < kThreads / 64; ++w) t += red[w];
      loss_out[0] = t * inv_rows;
    }
  }
}

__global__ __launch_bounds__(256) void fill_zero_kernel(uint32_t* __restrict__ p, size_t words) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < words; i += (size_t)gridDim.x * 256) p[i] = 0u;
}

}  // namespace

template <typename DZ>
static void enqueue_softmax_xent(const float* logits, int ldz, const int32_t* labels, int rows, int classes, DZ* dz, int lddz, float* row_loss,
                                 float* loss_out, hipStream_t stream) {
  if (classes <= 64) {
    int lpr = 1;
    while (lpr < classes) lpr <<= 1;
    // One workgroup and one launch while that is at most two passes over its 1024 threads: a pass is about 1.3 us of
    // latency, a second launch 2.4 us (4096 rows of 24 classes in one workgroup: 688 us; over 512 workgroups: 5 us).
    if ((long long)rows * lpr <= 2048) {
      hipLaunchKernelGGL((softmax_xent_few_kernel<DZ, true>), dim3(1), dim3(1024), 0, stream, logits, ldz, labels, rows, classes, lpr, dz, lddz, row_loss, loss_out);
      return;
    }
    const int per_block = 256 / lpr;
    hipLaunchKernelGGL((softmax_xent_few_kernel<DZ, false>), dim3((rows + per_block - 1) / per_block), dim3(256), 0, stream, logits, ldz, labels, rows, classes, lpr,
                       dz, lddz, row_loss, loss_out);
  } else if (classes <= 2048) {
#define SPB_XENT(VALS)                                                                                                                           \
  hipLaunchKernelGGL((softmax_xent_wave_kernel<DZ, VALS>), dim3((rows + 3) / 4), dim3(256), 0, stream, logits, ldz, labels, rows, classes, dz, \
                     lddz, row_loss)
    if (classes <= 128) SPB_XENT(2);
    else if (classes <= 256) SPB_XENT(4);
    else if (classes <= 512) SPB_XENT(8);
    else if (classes <= 1024) SPB_XENT(16);
    else SPB_XENT(32);
#undef SPB_XENT
  } else {
    const bool vec_ok = ldz % 4 == 0 && lddz % 4 == 0 && (reinterpret_cast<uintptr_t>(logits) & 15u) == 0 && (reinterpret_cast<uintptr_t>(dz) & 15u) == 0;
    const int width = ldz > lddz ? ldz : lddz;
#define SPB_XENT(VECS)                                                                                                                          \
  hipLaunchKernelGGL((softmax_xent_kernel<DZ, VECS>), dim3(rows), dim3(kXentThreads), 0, stream, logits, ldz, labels, rows, classes, dz, lddz, \
                     row_loss)
    if (!vec_ok || width > kXentThreads * 16 * 4)
      hipLaunchKernelGGL((softmax_xent_any_kernel<DZ>), dim3(rows), dim3(256), 0, stream, logits, ldz, labels, rows, classes, dz, lddz, row_loss);
    else if (width <= kXentThreads * 2 * 4) SPB_XENT(2);
    else if (width <= kXentThreads * 4 * 4) SPB_XENT(4);
    else if (width <= kXentThreads * 8 * 4) SPB_XENT(8);
    else SPB_XENT(16);
#undef SPB_XENT
  }
  hipLaunchKernelGGL(mean_kernel, dim3(1), dim3(256), 0, stream, row_loss, rows, loss_out);
}

hipError_t launch_softmax_xent(const float* logits, int ldz, const int32_t* labels, int rows, int classes,
                               void* dz, int lddz, DType dz_dtype, float* row_loss, float* loss_out,
                               hipStream_t stream) {
  if (!logits || !labels || !dz || !row_loss || !loss_out || rows <= 0 || classes <= 0 || ldz < classes || lddz < classes)
    return hipErrorInvalidValue;
  if (dz_dtype == DType::F32) enqueue_softmax_xent(logits, ldz, labels, rows, classes, static_cast<float*>(dz), lddz, row_loss, loss_out, stream);
  else enqueue_softmax_xent(logits, ldz, labels, rows, classes, static_cast<uint16_t*>(dz), lddz, row_loss, loss_out, stream);
  return hipGetLastError();
}

hipError_t launch_fill_zero(void* ptr, size_t bytes, hipStream_t stream) {
  if (!ptr || bytes % 4) return hipErrorInvalidValue;
  if (bytes == 0) return hipSuccess;
  const size_t words = bytes / 4;
  const int grid = (int)((words + 255) / 256 < 2048 ? (words + 255) / 256 : 2048);
  hipLaunchKernelGGL(fill_zero_kernel, dim3(grid), dim3(256), 0, stream, (uint32_t*)ptr, words);
  return hipGetLastError();
}

}  // namespace spb
