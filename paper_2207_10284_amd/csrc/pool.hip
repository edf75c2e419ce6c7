// Block means of Q, K, V: the scale-32 rows Q~, K~, V~ of MRA-2
// (Sec. 4.1 eq. recursive_pooling, Sec. 4.3 eq. recursive_pooling_V; five
// pairwise halvings of a 32-row block equal its plain mean).
//
// HBM-bound: every input byte is read once, 1/32 of it is written back.
// Two threads own one 16-byte column chunk of one 32-row block: one sums rows
// 0..15, the other rows 16..31 (each in row order, float32), and the mean is
// (first half + second half) / 32. A wave's load covers whole 128-byte row
// segments, so every HBM line fetched is fully used; two threads per chunk
// keep enough waves in flight to fill the GPU. No LDS, no barriers.
//
// The float32 gradient passes read Q, K, V and dZ as bfloat16 planes, which
// split_kernel writes.
#include "common.h"
#include "kernels.h"
#include "tile_ops.h"

namespace mra {

template <int DT>
__global__ __launch_bounds__(256) void pool_kernel(const void* __restrict__ x0,
                                                    const void* __restrict__ x1,
                                                    const void* __restrict__ x2,
                                                    float* __restrict__ y0,
                                                    float* __restrict__ y1,
                                                    float* __restrict__ y2,
                                                    long long chunks, int d) {
  const int which = blockIdx.y;
  const void* x = which == 0 ? x0 : (which == 1 ? x1 : x2);
  float* y = which == 0 ? y0 : (which == 1 ? y1 : y2);
  if (y == nullptr) return;
  constexpr int kPer = DT == BF16 ? 8 : 4;        // elements per 16-byte chunk
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int cpr = d / kPer;                        // chunks per row
  // thread t: block t / (2 cpr); within it, half (rows 16 half ..) and chunk
  const long long blk = t / (2 * cpr);
  const int i = (int)(t - blk * 2 * cpr), half = i / cpr, c = i - half * cpr;
  const bool active = t < 2 * chunks;              // whole (block, chunk) pairs: 2 cpr divides 64
  float acc[kPer];
#pragma unroll
  for (int e = 0; e < kPer; ++e) acc[e] = 0.0f;
  if (active) {
    const long long row0 = blk * kBlock + 16 * half;   // all heads flattened
    const u32x4* base = reinterpret_cast<const u32x4*>(x) + row0 * cpr + c;
#pragma unroll 8
    for (int r = 0; r < 16; ++r) {
      const u32x4 w = base[(long long)r * cpr];
      if constexpr (DT == BF16) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc[2 * e] += bf16_to_f32(w[e] & 0xFFFFu);
          acc[2 * e + 1] += bf16_to_f32(w[e] >> 16);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += __uint_as_float(w[e]);
      }
    }
  }
  // the second half's sums, from lane + cpr of the same wave
  float hi[kPer];
#pragma unroll
  for (int e = 0; e < kPer; ++e) hi[e] = __shfl_down(acc[e], cpr);
  if (!active || half != 0) return;
  constexpr float inv = 1.0f / kBlock;             // exact: power of two
  f32x4* out = reinterpret_cast<f32x4*>(y + blk * d + c * kPer);
#pragma unroll
  for (int v = 0; v < kPer / 4; ++v) {
    f32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (acc[4 * v + e] + hi[4 * v + e]) * inv;
    out[v] = o;
  }
}

// float32 tensors as three bfloat16 planes (split2), one thread per eight
// consecutive elements: reads 32 bytes, writes 16 to each plane. HBM-bound:
// 10 bytes per element.
__global__ __launch_bounds__(256) void split_kernel(const float* __restrict__ x0, const float* __restrict__ x1,
                                                    const float* __restrict__ x2, const float* __restrict__ x3,
                                                    u32x4* __restrict__ y0, u32x4* __restrict__ y1,
                                                    u32x4* __restrict__ y2, u32x4* __restrict__ y3,
                                                    long long chunks, int cpb) {
  const int which = blockIdx.y;
  const float* x = which == 0 ? x0 : (which == 1 ? x1 : (which == 2 ? x2 : x3));
  u32x4* y = which == 0 ? y0 : (which == 1 ? y1 : (which == 2 ? y2 : y3));
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  if (t >= chunks) return;
  const f32x4* src = reinterpret_cast<const f32x4*>(x) + 2 * t;
  const f32x4 a = src[0], b = src[1];
  const float v[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  u32x4 pl[3];
  split8(v, pl);
  const long long blk = t / cpb;                   // cpb: chunks of a 32-row block (4 d)
  u32x4* out = y + blk * 3 * cpb + (t - blk * cpb);
#pragma unroll
  for (int q = 0; q < 3; ++q) out[q * cpb] = pl[q];
}

hipError_t launch_split(const float* q, const float* k, const float* v, const float* g, void* qpl,
                        void* kpl, void* vpl, void* gpl, long long bh, int n, int d, hipStream_t stream) {
  const int cpb = kBlock * d / 8;
  const long long chunks = bh * (n / kBlock) * cpb;
  const dim3 grid((unsigned)((chunks + 255) / 256), 4);
  split_kernel<<<grid, 256, 0, stream>>>(q, k, v, g, static_cast<u32x4*>(qpl), static_cast<u32x4*>(kpl),
                                         static_cast<u32x4*>(vpl), static_cast<u32x4*>(gpl), chunks, cpb);
  return hipGetLastError();
}

hipError_t launch_pool(const void* q, const void* k, const void* v, float* qp, float* kp,
                       float* vp, long long bh, int n, int d, int dtype, hipStream_t stream) {
  const int per = dtype == BF16 ? 8 : 4;
  const long long chunks = bh * (n / kBlock) * (d / per);
  const int threads = 256;
  const long long blocks = (2 * chunks + threads - 1) / threads;   // two threads per chunk
  dim3 grid((unsigned)blocks, 3);
  if (dtype == BF16)
    pool_kernel<BF16><<<grid, threads, 0, stream>>>(q, k, v, qp, kp, vp, chunks, d);
  else
    pool_kernel<F32><<<grid, threads, 0, stream>>>(q, k, v, qp, kp, vp, chunks, d);
  return hipGetLastError();
}

// Debug aid (MRA_DEBUG_NANFILL, api.cpp): every 32-bit word of a buffer set to
// one pattern, grid-stride, plain vector stores.
__global__ void fill_u32_kernel(uint32_t* __restrict__ p, long long words, uint32_t pattern) {
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < words; i += stride) p[i] = pattern;
}

hipError_t launch_fill(void* p, size_t bytes, uint32_t pattern, hipStream_t stream) {
  const long long words = (long long)(bytes / 4);
  if (p == nullptr || words == 0) return hipSuccess;
  const int threads = 256;
  long long blocks = (words + threads - 1) / threads;
  if (blocks > 65536) blocks = 65536;
  fill_u32_kernel<<<(unsigned)blocks, threads, 0, stream>>>(static_cast<uint32_t*>(p), words, pattern);
  return hipGetLastError();
}

}  // namespace mra
