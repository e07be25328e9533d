// Image loss and dL/dI for the training step (L1 or L2 against a target).
#include "shade.h"

namespace g4d {
namespace {

using shade::loss_term;

// Bound by HBM for large images (33M values in 79 us, 5 TB/s); for small ones
// by the atomics, one per block, that meet on the loss's address (12 ns each).
// Hence few, larger blocks: 512 threads on at most 256 blocks, against 256 on
// 512 (as many threads in flight): 16.4 -> 13.6 us at 4.1M values, 7.3 -> 5.1
// at 0.4M, 79 either way at 33M. 1024 on 256: 12.4, 4.1, 81.5.
constexpr int kLossThreads = 512;
constexpr int kLossBlocks = 256;
__global__ void __launch_bounds__(kLossThreads) k_image_loss(int kind, uint64_t n, const float* __restrict__ img,
                                                             const float* __restrict__ tgt, float scale,
                                                             float* __restrict__ loss, float* __restrict__ grad) {
  __shared__ float s_part[kLossThreads / 64];
  float acc = 0.f;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  const uint64_t n4 = n / 4;
  const bool vec = ((reinterpret_cast<uintptr_t>(img) | reinterpret_cast<uintptr_t>(tgt) |
                     reinterpret_cast<uintptr_t>(grad)) & 15u) == 0;
  const uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (vec) {
    for (uint64_t i = i0; i < n4; i += stride) {
      const float4 a = reinterpret_cast<const float4*>(img)[i];
      const float4 b = reinterpret_cast<const float4*>(tgt)[i];
      float4 g;
      acc += loss_term(kind, a.x - b.x, scale, g.x);
      acc += loss_term(kind, a.y - b.y, scale, g.y);
      acc += loss_term(kind, a.z - b.z, scale, g.z);
      acc += loss_term(kind, a.w - b.w, scale, g.w);
      reinterpret_cast<float4*>(grad)[i] = g;
    }
  }
  // scalar path: everything when unaligned, else the tail after the float4 groups
  for (uint64_t i = (vec ? 4 * n4 : 0) + i0; i < n; i += stride) {
    float g;
    acc += loss_term(kind, img[i] - tgt[i], scale, g);
    grad[i] = g;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < kLossThreads / 64; ++w) t += s_part[w];
    atomicAdd(loss, scale * t);
  }
}

// One workgroup of 1024 threads: *loss += scale * (sum of the n per-tile
// partial sums), in a fixed order. Each thread keeps four 16-byte loads in
// flight per step (a single workgroup is latency-bound, not bandwidth-bound).
__global__ void __launch_bounds__(1024) k_loss_partials(const float* __restrict__ part, uint32_t n, float scale,
                                                         float* __restrict__ loss) {
  __shared__ float s_part[16];
  float acc = 0.f;
  const uint32_t n4 = n / 4;  // part is 256-byte aligned
  const float4* p4 = reinterpret_cast<const float4*>(part);
  for (uint32_t i0 = threadIdx.x; i0 < n4; i0 += 4 * 1024) {
    float4 q[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t i = i0 + (uint32_t)j * 1024;
      q[j] = i < n4 ? p4[i] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) acc += (q[j].x + q[j].y) + (q[j].z + q[j].w);
  }
  if (threadIdx.x < n - 4 * n4) acc += part[4 * n4 + threadIdx.x];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) t += s_part[w];
    *loss += scale * t;
  }
}

}  // namespace

void launch_loss_partials(const float* part, uint32_t n, float scale, float* loss, hipStream_t s) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_loss_partials, dim3(1), dim3(1024), 0, s, part, n, scale, loss);
}

void launch_image_loss(int kind, uint64_t n, const float* img, const float* tgt, float scale, float* loss,
                       float* grad, hipStream_t s) {
  if (n == 0) return;
  uint64_t g = (n / 4 + kLossThreads - 1) / kLossThreads;
  if (g > kLossBlocks) g = kLossBlocks;
  if (g < 1) g = 1;
  hipLaunchKernelGGL(k_image_loss, dim3((unsigned)g), dim3(kLossThreads), 0, s, kind, n, img, tgt, scale, loss, grad);
}

}  // namespace g4d
