// Elementwise parts of a decoder layer for the selected rows: RMSNorm and the
// rotary table at linked positions (the rotation itself runs in the epilogue of
// the fused Q|K|V projection, gemm.hip).
//
// RMSNorm: y = x / sqrt(mean(x^2) + eps) * w, fp32 statistics.
// Rotary embedding: the pair (i, i + D/2) of a head is rotated by angle
// pos * theta^(-2i/D), pos = the row's LINKED position (its place in the
// concatenated sequence), so recomputed chunk tokens see their non-initial
// positions (Sec. 4.2).  Angles are formed in float64: in float32,
// pos * inv_freq at pos ~ 1e5 would be off by ~1e-2 rad.
#include <algorithm>
#include <cmath>

#include "device_common.h"
#include "kernels.h"
#include "stream_sum.h"

namespace epic {

namespace {

constexpr int kNormThreads = 256;

struct RopeTable {
  const int32_t* s_pos;
  float2* cs;                // [n_rows][half_dim]
  int n_rows, half_dim;
  double log2_theta;
};

__device__ __forceinline__ float block_sum(float v, float* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) red[wave] = v;
  __syncthreads();
  float s = 0.0f;
#pragma unroll
  for (int w = 0; w < kNormThreads / 64; ++w) s += red[w];
  return s;
}

// The residual stream's pass between a GEMM that left partial sums and the next norm:
// h += the sums, then y = RMSNorm(h) w, the row kept in registers between the two.  One
// workgroup of 1024 threads per row: there are few rows, and a row's planes are many
// independent loads, so what bounds it is load latency.  The squares are added in
// rmsnorm_kernel's order (through LDS), so that a layer run on its own, whose last sum
// and next norm are separate launches, gives the same bits as inside a model call.
constexpr int kSumThreads = 1024;
constexpr int kSumKeep = 2;                             // float4 per thread: hidden <= 8192
__global__ __launch_bounds__(kSumThreads) void rmsnorm_sum_kernel(StreamSum s, float* __restrict__ x,
                                                                  const uint16_t* __restrict__ w,
                                                                  uint16_t* __restrict__ out_bf16,
                                                                  float* __restrict__ out_f32, float eps) {
  __shared__ float red[kNormThreads / 64];
  __shared__ float sq[kSumKeep * kSumThreads];
  const int row = blockIdx.x, hidden = s.N, n4 = hidden / 4;
  float4* xr = reinterpret_cast<float4*>(x + size_t(row) * hidden);
  float4 keep[kSumKeep];
#pragma unroll
  for (int k = 0; k < kSumKeep; ++k) {
    const int i = threadIdx.x + k * kSumThreads;
    if (i >= n4) break;
    const float4 o = xr[i], d = s.sum4(row, 4 * i);
    keep[k] = make_float4(o.x + d.x, o.y + d.y, o.z + d.z, o.w + d.w);
    xr[i] = keep[k];
    sq[i] = keep[k].x * keep[k].x + keep[k].y * keep[k].y + keep[k].z * keep[k].z + keep[k].w * keep[k].w;
  }
  __syncthreads();
  if (threadIdx.x < kNormThreads) {
    float ss = 0.0f;
    for (int i = threadIdx.x; i < n4; i += kNormThreads) ss += sq[i];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  }
  __syncthreads();
  float total = 0.0f;
#pragma unroll
  for (int v = 0; v < kNormThreads / 64; ++v) total += red[v];
  const float inv = 1.0f / sqrtf(total / float(hidden) + eps);
#pragma unroll
  for (int k = 0; k < kSumKeep; ++k) {
    const int i = threadIdx.x + k * kSumThreads;
    if (i >= n4) break;
    const uint2 wb = *reinterpret_cast<const uint2*>(w + 4 * i);
    const float y0 = keep[k].x * inv * bf16_to_f32(uint16_t(wb.x & 0xFFFFu));
    const float y1 = keep[k].y * inv * bf16_to_f32(uint16_t(wb.x >> 16));
    const float y2 = keep[k].z * inv * bf16_to_f32(uint16_t(wb.y & 0xFFFFu));
    const float y3 = keep[k].w * inv * bf16_to_f32(uint16_t(wb.y >> 16));
    if (out_bf16)
      *reinterpret_cast<uint2*>(out_bf16 + size_t(row) * hidden + 4 * i) =
          make_uint2(pack_bf16x2(y0, y1), pack_bf16x2(y2, y3));
    else
      *reinterpret_cast<float4*>(out_f32 + size_t(row) * hidden + 4 * i) = make_float4(y0, y1, y2, y3);
  }
}

// cs[row][i] = (cos, sin)(s_pos[row] * theta^(-2i/D)), float64 angle.
__device__ __forceinline__ void rope_entry(const RopeTable& t, int idx) {
  if (idx >= t.n_rows * t.half_dim) return;
  const int row = idx / t.half_dim, i = idx % t.half_dim;
  const double inv_freq = exp2(-double(2 * i) / double(2 * t.half_dim) * t.log2_theta);
  const double ang = double(t.s_pos[row]) * inv_freq;
  double s, c;
  sincos(ang, &s, &c);
  t.cs[idx] = make_float2(float(c), float(s));
}

// One workgroup per row; hidden % 4 == 0.  out_bf16 or out_f32 receives the row.
// START: the first norm of a call also fills the rotary table and clears the GEMM's
// counters, in workgroups past the rows' (each would be a dependent launch of its own,
// about 5 us in front of a layer).
template <bool START>
__global__ __launch_bounds__(kNormThreads) void rmsnorm_kernel(const float* __restrict__ x, const uint16_t* __restrict__ w,
                                                               uint16_t* __restrict__ out_bf16,
                                                               float* __restrict__ out_f32, int hidden, float eps,
                                                               RopeTable table, int* __restrict__ cnt, int n_cnt) {
  if constexpr (START) {
    const int extra = int(blockIdx.x) - table.n_rows;
    if (extra >= 0) {
      const int idx = extra * kNormThreads + threadIdx.x;
      rope_entry(table, idx);
      if (idx < n_cnt) cnt[idx] = 0;
      return;
    }
  }
  // The row stays in registers between the two passes (up to kKeep float4 per
  // thread, hidden <= 8192 at 256 threads); a longer row is read again.  The kept
  // part's loads, and its weights, are issued together from clamped indices (no
  // branch between them, so one wait covers them all); slots past the row add an
  // exact 0 to the sum of squares, which leaves it as the in-order sum of the row.
  constexpr int kKeep = 8;
  __shared__ float red[kNormThreads / 64];
  const int row = blockIdx.x;
  const float4* xr = reinterpret_cast<const float4*>(x + size_t(row) * hidden);
  const int n4 = hidden / 4;
  float4 keep[kKeep];
  uint2 keep_w[kKeep];
#pragma unroll
  for (int k = 0; k < kKeep; ++k) {
    const int i = min(int(threadIdx.x) + k * kNormThreads, n4 - 1);
    keep[k] = xr[i];
    keep_w[k] = *reinterpret_cast<const uint2*>(w + 4 * i);
  }
  float ss = 0.0f;
#pragma unroll
  for (int k = 0; k < kKeep; ++k) {
    const float sq = keep[k].x * keep[k].x + keep[k].y * keep[k].y + keep[k].z * keep[k].z + keep[k].w * keep[k].w;
    ss += int(threadIdx.x) + k * kNormThreads < n4 ? sq : 0.0f;
  }
  for (int i = threadIdx.x + kKeep * kNormThreads; i < n4; i += kNormThreads) {
    const float4 v = xr[i];
    ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
  }
  const float total = block_sum(ss, red);
  const float inv = 1.0f / sqrtf(total / float(hidden) + eps);
  auto put = [&](int i, const float4& v, const uint2& wb) {
    const float y0 = v.x * inv * bf16_to_f32(uint16_t(wb.x & 0xFFFFu));
    const float y1 = v.y * inv * bf16_to_f32(uint16_t(wb.x >> 16));
    const float y2 = v.z * inv * bf16_to_f32(uint16_t(wb.y & 0xFFFFu));
    const float y3 = v.w * inv * bf16_to_f32(uint16_t(wb.y >> 16));
    if (out_bf16) {
      *reinterpret_cast<uint2*>(out_bf16 + size_t(row) * hidden + 4 * i) =
          make_uint2(pack_bf16x2(y0, y1), pack_bf16x2(y2, y3));
    } else {
      *reinterpret_cast<float4*>(out_f32 + size_t(row) * hidden + 4 * i) = make_float4(y0, y1, y2, y3);
    }
  };
#pragma unroll
  for (int k = 0; k < kKeep; ++k) {
    const int i = threadIdx.x + k * kNormThreads;
    if (i < n4) put(i, keep[k], keep_w[k]);
  }
  for (int i = threadIdx.x + kKeep * kNormThreads; i < n4; i += kNormThreads)
    put(i, xr[i], *reinterpret_cast<const uint2*>(w + 4 * i));
}

}  // namespace

void launch_rmsnorm(const float* x, const uint16_t* w, uint16_t* out_bf16, float* out_f32, int rows, int hidden,
                    float eps, hipStream_t stream) {
  if (rows == 0) return;
  rmsnorm_kernel<false><<<rows, kNormThreads, 0, stream>>>(x, w, out_bf16, out_f32, hidden, eps, RopeTable{}, nullptr, 0);
}

void launch_rmsnorm_start(const float* x, const uint16_t* w, uint16_t* out_bf16, int rows, int hidden, float eps,
                          const int32_t* s_pos, float2* cs, int head_dim, double theta, int* cnt, int n_cnt,
                          hipStream_t stream) {
  if (rows == 0) return;
  const RopeTable t{s_pos, cs, rows, head_dim / 2, std::log2(theta)};
  const int extra = std::max(rows * (head_dim / 2), n_cnt);
  rmsnorm_kernel<true><<<rows + (extra + kNormThreads - 1) / kNormThreads, kNormThreads, 0, stream>>>(
      x, w, out_bf16, nullptr, hidden, eps, t, cnt, n_cnt);
}

void launch_rmsnorm_sum(const StreamSum& s, float* x, const uint16_t* w, uint16_t* out_bf16, float* out_f32, float eps,
                        hipStream_t stream) {
  if (s.N <= 4 * kSumKeep * kSumThreads) {
    rmsnorm_sum_kernel<<<s.M, kSumThreads, 0, stream>>>(s, x, w, out_bf16, out_f32, eps);
    return;
  }
  GemmArgs g{};                                         // longer rows: two passes
  g.C = x;
  launch_stream_finish(s, g, kResidual, stream);
  launch_rmsnorm(x, w, out_bf16, out_f32, s.M, s.N, eps, stream);
}

}  // namespace epic
