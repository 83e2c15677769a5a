// The result of a weight-streaming GEMM before its consumer: fp32 partial sums of C in
// planes [M][N], dealt as gemm_stream.hip describes.  A tile (tm rows x tn columns) has
// last worker - first worker + 1 planes, in K order.
#pragma once

#include <hip/hip_runtime.h>

#include "gemm.h"

namespace epic {

struct StreamSum {
  const float* partial;
  int M, N;
  int tm, tn, m_tiles, ks;   // rows and columns per tile, row tiles, K stages per tile (tile t = column tile * m_tiles + row tile)
  int units, G;          // K stages over all tiles, workers; units * G < 2^31
  int fixed;             // planes of every tile, where that is one number (the fields above are then unused)

  // worker w runs units [begin(w), begin(w + 1)); owner(v): the worker of unit v
  __host__ __device__ int begin(int w) const { return int(int64_t(w) * units / G); }
  __host__ __device__ int owner(int v) const {
    return int((uint32_t(v + 1) * uint32_t(G) + uint32_t(units) - 1) / uint32_t(units)) - 1;
  }
  __host__ __device__ int planes(int tile) const { return owner((tile + 1) * ks - 1) - owner(tile * ks) + 1; }

  // columns n .. n + 3 of row m (n % 4 == 0), the planes added in K order; four planes'
  // loads in flight at a time, the ones past the last repeating it and adding 0
  __device__ __forceinline__ float4 sum4(int m, int n) const {
    const int np = fixed > 0 ? fixed : planes(n / tn * m_tiles + m / tm);
    const size_t plane = size_t(M) * N;
    const float* p = partial + size_t(m) * N + n;
    float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int i = 0; i < np; i += 4) {
      float4 x[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) x[j] = *reinterpret_cast<const float4*>(p + (i + j < np ? i + j : np - 1) * plane);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bool ok = i + j < np;
        v.x += ok ? x[j].x : 0.0f;
        v.y += ok ? x[j].y : 0.0f;
        v.z += ok ? x[j].z : 0.0f;
        v.w += ok ? x[j].w : 0.0f;
      }
    }
    return v;
  }
};

// Enqueue the partial sums of g's product (g.partial: the GEMM workspace); returns how to sum them.
StreamSum launch_gemm_stream(const GemmArgs& g, hipStream_t stream);
// The same with 192- or 256-row tiles of 256 columns, each cut into equal parts of K
// (gemm_wide.hip); parts = 0 where that gives fewer than two.
struct WideSplit {
  int tm, parts;
};
WideSplit wide_split(const GemmArgs& g, int epi);
double wide_split_time(const WideSplit& s, int M, int N, int K);   // estimate in us, without the planes
StreamSum launch_gemm_wide_split(const GemmArgs& g, int epi, hipStream_t stream);
// The partial sums of a route that leaves them to the consumer.
inline bool is_partial(GemmRoute r) { return r == GemmRoute::kStream || r == GemmRoute::kSplit; }
inline StreamSum launch_gemm_partial(const GemmArgs& g, int epi, GemmRoute r, hipStream_t stream) {
  return r == GemmRoute::kSplit ? launch_gemm_wide_split(g, epi, stream) : launch_gemm_stream(g, stream);
}
// Whether the partial sums of a product of these sizes fit the GEMM workspace.
bool stream_fits(int M, int N, int K);
// Gate|up of a short row set in one round of whole tiles, with SwiGLU; whether it takes these sizes.
bool glu_fits(int M, int ffn, int K);
void launch_gemm_glu(const GemmArgs& g, hipStream_t stream);
// Enqueue the pass that sums the planes and runs g's epilogue.
void launch_stream_finish(const StreamSum& s, const GemmArgs& g, int epi, hipStream_t stream);
// The link write of a streamed Q|K|V product: the plan's private blocks and the layer's caches.
struct StreamWrite {
  const int32_t *priv_block, *priv_src, *priv_rows;
  int n_private;
  uint16_t *k_cache, *v_cache;
};
// Enqueue the rotary epilogue with k and v written to the private blocks (no re-rotation).
void launch_stream_rope_write(const StreamSum& s, const GemmArgs& g, const StreamWrite& w, hipStream_t stream);
// Enqueue x += the summed planes, then RMSNorm of x's rows into out_bf16 or out_f32.
void launch_rmsnorm_sum(const StreamSum& s, float* x, const uint16_t* w, uint16_t* out_bf16, float* out_f32, float eps,
                        hipStream_t stream);

}  // namespace epic
