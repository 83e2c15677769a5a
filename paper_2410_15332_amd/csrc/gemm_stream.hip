// Weight-streaming GEMMs of short row sets: partial sums of C[M x N] = A[M x K] . W[N x K]^T.
//
// With few rows the projection's cost is reading W once.  What has to be hidden is
// memory latency, and every CU has to stream the same share of W.  So:
//   - tiles are TM x TN (TM = 32, 64 or 128 rows, several row tiles past 128; TN = 64 or
//     128), K in stages of 64, and the tiles' K stages in tile order are dealt in G equal
//     contiguous shares, whatever N and K are;
//   - a share's part of a tile goes to memory as an fp32 partial in a plane of its own
//     (plane p = p-th worker of the tile), and the kernel that consumes C sums the
//     planes in K order (stream_sum.h): no counters, no waiting on another workgroup,
//     and the sum is fused into the pass that reads C anyway (residual + RMSNorm,
//     SwiGLU, rotary embedding);
//   - a stage's four k-slices add to accumulators of their own (two of them where the 64
//     columns of a wavefront leave no registers for four), added up at the end of a part:
//     a chain of additions then has a quarter of the length, and its error grows with the
//     square root of that.  Relative error against float64 with one chain -> now (256-row
//     tiles cut along K, which these kernels replaced): 500 rows, N 3072, K 2048 2.0e-7 ->
//     1.05e-7 (1.14e-7); 64 rows, 16384, 2048 2.7e-7 -> 1.3e-7 (1.9e-7); 256 rows, 4096, 14336
//     3.7e-7 -> 2.6e-7 (2.6e-7).  It costs 0.2 to 0.5 us of 10 to 20;
//   - LDS is a ring of NS stages, loads issued NS - 1 stages ahead of their use (144 KB
//     in flight per CU), and a wavefront reads a stage's fragments while the previous
//     stage is on the matrix cores.
// Measured with its finishing pass (K = 4096, N = 4096; the cut 256 x 128 tiles before):
// 32 rows 21.2 -> 12.8 us, 128 rows 29.1 -> 15.6; K = 14336: 36.1 -> 26.8 and 47.5 -> 34.4,
// where the kernel alone reads W at 5.0 and 4.0 TB/s (a plain read probe: 5.5).  At 128
// rows the LDS (fragment reads and stage writes, about 700 cycles a 64-column stage)
// comes within a factor of two of the pace; 128-column tiles need 500.
//
// Stage layout: (TM + TN) rows of 128 bytes, A rows then W rows, in groups of 8 rows
// (1 KB, one load instruction); the eight 16-byte chunks of row r are XOR-swizzled by
// (r / 2) % 8, so the 16 lanes of each ds_read_b128 group touch distinct banks.
// Rows past M are read as row M - 1 and never stored.
#include <algorithm>

#include "device_common.h"
#include "gemm.h"
#include "gemm_device.h"
#include "link_tile.h"
#include "stream_sum.h"

namespace epic {

namespace {

constexpr int kBK = 64;
constexpr int kWorkers = 256;                           // one workgroup per CU
constexpr int kMinUnits = 4;                            // K stages per worker, at least

struct StreamArgs {
  const uint16_t* A;
  const uint16_t* W;
  float* partial;       // [planes][M][N]
  int M, N, K;
  StreamSum s;
  uint16_t* act;        // whole gate|up tiles: their result
  int ffn;
};

__device__ __forceinline__ float silu(float x) { return x * __builtin_amdgcn_rcpf(1.0f + fast_exp2(-x * kLog2e)); }

// GLU: a tile's columns are TN / 2 gate columns and the same up columns; worker w has the
// whole tile w and stores silu(gate) * up itself.  It starts at K stage w % ks and wraps:
// rows of W a multiple of 4 KB apart put the same stage of every row on the same few
// memory channels, so the workers have to be at different stages.  K = 4096, ffn 14336 (235
// MB): 32 rows 44.6 us (5.3 TB/s), all starting at stage 0 53.1; before, one round of 96 x 128
// tiles 47.4, and partial sums would take 51.8; 128 rows 51.0, 128 x 128 tiles 52.2, partial
// sums 63.1.
// All bounds say 512 threads: for fewer, the compiler has more than 256 registers, puts the
// accumulators into AGPRs and moves them there and back for every part (0.4 us more).
template <int TM, int TN, int NW, int CT, int NS, int NA, bool GLU = false>
__global__ __launch_bounds__(512, 1) void gemm_stream_kernel(StreamArgs g) {
  constexpr int NG = (TM + TN) / 8;                    // 1 KB row groups per stage
  constexpr int NL = NG / NW;                           // ... per wavefront
  static_assert(NG % NW == 0, "row groups per wavefront");
  static_assert((TM / 32) * (TN / 32 / CT) == NW, "a wavefront per 32 rows x 32 CT columns");
  static_assert(!GLU || CT == 2, "a wavefront holds the gate and up of its columns");
  constexpr int SB = (TM + TN) * 128;                  // bytes per stage
  __shared__ __attribute__((aligned(1024))) char lds[NS][SB];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int w = blockIdx.x, G = g.s.G;
  const int wr = G % 8 == 0 ? (w % 8) * (G / 8) + w / 8 : w;   // XCD-contiguous worker index
  const int ks = g.s.ks, m_tiles = g.s.m_tiles;
  const int u0 = g.s.begin(wr), u1 = g.s.begin(wr + 1);
  if (u0 >= u1) return;

  // ---- loads: row group gi of a stage, A rows first
  const int row_bytes = g.K * 2;
  const int lrow = lane >> 3;
  __amdgpu_buffer_rsrc_t rs[NL];
  int vo[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const bool is_a = wv * NL + i < TM / 8;
    rs[i] = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(is_a ? g.A : g.W), 0,
                                              (is_a ? g.M : g.N) * row_bytes, kBufWord3);
  }
  auto setup = [&](int tile) __attribute__((always_inline)) {
    const int nt = tile / m_tiles, mt = tile - nt * m_tiles;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int gi = wv * NL + i;
      const bool is_a = gi < TM / 8;
      const int row = (is_a ? gi : gi - TM / 8) * 8 + lrow;
      int gr = is_a ? min(mt * TM + row, g.M - 1) : nt * TN + row;
      if (GLU && !is_a) gr = nt * (TN / 2) + row % (TN / 2) + (row >= TN / 2 ? g.ffn : 0);
      vo[i] = gr * row_bytes + ((lane & 7) ^ ((row >> 1) & 7)) * 16;
    }
  };
  int du = u0, dtile = u0 / ks, dkt = u0 - dtile * ks;   // next unit to load
  setup(dtile);
  if (GLU) dkt = wr % ks;
  auto dma_next = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NL; ++i) dma16(rs[i], lds[buf] + (wv * NL + i) * 1024, vo[i], dkt * (kBK * 2));
    if (du + 1 < u1) {                                  // past the last unit: that one again
      ++du;
      if (++dkt == ks) {
        dkt = 0;
        if (!GLU) setup(++dtile);
      }
    }
  };

  // ---- compute: wavefront -> row block rt, first column block ct
  constexpr int WC = TN / 32 / CT;                      // wavefronts along N
  const int rt = wv / WC, ct = wv % WC * (GLU ? 1 : CT);
  constexpr int CS = GLU ? WC : 1;                      // 32-column blocks between a wavefront's CT
  const int lbase = (lane & 31) * 128, lsw = (lane >> 1) & 7, half = lane >> 5;
  const int abase = rt * 4096 + lbase, bbase = (TM / 32 + ct) * 4096 + lbase;

#pragma unroll
  for (int b = 0; b < NS - 1; ++b) dma_next(b);
  int buf = 0, u = u0, tile = u0 / ks;
  while (u < u1) {
    const int ue = min(u1, (tile + 1) * ks);
    f32x16 sums[NA][CT];                                // k-slice i of a stage adds to sums[i % NA]
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int j = 0; j < CT; ++j) sums[i][j] = f32x16{};
    // the k-slices of unit u are read while unit u - 1 is on the matrix cores
    struct Frags {
      bf16x8 a[4], b[4][CT];
    } f0, f1;
    auto fetch = [&](Frags& f) __attribute__((always_inline)) {
      wait_vmem<(NS - 2) * NL>();                     // this wavefront's loads of unit u
      barrier_lds();                                 // everyone's; and unit u - 1 is read
      dma_next(buf == 0 ? NS - 1 : buf - 1);            // unit u + NS - 1, where u - 1 was
      const char* p = lds[buf];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int c = ((2 * i + half) ^ lsw) * 16;
        f.a[i] = *reinterpret_cast<const bf16x8*>(p + abase + c);
#pragma unroll
        for (int j = 0; j < CT; ++j) f.b[i][j] = *reinterpret_cast<const bf16x8*>(p + bbase + j * CS * 4096 + c);
      }
      buf = buf + 1 == NS ? 0 : buf + 1;
      __builtin_amdgcn_sched_barrier(0);
    };
    auto mma = [&](const Frags& f) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j) sums[i % NA][j] = mfma_32x32x16(f.a[i], f.b[i][j], sums[i % NA][j]);
      __builtin_amdgcn_sched_barrier(0);
    };
    fetch(f0);
    for (++u; u + 1 < ue; u += 2) {
      fetch(f1);
      mma(f0);
      fetch(f0);
      mma(f1);
    }
    if (u < ue) {
      ++u;
      fetch(f1);
      mma(f0);
      mma(f1);
    } else {
      mma(f0);
    }
    f32x16 acc[CT];
#pragma unroll
    for (int j = 0; j < CT; ++j) {
      acc[j] = sums[0][j];
      if constexpr (NA == 2) acc[j] += sums[1][j];
      if constexpr (NA == 4) acc[j] = (acc[j] + sums[1][j]) + (sums[2][j] + sums[3][j]);
    }
    // this worker's part of the tile: plane (worker - first worker of the tile)
    const int nt = tile / m_tiles, mt = tile - nt * m_tiles;
    const int m0 = mt * TM + rt * 32 + half * 4;
    if constexpr (GLU) {
      const __amdgpu_buffer_rsrc_t ro =
          __builtin_amdgcn_make_buffer_rsrc(g.act, 0, g.M * g.ffn * 2, kBufWord3);   // rows past M: dropped
      const int n = nt * (TN / 2) + ct * 32 + (lane & 31);
#pragma unroll
      for (int r = 0; r < 16; ++r)
        __builtin_amdgcn_raw_buffer_store_b16(uint16_t(pack_bf16x2(silu(acc[0][r]) * acc[1][r], 0.0f)), ro,
                                              ((m0 + (r >> 2) * 8 + (r & 3)) * g.ffn + n) * 2, 0, 0);
      ++tile;
      continue;
    }
    const int plane = wr - g.s.owner(tile * ks);
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
        g.partial + size_t(plane) * g.M * g.N, 0, g.M * g.N * 4, kBufWord3);   // rows past M: dropped
    const int n = nt * TN + ct * 32 + (lane & 31);
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
      for (int j = 0; j < CT; ++j) {
        const float x = acc[j][r];
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), ro,
                                              ((m0 + (r >> 2) * 8 + (r & 3)) * g.N + n + j * 32) * 4, 0, 0);
      }
    ++tile;
  }
  wait_vmem<0>();                                     // no load may land in LDS after the workgroup ends
}

// C = sum of the planes, stored (kStoreF32) or added (kResidual): four columns per thread.
template <int EPI>
__global__ __launch_bounds__(256) void stream_finish_kernel(StreamSum s, float* __restrict__ c, uint16_t* __restrict__ act,
                                                            int ffn) {
  const int n4 = (EPI == kSwiGLU ? ffn : s.N) / 4;
  const int idx = blockIdx.x * 256 + threadIdx.x;
  const int m = idx / n4, n = (idx - m * n4) * 4;
  if (m >= s.M) return;
  float4 v = s.sum4(m, n);
  if constexpr (EPI == kSwiGLU) {
    const float4 up = s.sum4(m, ffn + n);
    *reinterpret_cast<uint2*>(act + size_t(m) * ffn + n) =
        make_uint2(pack_bf16x2(silu(v.x) * up.x, silu(v.y) * up.y), pack_bf16x2(silu(v.z) * up.z, silu(v.w) * up.w));
  } else {
    float4* p = reinterpret_cast<float4*>(c + size_t(m) * s.N + n);
    if constexpr (EPI == kResidual) {
      const float4 o = *p;
      v = make_float4(o.x + v.x, o.y + v.y, o.z + v.z, o.w + v.w);
    }
    *p = v;
  }
}

// Four rotary pairs (i .. i + 3, i + D/2 ..) of a head of a row, summed and
// perhaps rotated by the row's table.
__device__ __forceinline__ void sum_pairs(const StreamSum& s, const float2* cs, int m, int col, int D, int i, bool rotate,
                                          uint2& lo, uint2& hi) {
  const int hd2 = D / 2;
  const float4 a = s.sum4(m, col + i), b = s.sum4(m, col + hd2 + i);
  float x1[4] = {a.x, a.y, a.z, a.w}, x2[4] = {b.x, b.y, b.z, b.w};
  if (rotate) {
    const float4* p = reinterpret_cast<const float4*>(cs + size_t(m) * hd2 + i);
    const float4 t0 = p[0], t1 = p[1];
    const float c[4] = {t0.x, t0.z, t1.x, t1.z}, sn[4] = {t0.y, t0.w, t1.y, t1.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float y1 = x1[e] * c[e] - x2[e] * sn[e], y2 = x2[e] * c[e] + x1[e] * sn[e];
      x1[e] = y1;
      x2[e] = y2;
    }
  }
  lo = make_uint2(pack_bf16x2(x1[0], x1[1]), pack_bf16x2(x1[2], x1[3]));
  hi = make_uint2(pack_bf16x2(x2[0], x2[1]), pack_bf16x2(x2[2], x2[3]));
}

// q, k, v of the fused Q|K|V projection: q and k heads rotated at each row's linked
// position (pairs (i, i + D/2)), v heads as they are; bf16.  A thread takes four pairs.
__global__ __launch_bounds__(256) void stream_rope_kernel(StreamSum s, GemmArgs g) {
  const int D = g.head_dim, hd2 = D / 2, per_row = s.N / 8;
  const int idx = blockIdx.x * 256 + threadIdx.x;
  const int m = idx / per_row, r = idx - m * per_row;
  if (m >= s.M) return;
  const int head = r / (hd2 / 4), i = (r - head * (hd2 / 4)) * 4;
  uint16_t* base;
  int heads, hd;
  if (head < g.hq) base = g.q, heads = g.hq, hd = head;
  else if (head < g.hq + g.hkv) base = g.k, heads = g.hkv, hd = head - g.hq;
  else base = g.v, heads = g.hkv, hd = head - g.hq - g.hkv;
  uint2 lo, hi;
  sum_pairs(s, g.cs, m, head * D, D, i, head < g.hq + g.hkv, lo, hi);
  uint16_t* o = base + (size_t(m) * heads + hd) * D + i;
  *reinterpret_cast<uint2*>(o) = lo;
  *reinterpret_cast<uint2*>(o + hd2) = hi;
}

// The same fused with the link write: k and v go straight to the private blocks of the
// linked cache, which a launch of their own wrote before (about 5 us of a 155 us decode
// layer, as long as any dependent launch takes).  The first n_private * hkv workgroups
// build a (block, KV head) each, as link_write_kernel does; the rest write q.
template <int D>
__global__ __launch_bounds__(2 * D) void stream_rope_write_kernel(StreamSum s, GemmArgs g, StreamWrite w) {
  __shared__ VTile<D> vt;
  const int tid = threadIdx.x;
  const int n_kv = w.n_private * g.hkv;
  if (int(blockIdx.x) >= n_kv) {              // q: four pairs per thread
    const int per_row = g.hq * (D / 8);
    const int idx = (blockIdx.x - n_kv) * 2 * D + tid;
    const int m = idx / per_row, r = idx - m * per_row;
    if (m >= s.M) return;
    const int head = r / (D / 8), i = (r - head * (D / 8)) * 4;
    uint2 lo, hi;
    sum_pairs(s, g.cs, m, head * D, D, i, true, lo, hi);
    uint16_t* o = g.q + (size_t(m) * g.hq + head) * D + i;
    *reinterpret_cast<uint2*>(o) = lo;
    *reinterpret_cast<uint2*>(o + D / 2) = hi;
    return;
  }
  const int pv = blockIdx.x / g.hkv, h = blockIdx.x % g.hkv;
  const int dst = w.priv_block[pv], src = w.priv_src[pv];
  const int o = tid / (D / 8), c = tid % (D / 8);          // slot; K pairs 4 c .., V dims 8 c ..
  const int r = w.priv_rows[pv * 16 + o];
  const size_t at = ((size_t(src < 0 ? 0 : src) * g.hkv + h) * 16) * D;
  uint2 lo = make_uint2(0, 0), hi = lo;
  uint4 v = make_uint4(0, 0, 0, 0);
  if (r >= 0) {
    sum_pairs(s, g.cs, r, (g.hq + h) * D, D, c * 4, true, lo, hi);
    const int col = (g.hq + g.hkv + h) * D + c * 8;
    const float4 x = s.sum4(r, col), y = s.sum4(r, col + 4);
    v = make_uint4(pack_bf16x2(x.x, x.y), pack_bf16x2(x.z, x.w), pack_bf16x2(y.x, y.y), pack_bf16x2(y.z, y.w));
  } else if (src >= 0) {
    lo = *reinterpret_cast<const uint2*>(w.k_cache + at + o * D + c * 4);
    hi = *reinterpret_cast<const uint2*>(w.k_cache + at + o * D + D / 2 + c * 4);
  }
  if (src >= 0) {
    vt.load(w.v_cache + at, tid);
    __syncthreads();
  }
  if (r >= 0 || src < 0) vt.put(o, c * 8, v);
  __syncthreads();
  const size_t to = ((size_t(dst) * g.hkv + h) * 16) * D;
  *reinterpret_cast<uint2*>(w.k_cache + to + o * D + c * 4) = lo;
  *reinterpret_cast<uint2*>(w.k_cache + to + o * D + D / 2 + c * 4) = hi;
  vt.store(w.v_cache + to, tid);
}

int cdiv(int a, int b) { return (a + b - 1) / b; }

StreamSum make_sum(int M, int N, int K, int TM, int TN, const float* partial) {
  StreamSum s{};
  s.partial = partial;
  s.M = M, s.N = N;
  s.tm = TM, s.tn = TN;
  s.m_tiles = cdiv(M, TM);
  s.ks = K / kBK;
  s.units = s.m_tiles * (N / TN) * s.ks;
  s.G = s.units < kWorkers * kMinUnits ? cdiv(s.units, kMinUnits) : kWorkers;
  return s;
}

// Rows past 64: 128-column tiles where every worker then still gets kWideUnits stages.
// They read and stage two thirds of the operand bytes of 64-column tiles per product,
// but cut each tile into twice the planes (128 rows, K = 14336: 39.3 -> 35.7 us; K = 4096,
// 8 stages per worker: 18.1 -> 19.9).
constexpr int kWideUnits = 16;
bool wide_tiles(int M, int N, int K) {
  return int64_t(cdiv(M, 128)) * (N / 128) * (K / kBK) >= int64_t(kWideUnits) * kWorkers;
}

template <int TM, int TN, int NW, int CT, int NS, int NA>
StreamSum launch_tm(const GemmArgs& g, hipStream_t stream) {
  StreamArgs a{};
  a.A = g.A, a.W = g.W, a.partial = g.partial, a.M = g.M, a.N = g.N, a.K = g.K;
  a.s = make_sum(g.M, g.N, g.K, TM, TN, g.partial);
  gemm_stream_kernel<TM, TN, NW, CT, NS, NA><<<a.s.G, NW * 64, 0, stream>>>(a);
  return a.s;
}

}  // namespace

// Planes of a tile: at most ceil(ks / stages per worker) + 1 workers.  They have half of the
// workspace: products whose planes need more were not measured here.
bool stream_fits(int M, int N, int K) {
  const int tm = M <= 32 ? 32 : M <= 64 ? 64 : 128;
  const int64_t units = int64_t(cdiv(M, tm)) * (N / 64) * (K / kBK);
  if (units >= (1 << 23)) return false;                 // 32-bit arithmetic of StreamSum::owner
  const int64_t per = std::max<int64_t>(units / 2 / kWorkers, 1);   // of either tile width
  const int64_t planes = (K / kBK + per - 1) / per + 1;
  return 2 * planes * M * N <= int64_t(gemm_partial_floats());
}

StreamSum launch_gemm_stream(const GemmArgs& g, hipStream_t stream) {
  // One wavefront per 32 rows x 32 or 64 columns, so a 32- or 64-row stage costs few barriers
  // and LDS reads (W_down of 32 rows: 2 wavefronts 29.2 us, 4 that share the k-slices of a
  // stage 32.7; of 64 rows: 4 wavefronts 31.8, 8 33.0).
  if (g.M <= 32) return launch_tm<32, 64, 2, 1, 12, 4>(g, stream);
  if (g.M <= 64) return launch_tm<64, 64, 4, 1, 9, 4>(g, stream);
  if (wide_tiles(g.M, g.N, g.K)) return launch_tm<128, 128, 8, 2, 4, 2>(g, stream);
  return launch_tm<128, 64, 8, 1, 6, 4>(g, stream);
}

// Gate|up of up to 128 rows where its 64 + 64-column tiles make one round that fills at
// least 3/4 of the CUs, and W's rows are a multiple of 4 KB apart, so that the memory
// channels are the bound.  Against what else would run (us, 1 / 32 / 64 / 128 rows):
//   K = 2048, ffn 12416: 23.4 / 23.4 / 24.1 / 26.8, one round of narrow tiles 25.9 / 26.2 / 26.5 / 28.8
//   K = 6144, ffn 14336: 61 / 64 / 68 / 79, narrow tiles 73 / 75 / 78 / 87
//   K = 8192, ffn 16384: 90 / 90 / 90 / 99, partial sums 117 / 115 / 117 / 140
// Not K = 5120, ffn 13824: 50.6 / 52.6 / 56.6 / 65.4, narrow tiles 49.3 / 51.8 / 55.4 / 65.2.
bool glu_fits(int M, int ffn, int K) {
  return M <= 128 && ffn / 64 >= 192 && ffn / 64 <= 256 && K % 2048 == 0;
}

template <int TM, int NW, int NS>
static void launch_glu(const GemmArgs& g, hipStream_t stream) {
  StreamArgs a{};
  a.A = g.A, a.W = g.W, a.M = g.M, a.N = g.N, a.K = g.K, a.act = g.act, a.ffn = g.ffn;
  a.s.M = g.M, a.s.N = g.N, a.s.tm = TM, a.s.tn = 128, a.s.m_tiles = 1;
  a.s.ks = g.K / kBK;
  a.s.G = g.ffn / 64;
  a.s.units = a.s.G * a.s.ks;
  gemm_stream_kernel<TM, 128, NW, 2, NS, 1, true><<<a.s.G, NW * 64, 0, stream>>>(a);
}

void launch_gemm_glu(const GemmArgs& g, hipStream_t stream) {
  if (g.M <= 32) launch_glu<32, 2, 7>(g, stream);
  else if (g.M <= 64) launch_glu<64, 4, 6>(g, stream);
  else launch_glu<128, 8, 4>(g, stream);
}

void launch_stream_finish(const StreamSum& s, const GemmArgs& g, int epi, hipStream_t stream) {
  if (epi == kRope) {
    stream_rope_kernel<<<cdiv(s.M * (s.N / 8), 256), 256, 0, stream>>>(s, g);
    return;
  }
  const int grid = cdiv(s.M * ((epi == kSwiGLU ? g.ffn : s.N) / 4), 256);
  if (epi == kStoreF32) stream_finish_kernel<kStoreF32><<<grid, 256, 0, stream>>>(s, g.C, g.act, g.ffn);
  else if (epi == kResidual) stream_finish_kernel<kResidual><<<grid, 256, 0, stream>>>(s, g.C, g.act, g.ffn);
  else stream_finish_kernel<kSwiGLU><<<grid, 256, 0, stream>>>(s, g.C, g.act, g.ffn);
}

void launch_stream_rope_write(const StreamSum& s, const GemmArgs& g, const StreamWrite& w, hipStream_t stream) {
  const int D = g.head_dim;
  const int grid = w.n_private * g.hkv + cdiv(s.M * g.hq * (D / 8), 2 * D);
  if (D == 128) stream_rope_write_kernel<128><<<grid, 256, 0, stream>>>(s, g, w);
  else stream_rope_write_kernel<64><<<grid, 128, 0, stream>>>(s, g, w);
}

}  // namespace epic
