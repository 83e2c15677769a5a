// Whole-tile GEMMs of many rows: C[M x N] = A[M x K] . W[N x K]^T, tiles of 256 or 192
// rows x 256 columns, one workgroup of four wavefronts per CU, epilogues fused.
//
// What bounds it: at 20 560 rows the chip runs at its power limit (1.65 GHz of 2.4), so
// beside the MFMAs it is the operand traffic that costs.  Hence
//   - a wavefront owns TM/2 x 128 outputs (4 x 4 or 3 x 4 MFMA tiles of 32 x 32, the
//     accumulators in AGPRs): 0.5 KB of LDS reads per MFMA, where eight wavefronts of
//     128 x 64 read 0.75 KB and kept the LDS as busy as the matrix cores;
//   - one wavefront per SIMD has nothing beside it to hide latency, so the schedule is
//     fixed: each k-slice of 16 issues its MFMAs with the next slice's fragment reads
//     and a quarter of a stage's loads between them;
//   - LDS is a ring of five half stages (one operand, 64 of K, 32 KB each).  The two
//     that a stage frees take the W half of the stage after next and the A half of the
//     one after that, four loads per slice and wavefront: evenly spread, since loads
//     issued together queue behind each other and hold the wavefront up (all 16 in one
//     slice, two whole stages in the LDS: W_down 1929 -> 2161 us);
//   - a multiple of eight workgroups in XCD-contiguous order, so that concurrent tiles
//     share operands through their XCD's L2 (252 workgroups dealt in tile order missed
//     it 2.6 times as often: gate|up 3948 -> 3752 us).
// Measured against the eight-wavefront kernel (same box, 20 560 rows): gate|up (N 28672,
// K 4096) 3752 -> 3580 us, W_down (K 14336) 2110 -> 1929, Q|K|V 861 -> 809, W_O 668 -> 628;
// 736 rows, gate|up 202 -> 167.  MFMA busy 79% of cycles (73% before).
//
// With few tiles and a long K the same kernel runs equal parts of K of every tile, one
// workgroup each, into fp32 planes that the consumer adds (stream_sum.h): the part index
// is the slow one, so the workgroups of an XCD are at the same K and share operands
// (shares cut anywhere in the tile order, and thus at as many K offsets as workgroups:
// 736 rows, N = K = 4096 43 -> 48 us, Q|K|V 59 -> 67).  W_down of 736 rows, against cut 256 x 128 tiles with
// arrival counters: 117 -> 93 us with the pass that sums.
//
// Half-stage layout: rows of 128 bytes in groups of 8 (1 KB, one load instruction); the
// eight 16-byte chunks of row r are XOR-swizzled by (r / 2) % 8, so the 16 lanes of each
// ds_read_b128 group touch distinct banks.  For kSwiGLU the W rows of a tile are gate and
// up in turn, 32 rows each; for kRope with D = 128 each 128-column head is staged as
// (i.., i+64.., i+32.., i+96..) in 32-row groups, so that MFMA tiles 2 q and 2 q + 1 of a
// wavefront hold gate and up, or the two halves of rotary pairs (D = 64 needs no order).
// Rows past M and columns past N are read clamped and never stored.
#include <algorithm>
#include <cmath>

#include "device_common.h"
#include "gemm.h"
#include "gemm_device.h"
#include "stream_sum.h"

namespace epic {

namespace {

constexpr int kBK = 64, kTN = 256;
constexpr int kMaxWorkers = 256;

struct WidePlan {
  int m_tiles, n_tiles, tiles;
  int ks;                      // K stages per tile
  int gm;                      // row tiles per ordering group
  int G;                       // workgroups, a multiple of 8
  int parts;                   // kPlanes: equal parts of K per tile, a workgroup each
  int chains;                  // kResidual: parts of K added to the output one after the other
  int fresh;                   // kResidual: the output holds nothing yet
};
constexpr int kPlanes = 4;     // epilogue: fp32 partial sums into planes (stream_sum.h)

template <int EPI, int TM>
__global__ __launch_bounds__(256, 1) void gemm_wide_kernel(GemmArgs g, WidePlan p) {
  constexpr int I = TM / 64, J = 4;                     // 32 x 32 MFMA tiles per wavefront
  constexpr int NLA = TM / 32, NLB = kTN / 32;          // 1 KB row groups per wavefront and stage
  constexpr int SLOTS = 5, SLOT = kTN * 128;            // half stages (one operand, 64 of K)
  __shared__ __attribute__((aligned(1024))) char lds[SLOTS][SLOT];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wv >> 1, wn = wv & 1;
  const int w = blockIdx.x;
  const int wr = (w % 8) * (p.G / 8) + w / 8;           // XCD-contiguous worker index (G % 8 == 0)
  // This worker's K stages: whole tiles wr, wr + G, ..; with kPlanes part wr / tiles of
  // tile wr % tiles, so that the workgroups of an XCD are at the same K.
  constexpr bool SPLIT = EPI == kPlanes;
  if (wr >= (SPLIT ? p.parts * p.tiles : p.tiles)) return;
  const int part = SPLIT ? wr / p.tiles : 0;
  const int tile0 = SPLIT ? wr - part * p.tiles : wr;
  const int kt0 = SPLIT ? part * p.ks / p.parts : 0;
  const int n_units = SPLIT ? (part + 1) * p.ks / p.parts - kt0 : (p.tiles - wr + p.G - 1) / p.G * p.ks;

  auto tile_mn = [&](int t, int& mt, int& nt) __attribute__((always_inline)) {
    if constexpr (SPLIT) {
      nt = t / p.m_tiles;
      mt = t - nt * p.m_tiles;
      return;
    }
    const int per_group = p.gm * p.n_tiles;
    const int grp = t / per_group;
    const int first = grp * p.gm;
    const int gsz = min(p.m_tiles - first, p.gm);
    const int r = t - grp * per_group;
    mt = first + r % gsz;
    nt = r / gsz;
  };

  // ---- loads: this wavefront stages A row groups NLA wv .., W row groups NLB wv ..
  const int lrow = lane >> 3;
  const int row_bytes = g.K * 2;
  const int w_rows = EPI == kSwiGLU ? 2 * g.ffn : g.N;
  const __amdgpu_buffer_rsrc_t rsa =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(g.A), 0, g.M * row_bytes, kBufWord3);
  const __amdgpu_buffer_rsrc_t rsb =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(g.W), 0, w_rows * row_bytes, kBufWord3);
  int va[NLA], vb[NLB];
  struct Cursor {
    int tile, kt, slot, left;
  };
  Cursor ca{tile0, kt0, 0, n_units}, cb{tile0, kt0, 1, n_units};   // next half stages to load
  auto setup_a = [&]() __attribute__((always_inline)) {
    int mt, nt;
    tile_mn(ca.tile, mt, nt);
#pragma unroll
    for (int i = 0; i < NLA; ++i) {
      const int row = (NLA * wv + i) * 8 + lrow;
      va[i] = min(mt * TM + row, g.M - 1) * row_bytes + ((lane & 7) ^ ((row >> 1) & 7)) * 16;
    }
  };
  auto setup_b = [&]() __attribute__((always_inline)) {
    int mt, nt;
    tile_mn(cb.tile, mt, nt);
#pragma unroll
    for (int i = 0; i < NLB; ++i) {
      const int row = (NLB * wv + i) * 8 + lrow;
      int gr;
      if constexpr (EPI == kSwiGLU)
        gr = ((row >> 5) & 1) * g.ffn + nt * (kTN / 2) + (row >> 6) * 32 + (row & 31);
      else if constexpr (EPI == kRope) {
        const int hc = g.head_dim == 128 ? (row & ~127) + ((row >> 5) & 1) * 64 + ((row >> 6) & 1) * 32 + (row & 31)
                                         : row;
        gr = min(nt * kTN + hc, g.N - 1);
      } else gr = min(nt * kTN + row, g.N - 1);
      vb[i] = gr * row_bytes + ((lane & 7) ^ ((row >> 1) & 7)) * 16;
    }
  };
  setup_a();
  setup_b();
  auto bump = [&](int slot) __attribute__((always_inline)) { return slot >= SLOTS - 2 ? slot + 2 - SLOTS : slot + 2; };
  // to the next half stage; past the last, that one again.  True: another tile
  auto advance = [&](Cursor& c) __attribute__((always_inline)) {
    c.slot = bump(c.slot);
    if (--c.left <= 0) return false;
    if (++c.kt < p.ks) return false;
    c.tile += p.G;
    c.kt = 0;
    return true;
  };
  auto dma_a = [&](int i) __attribute__((always_inline)) {
    dma16(rsa, lds[ca.slot] + (NLA * wv + i) * 1024, va[i], ca.kt * 128);
    if (i == NLA - 1 && advance(ca)) setup_a();
  };
  auto dma_b = [&](int i) __attribute__((always_inline)) {
    dma16(rsb, lds[cb.slot] + (NLB * wv + i) * 1024, vb[i], cb.kt * 128);
    if (i == NLB - 1 && advance(cb)) setup_b();
  };

  // ---- fragments
  const int half = lane >> 5, lsw = (lane >> 1) & 7;
  const int la = wm * (TM / 2) * 128 + (lane & 31) * 128;
  const int lb = wn * 128 * 128 + (lane & 31) * 128;
  int sw[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) sw[s] = ((2 * s + half) ^ lsw) * 16;
  struct Frags {
    bf16x8 a[I], b[J];
  } f0, f1;
  auto read1 = [&](Frags& f, const char* sa, const char* sb, int s, int i) __attribute__((always_inline)) {   // a0 b0 .. b3 a1 ..
    if (i == 0) f.a[0] = *reinterpret_cast<const bf16x8*>(sa + la + sw[s]);
    else if (i <= J) f.b[i <= J && i > 0 ? i - 1 : 0] = *reinterpret_cast<const bf16x8*>(sb + lb + (i - 1) * 4096 + sw[s]);
    else f.a[i > J ? i - J : 0] = *reinterpret_cast<const bf16x8*>(sa + la + (i - J) * 4096 + sw[s]);
  };

  f32x16 acc[I][J];
  constexpr int NM = I * J;
  // one k-slice: its MFMAs on f; the fragments of the next slice (slice s of the stage at
  // sa, sb) read into fn beside the first of them, and a quarter of the stage's loads
  auto slice = [&](const Frags& f, Frags& fn, const char* sa, const char* sb, int s, auto load) __attribute__((always_inline)) {
    constexpr int L = decltype(load)::value;            // this slice's loads: half of W (0, 1) or of A (2, 3)
    constexpr int NL = (L < 2 ? NLB : NLA) / 2;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      acc[m / J][m % J] = mfma_32x32x16(f.a[m / J], f.b[m % J], acc[m / J][m % J]);
      if (m < I + J) read1(fn, sa, sb, s, m);
#pragma unroll
      for (int i = 0; i < NL; ++i)
        if (m == i * NM / NL + 1) {
          if constexpr (L < 2) dma_b(L * NL + i);
          else dma_a((L - 2) * NL + i);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // the next stage's loads landed, everyone's (the A loads past it stay in flight), and
  // this stage is read
  auto sync = [&]() __attribute__((always_inline)) {
    wait_vmem<NLA>();
    barrier_lds();
  };

#pragma unroll
  for (int i = 0; i < NLA; ++i) dma_a(i);
#pragma unroll
  for (int i = 0; i < NLB; ++i) dma_b(i);
#pragma unroll
  for (int i = 0; i < NLA; ++i) dma_a(i);
#pragma unroll
  for (int i = 0; i < NLB / 2; ++i) dma_b(i);
  wait_vmem<NLA + NLB / 2>();                           // stage 0
  __asm__ volatile("s_barrier" ::: "memory");
#pragma unroll
  for (int i = 0; i < I + J; ++i) read1(f0, lds[0], lds[1], 0, i);

  int sa = 0, sb = 1;
  constexpr bool CHAINS = EPI == kResidual;
  int chain = 0;
  for (int tile = tile0, left = n_units; left > 0;) {
    // stages until the sums go to the output: the tile's, or its next chain's
    const int n = SPLIT ? n_units : CHAINS ? (chain + 1) * p.ks / p.chains - chain * p.ks / p.chains : p.ks;
#pragma unroll
    for (int i = 0; i < I; ++i)
#pragma unroll
      for (int j = 0; j < J; ++j) acc[i][j] = f32x16{};
    for (int kt = 0; kt < n; ++kt) {
      const char *pa = lds[sa], *pb = lds[sb];
      slice(f0, f1, pa, pb, 1, std::integral_constant<int, 1>{});
      slice(f1, f0, pa, pb, 2, std::integral_constant<int, 2>{});
      slice(f0, f1, pa, pb, 3, std::integral_constant<int, 3>{});
      sync();
      sa = bump(sa);
      sb = bump(sb);
      slice(f1, f0, lds[sa], lds[sb], 0, std::integral_constant<int, 0>{});
    }
    // ---- epilogue (rows past M fall outside the descriptors)
    int mt, nt;
    tile_mn(tile, mt, nt);
    const int col = lane & 31;
    const int m0 = mt * TM + wm * (TM / 2) + half * 4;   // register r of row block i: row m0 + 32 i + 8 (r / 4) + r % 4
    // The offsets of a block of stores start from a value the compiler cannot see
    // through, or it computes all of them ahead and spills.
    auto hide = [](int x) __attribute__((always_inline)) {
      __asm__ volatile("" : "+v"(x));
      return x;
    };
    if constexpr (EPI == kSwiGLU) {
      const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(g.act, 0, g.M * g.ffn * 2, kBufWord3);
      const int n = nt * (kTN / 2) + wn * 64 + col;
#pragma unroll
      for (int i = 0; i < I; ++i)
#pragma unroll
        for (int j = 0; j < J; j += 2) {
          const int o = hide(((m0 + i * 32) * g.ffn + n + j * 16) * 2);
#pragma unroll
          for (int r = 0; r < 16; r += 2) {
            float act[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const float gt = acc[i][j][r + e], up = acc[i][j + 1][r + e];
              act[e] = gt * __builtin_amdgcn_rcpf(1.0f + fast_exp2(-gt * kLog2e)) * up;
            }
            const uint32_t two = pack_bf16x2(act[0], act[1]);
            const int row = (r >> 2) * 8 + (r & 3);
            __builtin_amdgcn_raw_buffer_store_b16(uint16_t(two), ro, o + row * g.ffn * 2, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b16(uint16_t(two >> 16), ro, o + (row + 1) * g.ffn * 2, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
    } else if constexpr (EPI == kRope) {
      // blocks of one row block and one pair of column tiles (2 q, 2 q + 1); the cos / sin
      // of DEPTH blocks are in flight (a load is not moved above an earlier store)
      constexpr int NB = I * (J / 2), DEPTH = 3;
      const int D = g.head_dim, hd2 = D >> 1;
      const __amdgpu_buffer_rsrc_t rc =
          __builtin_amdgcn_make_buffer_rsrc(const_cast<float2*>(g.cs), 0, g.M * hd2 * 8, kBufWord3);
      // D = 128: both pairs of a wavefront lie in one head (ip, ip + 64); D = 64: a head each
      auto head_of = [&](int q) __attribute__((always_inline)) { return D == 128 ? (nt * kTN >> 7) + wn : (nt * kTN >> 6) + 2 * wn + q; };
      auto ip_of = [&](int q) __attribute__((always_inline)) { return (D == 128 ? q * 32 : 0) + col; };
      float2 t[DEPTH][16];
      auto fetch = [&](int b) __attribute__((always_inline)) {
        const int i = b / (J / 2), q = b % (J / 2);
        const int o = hide(((m0 + i * 32) * hd2 + ip_of(q)) * 8);
#pragma unroll
        for (int r = 0; r < 16; ++r)
          t[b % DEPTH][r] = __builtin_bit_cast(
              float2, __builtin_amdgcn_raw_buffer_load_b64(rc, o + ((r >> 2) * 8 + (r & 3)) * hd2 * 8, 0, 0));
        __builtin_amdgcn_sched_barrier(0);
      };
#pragma unroll
      for (int b = 0; b < DEPTH && b < NB; ++b) fetch(b);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int i = b / (J / 2), q = b % (J / 2), j = 2 * q;
        const int head = head_of(q);
        uint16_t* base;
        int heads, hd;
        bool rotate = true;
        if (head < g.hq) base = g.q, heads = g.hq, hd = head;
        else if (head < g.hq + g.hkv) base = g.k, heads = g.hkv, hd = head - g.hq;
        else base = g.v, heads = g.hkv, hd = head - g.hq - g.hkv, rotate = false;
        // columns past N: an empty range drops the stores
        const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
            base, 0, head < g.hq + 2 * g.hkv ? g.M * heads * D * 2 : 0, kBufWord3);
        const int o = hide((((m0 + i * 32) * heads + hd) * D + ip_of(q)) * 2);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float x1 = acc[i][j][r], x2 = acc[i][j + 1][r];
          const float c = rotate ? t[b % DEPTH][r].x : 1.0f, sn = rotate ? t[b % DEPTH][r].y : 0.0f;
          const float y1 = rotate ? x1 * c - x2 * sn : x1, y2 = rotate ? x2 * c + x1 * sn : x2;
          const uint32_t two = pack_bf16x2(y1, y2);
          const int e = o + ((r >> 2) * 8 + (r & 3)) * heads * D * 2;
          __builtin_amdgcn_raw_buffer_store_b16(uint16_t(two), ro, e, 0, 0);
          __builtin_amdgcn_raw_buffer_store_b16(uint16_t(two >> 16), ro, e + hd2 * 2, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (b + DEPTH < NB) fetch(b + DEPTH);
      }
    } else {
      // blocks of one MFMA tile; for the residual add the old values of DEPTH blocks are
      // in flight (a load is not moved above an earlier store)
      constexpr int DEPTH = 4;
      float* c = g.C;
      if constexpr (SPLIT) c = g.partial + size_t(part) * g.M * g.N;
      const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(c, 0, g.M * g.N * 4, kBufWord3);
      // what to add to: nothing (an empty range reads as 0) for the first chain of a plain product
      const __amdgpu_buffer_rsrc_t ri =
          __builtin_amdgcn_make_buffer_rsrc(c, 0, chain == 0 && p.fresh ? 0 : g.M * g.N * 4, kBufWord3);
      const int nw = nt * kTN + wn * 128;
      if (nw < g.N) {                                   // N % 128 == 0: all of the wavefront's columns, or none
        auto at = [&](int b) __attribute__((always_inline)) {
          return hide(((m0 + b / J * 32) * g.N + nw + col + b % J * 32) * 4);
        };
        float old[DEPTH][16];
        auto fetch = [&](int b) __attribute__((always_inline)) {
          if constexpr (EPI == kResidual) {
            const int o = at(b);
#pragma unroll
            for (int r = 0; r < 16; ++r)
              old[b % DEPTH][r] = __builtin_bit_cast(
                  float, __builtin_amdgcn_raw_buffer_load_b32(ri, o + ((r >> 2) * 8 + (r & 3)) * g.N * 4, 0, 0));
            __builtin_amdgcn_sched_barrier(0);
          }
        };
#pragma unroll
        for (int b = 0; b < DEPTH; ++b) fetch(b);
#pragma unroll
        for (int b = 0; b < I * J; ++b) {
          const int o = at(b);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            float x = acc[b / J][b % J][r];
            if constexpr (EPI == kResidual) x += old[b % DEPTH][r];
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), ro,
                                                  o + ((r >> 2) * 8 + (r & 3)) * g.N * 4, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
          if (b + DEPTH < I * J) fetch(b + DEPTH);
        }
      }
    }
    left -= n;
    if (!CHAINS || ++chain == p.chains) {
      chain = 0;
      tile += p.G;
    }
  }
  wait_vmem<0>();                                       // no load may land in LDS after the workgroup ends
}

int cdiv(int a, int b) { return (a + b - 1) / b; }

template <int EPI, int TM>
void launch_wide_tm(const GemmArgs& g, hipStream_t stream) {
  WidePlan p{};
  p.m_tiles = cdiv(g.M, TM);
  p.n_tiles = EPI == kSwiGLU ? g.ffn / (kTN / 2) : cdiv(g.N, kTN);
  p.ks = g.K / kBK;
  p.gm = std::min(p.m_tiles, 8);
  p.tiles = p.m_tiles * p.n_tiles;
  p.G = cdiv(cdiv(p.tiles, cdiv(p.tiles, kMaxWorkers)), 8) * 8;
  if constexpr (EPI == kStoreF32 || EPI == kResidual) {
    p.chains = std::min(gemm_chains(g, EPI), p.ks);
    p.fresh = EPI == kStoreF32;
    if (EPI == kResidual || p.chains > 1) {
      gemm_wide_kernel<kResidual, TM><<<p.G, 256, 0, stream>>>(g, p);
      return;
    }
  }
  gemm_wide_kernel<EPI, TM><<<p.G, 256, 0, stream>>>(g, p);
}

}  // namespace

// Chains of additions that a tile's sums have to be made of, so that fp32 results are as exact as
// by what ran these sizes before.  A chain of L matrix instructions leaves a rounding error
// of sqrt(L).  Products of less than a round of 256-row tiles used to be 256 x 128 tiles cut along
// K into shares of x tiles; a tile's parts c_i (of L) left sqrt(L sum c_i^2), with a sum of x
// where the shares are parts of tiles, else on average x - x^2 / 3 up to a tile and
// 1 - 1 / (3 x) past it.  As many equal chains as the reciprocal of that leave no more.
// Relative error and us, cut -> one chain -> the chains needed:
//   whole tiles  3000 rows, N 4096, K 4096   3.59e-7 -> 3.95e-7 -> 2.72e-7, 109 -> 82 -> 94
//                3000, 4096, 14336           6.95e-7 -> 7.64e-7 -> 5.33e-7, 356 -> 259 -> 274
//                296, 28672, 4096            3.56e-7 -> 3.95e-7 -> 2.73e-7, 116 -> 83 -> 95
//   split tiles  912, 2176, 1024             0.94e-7 -> 1.28e-7 -> 0.88e-7, 33 -> 18 -> 26
// Two sets of accumulators instead, for which 192 rows leave the registers, are spilled.
int gemm_chains(const GemmArgs& g, int epi) {
  if ((epi != kStoreF32 && epi != kResidual) || g.in_layer) return 1;
  const int m_tiles = cdiv(g.M, 256);
  if (int64_t(m_tiles) * cdiv(g.N, kTN) >= kMaxWorkers) return 1;
  const int tiles = m_tiles * cdiv(g.N, 128);
  const int shares = int(std::min<int64_t>(kMaxWorkers, std::max<int64_t>(1, int64_t(tiles) * (g.K / kBK) / 4)));
  if (tiles % shares == 0) return 1;
  const double x = double(tiles) / shares;
  const double sum = shares % tiles == 0 ? x : x <= 1.0 ? x - x * x / 3 : 1.0 - 1.0 / (3 * x);
  return int(std::ceil(1.0 / sum - 1e-9));
}

// A stage takes longer with 256 rows than with 192, and the more CUs run; and what of the
// weights does not come from the L2 in time.
double wide_split_time(const WideSplit& s, int M, int N, int K) {
  const double w = double(K) * N * 2e-6, t = double(cdiv(M, s.tm)) * cdiv(N, kTN) * s.parts / kMaxWorkers;
  return 9.4 + cdiv(K / kBK, s.parts) * ((s.tm == 256 ? 1.14 : 0.78) + 0.36 * t) + 0.02 * w +
         0.045 * std::max(w - 120.0, 0.0);
}

// Equal parts of K per tile, a workgroup each, in one round; at least eight stages a part
// (fewer only where the sums need more chains), planes within the workspace.  The height by
// the time of the stages alone, 1.5 us with 256 rows and 1.25 with 192.  Up to 128 rows the
// tiles would mostly be padding.
WideSplit wide_split(const GemmArgs& g, int epi) {
  const int M = g.M, N = g.N, K = g.K, chains = gemm_chains(g, epi);
  WideSplit best{};
  double best_time = 0.0;
  if (M <= 128) return best;
  for (const int tm : {256, 192}) {
    const int64_t tiles = int64_t(cdiv(M, tm)) * cdiv(N, kTN);
    if (tiles > kMaxWorkers / 2) continue;
    const int64_t fit = int64_t(gemm_partial_floats()) / (int64_t(M) * N);
    const int64_t most = std::min({kMaxWorkers / tiles, int64_t(K / kBK), fit});
    const int parts = int(std::min(most, std::max<int64_t>(K / kBK / 8, chains)));
    if (parts < 2 || parts < chains) continue;
    const double time = cdiv(K / kBK, parts) * (tm == 256 ? 1.5 : 1.25);
    if (best.parts == 0 || time < best_time) best = WideSplit{tm, parts}, best_time = time;
  }
  return best;
}

StreamSum launch_gemm_wide_split(const GemmArgs& g, int epi, hipStream_t stream) {
  const WideSplit w = wide_split(g, epi);
  WidePlan p{};
  p.m_tiles = cdiv(g.M, w.tm);
  p.n_tiles = cdiv(g.N, kTN);
  p.ks = g.K / kBK;
  p.tiles = p.m_tiles * p.n_tiles;
  p.parts = w.parts;
  p.G = cdiv(p.tiles * p.parts, 8) * 8;
  StreamSum s{};
  s.partial = g.partial;
  s.M = g.M, s.N = g.N, s.fixed = p.parts;
  if (w.tm == 192) gemm_wide_kernel<kPlanes, 192><<<p.G, 256, 0, stream>>>(g, p);
  else gemm_wide_kernel<kPlanes, 256><<<p.G, 256, 0, stream>>>(g, p);
  return s;
}

void launch_gemm_wide(const GemmArgs& g, int epi, int tm, hipStream_t stream) {
  if (tm == 256) {
    if (epi == kStoreF32) launch_wide_tm<kStoreF32, 256>(g, stream);
    else if (epi == kResidual) launch_wide_tm<kResidual, 256>(g, stream);
    else if (epi == kSwiGLU) launch_wide_tm<kSwiGLU, 256>(g, stream);
    else launch_wide_tm<kRope, 256>(g, stream);
  } else {
    if (epi == kStoreF32) launch_wide_tm<kStoreF32, 192>(g, stream);
    else if (epi == kResidual) launch_wide_tm<kResidual, 192>(g, stream);
    else if (epi == kSwiGLU) launch_wide_tm<kSwiGLU, 192>(g, stream);
    else launch_wide_tm<kRope, 192>(g, stream);
  }
}

}  // namespace epic
