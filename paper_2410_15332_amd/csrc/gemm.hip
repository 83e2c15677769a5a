// Row-set GEMMs of the link step on MFMA: C[M x N] = A[M x K] . W[N x K]^T.
//
// A holds the selected rows' activations (bf16, K contiguous), W a weight
// matrix in [out][in] layout (bf16), so both MFMA operands are read along K.
// Epilogues are fused:
//   kStoreF32 : C -> fp32 [M][N]                     (the plain projection of epic_gemm)
//   kResidual : h[M][N] += C                         (W_O and W_down; fp32 residual stream)
//   kSwiGLU   : act[M][N/2] = silu(gate) * up, bf16  (W_gate_up; gate rows [0, F), up rows [F, 2F))
//   kRope     : the fused Q|K|V projection: q and k heads rotated at each row's linked
//               position (rotary pairs (i, i + D/2)), v heads as they are; bf16 q, k, v
//
// Three families of kernels, chosen by gemm_route below:
//   - many rows: whole 256- or 192-row tiles of 256 columns, or equal parts of K of
//     them (gemm_wide.hip);
//   - short row sets: small tiles, K dealt in equal shares, sums in the consumer; gate|up
//     of up to 128 rows in whole tiles (gemm_stream.hip);
//   - in between (this file): 128-column tiles, whole where one round of them fills the
//     chip, else cut along K.
//
// Tiling here: workgroup tile TM x 128 (TM = 256, 128 or 96), 8 wavefronts of 64 columns
// each (4 x 2 wavefronts of TM/4 x 64, and at TM = 96 3 x 2 of 32 x 64 while the other
// two only stage operands).  K runs in stages of 64 staged in LDS by direct buffer->LDS
// loads, three stages in LDS (loads issued two stages ahead of use).  An operand stage is
// groups of 8 rows of 128 bytes
// (one whole cache line per row: a load instruction that covers 16 half lines moves
// about 0.6x the bytes per cycle of one that covers 8 whole lines); row r sits at byte
// 128 r with its eight 16-byte chunks XOR-swizzled by (r / 2) % 8, so one load
// instruction fills one group (1 KB) and the 16 lanes of each ds_read_b128 group
// touch distinct banks.  For kSwiGLU the weight rows of a tile are gate/up in
// 32-row groups (gate j.., up j.., gate j+32.., ...), so a wavefront's two
// 32-column MFMA tiles hold gate and up of the same 32 outputs.  For kRope the two
// 32-column MFMA tiles of a wavefront hold the two halves of rotary pairs: with
// D = 64 that is the natural order (a wavefront's 64 columns are one head); with
// D = 128 each 128-column head is staged as (i.., i+64.., i+32.., i+96..) in
// 32-row groups, i = 0.., so lane column c of tile 0 and tile 1 are head
// columns ip and ip + 64.
//
// Scheduling: at most one workgroup per CU (G of them), persistent.  Whole 96 x 128 or
// 128 x 128 tiles run in one round; of the 256 x 128 tiles the ones that do not fill
// whole rounds (the last partial round plus one full round, or all of them) are cut along
// K into G equal shares of K stages, one per workgroup, so every CU gets the same work.  A
// share runs its last segment (the one that starts a tile) first.
// A tile cut across workgroups: each wavefront part of it has an arrival counter.
// The owner of the tile's last K stage polls it (a bounded number of times) until
// the other parts have written their fp32 partials, then adds them to its own
// accumulators and runs the epilogue; if the polls run out it writes its partial
// too, and the last wavefront to arrive finishes.  Either way the parts are summed
// in one fixed order, so the result does not depend on arrival order.  Workgroups
// are dealt round-robin to the 8 XCDs; worker indices are arranged so that each XCD
// works on a contiguous run of tiles, and tiles are ordered in groups of up to 8 row
// tiles per weight tile, so concurrent workgroups on an XCD share operands through
// its L2.
// Rows past M and columns past N are computed from clamped rows and never stored.
#include <algorithm>
#include <cstdlib>

#include "device_common.h"
#include "gemm.h"
#include "gemm_device.h"
#include "stream_sum.h"

namespace epic {

namespace {

constexpr int kTM = 256, kBK = 64;
constexpr int kThreads = 512;
constexpr int kMaxWorkers = 256;                        // one workgroup per CU
constexpr int kPartialFloats = kTM * 256;               // per partial slot (twice a 256 x 128 tile)
constexpr int kMaxSplitTiles = 2 * kMaxWorkers;
constexpr int kCounters = kMaxSplitTiles * (kThreads / 64);   // one per (cut tile, wavefront)
constexpr int kMinUnits = 4;                            // K stages per workgroup, at least
constexpr int kStreamRows = 512;                        // most rows of a streamed product

constexpr int TN = 128;                                 // columns of a workgroup tile

template <int TM>
struct Shape {
  static_assert(TM == 256 || TM == 128 || TM == 96, "tile shape");
  static constexpr int NS = 3;                          // LDS stages (144 / 96 / 84 KB)
  // wavefronts along M (TM = 96: 3 x 2 wavefronts compute, the other two only stage
  // operands and meet the barriers)
  static constexpr int WAVES_M = TM >= 128 ? 4 : TM / 32;
  static constexpr int WM = TM / WAVES_M;               // rows per wavefront
  static constexpr int I = WM / 32;                     // 32-row MFMA tiles per wavefront
  static constexpr int J = 2;                           // 32-column MFMA tiles per wavefront
  static constexpr int A_STAGE = TM * kBK * 2;          // bytes per stage
  static constexpr int B_STAGE = TN * kBK * 2;
  static constexpr int NLA = TM / 32;                   // A row groups (8 rows) per loading wavefront
  static constexpr int NLB = TN / 32;                   // W row groups per loading wavefront
  static constexpr int NL = NLA > NLB ? NLA : NLB;
};

struct GemmPlan {
  int m_tiles, n_tiles, ks;    // tiles along M and N, K stages per tile
  int gm;                      // row tiles per ordering group
  int G;                       // workgroups
  int dp_rounds, dp_tiles;     // whole-tile rounds and the tiles they cover (tiles 0 .. dp_tiles-1)
  int sk_units;                // K stages of the cut tiles (tiles dp_tiles ..)
  int polls;                   // counter polls of a cut tile's last-stage owner before it falls back
};

template <int TM>
struct GemmLds {
  char a[Shape<TM>::NS][Shape<TM>::A_STAGE];
  char b[Shape<TM>::NS][Shape<TM>::B_STAGE];
};

// Position in a workgroup's sequence of K stages: tile, stage, and the stage range
// [kbeg, kend) of the current segment (the part of the tile this workgroup owns).
struct Cursor {
  int u, tile, kt, kbeg, kend;
};

template <int EPI, int TM>
__global__ __launch_bounds__(kThreads, 1) void gemm_kernel(GemmArgs g, GemmPlan p) {
  using SH = Shape<TM>;
  constexpr int NS = SH::NS, I = SH::I, J = SH::J, NLA = SH::NLA, NLB = SH::NLB, NL = SH::NL;
  __shared__ __attribute__((aligned(1024))) GemmLds<TM> lds;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // wavefront tile: rows wm*WM.., columns wn*64..  The two wavefronts of
  // each SIMD (wavefronts w and w + 4) take different row halves, so a tile whose
  // rows past M leave half the wavefronts idle still keeps every SIMD busy.  Wavefronts
  // with wm >= WAVES_M (TM = 96: wavefronts 6 and 7) compute and store nothing.
  const int wm = wv >> 1;
  const int wn = wv & 1;
  const int w = blockIdx.x;
  const int wr = p.G % 8 == 0 ? (w % 8) * (p.G / 8) + w / 8 : w;   // XCD-contiguous worker index
  const int64_t su = p.sk_units;
  const int s0 = int(int64_t(wr) * su / p.G), s1 = int(int64_t(wr + 1) * su / p.G);
  // whole tiles wr, wr + G, .. below dp_tiles (the last round may be short), then the K share
  const int dp_units = (wr < p.dp_tiles ? (p.dp_tiles - wr + p.G - 1) / p.G : 0) * p.ks;
  const int n_units = dp_units + (s1 - s0);
  if (n_units == 0) return;             // (no such workgroup is launched; kept as a guard)
  // The K share runs its last segment first: that segment starts a tile (K stage 0)
  // and the rest ends one (the last stage), so the workgroups of an XCD that cross a
  // tile boundary sit at two K offsets at any time instead of one each, and their
  // operand stages are shared in the L2.  sh: first unit of the last segment.
  const int sh = max(s0, s1 > s0 ? (s1 - 1) / p.ks * p.ks : s0);

  auto tile_mn = [&](int t, int& mt, int& nt) __attribute__((always_inline)) {
    const int per_group = p.gm * p.n_tiles;
    const int grp = t / per_group;
    const int first = grp * p.gm;
    const int gsz = min(p.m_tiles - first, p.gm);
    const int r = t - grp * per_group;
    mt = first + r % gsz;
    nt = r / gsz;
  };
  auto seek = [&](Cursor& c, int u) __attribute__((always_inline)) {   // u: first unit of a segment
    c.u = u;
    if (u < dp_units) {
      c.tile = (u / p.ks) * p.G + wr;
      c.kbeg = 0;
      c.kend = p.ks;
    } else {
      const int i = u - dp_units;           // position in the share's processing order
      const bool first = i < s1 - sh;       // in the last segment, run first
      const int v = first ? sh + i : s0 + (i - (s1 - sh));
      const int q = v / p.ks;
      c.tile = p.dp_tiles + q;
      c.kbeg = v - q * p.ks;
      c.kend = min(p.ks, (first ? s1 : sh) - q * p.ks);
    }
    c.kt = c.kbeg;
  };
  auto advance = [&](Cursor& c) __attribute__((always_inline)) {      // to the next unit; stays on the last one
    if (c.u + 1 >= n_units) return;
    ++c.u;
    if (++c.kt == c.kend) seek(c, c.u);
  };

  // ---- buffer->LDS loads: wavefronts 0..3 stage the TM / 8 A row groups (NLA each),
  // 4..7 the TN / 8 W row groups (NLB each).
  const bool a_wave = wv < 4;
  // With M <= 128 (one row tile) the A row groups 16..31 hold no row of A: their
  // loading wavefronts issue nothing (none of their waits then has anything to wait for).
  const bool dma_idle = TM == 256 && a_wave && g.M <= 128 && wv >= 2;
  const int nl = a_wave ? NLA : NLB;                   // loads per stage of this wavefront
  const int grp0 = nl * (wv & 3);
  const int lrow = lane >> 3;                              // row within an 8-row group
  const int row_bytes = g.K * 2;
  const int w_rows = EPI == kSwiGLU ? 2 * g.ffn : g.N;
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(a_wave ? g.A : g.W), 0, (a_wave ? g.M : w_rows) * row_bytes, kBufWord3);
  int vo[NL];                                           // lane byte offsets of the row groups (nl)
  // load i of a stage: issued by this wavefront (i < nl; the bound is a constant for
  // the i below both counts)
  auto has_load = [&](int i) __attribute__((always_inline)) { return a_wave ? i < NLA : i < NLB; };
  auto dma_setup = [&](int tile) __attribute__((always_inline)) {
    int mt, nt;
    tile_mn(tile, mt, nt);
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int row = (grp0 + i) * 8 + lrow;               // row of the operand tile
      const int lchunk = (lane & 7) ^ ((row >> 1) & 7);    // 16-byte chunk of that row this lane loads
      int gr;
      if (a_wave) gr = min(mt * TM + row, g.M - 1);
      else if constexpr (EPI == kSwiGLU)
        gr = ((row >> 5) & 1) * g.ffn + nt * (TN / 2) + (row >> 6) * 32 + (row & 31);
      else if constexpr (EPI == kRope) {
        // D = 128: LDS row p = wn' * 64 + j * 32 + r of a head holds head column
        // j * 64 + wn' * 32 + r (wn' = wavefront column half within the head)
        const int hc = g.head_dim == 128 ? (row & ~127) + ((row >> 5) & 1) * 64 + ((row >> 6) & 1) * 32 + (row & 31)
                                         : row;
        gr = min(nt * TN + hc, g.N - 1);
      } else gr = min(nt * TN + row, g.N - 1);
      vo[i] = gr * row_bytes + lchunk * 16;
    }
  };
  char* const dma_base = a_wave ? lds.a[0] + grp0 * 1024 : lds.b[0] + grp0 * 1024;
  const int dma_stage = a_wave ? SH::A_STAGE : SH::B_STAGE;
  auto dma = [&](int buf, int kt) __attribute__((always_inline)) {
    if (dma_idle) return;
    char* dst = dma_base + buf * dma_stage;
#pragma unroll
    for (int i = 0; i < NL; ++i)
      if (has_load(i)) dma16(rs, dst + i * 1024, vo[i], kt * (kBK * 2));
  };

  // ---- MFMA operands: for k-slice ks (16 wide, 4 per stage) lane l reads row l % 32
  // of a 32-row tile, 16-byte chunk 2 ks + l / 32, stored at chunk position
  // chunk ^ ((l % 32) / 2 % 8).
  const int lrow32 = (lane & 31) * 128;
  const int lsw = (lane >> 1) & 7;
  const int lb0 = lrow32 + (((0 + (lane >> 5)) ^ lsw) * 16);
  const int lb1 = lrow32 + (((2 + (lane >> 5)) ^ lsw) * 16);
  const int lb2 = lrow32 + (((4 + (lane >> 5)) ^ lsw) * 16);
  const int lb3 = lrow32 + (((6 + (lane >> 5)) ^ lsw) * 16);
  const char* const pa = lds.a[0] + wm * SH::WM * 128;
  const char* const pb = lds.b[0] + wn * 64 * 128;
  struct Frags {
    bf16x8 a[I], b[J];
  };
  auto read = [&](Frags& f, int buf, int ks) __attribute__((always_inline)) {
    const int lb = ks == 0 ? lb0 : ks == 1 ? lb1 : ks == 2 ? lb2 : lb3;
    const char* a = pa + buf * SH::A_STAGE + lb;
    const char* b = pb + buf * SH::B_STAGE + lb;
#pragma unroll
    for (int i = 0; i < I; ++i) f.a[i] = *reinterpret_cast<const bf16x8*>(a + i * 4096);
#pragma unroll
    for (int j = 0; j < J; ++j) f.b[j] = *reinterpret_cast<const bf16x8*>(b + j * 4096);
  };

  f32x16 acc[I][J];
  auto zero_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < I; ++i)
#pragma unroll
      for (int j = 0; j < J; ++j) acc[i][j] = f32x16{};
  };
  auto mma = [&](const Frags& f) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < I; ++i)
#pragma unroll
      for (int j = 0; j < J; ++j) acc[i][j] = mfma_32x32x16(f.a[i], f.b[j], acc[i][j]);
  };
  // mma(f) with the loads of unit kt into buffer buf between its MFMAs (NL / (I J)
  // after each, same MFMA order as mma): issued together after the barrier, the
  // workgroup's 64 loads of 1 KB queued behind each other while no MFMA was issued.
  auto mma_dma = [&](const Frags& f, int buf, int kt) __attribute__((always_inline)) {
    constexpr int NM = I * J;
    char* const dst = dma_base + buf * dma_stage;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      acc[m / J][m % J] = mfma_32x32x16(f.a[m / J], f.b[m % J], acc[m / J][m % J]);
#pragma unroll
      for (int i = m * NL / NM; i < (m + 1) * NL / NM; ++i)
        if (!dma_idle && has_load(i)) dma16(rs, dst + i * 1024, vo[i], kt * (kBK * 2));
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // ---- epilogue through buffer descriptors: rows past M fall outside the
  // descriptor's range (loads read 0, stores are dropped).  Accumulator tile
  // t = i*J + j, register r: row wm*WM + i*32 + (r/4)*8 + half*4 + r%4, column
  // wn*64 + j*32 + col of the workgroup tile.  Written CT = 2 tiles (one row block)
  // at a time, so the fixup below holds two tiles of sums and one partial's two tiles
  // in flight (with four, the 128-wide kernels ran out of registers and the compiler
  // reloaded each 1 KB of a partial into the same registers, one round trip each).
  constexpr int NT = I * J, CT = 2, NCH = NT / CT;
  const int col = lane & 31, half = lane >> 5;
  auto epilogue_part = [&](int mt, int nt, int h, const f32x16 (&v)[CT]) __attribute__((always_inline)) {
    const int m0 = mt * TM + wm * SH::WM + half * 4;
    if constexpr (EPI == kSwiGLU) {
      const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(g.act, 0, g.M * g.ffn * 2, kBufWord3);
      const int n = nt * (TN / 2) + wn * 32 + col;
#pragma unroll
      for (int ii = 0; ii < CT / J; ++ii)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int m = m0 + (h * (CT / J) + ii) * 32 + (r >> 2) * 8 + (r & 3);
          const float gt = v[ii * J + 0][r], up = v[ii * J + 1][r];
          const float act = gt * __builtin_amdgcn_rcpf(1.0f + fast_exp2(-gt * kLog2e)) * up;
          __builtin_amdgcn_raw_buffer_store_b16(uint16_t(pack_bf16x2(act, 0.0f) & 0xFFFFu), ro, (m * g.ffn + n) * 2,
                                                0, 0);
        }
    } else if constexpr (EPI == kRope) {
      // this wavefront's 64 columns: one head (D = 64) or half of one (D = 128, the
      // pairs ip, ip + 64 with ip in [32 (wn % 2), + 32))
      const int D = g.head_dim, half = D >> 1;
      const int head = D == 128 ? (nt * TN >> 7) + (wn >> 1) : (nt * TN >> 6) + wn;
      if (head >= g.hq + 2 * g.hkv) return;               // columns past N
      const int ip = (D == 128 ? (wn & 1) * 32 : 0) + col;
      uint16_t* base;
      int heads, hd;
      bool rotate = true;
      if (head < g.hq) {
        base = g.q, heads = g.hq, hd = head;
      } else if (head < g.hq + g.hkv) {
        base = g.k, heads = g.hkv, hd = head - g.hq;
      } else {
        base = g.v, heads = g.hkv, hd = head - g.hq - g.hkv, rotate = false;
      }
      const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(base, 0, g.M * heads * D * 2, kBufWord3);
      const __amdgpu_buffer_rsrc_t rc =
          __builtin_amdgcn_make_buffer_rsrc(const_cast<float2*>(g.cs), 0, g.M * half * 8, kBufWord3);
#pragma unroll
      for (int ii = 0; ii < CT / J; ++ii) {
        // the row block's cos / sin first, so the 16 loads are in flight together (a
        // load is not moved above an earlier buffer store)
        float2 t[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int m = m0 + (h * (CT / J) + ii) * 32 + (r >> 2) * 8 + (r & 3);
          t[r] = rotate ? __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rc, (m * half + ip) * 8, 0, 0))
                        : make_float2(1.0f, 0.0f);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int m = m0 + (h * (CT / J) + ii) * 32 + (r >> 2) * 8 + (r & 3);
          const float x1 = v[ii * J + 0][r], x2 = v[ii * J + 1][r];
          float y1 = x1, y2 = x2;
          if (rotate) {
            y1 = x1 * t[r].x - x2 * t[r].y;
            y2 = x2 * t[r].x + x1 * t[r].y;
          }
          const int e = ((m * heads + hd) * D + ip) * 2;
          __builtin_amdgcn_raw_buffer_store_b16(uint16_t(pack_bf16x2(y1, 0.0f) & 0xFFFFu), ro, e, 0, 0);
          __builtin_amdgcn_raw_buffer_store_b16(uint16_t(pack_bf16x2(y2, 0.0f) & 0xFFFFu), ro, e + half * 2, 0, 0);
        }
      }
    } else {
      if (nt * TN + wn * 64 >= g.N) return;                // this wavefront's columns are past N
      const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(g.C, 0, g.M * g.N * 4, kBufWord3);
      const int n = nt * TN + wn * 64 + col;
#pragma unroll
      for (int ii = 0; ii < CT / J; ++ii) {
        // residual: every load of the row block first, so they are in flight together
        // (a load may not move above an earlier store through the same descriptor)
        float cin[16][J];
        if constexpr (EPI == kResidual) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int m = m0 + (h * (CT / J) + ii) * 32 + (r >> 2) * 8 + (r & 3);
#pragma unroll
            for (int j = 0; j < J; ++j)
              cin[r][j] = __builtin_bit_cast(float,
                                             __builtin_amdgcn_raw_buffer_load_b32(ro, (m * g.N + n + j * 32) * 4, 0, 0));
          }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int m = m0 + (h * (CT / J) + ii) * 32 + (r >> 2) * 8 + (r & 3);
#pragma unroll
          for (int j = 0; j < J; ++j) {
            float x = v[ii * J + j][r];
            if constexpr (EPI == kResidual) x += cin[r][j];
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), ro, (m * g.N + n + j * 32) * 4, 0, 0);
          }
        }
      }
    }
  };

  // End of a segment: a whole tile goes straight to the epilogue; a cut tile
  // through the partial buffers and its arrival counter.
  constexpr int kWaveFloats = NT * 16 * 64;
  auto finish = [&](const Cursor& c) __attribute__((always_inline)) {
    int mt, nt;
    tile_mn(c.tile, mt, nt);
    // no rows of this part (past the tile, or every row past M): nothing to write
    if (wm >= SH::WAVES_M || mt * TM + wm * SH::WM >= g.M) return;
    if (c.kbeg == 0 && c.kend == p.ks) {
#pragma unroll
      for (int h = 0; h < NCH; ++h) {
        f32x16 v[CT];
#pragma unroll
        for (int t = 0; t < CT; ++t) v[t] = acc[(h * CT + t) / J][(h * CT + t) % J];
        epilogue_part(mt, nt, h, v);
      }
      return;
    }
    // Only 256-row tiles are ever cut, so the others carry no partial protocol (and its registers).
    if constexpr (TM != 256) return;
    const int q = c.tile - p.dp_tiles;
    const int64_t U = p.sk_units;
    auto owner = [&](int64_t v) __attribute__((always_inline)) { return int(((v + 1) * p.G + U - 1) / U - 1); };
    const int wf = owner(int64_t(q) * p.ks), wl = owner(int64_t(q + 1) * p.ks - 1);
    // worker x's partial of this tile (this wavefront's part): its last segment if
    // it owns the tile's first stage (slot 2x + 1), else its first segment (slot 2x).
    // Layout: [wavefront][tile t][register quad][lane][4] floats, so each access is
    // 16 bytes per lane, 1 KB per instruction.  Partials are written and read with
    // agent-scope accesses (cache policy sc1 = device scope on gfx950), which go past
    // the XCD's L2, so no cache-wide write-back or invalidate is needed.
    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
        g.partial, 0, 2 * kMaxWorkers * kPartialFloats * 4, kBufWord3);
    auto slot_off = [&](int x) __attribute__((always_inline)) {   // bytes
      return int((2 * x + (x == wf ? 1 : 0)) * kPartialFloats + wv * kWaveFloats) * 4 + lane * 16;
    };
    constexpr int kSc1 = 16;             // cache policy sc1 alone: agent (device) scope
    typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
    int* cnt = g.tile_count + q * (kThreads / 64) + wv;
    // The tile's sum in a fixed order: the part of the owner of the tile's last
    // stage (worker wl) first, then the partials of workers wf .. wl - 1 in K order;
    // then the epilogue.  own: this wavefront is that owner and starts from its
    // accumulators, else it starts from the owner's partial.  Each partial's loads
    // are issued together, so a partial costs one round trip.
    auto fixup = [&](bool own) __attribute__((always_inline)) {
#pragma unroll
      for (int h = 0; h < NCH; ++h) {
        f32x16 v[CT];
        auto load_part = [&](int x, f32x4 (&p4)[CT * 4]) __attribute__((always_inline)) {
          const int off = slot_off(x);
#pragma unroll
          for (int c = 0; c < CT * 4; ++c)
            p4[c] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rp, off + (h * CT * 4 + c) * 1024, 0, kSc1));
        };
        if (own) {
#pragma unroll
          for (int t = 0; t < CT; ++t) v[t] = acc[(h * CT + t) / J][(h * CT + t) % J];
        } else {
          f32x4 p4[CT * 4];
          load_part(wl, p4);
#pragma unroll
          for (int c = 0; c < CT * 4; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[c >> 2][4 * (c & 3) + e] = p4[c][e];
        }
        for (int x = wf; x < wl; ++x) {
          f32x4 p4[CT * 4];
          load_part(x, p4);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int c = 0; c < CT * 4; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[c >> 2][4 * (c & 3) + e] += p4[c][e];
        }
        epilogue_part(mt, nt, h, v);
      }
      if (lane == 0) __hip_atomic_exchange(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next launch
    };
    // The owner of the tile's last stage runs that segment last (its K share runs the
    // segment that starts a tile first), so the others' partials are usually written
    // by then: it polls the counter, a bounded number of times, until the other
    // wl - wf parts have arrived, and finishes from its registers without writing its
    // own partial.  The others never see the count reach wl - wf before it, so none of
    // them finishes the tile.  If they are not all there in time it falls back to the
    // protocol below (write, count, the last to arrive finishes); the sums are the same
    // on both paths.
    if (wr == wl) {
      int seen = 0;
      for (int it = 0; it < p.polls; ++it) {
        if (lane == 0) seen = __hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        seen = __builtin_amdgcn_readfirstlane(seen);
        if (seen == wl - wf) break;
        __builtin_amdgcn_s_sleep(2);
      }
      __atomic_signal_fence(__ATOMIC_SEQ_CST);
      if (seen == wl - wf) {
        fixup(true);
        return;
      }
    }
    const int mine = slot_off(wr);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        const f32x16& a16 = acc[t / J][t % J];
        const f32x4 v4 = {a16[4 * qd], a16[4 * qd + 1], a16[4 * qd + 2], a16[4 * qd + 3]};
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4v, v4), rp, mine + (t * 4 + qd) * 1024, 0,
                                               kSc1);
      }
    // Each wavefront keeps its own arrival counter for the tile (its part of the
    // tile depends only on the same wavefront's part of the other partials), so no
    // workgroup barrier is needed: the last wavefront to arrive finishes that part.
    // The counter bump is an agent-scope atomic.  The hardware wait orders it after this
    // wavefront's partial stores; the compiler-only fences on both sides keep the
    // compiler from moving the stores below it or the partial loads above it (they
    // emit no instruction, so no L2 write-back).
    wait_vmem<0>();                      // this wavefront's partial has landed
    int before = 0;
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    if (lane == 0) before = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    before = __builtin_amdgcn_readfirstlane(before);
    if (before != wl - wf) return;       // not the last to arrive
    fixup(false);                        // the last to arrive: every part from the partials
  };

  // ---- pipeline: unit u (one K stage of one tile) lives in LDS buffer u % NS.
  // Step u reads each k-slice while the previous one runs on the matrix cores,
  // waits for this wavefront's loads of unit u + 1, and after the barrier (all
  // loads of u + 1 visible, every read of buffer u % NS done) refills that buffer
  // with unit u + NS and reads the first k-slice of u + 1.  Loads past the last
  // unit repeat it, so every step leaves the same number in flight.  (One barrier
  // per two units measured slower.)
  Cursor cc, dc;
  seek(cc, 0);
  dc = cc;
  int dtile = dc.tile;
  dma_setup(dtile);
  auto dma_advance = [&]() __attribute__((always_inline)) {
    advance(dc);
    if (dc.tile != dtile) {
      dtile = dc.tile;
      dma_setup(dtile);
    }
  };
  auto dma_next = [&](int buf) __attribute__((always_inline)) {
    dma(buf, dc.kt);
    dma_advance();
  };
#pragma unroll
  for (int b = 0; b < NS; ++b) dma_next(b);
  if (a_wave) wait_vmem<(NS - 1) * NLA>();      // unit 0 of this wavefront
  else wait_vmem<(NS - 1) * NLB>();
  barrier_lds();                                    // ... of every wavefront
  Frags f0, f1;
  read(f0, 0, 0);
  zero_acc();
  // rows of this wavefront's part of the current tile exist (else it only stages and
  // syncs)
  auto live_in = [&](int tile) __attribute__((always_inline)) {
    int mt, nt;
    tile_mn(tile, mt, nt);
    return __builtin_amdgcn_readfirstlane(int(wm < SH::WAVES_M && mt * TM + wm * SH::WM < g.M)) != 0;
  };
  bool live = live_in(cc.tile);
  int u = 0, buf = 0;
  while (true) {
    // the units of one segment (the epilogue stays out of the hot loop)
    for (const int ue = u + (cc.kend - cc.kt); u < ue; ++u) {
      const int nbuf = buf + 1 == NS ? 0 : buf + 1;
      if (live) {
        read(f1, buf, 1);
        mma(f0);
        read(f0, buf, 2);
        mma(f1);
        read(f1, buf, 3);
        mma(f0);
      }
      if (a_wave) wait_vmem<(NS - 2) * NLA>();  // this wavefront's loads of unit u + 1
      else wait_vmem<(NS - 2) * NLB>();
      barrier_lds();
      if (live) {
        read(f0, nbuf, 0);
        mma_dma(f1, buf, dc.kt);                  // unit u + NS into buf, between the MFMAs
      } else {
        dma(buf, dc.kt);
      }
      dma_advance();
      buf = nbuf;
    }
    finish(cc);
    if (u >= n_units) break;
    zero_acc();
    seek(cc, u);
    const bool was_live = live;
    live = live_in(cc.tile);
    // f0 (first k-slice of unit u, in buffer buf: loaded and published at the last
    // barrier) was only prefetched if the previous segment was live
    if (live && !was_live) read(f0, buf, 0);
  }
  wait_vmem<0>();                       // no load may land in LDS after the workgroup ends
}

__global__ void gemm_clear_kernel(int* cnt) {
  for (int i = threadIdx.x; i < kCounters; i += blockDim.x) cnt[i] = 0;
}

int cdiv(int a, int b) { return (a + b - 1) / b; }

// Counter polls of a cut tile's last-stage owner (about 0.3 ms at the default).  The
// environment variable EPIC_GEMM_FINISH_POLLS overrides it (0 forces the fallback
// protocol: a test hook); read at every launch.
int finish_polls() {
  const char* e = std::getenv("EPIC_GEMM_FINISH_POLLS");
  if (e == nullptr || *e == 0) return 4096;
  const long v = std::strtol(e, nullptr, 10);
  return int(std::min<long>(std::max<long>(v, 0), 1 << 20));
}

template <int EPI, int TM>
void launch_tn(const GemmArgs& g, bool whole_tiles, hipStream_t stream) {
  GemmPlan p{};
  p.m_tiles = cdiv(g.M, TM);
  p.n_tiles = EPI == kSwiGLU ? g.ffn / (TN / 2) : cdiv(g.N, TN);
  p.ks = g.K / kBK;
  p.gm = p.m_tiles < 8 ? p.m_tiles : 8;
  const int64_t tiles = int64_t(p.m_tiles) * p.n_tiles;
  if (whole_tiles) {
    // one round of whole tiles (a multiple of 8 workgroups, for the XCD-contiguous order)
    p.G = int((tiles + 7) / 8 * 8);
    p.dp_rounds = 1;
    p.dp_tiles = int(tiles);                         // a short last round leaves some workgroups idle
    p.sk_units = 0;
  } else {
    const int64_t units = tiles * p.ks;
    p.G = int(std::min<int64_t>(kMaxWorkers, std::max<int64_t>(1, units / kMinUnits)));
    const int64_t full = tiles / p.G, rem = tiles % p.G;
    p.dp_rounds = int(rem == 0 ? full : std::max<int64_t>(full - 1, 0));
    p.dp_tiles = p.dp_rounds * p.G;
    p.sk_units = int((tiles - p.dp_tiles) * p.ks);
  }
  p.polls = finish_polls();
  gemm_kernel<EPI, TM><<<dim3(p.G), kThreads, 0, stream>>>(g, p);
}

template <int EPI>
void launch_epi(const GemmArgs& g, GemmRoute r, hipStream_t stream) {
  if (r == GemmRoute::kWhole96) launch_tn<EPI, 96>(g, true, stream);
  else if (r == GemmRoute::kWhole128) launch_tn<EPI, 128>(g, true, stream);
  else launch_tn<EPI, 256>(g, false, stream);
}

}  // namespace

GemmRoute gemm_route(const GemmArgs& g, int epi) {
  // At least a round of 256 x 256 tiles: whole tiles only (measured: cutting tiles
  // along K costs about one tile time in partial traffic, more than a short last
  // round).  The tiles are 256 or 192 rows high, whichever takes less time: a round
  // of 192-row tiles takes 0.77-0.84 of one of 256-row tiles (gate|up, W_down, W_O and
  // Q|K|V of 20 560 rows), counted as 13/16.  So W_down and W_O of 20 560 rows run 7 rounds
  // of 192 rows (1925 and 618 us) instead of 6 of 256 (1961 and 634), gate|up 36 rounds
  // of 256 (3607 us) instead of 48 of 192 (3755), and gate|up of 736 rows 2 rounds of
  // 192 rows on 224 CUs instead of 2 of 256 on 168.
  const bool swiglu = epi == kSwiGLU;
  const int m_tiles = cdiv(g.M, kTM);
  const int n256 = swiglu ? (g.ffn % 128 == 0 ? g.ffn / 128 : 0) : cdiv(g.N, 256);
  if (int64_t(m_tiles) * n256 >= kMaxWorkers) {
    const int64_t r256 = (int64_t(m_tiles) * n256 + kMaxWorkers - 1) / kMaxWorkers;
    const int64_t r192 = (int64_t(cdiv(g.M, 192)) * n256 + kMaxWorkers - 1) / kMaxWorkers;
    return r192 * 13 < r256 * 16 ? GemmRoute::kWhole192 : GemmRoute::kWhole256;
  }
  if (swiglu && glu_fits(g.M, g.ffn, g.K)) return GemmRoute::kGlu;
  // Fewer: with a short K and one round of 96 x 128 or 128 x 128 tiles that fills at
  // least 3/4 of the CUs, those tiles whole (96 rows where they make such a round: more
  // CUs, fewer bytes each); else 256 x 128 tiles cut along K so that every CU gets a
  // share.  Measured at 736 rows, N = 4096: whole 128 x 128 tiles take about 0.57 us per
  // K stage on 192 CUs, the cut tiles about 0.45 us per stage of a tile's K plus about
  // 15 us of partial traffic and fixup, so whole tiles win up to about 100 stages (W_O,
  // K = 4096: 48.0 -> 40.2 us; W_down, K = 14336: 103.8 -> 127.7 us).  96 x 128 tiles on
  // 256 CUs took W_O about 1 us further (the c3 link step 0.3% faster on one box).
  const int64_t n128 = swiglu ? g.ffn / 64 : cdiv(g.N, 128);
  const int64_t t128 = int64_t(cdiv(g.M, 128)) * n128, t96 = int64_t(cdiv(g.M, 96)) * n128;
  auto one_round = [](int64_t t) { return t >= 3 * kMaxWorkers / 4 && t <= kMaxWorkers; };
  if (g.K / kBK <= 96) {
    if (one_round(t96)) return GemmRoute::kWhole96;
    if (one_round(t128)) return GemmRoute::kWhole128;
  }
  // Else the least estimated time (us).  The estimates are fitted to every route at 1486
  // sizes (N 1024-32768, K 512-14336, 1-7000 rows; relative deviation 4-8%), of which they
  // take routes 0.5% (geometric mean) behind the best one, and 27% ahead of cutting always.
  // w: MB of weights, u: K stages per workgroup.  Measured examples (K x N, rows: us):
  //   streamed weights  4096 x 4096, 128: 15.6, 384: 29; 14336 x 4096, 128: 31, 384: 53
  //   whole wide tiles  4096 x 28672, 300: 87 (cut 115), 512: 115 (150); 4096 x 6144, 1500: 68 (84; 77 in two chains)
  //   split wide tiles  14336 x 4096, 363: 57 (streamed 75), 736: 92 (cut 110), 2000: 206 (249);
  //                     8192 x 2048, 600: 42 (53)
  //   cut tiles         4096 x 4096, 1472: 61-66 (split 66-69); 14336 x 16384, 64: 90 (streamed 114)
  //   ... a whole number of rounds of them, none cut: 2048 x 16384, 300: 37 (whole wide tiles 40),
  //                     4096 x 8192, 769: 64 (split 71), 2048 x 32768, 129: 40 (53)
  // In a layer the pass that sums partials replaces a norm or a link write (bonus).
  constexpr double kNever = 1e30;
  const double bonus = !g.in_layer ? 0.0 : epi == kResidual ? 5.0 : epi == kRope ? 10.0 : 0.0;
  const double w = double(g.K) * g.N * 2e-6, plane = double(g.M) * g.N * 4e-6;
  const int64_t ks = g.K / kBK;
  const double per_mb = g.M <= 32 ? 0.12 : g.M <= 64 ? 0.14 : g.M <= 128 ? 0.155 : g.M <= 256 ? 0.27 : g.M <= 384 ? 0.52 : 0.66;
  const double stream = g.M <= kStreamRows && stream_fits(g.M, g.N, g.K)
                            ? 9.0 + w * per_mb + 0.08 * std::max(w - 100.0, 0.0) + 0.38 * plane - bonus
                            : kNever;
  const WideSplit sp = wide_split(g, epi);
  const double split = sp.parts >= 2 ? wide_split_time(sp, g.M, g.N, g.K) + 0.24 * sp.parts * plane - bonus : kNever;
  const int chains = std::min<int64_t>(gemm_chains(g, epi), ks);
  auto whole = [&](int tm) {     // one round; a stage takes longer the more CUs run; a further chain is a tile written and read
    const int64_t tiles = int64_t(cdiv(g.M, tm)) * n256;
    if (n256 == 0 || tiles > kMaxWorkers) return kNever;
    const double t = double(tiles) / kMaxWorkers;
    return 5.8 + ks * (tm == 256 ? 0.90 + 0.44 * t : 0.69 + 0.37 * t) + 0.05 * w + 0.067 * plane +
           (chains - 1) * (tm == 256 ? 8.0 + 0.15 * plane : 8.0 + 0.12 * plane);
  };
  const double whole256 = whole(256), whole192 = whole(192);
  // A stage of a 256 x 128 tile: less where wavefronts have no rows (64 each) if that holds
  // for a whole round; a stage of one row tile's waits for weights that no other tile shares.
  const int64_t cut_tiles = int64_t(m_tiles) * n128;
  const double live = double(cdiv(g.M, 64) * 64) / (m_tiles * kTM);
  const bool rounds = cut_tiles % kMaxWorkers == 0;     // whole rounds: nothing is cut
  const double stage = m_tiles == 1 ? (0.61 + 0.45 * live) * (rounds || kMaxWorkers % cut_tiles == 0 ? 1.0 : 1.12)
                                    : rounds ? 0.46 + 0.54 * live : 1.11;
  const double cut = 10.2 + stage * double(cut_tiles * ks) / kMaxWorkers + (rounds ? 0.0 : 2.5 * kMaxWorkers / double(cut_tiles));
  const double best = std::min({stream, split, whole256, whole192, cut});
  if (best == stream) return GemmRoute::kStream;
  if (best == split) return GemmRoute::kSplit;
  if (best == whole192) return GemmRoute::kWhole192;
  if (best == whole256) return GemmRoute::kWhole256;
  return GemmRoute::kCut;
}

const char* gemm_route_name(GemmRoute r) {
  switch (r) {
    case GemmRoute::kWhole256: return "whole256";
    case GemmRoute::kWhole192: return "whole192";
    case GemmRoute::kWhole128: return "whole128";
    case GemmRoute::kWhole96: return "whole96";
    case GemmRoute::kCut: return "cut";
    case GemmRoute::kStream: return "stream";
    case GemmRoute::kSplit: return "split";   // epic_gemm_route_name adds the tile height
    case GemmRoute::kGlu: return "glu";
  }
  return "";
}

size_t gemm_partial_floats() { return size_t(2 * kMaxWorkers) * kPartialFloats; }

int gemm_counters() { return kCounters; }

size_t gemm_workspace_bytes() { return gemm_partial_floats() * sizeof(float) + kCounters * sizeof(int); }

void gemm_workspace(void* base, float** partial, int** tile_count) {
  *partial = static_cast<float*>(base);
  *tile_count = reinterpret_cast<int*>(static_cast<char*>(base) + size_t(2 * kMaxWorkers) * kPartialFloats * 4);
}

void launch_gemm_clear(int* tile_count, hipStream_t stream) {
  gemm_clear_kernel<<<1, 256, 0, stream>>>(tile_count);
}

void launch_gemm(const GemmArgs& g, int epi, GemmRoute r, hipStream_t stream) {
  if (g.M == 0) return;
  if (is_partial(r))
    launch_stream_finish(launch_gemm_partial(g, epi, r, stream), g, epi, stream);
  else if (r == GemmRoute::kGlu)
    launch_gemm_glu(g, stream);
  else if (r == GemmRoute::kWhole256 || r == GemmRoute::kWhole192)
    launch_gemm_wide(g, epi, r == GemmRoute::kWhole256 ? 256 : 192, stream);
  else if (epi == kStoreF32)
    launch_epi<kStoreF32>(g, r, stream);
  else if (epi == kRope)
    launch_epi<kRope>(g, r, stream);
  else if (epi == kResidual)
    launch_epi<kResidual>(g, r, stream);
  else
    launch_epi<kSwiGLU>(g, r, stream);
}

}  // namespace epic
