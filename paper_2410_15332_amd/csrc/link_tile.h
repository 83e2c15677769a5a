// One block's V slab [D][16] (bf16) in LDS, filled by rows and stored transposed.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace epic {

// Rows of 18 values: 2-byte stores of one chunk's dims fall in distinct banks, and the
// 16 slots of a dim leave as four-byte reads.
template <int D>
struct VTile {
  static constexpr int LD = 18;
  alignas(4) uint16_t e[D * LD];               // read and written four bytes at a time too

  // thread tid (of 2 D) moves dim tid / 2, slots 8 (tid % 2) .. + 7
  __device__ __forceinline__ void load(const uint16_t* slab, int tid) {
    const uint4 x = *reinterpret_cast<const uint4*>(slab + tid * 8);
    uint32_t* p = reinterpret_cast<uint32_t*>(e + (tid >> 1) * LD + (tid & 1) * 8);
    p[0] = x.x, p[1] = x.y, p[2] = x.z, p[3] = x.w;
  }
  __device__ __forceinline__ void store(uint16_t* slab, int tid) const {
    const uint32_t* p = reinterpret_cast<const uint32_t*>(e + (tid >> 1) * LD + (tid & 1) * 8);
    *reinterpret_cast<uint4*>(slab + tid * 8) = make_uint4(p[0], p[1], p[2], p[3]);
  }
  // dims d .. d + 7 of slot o
  __device__ __forceinline__ void put(int o, int d, const uint4& x) {
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      e[(d + 2 * i) * LD + o] = uint16_t(w[i] & 0xFFFFu);
      e[(d + 2 * i + 1) * LD + o] = uint16_t(w[i] >> 16);
    }
  }
};

}  // namespace epic
