// Shared by the grouped GEMMs of a multi-token call (kernels.hip, wide.h): the
// experts of a launch, its M-tiles, operand types and block decoding helpers.
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstdint>

#include "kernels.h"

namespace moecache {

constexpr int kWave = 64;

// MFMA operand and accumulator vectors.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float half_bits_to_float(uint32_t bits16) {
  _Float16 h;
  uint16_t b = (uint16_t)bits16;
  __builtin_memcpy(&h, &b, 2);
  return (float)h;
}

// A pair is only 4-byte aligned; the 16-byte loads below rely on the
// unaligned global access that gfx9 runtimes enable (one dwordx4 instead of
// four dword loads: a quarter of the address work per byte).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_a4 __attribute__((aligned(4)));
// Weight pointers come out of the work lists as generic pointers; loads
// through them would be flat loads, which also count against the LDS wait
// counter (every LDS wait would then wait for the weights as well).  Slots
// are device memory: the weights are read through global-address-space
// pointers.
typedef __attribute__((address_space(1))) const u32x4_a4 g_u32x4_a4;
typedef __attribute__((address_space(1))) const uint32_t g_u32;

// One wave's experts for the grouped GEMMs (kernel argument, 3.3 KB; all arguments of a
// launch together have to stay within 4 KB).
constexpr int kPfMaxExperts = 128;
constexpr int kPfMaxTiles = 512;  // 128 experts of up to 576 rows in tiles of 144
struct PfExperts {
  const uint8_t *payload[kPfMaxExperts];
  int32_t row0[kPfMaxExperts];  // first row of the expert's pairs in perm / Ab
  int32_t n[kPfMaxExperts];     // pairs (tokens) routed to it
  int16_t rt[kPfMaxExperts];    // rows of each of its M-tiles but the last
  int32_t count;
  // flat M-tile t: expert in the low byte, the expert's M-tile in the high
  // byte; ntiles == 0 when the launch's tiles do not fit (then a scan)
  int32_t ntiles;
  uint16_t tile[kPfMaxTiles];
};

constexpr int kPfBM = 128;  // tokens per tile
constexpr int kPfBK = 64;   // one pair of weight blocks per row
// Rows of the wide and the slim kernels' largest tile.
constexpr int kWideBM = 144, kSlimBM = 64;

// (expert, first row) of a flat M-tile index; returns false past the end.  One
// lookup in the launch's tile table (a scan over the experts, one dependent
// scalar load each, took microseconds for the last tiles of a launch).
__device__ __forceinline__ bool pf_tile(const PfExperts &X, int mt, int &j, int &m0) {
  if (X.ntiles > 0) {
    if (mt >= X.ntiles) return false;
    const uint32_t v = X.tile[mt];
    j = (int)(v & 0xffu);
    m0 = (int)(v >> 8) * X.rt[j];
    return true;
  }
  for (j = 0; j < X.count; ++j) {
    const int rt = X.rt[j], tiles = (X.n[j] + rt - 1) / rt;
    if (mt < tiles) {
      m0 = mt * rt;
      return true;
    }
    mt -= tiles;
  }
  return false;
}

struct GmParams {
  PfExperts X;
  const int32_t *perm;
  const __bf16 *A;  // gate/up: xb [2][T][H]; down: ab [2][pairs][I] (hi then lo planes)
  __bf16 *ab;       // gate/up output [2][pairs][I]
  const float *w;   // down: routing weights [pairs]
  float *P;         // down output [pairs][H]
  int T, pairs, H, I, k;
  int64_t mat, down_off;  // bytes of W_gate; offset of W_down in a payload
  int64_t rowb;           // bytes of a weight row of the format (gate/up: H inputs; down: I)
};

// The wide-tile kernels (wide.h), one translation unit per weight format.
template <int FMT>
hipError_t wide_gateup(bool slim, dim3 grid, const GmParams &a, hipStream_t s, const Timing &t);
template <int FMT>
hipError_t wide_down(bool slim, dim3 grid, const GmParams &a, hipStream_t s, const Timing &t);

}  // namespace moecache
