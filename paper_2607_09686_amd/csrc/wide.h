// The grouped GEMMs' wide-tile kernels (a multi-token call's gate/up and down over
// many rows per expert), templates over the weight format; each format is its own
// translation unit (wide_*.hip), so that they compile side by side.
#pragma once
#include <type_traits>

#include "grouped.h"

namespace moecache {
namespace {

// SiLU for the grouped GEMMs' epilogue: the hardware base-2 exponential and
// reciprocal (about 1 ulp each) instead of the library exp and an IEEE divide,
// which took a fifth of a tile's time there.
__device__ __forceinline__ float silu_fast(float s) {
  return s * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * s));
}

typedef __attribute__((address_space(3))) void lds_void;

// Direct global -> LDS load of 16 bytes per lane from a buffer: lane l's bytes, at
// byte offset off + base of the buffer (off per lane, base uniform), land at
// dst + 16 l (dst wave-uniform).  (The buffer form: after a flat-encoded direct load
// the compiler takes every later wait for a loaded register as a wait for all.)
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t buf, uint32_t off, uint32_t base, void *dst) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(buf, (lds_void *)dst, 16, (int)off, (int)base, 0, 0);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t wide_buffer(const void *p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}

// Two kernels for each of gate/up and down, both over tiles of rows x 256 weight rows
// with K steps of 64.  The activation tile (both planes) goes straight from global
// memory into LDS with direct loads.  Every multiplying wave takes all of a tile's rows
// in 16-row subtiles against 64 of its 256 weight rows, so a tile's MFMAs follow its
// rows.  An expert's rows are split evenly over ceil(n / 144) tiles.
//   wide (tiles of up to 144 rows): 512 threads, one block per CU.  Waves 0-3 multiply
//     the current step, waves 4-7 stage the next one: the direct loads and the weight
//     tile, dequantised into LDS.
//   slim (launches whose tiles have at most 64 rows, at least three K steps, not Q6_K): 256
//     threads, two blocks per CU.
//     Each wave loads and dequantises its own 64 weight rows into its MFMA operand
//     registers (nothing of a weight goes through LDS), with the loads of later steps
//     in flight and the activations two steps ahead in three LDS stages.
// Both multiply the same products in the same order into an accumulator, so that a row's
// result does not depend on which of them, or which tile of it, computes the row.
// The line between them lies at 64 rows: whole warm calls of 12 to 120 tokens over 128
// experts take 3 to 5 % less with slim tiles than with wide ones (61 tokens: Q4_0 213 us
// against 221, Q8_0 243 against 255, Q4_K 219 against 228), 200 to 300 tokens the same
// within 3 %; above, splitting experts into 64-row tiles loses (Q8_0, 1200 tokens: 442 us
// against 393), as a wave's vector instructions do not hide behind its own MFMAs.  Q6_K has
// no slim kernels: its dequantisation is the longest, and the wide kernels' staging waves are
// as fast at few rows and faster at many (kernels.hip, wide_launch).
// A warm call over 128 experts of 768 x 2048 (Q8_0), gate/up + down: 4096 tokens 536 +
// 327 us with 128-row tiles and a weight row per staging lane, 467 + 284 us wide (883
// TFLOP/s of gate/up MFMAs on real rows; a large library bf16 product: 1118); 61 tokens
// 198 + 104 -> 116 + 62 us slim (3.5 TB/s of weights).  Q4_K gate/up + Q6_K down: 527 + 376
// -> 470 + 328 us; 61 tokens 178 + 117 -> 101 us slim + 81 us wide.
// Each LDS stage is its own array, so that the compiler sees the reads of one stage not
// alias the loads into the other.  The 1-D grid runs the column tiles of an M-tile, then
// an expert's M-tiles, one after the other on the same XCD (block L runs on XCD L % 8), so
// that their shared activation rows and weights come from that XCD's L2.
constexpr int kWideThreads = 512, kSlimThreads = 256;
template <int ROWS>
using ActTile = __bf16[2][ROWS][64];  // [plane][row][k], 16-byte chunks swizzled by row
typedef __bf16 WeightTile[256][kPfBK + 8];

// A lane's raw bytes of one K step and weight row.  Lane l works on quarter g = l % 4 (16
// weights) of weight row l / 4, so that four consecutive lanes read one row's 64 to 80
// bytes: with the MFMA operands' own order (row l % 16) every 16 lanes touch 16 rows and a
// load takes 64 cycles of address work.  Every format takes 20 bytes per lane, two load
// instructions (16 + 4 bytes): what several quarters need of a K-quant's super-block, one
// lane of the four loads and the others get by quad permutation.  (With each lane loading
// all it needs, 12 dwords in six instructions for Q6_K and 8 in two for Q4_K, the slim kernels
// spilled 312 to 357 and 8 to 10 registers; warm calls of 61 tokens over 128 experts took 376
// us in Q6_K and 235 in Q4_K, now 288 and 217, and a Q4_K_M call of 4096 tokens 937, now 870.)
constexpr int kRawDw = 5, kRawLoads = 2;
typedef uint32_t RawStep[kRawDw];
// Another lane's value of the four that share a row: quad_perm [C % 4, C / 4 % 4, ...].
template <int C>
__device__ __forceinline__ uint32_t quad(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, C, 0xf, 0xf, true);
}
// Keeps the compiler from masking and shifting each byte of q by itself: four bytes masked
// at once, then one byte conversion each (80 of Q4_K's 395 vector instructions in a step).
__device__ __forceinline__ void keep_bytes(uint32_t &q) { asm("" : "+v"(q)); }
// K order of the steps.  A step multiplies 64 inputs; the sum over K does not
// depend on the order in which they are visited, so a format may visit them in the
// order its bytes hold them, as long as activations and weights use the same one.
// Step kt, 16-byte chunk c of the activation tile's row (eight inputs) covers K
// indices wide_kbase(kt) + wide_kchunk(c) + 0..7; quarter g of a weight row's step
// meets chunks 2 g and 2 g + 1.
// Q6_K: a step is one quarter (n, j) of a super-block, n = the half (128
// weights), j = which 16 of each of its four 32-weight groups: the weights
// 128 n + 32 g + 16 j + l (g < 4, l < 16), whose low bits sit in 16 bytes of
// ql for g = 0, 2 (low and high nibbles), 16 bytes for g = 1, 3, and whose high
// bits sit in 16 bytes of qh (two bits per group).  So every loaded byte is
// used by one step only.
template <int FMT>
__device__ __forceinline__ uint32_t wide_kbase(int kt) {
  if constexpr (FMT == 14) return 256u * (uint32_t)(kt >> 2) + 128u * (uint32_t)((kt >> 1) & 1) + 16u * (uint32_t)(kt & 1);
  return (uint32_t)(kt * kPfBK);
}
template <int FMT>
__device__ __forceinline__ uint32_t wide_kchunk(int c) {
  if constexpr (FMT == 14) return 32u * (uint32_t)(c >> 1) + 8u * (uint32_t)(c & 1);
  return 8u * (uint32_t)c;
}
// Every load stays inside the row's step (Q8_0, Q4_0), inside the super-block (Q4_K) or,
// for Q6_K (210-byte super-blocks, 2-byte aligned; a: the address rounded down to a dword),
// inside [a, a + 212): a payload starts and ends 16-byte aligned, so its last super-block
// starts at an address 2 mod 4 and ends at a + 212.
// base, off: see WeightRows.
template <int FMT>
__device__ __forceinline__ void wide_load(const uint8_t *base, uint32_t off, int kt, int g, RawStep &v) {
  uint32_t p, last;  // 16 bytes and the fifth dword
  if constexpr (FMT == 8) {
    // block g / 2 of the 68-byte pair: the five dwords around the 16 q bytes (its d is
    // in the first dword of the even quarter)
    p = off + (uint32_t)kt * 68u + 16u * (uint32_t)g;
    last = p + 16;
  } else if constexpr (FMT == 2) {
    p = off + (uint32_t)kt * 36u + 16u * (uint32_t)(g >> 1);
    last = p + 16;
  } else if constexpr (FMT == 12) {
    // the quarter's 16 q bytes; dword g of the super-block's header
    const uint32_t b = off + (uint32_t)(kt >> 2) * 144u;
    p = b + 16u + 32u * (uint32_t)(kt & 3) + 16u * (uint32_t)(g & 1);
    last = b + 4u * (uint32_t)g;
  } else {
    // quarters 0 and 1: the 16 ql bytes of groups g and g + 2, at 64 n + 32 g + 16 j; 2: the
    // 16 qh bytes of all groups, at 128 + 32 n + 16 j; 3: the super-block's 16 scales and d,
    // at 192; with what lies before and behind them in the same dwords
    const uint32_t n = (kt >> 1) & 1, j = kt & 1;
    p = ((off + (uint32_t)(kt >> 2) * 210u) & ~3u) +
        (((0xc0802000u + n * 0x00204040u + j * 0x00101010u) >> (8 * g)) & 0xffu);
    last = p + 16;
  }
  v[4] = *(const g_u32 *)(base + last);
  // (the single dword of each row first: with all the 16-byte loads first a warm Q8_0 call of
  // 61 tokens took 265 us instead of 243, with each row's 16 bytes first 253)
  asm volatile("" ::: "memory");
  const u32x4 q = *(g_u32x4_a4 *)(base + p);
  v[0] = q.x;
  v[1] = q.y;
  v[2] = q.z;
  v[3] = q.w;
  asm volatile("" ::: "memory");
}
// The quarter's 16 weights as bf16 (nearest even, from the fp32 value), eight per
// MFMA operand.  Q8_0: d q.  Q4_0: the nibbles as signed bytes 16 (n - 8) times d / 16,
// both exact, so d (n - 8) rounded once.  Q4_K: d sc q - dmin m, one fused multiply-add.
// Q6_K: ds (q - 32) = fma(ds, q, -32 ds) (32 ds is exact).
// The choices that depend on kt (the same for every lane) are byte permutes and shifts: as
// selects they become branches, which the scheduling groups of slim_gemm cannot cross.
template <int FMT>
__device__ __forceinline__ void wide_dequant(const RawStep &v, uint32_t off, int kt, int g, bf16x8 (&o)[2]) {
  if constexpr (FMT == 8 || FMT == 2) {
    // block 0's q bytes start two bytes into the loaded dwords, block 1's one dword in
    const bool b1 = g >> 1;
    const uint32_t sel = b1 ? 0x07060504u : 0x05040302u;
    // Q8_0: the first dword of the block, from the lane of its even quarter
    const uint32_t dd = FMT == 8 ? quad<0xa0>(v[0]) : v[0];
    const float d0 = half_bits_to_float(b1 ? dd >> 16 : dd & 0xffffu);
    const float d = FMT == 8 ? d0 : 0.0625f * d0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint32_t w = __builtin_amdgcn_perm(v[j + 1], v[j], sel);
      if constexpr (FMT == 2) w = ((w << ((g & 1) ? 0 : 4)) & 0xf0f0f0f0u) ^ 0x80808080u;
#pragma unroll
      for (int b = 0; b < 4; ++b)
        o[j >> 1][4 * (j & 1) + b] = (__bf16)(d * (float)(int8_t)((w >> (8 * b)) & 0xffu));
    }
  } else if constexpr (FMT == 12) {
    // sub-block s = 2 (kt % 4) + g / 2 of the eight (low nibbles for g < 2, high for g >= 2);
    // header: d and dmin, then the six-bit scales and mins of sub-blocks 0..3 in bytes s of B0
    // and B1; of 4..7 the low four bits in byte s - 4 of B2, the high two in the upper bits of
    // bytes s - 4 of B0 and B1
    const uint32_t D = quad<0x00>(v[4]), B0 = quad<0x55>(v[4]), B1 = quad<0xaa>(v[4]), B2 = quad<0xff>(v[4]);
    const int s = 2 * (kt & 3) + (g >> 1), up = 8 * (s & 3) + (kt & 2);
    const uint32_t low = 0x0c0c0c00u | (uint32_t)s;  // byte s of eight, zero extended
    const uint32_t sc = (__builtin_amdgcn_perm(B2, B0, low) & 0x0fu) | ((B0 >> up) & 0x30u);
    const uint32_t mn = ((__builtin_amdgcn_perm(B2, B1, low) >> ((2 * kt) & 4)) & 0x0fu) | ((B1 >> up) & 0x30u);
    const float d = half_bits_to_float(D & 0xffffu), dmin = half_bits_to_float(D >> 16);
    const float ds = d * (float)sc, dm = dmin * (float)mn;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint32_t q = (v[j] >> (4 * (g >> 1))) & 0x0f0f0f0fu;
      keep_bytes(q);
#pragma unroll
      for (int b = 0; b < 4; ++b)
        o[j >> 1][4 * (j & 1) + b] = (__bf16)fmaf(ds, (float)((q >> (8 * b)) & 0xffu), -dm);
    }
  } else {
    // the lane's own bytes at their place, then low four bits from the low (g < 2) or high
    // nibbles of lane g % 2, high two from bits 2 g, 2 g + 1 of lane 2, scale 8 n + 2 g + j
    // and d from lane 3
    const int sh = (int)((off + 2u * (uint32_t)(kt >> 2)) & 3u), n = (kt >> 1) & 1, j0 = kt & 1;
    uint32_t a[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] = __builtin_amdgcn_alignbyte(v[j + 1], v[j], sh);
    const uint32_t half = n ? 0x07060504u : 0x03020100u;
    const uint32_t s0 = quad<0xff>(__builtin_amdgcn_perm(a[2], a[0], half));
    const uint32_t s1 = quad<0xff>(__builtin_amdgcn_perm(a[3], a[1], half));
    const float d = half_bits_to_float(quad<0xff>(v[4] >> (8 * sh)) & 0xffffu);
    const float ds = d * (float)(int8_t)__builtin_amdgcn_perm(s1, s0, 0x0c0c0c00u | (uint32_t)(2 * g + j0));
    const float dm = -32.f * ds;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t lq = quad<0x44>(a[j]), hq = quad<0xaa>(a[j]);
      uint32_t q = ((lq >> (4 * (g >> 1))) & 0x0f0f0f0fu) | (((hq >> (2 * g)) & 0x03030303u) << 4);
      keep_bytes(q);
#pragma unroll
      for (int b = 0; b < 4; ++b)
        o[j >> 1][4 * (j & 1) + b] = (__bf16)fmaf(ds, (float)((q >> (8 * b)) & 0xffu), dm);
    }
  }
}

// A wave's 64 weight rows as four subtiles of 16, two from `first` and two `second` bytes on:
// base[q], the same for every lane, is the start of subtile q and off the distance from
// there to the lane's row.  Payloads are 16-byte aligned and 16 rows of any format a
// multiple of four bytes, so every base is dword aligned.  (A pointer per lane and subtile
// took eight registers and a 64-bit sum for each load.)
struct WeightRows {
  const uint8_t *base[4];
  uint32_t off;
  __device__ __forceinline__ WeightRows(const uint8_t *first, int64_t rowb, int64_t second, int lane)
      : base{first, first + 16 * rowb, first + second, first + second + 16 * rowb},
        off((uint32_t)(lane >> 2) * (uint32_t)rowb) {}
};

// (slim kernels) Brings the quarters of row r, held by lanes 4 r .. 4 r + 3, into the MFMA
// operand order of the wide kernels: o[ks] of lane 16 g + r gets the eight weights that
// meet chunk 4 ks + g, half g % 2 of quarter 2 ks + g / 2.  Lane group g fetches both
// halves of quarter 0, 2, 1, 3; swapping the odd groups of the first halves with the
// even groups of the second ones then leaves the chunks in order.
__device__ __forceinline__ void slim_fetch(bf16x8 (&o)[2]) {
  const int lane = threadIdx.x & (kWave - 1), g = lane >> 4;
  const int src = 4 * (4 * (lane & 15) + 2 * (g & 1) + (g >> 1));
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    u32x4 d = __builtin_bit_cast(u32x4, o[h]);
#pragma unroll
    for (int i = 0; i < 4; ++i) d[i] = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)d[i]);
    o[h] = __builtin_bit_cast(bf16x8, d);
  }
}
__device__ __forceinline__ void slim_swap(bf16x8 (&o)[2]) {
  u32x4 d0 = __builtin_bit_cast(u32x4, o[0]), d1 = __builtin_bit_cast(u32x4, o[1]);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const auto r = __builtin_amdgcn_permlane16_swap(d0[i], d1[i], false, false);
    d0[i] = r[0];
    d1[i] = r[1];
  }
  o[0] = __builtin_bit_cast(bf16x8, d0);
  o[1] = __builtin_bit_cast(bf16x8, d1);
}

// The (M-tile, column tile) of this block in the XCD-grouped order.
__device__ __forceinline__ void wide_tile(int NT, int &mt, int &nt) {
  const int total = gridDim.x, L = blockIdx.x, x = L % 8, idx = L / 8, per = total / 8, rem = total % 8;
  const int w = x * per + min(x, rem) + idx;
  mt = w / NT;
  nt = w % NT;
}

// Waits until at most N vector memory operations of the wave are outstanding and its
// LDS reads are done, then for the block.  (No fence: it would wait for every load in
// flight.  What crosses the barrier is LDS written by direct loads, which the wait
// covers, and stages read by finished LDS reads.)
template <int N>
__device__ __forceinline__ void wide_sync() {
  static_assert(N < 64, "the wait counter has six bits");
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));  // vmcnt(N) lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// One tile of NI 16-row subtiles (KT >= 3 K steps): acc[i][q] = subtile i times the
// wave's weight subtile q.  base[q], off: where the row of weight subtile q that this lane loads starts; A: the
// activation plane the wave loads from (wave wv: rows 16 u + 8 (wv / 2) .. +7 of
// plane wv % 2); asrc(u): byte offset there of this lane's 16 bytes of subtile u.
//
// Order of a wave's vector memory operations in step kt: the direct loads of
// kt + 2 (NI instructions), then the raw weights of kt + 3 (at least LW).  At
// the start of step kt the direct loads of kt have to be in: issued in step kt - 2,
// they are followed by two steps' weights and one step's direct loads, so a wait
// for at most 2 LW + NI outstanding operations covers them.  Three LDS stages rotate;
// the loop's head runs KT % 3 steps so that the last three steps are a fixed tail.
template <int FMT, int NI, class Src>
__device__ __forceinline__ void slim_gemm(f32x4 (&acc)[NI][4], __amdgpu_buffer_rsrc_t A, Src asrc,
                                          const uint8_t *const (&base)[4], uint32_t off, int KT, int wv, int lane,
                                          ActTile<kSlimBM> &As0, ActTile<kSlimBM> &As1, ActTile<kSlimBM> &As2) {
  constexpr int LW = 4 * kRawLoads;
  const int g = lane >> 4;
  uint32_t src[NI];
#pragma unroll
  for (int u = 0; u < NI; ++u) src[u] = asrc(u);
  RawStep W[3][4];
  bf16x8 bf[3][4][2];
  auto aload = [&](int kt, ActTile<kSlimBM> &As) {
#pragma unroll
    for (int u = 0; u < NI; ++u)
      dma16(A, src[u], 2 * wide_kbase<FMT>(kt), &As[wv & 1][16 * u + 8 * (wv >> 1)][0]);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
  };
  auto wload = [&](int kt, RawStep (&w)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) wide_load<FMT>(base[q], off, kt, lane & 3, w[q]);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto dequant = [&](int kt, const RawStep (&w)[4], bf16x8 (&b)[4][2]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      wide_dequant<FMT>(w[q], off, kt, lane & 3, b[q]);
      slim_fetch(b[q]);
      if (q > 0) slim_swap(b[q - 1]);  // (its fetches have come back by now)
    }
    slim_swap(b[3]);
  };
  // A subtile's operands are read one subtile ahead of its eight MFMAs; the scheduling
  // groups spread the step's dequantisation between the MFMAs (VMFMA of its vector
  // instructions behind each), which leaves it in their shadow.
  constexpr int kVector = FMT == 8 ? 210 : FMT == 2 ? 240 : 320;  // vector instructions of a step
  constexpr int VMFMA = (kVector + 16 * NI - 1) / (16 * NI);
  auto mma = [&](const ActTile<kSlimBM> &As, const bf16x8 (&b)[4][2]) {
    bf16x8 hi[2], lo[2];
    auto aread = [&](int s) {
      const int r = 16 * (s % NI) + (lane & 15);
      const int c = (4 * (s / NI) + g) ^ (r & 7);
      hi[s & 1] = *reinterpret_cast<const bf16x8 *>(&As[0][r][8 * c]);
      lo[s & 1] = *reinterpret_cast<const bf16x8 *>(&As[1][r][8 * c]);
    };
    aread(0);
    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
    for (int s = 0; s < 2 * NI; ++s) {
      const int i = s % NI, ks = s / NI;
      if (s + 1 < 2 * NI) {
        aread(s + 1);
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        acc[i][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi[s & 1], b[q][ks], acc[i][q], 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        acc[i][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo[s & 1], b[q][ks], acc[i][q], 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x2, VMFMA, 0);
      }
    }
  };
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[i][q] = f32x4{0.f, 0.f, 0.f, 0.f};
  // step kt: operands bf[S], stage AC; bf[S1] takes kt + 1's weights from W[S1]; stage
  // AN takes the activations of kt + 2; W[S] the raw weights of kt + 3
#define SLIM_STEP(S, AC, AN, kt)                            \
  do {                                                      \
    wide_sync<2 * LW + NI>();                               \
    aload((kt) + 2, AN);                                    \
    wload((kt) + 3, W[S]);                                  \
    dequant((kt) + 1, W[((S) + 1) % 3], bf[((S) + 1) % 3]); \
    mma(AC, bf[S]);                                         \
  } while (0)
#define SLIM_HEAD(S, A0, A1)                                     \
  do {                                                           \
    wload(0, W[S]);                                              \
    aload(0, A0);                                                \
    wload(1, W[((S) + 1) % 3]);                                  \
    aload(1, A1);                                                \
    wload(2, W[((S) + 2) % 3]);                                  \
    dequant(0, W[S], bf[S]);                                     \
  } while (0)
  const int lead = KT % 3;
  int kt = 0;
  // (a first step whose earlier operations are fewer than its wait allows would not
  // wait for its own stage: the first two stages are waited for here)
  if (lead == 0) {
    SLIM_HEAD(0, As0, As1);
  } else if (lead == 2) {
    SLIM_HEAD(1, As1, As2);
  } else {
    SLIM_HEAD(2, As2, As0);
  }
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
  if (lead == 2) {
    SLIM_STEP(1, As1, As0, 0);
    kt = 1;
  }
  if (lead != 0) {
    SLIM_STEP(2, As2, As1, kt);
    ++kt;
  }
  for (; kt < KT - 3; kt += 3) {
    SLIM_STEP(0, As0, As2, kt);
    SLIM_STEP(1, As1, As0, kt + 1);
    SLIM_STEP(2, As2, As1, kt + 2);
  }
  // the last three steps: nothing past the end is loaded
  wide_sync<2 * LW + NI>();
  aload(KT - 1, As2);
  dequant(KT - 2, W[1], bf[1]);
  mma(As0, bf[0]);
  wide_sync<LW + NI>();
  dequant(KT - 1, W[2], bf[2]);
  mma(As1, bf[1]);
  wide_sync<0>();
  mma(As2, bf[2]);
#undef SLIM_STEP
#undef SLIM_HEAD
}

// The wide kernels' producer waves: stage kt + 1 while the consumers multiply kt.
// base, off: the weight rows this lane loads a quarter of; asrc(u): as in slim_gemm.  At the end of a step the direct loads of kt + 1 have to be
// in; the raw weights of kt + 2 (at least LW instructions, issued after them) may stay
// in flight.
template <int FMT, class Src>
__device__ __forceinline__ void wide_produce(__amdgpu_buffer_rsrc_t A, Src asrc, int ni,
                                             const uint8_t *const (&base)[4], uint32_t off, int KT, int pw, int lane,
                                             ActTile<kWideBM> &As0, ActTile<kWideBM> &As1, WeightTile &Bs0,
                                             WeightTile &Bs1) {
  constexpr int LW = 4 * kRawLoads, NU = kWideBM / 16;
  const int g = lane & 3;
  uint32_t src[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) src[u] = asrc(u);
  RawStep W0[4], W1[4];
  auto aload = [&](int kt, ActTile<kWideBM> &As) {
#pragma unroll
    for (int u = 0; u < NU; ++u)
      if (u < ni) dma16(A, src[u], 2 * wide_kbase<FMT>(kt), &As[pw & 1][16 * u + 8 * (pw >> 1)][0]);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
  };
  auto wload = [&](int kt, RawStep (&w)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) wide_load<FMT>(base[q], off, kt, g, w[q]);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto stage = [&](int kt, const RawStep (&w)[4], WeightTile &Bs) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      bf16x8 o[2];
      wide_dequant<FMT>(w[q], off, kt, g, o);
      __bf16 *dst = &Bs[64 * pw + 16 * q + (lane >> 2)][16 * g];
      *reinterpret_cast<bf16x8 *>(dst) = o[0];
      *reinterpret_cast<bf16x8 *>(dst + 8) = o[1];
    }
  };
  aload(0, As0);
  wload(0, W0);
  if (KT > 1) wload(1, W1);
  stage(0, W0, Bs0);
  wide_sync<0>();
  if (KT == 1) {
    wide_sync<0>();  // (the consumers' only step)
    return;
  }
  // step kt: the raw weights of kt + 1 are in WO, WS takes those of kt + 2
#define WIDE_PROD(WS, WO, AN, BN, kt) \
  do {                                \
    aload((kt) + 1, AN);              \
    wload((kt) + 2, WS);              \
    stage((kt) + 1, WO, BN);          \
    wide_sync<LW>();                  \
  } while (0)
  int kt = 0;
  for (; kt + 4 <= KT; kt += 2) {  // both steps' loads are used by a later step
    WIDE_PROD(W0, W1, As1, Bs1, kt);
    WIDE_PROD(W1, W0, As0, Bs0, kt + 1);
  }
  // two or three steps are left: KT - kt
  if (kt + 2 < KT) {
    WIDE_PROD(W0, W1, As1, Bs1, kt);
    aload(kt + 2, As0);
    stage(kt + 2, W0, Bs0);
  } else {
    aload(kt + 1, As1);
    stage(kt + 1, W1, Bs1);
  }
#undef WIDE_PROD
  wide_sync<0>();
  wide_sync<0>();
}

// The wide kernels' consumer waves: the K loop over a tile of NI subtiles.  brow[q]:
// the tile's weight row where the wave's weight subtile q starts.
template <int NI>
__device__ __forceinline__ void wide_consume(f32x4 (&acc)[NI][4], int KT, const ActTile<kWideBM> &As0,
                                             const ActTile<kWideBM> &As1, const WeightTile &Bs0,
                                             const WeightTile &Bs1, const int (&brow)[4], int lane) {
  auto mma = [&](const ActTile<kWideBM> &As, const WeightTile &Bs) {
    bf16x8 hi[2], lo[2], bf[2][4];
    auto aread = [&](int s) {
      const int r = 16 * (s % NI) + (lane & 15);
      const int c = (4 * (s / NI) + (lane >> 4)) ^ (r & 7);
      hi[s & 1] = *reinterpret_cast<const bf16x8 *>(&As[0][r][8 * c]);
      lo[s & 1] = *reinterpret_cast<const bf16x8 *>(&As[1][r][8 * c]);
    };
    auto bread = [&](int ks) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        bf[ks][q] = *reinterpret_cast<const bf16x8 *>(&Bs[brow[q] + (lane & 15)][32 * ks + 8 * (lane >> 4)]);
    };
    // every operand is read one subtile (eight MFMAs) before its use; without the
    // scheduling groups the compiler reads some right before their MFMAs (1 to 3 %)
    bread(0);
    aread(0);
    __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
    for (int s = 0; s < 2 * NI; ++s) {
      const int i = s % NI;
      if (s == NI - 1) {
        bread(1);
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
      }
      if (s + 1 < 2 * NI) {
        aread(s + 1);
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x8, 8, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        acc[i][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi[s & 1], bf[s / NI][q], acc[i][q], 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        acc[i][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo[s & 1], bf[s / NI][q], acc[i][q], 0, 0, 0);
    }
  };
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[i][q] = f32x4{0.f, 0.f, 0.f, 0.f};
  wide_sync<0>();
  int kt = 0;
  for (; kt + 2 <= KT; kt += 2) {
    mma(As0, Bs0);
    wide_sync<0>();
    mma(As1, Bs1);
    wide_sync<0>();
  }
  if (kt < KT) {
    mma(As0, Bs0);
    wide_sync<0>();
  }
}

// A tile of ni subtiles runs the smallest instance that covers it (rows past the
// tile's last are not stored).  MAX: the largest instance.
template <int MAX, class F>
__device__ __forceinline__ void wide_dispatch(int ni, F f) {
  if constexpr (MAX > 4) {
    if (ni > 8) return f(std::integral_constant<int, 9>{});
    if (ni > 6) return f(std::integral_constant<int, 8>{});
    if (ni > 4) return f(std::integral_constant<int, 6>{});
  }
  if (ni > 2) return f(std::integral_constant<int, 4>{});
  if (ni > 1) return f(std::integral_constant<int, 2>{});
  return f(std::integral_constant<int, 1>{});
}

// h = silu(g) u of the wave's 32 columns (acc[i][q] gate, acc[i][2 + q] up) as bf16 hi
// and lo terms; out: the tile's first row at the lane's column.
template <int NI>
__device__ __forceinline__ void gateup_store(const f32x4 (&acc)[NI][4], __bf16 *out, int64_t lo_plane, int I, int n,
                                             int lane) {
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = 16 * i + 4 * (lane >> 4) + r;
      if (m < n) {
        __bf16 *o = out + (int64_t)m * I;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const float v = silu_fast(acc[i][q][r]) * acc[i][2 + q][r];
          const __bf16 hi = (__bf16)v;
          o[16 * q] = hi;
          o[lo_plane + 16 * q] = (__bf16)(v - (float)hi);
        }
      }
    }
}
// P[pair] = w[pair] * row for the wave's 64 columns, the first of them at P; row(m): the pair of
// tile row m and its weight.  (The lane's column is added here: a pointer kept through the K
// loop cost the slim kernels spills.)
struct RowPair {
  int32_t pair;
  float w;
};
template <int NI, class Row>
__device__ __forceinline__ void down_store(const f32x4 (&acc)[NI][4], float *P, Row row, int H, int n, int lane) {
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    RowPair rp[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) rp[r] = row(min(16 * i + 4 * (lane >> 4) + r, n - 1));
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (16 * i + 4 * (lane >> 4) + r < n) {
        float *dst = P + (int64_t)rp[r].pair * H + (lane & 15);
#pragma unroll
        for (int q = 0; q < 4; ++q) dst[16 * q] = rp[r].w * acc[i][q][r];
      }
  }
}

// Gate/up (I a multiple of 128), wide: 128 columns of h per block, wave c's weight rows
// are W_gate rows n0 + 32 c .. +31 and the same rows of W_up; h = silu(g) u written
// as bf16 hi and lo terms at the pair's grouped row.
template <int FMT>
__global__ __launch_bounds__(kWideThreads, 1) void pf_gateup_wide_kernel(GmParams a) {
  __shared__ __align__(16) ActTile<kWideBM> As0, As1;
  __shared__ __align__(16) WeightTile Bs0, Bs1;
  int mt, nt, j, m0;
  wide_tile(a.I / 128, mt, nt);
  if (!pf_tile(a.X, mt, j, m0)) return;
  const int lane = threadIdx.x & (kWave - 1), wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), wv = wid & 3;
  const int row0 = a.X.row0[j] + m0, n = min(a.X.n[j] - m0, (int)a.X.rt[j]), n0 = nt * 128 + 32 * wv;
  const int32_t *perm = a.perm + row0;
  const int H = a.H, I = a.I, k = a.k;
  // the activation plane this wave loads (its bytes fit 32 bits, checked at launch)
  const uint32_t plane = 2u * (uint32_t)a.T * (uint32_t)H;
  const __amdgpu_buffer_rsrc_t A = wide_buffer(a.A + (wv & 1) * ((int64_t)a.T * H), plane);
  auto asrc = [&](int u) {
    const int r = min(16 * u + 8 * (wv >> 1) + (lane >> 3), n - 1);
    return 2 * ((uint32_t)(perm[r] / k) * (uint32_t)H + wide_kchunk<FMT>((lane & 7) ^ (lane >> 3)));
  };
  // producer wave c: rows 64 (c % 2) .. of W_gate (c < 2) or W_up
  const WeightRows W(a.X.payload[j] + (wv >= 2 ? a.mat : 0) + (int64_t)(nt * 128 + 64 * (wv & 1)) * a.rowb, a.rowb,
                     32 * a.rowb, lane);
  if (wid >= 4) {
    wide_produce<FMT>(A, asrc, (n + 15) / 16, W.base, W.off, H / kPfBK, wv, lane, As0, As1, Bs0, Bs1);
    return;
  }
  const int brow[4] = {32 * wv, 32 * wv + 16, 128 + 32 * wv, 128 + 32 * wv + 16};
  __bf16 *out = a.ab + (int64_t)row0 * I + n0 + (lane & 15);
  const int64_t lo_plane = (int64_t)a.pairs * I;
  wide_dispatch<kWideBM / 16>((n + 15) / 16, [&](auto ni) {
    constexpr int NI = decltype(ni)::value;
    f32x4 acc[NI][4];
    wide_consume<NI>(acc, H / kPfBK, As0, As1, Bs0, Bs1, brow, lane);
    gateup_store<NI>(acc, out, lo_plane, I, n, lane);
  });
}

// Down (H a multiple of 256), wide: wave c's weight rows are W_down rows n0 + 64 c .. +63;
// the activation rows are the expert's, contiguous in perm order; P[pair] = w * row.
template <int FMT>
__global__ __launch_bounds__(kWideThreads, 1) void pf_down_wide_kernel(GmParams a) {
  __shared__ __align__(16) ActTile<kWideBM> As0, As1;
  __shared__ __align__(16) WeightTile Bs0, Bs1;
  __shared__ RowPair rows[kWideBM];
  int mt, nt, j, m0;
  wide_tile(a.H / 256, mt, nt);
  if (!pf_tile(a.X, mt, j, m0)) return;
  const int lane = threadIdx.x & (kWave - 1), wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), wv = wid & 3;
  const int row0 = a.X.row0[j] + m0, n = min(a.X.n[j] - m0, (int)a.X.rt[j]), n0 = nt * 256 + 64 * wv;
  const int32_t *perm = a.perm + row0;
  const int H = a.H, I = a.I;
  // the activation plane this wave loads (its bytes fit 32 bits, checked at launch)
  const uint32_t plane = 2u * (uint32_t)a.pairs * (uint32_t)I;
  const __amdgpu_buffer_rsrc_t A = wide_buffer(a.A + (wv & 1) * ((int64_t)a.pairs * I), plane);
  auto asrc = [&](int u) {
    const int r = min(16 * u + 8 * (wv >> 1) + (lane >> 3), n - 1);
    return 2 * ((uint32_t)(row0 + r) * (uint32_t)I + wide_kchunk<FMT>((lane & 7) ^ (lane >> 3)));
  };
  const WeightRows W(a.X.payload[j] + a.down_off + (int64_t)n0 * a.rowb, a.rowb, 32 * a.rowb, lane);
  if (wid >= 4) {
    wide_produce<FMT>(A, asrc, (n + 15) / 16, W.base, W.off, I / kPfBK, wv, lane, As0, As1, Bs0, Bs1);
    return;
  }
  // the rows' pairs and weights, while the first step is staged: loaded in the epilogue, each
  // subtile's two dependent loads made it the longest part of a tile of one or two K steps
  if ((int)threadIdx.x < n) {
    const int pair = perm[threadIdx.x];
    rows[threadIdx.x] = {pair, a.w[pair]};
  }
  const int brow[4] = {64 * wv, 64 * wv + 16, 64 * wv + 32, 64 * wv + 48};
  float *P = a.P + n0;
  wide_dispatch<kWideBM / 16>((n + 15) / 16, [&](auto ni) {
    constexpr int NI = decltype(ni)::value;
    f32x4 acc[NI][4];
    wide_consume<NI>(acc, I / kPfBK, As0, As1, Bs0, Bs1, brow, lane);
    down_store<NI>(acc, P, [&](int m) { return rows[m]; }, H, n, lane);
  });
}

// Gate/up (I a multiple of 128), slim: 128 columns of h per block, wave c's weight rows
// are W_gate rows n0 + 32 c .. +31 and the same rows of W_up; h = silu(g) u written
// as bf16 hi and lo terms at the pair's grouped row.
template <int FMT>
__global__ __launch_bounds__(kSlimThreads, 2) void pf_gateup_slim_kernel(GmParams a) {
  __shared__ __align__(16) ActTile<kSlimBM> As0, As1, As2;
  int mt, nt, j, m0;
  wide_tile(a.I / 128, mt, nt);
  if (!pf_tile(a.X, mt, j, m0)) return;
  const int lane = threadIdx.x & (kWave - 1), wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), wv = wid & 3;
  const int row0 = a.X.row0[j] + m0, n = min(a.X.n[j] - m0, (int)a.X.rt[j]), n0 = nt * 128 + 32 * wv;
  const int32_t *perm = a.perm + row0;
  const int H = a.H, I = a.I, k = a.k;
  // the activation plane this wave loads (its bytes fit 32 bits, checked at launch)
  const uint32_t plane = 2u * (uint32_t)a.T * (uint32_t)H;
  const __amdgpu_buffer_rsrc_t A = wide_buffer(a.A + (wv & 1) * ((int64_t)a.T * H), plane);
  auto asrc = [&](int u) {
    const int r = min(16 * u + 8 * (wv >> 1) + (lane >> 3), n - 1);
    return 2 * ((uint32_t)(perm[r] / k) * (uint32_t)H + wide_kchunk<FMT>((lane & 7) ^ (lane >> 3)));
  };
  const WeightRows W(a.X.payload[j] + (int64_t)n0 * a.rowb, a.rowb, a.mat, lane);
  __bf16 *out = a.ab + (int64_t)row0 * I + n0 + (lane & 15);
  const int64_t lo_plane = (int64_t)a.pairs * I;
  wide_dispatch<kSlimBM / 16>((n + 15) / 16, [&](auto ni) {
    constexpr int NI = decltype(ni)::value;
    f32x4 acc[NI][4];
    slim_gemm<FMT, NI>(acc, A, asrc, W.base, W.off, H / kPfBK, wv, lane, As0, As1, As2);
    gateup_store<NI>(acc, out, lo_plane, I, n, lane);
  });
}

// Down (H a multiple of 256), slim: wave c's weight rows are W_down rows n0 + 64 c .. +63;
// the activation rows are the expert's, contiguous in perm order; P[pair] = w * row.
template <int FMT>
__global__ __launch_bounds__(kSlimThreads, 2) void pf_down_slim_kernel(GmParams a) {
  __shared__ __align__(16) ActTile<kSlimBM> As0, As1, As2;
  int mt, nt, j, m0;
  wide_tile(a.H / 256, mt, nt);
  if (!pf_tile(a.X, mt, j, m0)) return;
  const int lane = threadIdx.x & (kWave - 1), wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), wv = wid & 3;
  const int row0 = a.X.row0[j] + m0, n = min(a.X.n[j] - m0, (int)a.X.rt[j]), n0 = nt * 256 + 64 * wv;
  const int32_t *perm = a.perm + row0;
  const int H = a.H, I = a.I;
  // the activation plane this wave loads (its bytes fit 32 bits, checked at launch)
  const uint32_t plane = 2u * (uint32_t)a.pairs * (uint32_t)I;
  const __amdgpu_buffer_rsrc_t A = wide_buffer(a.A + (wv & 1) * ((int64_t)a.pairs * I), plane);
  auto asrc = [&](int u) {
    const int r = min(16 * u + 8 * (wv >> 1) + (lane >> 3), n - 1);
    return 2 * ((uint32_t)(row0 + r) * (uint32_t)I + wide_kchunk<FMT>((lane & 7) ^ (lane >> 3)));
  };
  const WeightRows W(a.X.payload[j] + a.down_off + (int64_t)n0 * a.rowb, a.rowb, 32 * a.rowb, lane);
  float *P = a.P + n0;
  const float *w = a.w;
  wide_dispatch<kSlimBM / 16>((n + 15) / 16, [&](auto ni) {
    constexpr int NI = decltype(ni)::value;
    f32x4 acc[NI][4];
    slim_gemm<FMT, NI>(acc, A, asrc, W.base, W.off, I / kPfBK, wv, lane, As0, As1, As2);
    down_store<NI>(acc, P, [&](int m) { return RowPair{perm[m], w[perm[m]]}; }, H, n, lane);
  });
}

}  // namespace

// The slim kernels take Q8_0, Q4_0 and Q4_K.
template <int FMT>
hipError_t wide_gateup(bool slim, dim3 grid, const GmParams &a, hipStream_t s, const Timing &t) {
  if constexpr (FMT != 14)
    if (slim) {
      hipExtLaunchKernelGGL(pf_gateup_slim_kernel<FMT>, grid, dim3(kSlimThreads), 0, s, t.start, t.stop, 0, a);
      return hipGetLastError();
    }
  hipExtLaunchKernelGGL(pf_gateup_wide_kernel<FMT>, grid, dim3(kWideThreads), 0, s, t.start, t.stop, 0, a);
  return hipGetLastError();
}
template <int FMT>
hipError_t wide_down(bool slim, dim3 grid, const GmParams &a, hipStream_t s, const Timing &t) {
  if constexpr (FMT != 14)
    if (slim) {
      hipExtLaunchKernelGGL(pf_down_slim_kernel<FMT>, grid, dim3(kSlimThreads), 0, s, t.start, t.stop, 0, a);
      return hipGetLastError();
    }
  hipExtLaunchKernelGGL(pf_down_wide_kernel<FMT>, grid, dim3(kWideThreads), 0, s, t.start, t.stop, 0, a);
  return hipGetLastError();
}

}  // namespace moecache
