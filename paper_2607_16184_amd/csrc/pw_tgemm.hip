// Paged GEMMs for more than a few slots per expert, gfx950: the tiled kernel
// (k_tgemm, from about 49 slots per expert to prefill batches) and, further
// down, the streaming kernel (k_sgemm).
//
// Tiled kernel. A workgroup of 8 waves (two per SIMD, one workgroup per CU)
// computes a 256-row x TM-slot tile of D = W X^T for one expert (TM = 256 or
// 128): gate/up tiles are 128 rows of gate plus the same 128 rows of up, down
// tiles are 256 rows of the down projection. A wave owns 128 rows x 64 slots
// (TM = 256) or 64 x 64 in 16x16x32 MFMA tiles; a gate/up wave holds the same
// rows of both projections, so SwiGLU needs no exchange. K advances in stages
// of 32 (one MFMA step).
//
// Data movement. Global loads write LDS directly (lds_load16): activations
// and 16-bit pages in their final place, 8- and 4-bit codes in a small buffer
// of the wave's own, from which the wave dequantizes its 32 weight rows once
// per tile to fl32(z + c s) rounded to the activation dtype. The page format's
// tiles are MFMA operand fragments, so weights lie in LDS as they lie in the
// page; activations come as whole 128-byte lines (8 rows x 64 values per load;
// half lines cost 50 % more L1-to-L2 requests, 1.90 against 1.77 ms for the
// 4096-token gate/up at 16 bits) with the 16-byte pieces of a row permuted by
// the row index, which keeps the operand reads free of bank conflicts. Weights
// of stage s + 3 are loaded while stage s is multiplied (four LDS slots),
// activations two 64-value units ahead (two slots).
//
// Schedule. One barrier per stage. In iteration s a wave issues the MFMAs of
// stage s from registers and reads each operand register's successor (stage
// s + 1) from LDS as soon as its last MFMA is issued, so the LDS reads, the
// loads, the dequantization and the other wave of the SIMD all run under the
// MFMAs. Against the kernel this one replaced (loads into registers, then
// LDS writes, two waves in alternating phases): 4096 tokens over 8 experts of
// 4096 x 14336, pages 50/25/25 % at 16/8/4 bits, gate/up 2.30 -> 1.82 ms, down
// 1.18 -> 0.96 ms; 64 experts of 2048 x 1408, top-6, 4096 tokens: 0.63 -> 0.38
// and 0.32 -> 0.24 ms. With no loads at all the gate/up loop takes 1.40 ms at
// 16 bits: what is left is mostly the clock (2.0 GHz under this load, 2.2
// without the loads) and the L2 misses. A form with the two waves of a SIMD
// in alternating phases ran at the same speed, four waves of 128 x 128 12 %
// slower, 32x32x16 MFMAs 4 % slower, lines touched ahead of their loads 15 %
// slower (the L1's request rate bounds it), and the dequantization placed
// between the MFMAs made no difference.
#include "pw_device.hpp"
#include "pw_internal.hpp"

namespace pw {
namespace {

constexpr int kWaves = 8;                   // waves of a tile's workgroup
constexpr int kTN = 256;                    // weight rows per tile
constexpr int kStK = 32;                    // K per stage: one MFMA k-step
constexpr int kRing = 4;                    // weight stages in LDS
constexpr int kTK = 64;                     // K per stage of the streaming kernel
constexpr int kGN = 4;                      // weight blocks per group of tiles

// A wave's weight share of a stage: 32 rows (two 16-row tiles) of one page as
// four fragments f = 2 * tile + step.
template <int B> struct WStage;
template <> struct WStage<16> { u32x4 v[4]; };                 // fragment f at v[f]
template <> struct WStage<8> { u32x4 v[2]; uint32_t sz[2]; };  // tile t: both steps
template <> struct WStage<4> { u32x2 v[2]; uint32_t sz[2]; };  // tile t: one word per step

// Nested bit-plane pages (format codes 108 and 104: 8 and 4 planes). Per row
// tile and 128-value block, lane l holds one 32-bit word per plane covering
// its four k-steps; `lut` points at the wave's 32 LUT rows staged in LDS.
// The LUT pointer is held in the LDS address space, so lookups are LDS reads
// with 32-bit addresses (a generic pointer would make them flat loads).
constexpr int kApl8 = 108, kApl4 = 104;
template <int B> constexpr int apl_planes() { return B == kApl8 ? 8 : 4; }
typedef const __attribute__((address_space(3))) uint16_t* lds_lut_t;
template <> struct WStage<kApl8> { uint32_t p[2][8]; int hh; lds_lut_t lut; };
template <> struct WStage<kApl4> { uint32_t p[2][4]; int hh; lds_lut_t lut; };

// Weights are re-read by the other slot tiles of the expert: plain (cached) loads.
// For nested bit-plane pages tile0 is the page base plus the wave's row-tile
// offset inside a plane, and szrow carries the wave's LUT rows in LDS.
template <int B>
__device__ __forceinline__ void w_fetch(WStage<B>& w, const uint8_t* tile0, const uint8_t* szrow, int kb, int hh,
                                        int g, int nkb, int R) {
  const int lane = lane_id();
  if constexpr (B == kApl8 || B == kApl4) {
    const size_t rk8 = static_cast<size_t>(R) * nkb * 16;
#pragma unroll
    for (int j = 0; j < apl_planes<B>(); ++j) {
      const size_t pb = j < 4 ? j * rk8 : 4 * rk8 + 32 * static_cast<size_t>(R) + (j - 4) * rk8;
#pragma unroll
      for (int t = 0; t < 2; ++t)
        w.p[t][j] = *reinterpret_cast<const uint32_t*>(tile0 + pb + (static_cast<size_t>(t) * nkb + kb) * 256 +
                                                       4 * lane);
    }
    w.hh = hh;
    w.lut = (lds_lut_t)szrow;   // szrow points into LDS for these pages (generic to LDS: a C-style cast)
    (void)g;
  } else {
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const uint8_t* tp = tile0 + (static_cast<size_t>(t) * nkb + kb) * tile_bytes<B>() + 16 * lane;
    if constexpr (B == 16) {
      w.v[2 * t] = ld16(tp + 2 * hh * 1024);
      w.v[2 * t + 1] = ld16(tp + (2 * hh + 1) * 1024);
    } else if constexpr (B == 8) {
      w.v[t] = ld16(tp + hh * 1024);
    } else {
      w.v[t] = *reinterpret_cast<const u32x2*>(tp + 8 * hh);
    }
  }
  if constexpr (B != 16) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
      w.sz[t] = *reinterpret_cast<const uint32_t*>(szrow + (static_cast<size_t>(g) * R + 16 * t) * 4);
  }
  }
}

// Two fp32 values -> a packed 16-bit word (round to nearest even).
template <int ACT>
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  typedef _Float16 h2 __attribute__((ext_vector_type(2)));
  const f2 p = {a, b};
  if constexpr (ACT == PW_BF16) return __builtin_bit_cast(uint32_t, __builtin_convertvector(p, b2));
  else return __builtin_bit_cast(uint32_t, __builtin_convertvector(p, h2));
}

// Eight fp32 values -> four packed 16-bit words.
template <int ACT>
__device__ __forceinline__ u32x4 pack8(const float (&v)[8]) {
  u32x4 o;
#pragma unroll
  for (int q = 0; q < 4; ++q) o[q] = pack2<ACT>(v[2 * q], v[2 * q + 1]);
  return o;
}

// Fragment f of the wave's weights in the activation dtype: quantized codes
// become fl32(z + c s) (c s is exact in fp32, so one fma rounds once).
template <int ACT, int SDT, int B>
__device__ __forceinline__ u32x4 w_piece(const WStage<B>& w, int f) {
  if constexpr (B == kApl8 || B == kApl4) {
    // plane j's eight bits of this k-step (byte bs of its word) go to byte
    // 7 - j of a 64-bit word (8-bit pages; 4-bit pages: byte 3 - j of a
    // 32-bit word), gathered with byte permutes; a bit transpose then brings
    // each element's plane bits together (plane 0 the most significant)
    const int t = f >> 1;
    const uint32_t bs = static_cast<uint32_t>(2 * w.hh + (f & 1));
    const uint32_t pair = 0x0C0C0000u | ((4u + bs) << 8) | bs;   // (S0.byte bs, S1.byte bs) -> bytes 1, 0
    const uint32_t hi = __builtin_amdgcn_perm(__builtin_amdgcn_perm(w.p[t][0], w.p[t][1], pair),
                                              __builtin_amdgcn_perm(w.p[t][2], w.p[t][3], pair), 0x05040100u);
    constexpr int nl = B == kApl8 ? 256 : 16;
    const lds_lut_t lut = w.lut + (16 * t + (lane_id() & 15)) * nl;
    uint32_t idx[8];
    if constexpr (B == kApl8) {
      const uint32_t lo = __builtin_amdgcn_perm(__builtin_amdgcn_perm(w.p[t][4], w.p[t][5], pair),
                                                __builtin_amdgcn_perm(w.p[t][6], w.p[t][7], pair), 0x05040100u);
      // 8 x 8 transpose (three delta swaps): element e's code in byte e
      uint64_t x = (static_cast<uint64_t>(hi) << 32) | lo;
      uint64_t y = (x ^ (x >> 7)) & 0x00AA00AA00AA00AAull;
      x = x ^ y ^ (y << 7);
      y = (x ^ (x >> 14)) & 0x0000CCCC0000CCCCull;
      x = x ^ y ^ (y << 14);
      y = (x ^ (x >> 28)) & 0x00000000F0F0F0F0ull;
      x = x ^ y ^ (y << 28);
#pragma unroll
      for (int e = 0; e < 8; ++e) idx[e] = static_cast<uint32_t>(x >> (8 * e)) & 0xFFu;
    } else {
      // 4 x 8 transpose: bit 8 r + e (row r = byte r, element e) goes to bit
      // 4 n + r with n = 4 e1 + 2 e0 + e2 (the bits of e rotated), which two
      // delta swaps of index bits (0 with 3, 1 with 4) do: element e's 4-bit
      // code in nibble n
      uint32_t x = hi;
      uint32_t y = (x ^ (x >> 7)) & 0x00AA00AAu;
      x = x ^ y ^ (y << 7);
      y = (x ^ (x >> 14)) & 0x0000CCCCu;
      x = x ^ y ^ (y << 14);
      constexpr int nib[8] = {0, 2, 4, 6, 1, 3, 5, 7};
#pragma unroll
      for (int e = 0; e < 8; ++e) idx[e] = (x >> (4 * nib[e])) & 0xFu;
    }
    u32x4 o;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      o[q] = static_cast<uint32_t>(lut[idx[2 * q]]) | (static_cast<uint32_t>(lut[idx[2 * q + 1]]) << 16);
    return o;
  } else if constexpr (B == 16) {
    return w.v[f];
  } else {
    const int t = f >> 1, i = f & 1;
    const float s = val16(w.sz[t], SDT), z = val16(w.sz[t] >> 16, SDT);
    float v[8];
    if constexpr (B == 8) {
      const uint32_t d0 = w.v[t][2 * i], d1 = w.v[t][2 * i + 1];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        v[q] = __builtin_fmaf(static_cast<float>((d0 >> (8 * q)) & 0xFFu), s, z);
        v[4 + q] = __builtin_fmaf(static_cast<float>((d1 >> (8 * q)) & 0xFFu), s, z);
      }
    } else {
      // codes 2u at bits 4u, 2u + 1 at bits 16 + 4u: split the nibbles into bytes
      const uint32_t d = w.v[t][i];
      const uint32_t lo = d & 0x0F0F0F0Fu, hi = (d >> 4) & 0x0F0F0F0Fu;
      const uint32_t src[8] = {lo, lo >> 16, hi, hi >> 16, lo >> 8, lo >> 24, hi >> 8, hi >> 24};
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = __builtin_fmaf(static_cast<float>(src[q] & 0xFFu), s, z);
    }
    return pack8<ACT>(v);
  }
}

#define PW_LDS __attribute__((address_space(3)))
typedef PW_LDS uint8_t* lds_u8_t;
__device__ __forceinline__ u32x4 lds16(lds_u8_t p) { return *reinterpret_cast<const PW_LDS u32x4*>(p); }

// ---- LDS-direct loads -------------------------------------------------------
// A wave-wide load that lands in LDS: lane l's 16 (or 4) bytes from base +
// voff go to LDS byte address `dst` + 16 l (4 l), wave-uniform base and dst.
// Written as asm because the compiler, which cannot tell what such a load
// writes, waits for all of them before any LDS access; here the waits are
// counted by hand (wait_vm). No register receives data, so nothing can be
// reallocated under a load in flight. (M0 holds the LDS address; one wait
// state between its write and the load.)
__device__ __forceinline__ void lds_load16(uint32_t dst, uint32_t voff, const uint8_t* base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(dst), "v"(voff), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void lds_load4(uint32_t dst, uint32_t voff, const uint8_t* base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
               :: "s"(dst), "v"(voff), "s"(base) : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_lds() {
  asm volatile("s_waitcnt lgkmcnt(%0)" :: "n"(N) : "memory");
}
__device__ __forceinline__ void wg_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ const uint8_t* uniform_ptr(const uint8_t* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
  return reinterpret_cast<const uint8_t*>((static_cast<uint64_t>(hi) << 32) | lo);
}

// Geometry of a tile of kTN weight rows x TM slots: the waves' grid (WN x WM),
// each wave's 16 x 16 tiles (NR x NC), and what it stages: RT weight row tiles
// per stage and NX activation loads per two stages.
template <int TM>
struct TileGeo {
  static constexpr int WN = TM == 256 ? 2 : 4, WM = kWaves / WN;
  static constexpr int NR = kTN / 16 / WN, NC = TM / 16 / WM;
  static constexpr int RT = kTN / 16 / kWaves, NX = TM / 8 / kWaves;
  static constexpr int kSlot = kTN * kStK * 2;                 // weights of one stage
  static constexpr int kXSlot = TM * 128;                      // activations of two stages
  static constexpr int kXOff = kRing * kSlot;
  static constexpr int kRawW = RT * 1024, kSzW = RT * 128;     // per wave: codes and scale/zero pairs of a unit
  static constexpr int kRaw = kXOff + 2 * kXSlot;
  static constexpr int kSz = kRaw + kWaves * kRawW;
  static constexpr int kLds = kSz + kWaves * kSzW;
};

// What a wave stages and computes. Its weight rows (16 RT, all in one page of
// format B) and 8 NX slots are its staging share; the tile it multiplies is
// set by (wn, wm).
//
// Waits. Vector-memory operations complete in order, so "at most N of them
// outstanding" (wait_vm<N>) means that everything older than the newest N has
// landed; N is counted from the fixed order of issue. Iteration s issues
// [activations of stages s + 3, s + 4 if s is odd][16-bit weights of stage
// s + 3][the next unit of codes if one was picked up]; its barrier publishes
// stage s + 2, whose loads were issued in iteration s - 1. A slot is refilled
// only after a barrier that follows every wave's last read of it: weights of
// stage s - 1 (read in iteration s - 2, consumed in s - 1) by iteration s;
// activations of unit u (last read in iteration 2 u, waited for before its
// barrier) by iteration 2 u + 1.
template <int ACT, int SDT, int B, bool GATEUP, int TM>
struct TileLoop {
  typedef TileGeo<TM> Geo;
  static constexpr int NR = Geo::NR, NC = Geo::NC, NX = Geo::NX, RT = Geo::RT;
  static constexpr int NW = B == 16 ? RT : 0;    // weight loads per stage
  // stages of one unit of codes: 8-bit pages keep two k-steps in a lane's 16
  // bytes, 4-bit pages four; loads of a unit
  static constexpr int UNIT = B == 8 ? 2 : 4;
  static constexpr int NRAW = RT + 1;
  // a unit is picked up three stages before its first
  static constexpr bool pickup(int j) { return B != 16 && ((j + 3) & 3) % UNIT == 0; }
  // operations younger than the codes picked up at the start of an iteration
  // (only activations come between), and than the stage its barrier publishes
  static constexpr int younger_raw() { return UNIT == 4 ? NX : 0; }
  static constexpr int younger_next(int j) {
    return (j & 1 ? NX : 0) + NW + NRAW * ((pickup(j) ? 1 : 0) + (pickup((j + 3) & 3) ? 1 : 0));
  }

  lds_u8_t lds;
  uint32_t lds0;                 // LDS byte address of `lds`
  const uint8_t* xbase;          // activations, K offset of the range included
  uint32_t xoff[NX];
  const uint8_t* wbase;          // first 16-row tile of the wave, first block of the range
  size_t tstride;
  const uint8_t* szbase;         // scale/zero pair of the wave's first row, group 0
  uint32_t szoff;
  int kstart, R, gshift;         // first k of the range, rows per page, log2 G
  int nstage, wave, wn, wm, lane;
  bool live;
  int boff;                      // lane part of the activation reads

  u32x4 a[NR], b[2][NC];
  u32x4 raw[RT], dq[RT];
  uint32_t sz[2][RT];
  f32x4 acc[NR][NC];

  // The q-th load of the activations of stages 2 u and 2 u + 1: 8 rows x 128
  // bytes (whole cache lines); row r's 16-byte piece p lies at place p ^ (r mod 8).
  // (Loads past the end repeat the last unit, here and below.)
  __device__ __forceinline__ void load_x(int u, int q) {
    const uint8_t* p = xbase + static_cast<size_t>(min(u, nstage / 2 - 1)) * 128;
    lds_load16(lds0 + Geo::kXOff + (u & 1) * Geo::kXSlot + wave * NX * 1024 + 1024 * q, xoff[q], p);
  }
  __device__ __forceinline__ void load_x(int u) {
#pragma unroll
    for (int q = 0; q < NX; ++q) load_x(u, q);
  }
  // 16-bit weights of stage s
  __device__ __forceinline__ void load_w(int s, int slot) {
    if constexpr (B == 16) {
      const uint8_t* p = wbase + static_cast<size_t>(min(s, nstage - 1)) * 1024;
      const uint32_t d = lds0 + slot * Geo::kSlot + wave * RT * 1024;
#pragma unroll
      for (int t = 0; t < RT; ++t) lds_load16(d + 1024 * t, 16u * lane, p + t * tstride);
    }
  }
  // codes and scale/zero pairs of unit u (stages UNIT u .. + UNIT - 1)
  __device__ __forceinline__ void load_raw(int u) {
    const int v = min(u, nstage / UNIT - 1);
    const uint8_t* p = wbase + static_cast<size_t>(v) * 1024;
    const int g = (kstart + v * (UNIT * kStK)) >> gshift;
    const uint32_t d = lds0 + Geo::kRaw + wave * Geo::kRawW;
#pragma unroll
    for (int t = 0; t < RT; ++t) lds_load16(d + 1024 * t, 16u * lane, p + t * tstride);
    lds_load4(lds0 + Geo::kSz + wave * Geo::kSzW, szoff, szbase + static_cast<size_t>(g) * R * 4);
  }
  __device__ __forceinline__ void pick_raw() {
    lds_u8_t p = lds + Geo::kRaw + wave * Geo::kRawW + 16 * lane;
#pragma unroll
    for (int t = 0; t < RT; ++t) raw[t] = lds16(p + 1024 * t);
    const PW_LDS uint32_t* q = reinterpret_cast<const PW_LDS uint32_t*>(lds + Geo::kSz + wave * Geo::kSzW) + (lane & 15);
#pragma unroll
    for (int g = 0; g < (B == 4 ? 2 : 1); ++g)
#pragma unroll
      for (int t = 0; t < RT; ++t) sz[g][t] = q[16 * (RT * g + t)];
  }
  // the wave's weights of the stage at position j of its 128-block (its codes
  // are in `raw`), as fl32(z + c s) rounded to the activation dtype
  __device__ __forceinline__ void dequant(int j) {
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const uint32_t szw = B == 4 && gshift == 6 && j >= 2 ? sz[1][t] : sz[0][t];
      const float s = val16(szw, SDT), z = val16(szw >> 16, SDT);
      float v[8];
      if constexpr (B == 8) {
        const uint32_t d0 = raw[t][2 * (j & 1)], d1 = raw[t][2 * (j & 1) + 1];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          v[q] = __builtin_fmaf(static_cast<float>((d0 >> (8 * q)) & 0xFFu), s, z);
          v[4 + q] = __builtin_fmaf(static_cast<float>((d1 >> (8 * q)) & 0xFFu), s, z);
        }
      } else {
        // codes 2u at bits 4u, 2u + 1 at bits 16 + 4u: split the nibbles into bytes
        const uint32_t d = raw[t][j];
        const uint32_t lo = d & 0x0F0F0F0Fu, hi = (d >> 4) & 0x0F0F0F0Fu;
        const uint32_t src[8] = {lo, lo >> 16, hi, hi >> 16, lo >> 8, lo >> 24, hi >> 8, hi >> 24};
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = __builtin_fmaf(static_cast<float>(src[q] & 0xFFu), s, z);
      }
      dq[t] = pack8<ACT>(v);
    }
  }
  __device__ __forceinline__ void store_dq(int slot) {
    lds_u8_t d = lds + slot * Geo::kSlot + wave * RT * 1024 + 16 * lane;
#pragma unroll
    for (int t = 0; t < RT; ++t) *reinterpret_cast<PW_LDS u32x4*>(d + 1024 * t) = dq[t];
  }
  // weight fragment of the wave's r-th row tile: a gate/up wave holds the same
  // rows of both projections (r < NR / 2: gate)
  __device__ __forceinline__ u32x4 read_a(int slot, int r) const {
    const int f = GATEUP ? (r < NR / 2 ? (NR / 2) * wn + r : kTN / 32 + (NR / 2) * wn + r - NR / 2) : NR * wn + r;
    return lds16(lds + slot * Geo::kSlot + 16 * lane + 1024 * f);
  }
  __device__ __forceinline__ u32x4 read_b(int slot, int c) const {
    return lds16(lds + Geo::kXOff + (slot >> 1) * Geo::kXSlot + (slot & 1 ? boff ^ 64 : boff) + 2048 * (NC * wm + c));
  }

  // Iteration s, at position J = s mod 4 of its 128-block: stage s's MFMAs
  // (operands in registers), stage s + 1's operands read as registers come
  // free, stage s + 2's dequantized weights written, stage s + 3's loads issued
  // and its weights dequantized.
  template <int J, bool LIVE>
  __device__ __forceinline__ void step(int s) {
    if constexpr (pickup(J)) {
      wait_vm<younger_raw()>();
      pick_raw();
    }
    if constexpr (B != 16) store_dq((J + 2) & 3);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (B != 16) dequant((J + 3) & 3);
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      if constexpr (LIVE) {
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[r][c] = mma<ACT>(a[r], b[J & 1][c], acc[r][c]);
        a[r] = read_a((J + 1) & 3, r);
        if (r < NC) b[(J + 1) & 1][r] = read_b((J + 1) & 3, r);
      }
      if ((J & 1) && r < NX) load_x((s + 3) >> 1, r);
      if (r == NR - 2) load_w(s + 3, (J + 3) & 3);
    }
    __builtin_amdgcn_sched_barrier(0);
    // At an odd stage, the LDS operations before the NR + NC >= 8 operand reads
    // (codes picked up, weights stored) are done; at an even one, whose reads
    // were the last of an activation slot that the next iteration refills, all.
    if constexpr (J & 1) {
      if constexpr (B != 16) wait_lds<LIVE ? 8 : 0>();
    } else {
      wait_lds<0>();
    }
    if constexpr (pickup(J)) load_raw((s + 3) / UNIT + 1);
    wait_vm<younger_next(J)>();
    wg_barrier();
  }

  template <bool LIVE>
  __device__ __forceinline__ void loop() {
    for (int s = 0; s < nstage; s += 4) {
      step<0, LIVE>(s);
      step<1, LIVE>(s + 1);
      step<2, LIVE>(s + 2);
      step<3, LIVE>(s + 3);
    }
  }

  __device__ __forceinline__ void run() {
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the loads in the order in which iterations -3, -2, -1 would issue them,
    // so that the loop's counted waits hold from the first iteration on
    if constexpr (B != 16) load_raw(0);
    load_x(0);
    load_w(0, 0);
    if constexpr (B != 16) {
      wait_vm<NX>();
      pick_raw();
      wait_lds<0>();
      load_raw(1);
      dequant(0);
      store_dq(0);
      dequant(1);
      store_dq(1);
    }
    load_w(1, 1);
    if constexpr (B == 8) {
      wait_vm<0>();
      pick_raw();
      wait_lds<0>();
    }
    load_x(1);
    load_w(2, 2);
    if constexpr (B == 8) load_raw(2);
    if constexpr (B != 16) dequant(2);
    wait_lds<0>();
    wait_vm<younger_next(3)>();
    wg_barrier();
    if (live) {
#pragma unroll
      for (int r = 0; r < NR; ++r) a[r] = read_a(0, r);
#pragma unroll
      for (int c = 0; c < NC; ++c) b[0][c] = read_b(0, c);
      loop<true>();
    } else {
      loop<false>();
    }
    wait_vm<0>();                // the clamped loads past the end
  }
};

// A workgroup's tile. The tiles of a launch are ordered expert by expert; an
// expert's tiles in groups of kGN weight blocks, inside a group slot tile by
// slot tile with the weight block fastest. Workgroups are dealt to the eight
// XCDs in turn (blockIdx mod 8); XCD x takes the x-th eighth of that order, so
// the 32 or so workgroups resident on an XCD share one expert's kGN weight
// blocks and its slot tiles in the XCD's L2, and every XCD has the same
// number of tiles whatever the routing. Lane l holds the tile count of expert
// e0 + 64 c + l; wave-wide sums and prefix sums find the expert.
template <int TM>
__device__ __forceinline__ bool find_tile(const GemmArgs& a, int nblk, int* e_out, int* off_e, int* n_e, int* m0,
                                          int* nb) {
  const int lane = lane_id();
  auto tiles = [&](int c, int& o, int& n) {
    const int i = c + lane;
    o = clampi(a.offsets[a.e0 + min(i, a.ne)], 0, a.S);
    n = i < a.ne ? clampi(a.offsets[a.e0 + i + 1], o, a.S) - o : 0;
    return (n + TM - 1) / TM;
  };
  auto prefix = [&](int v) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int up = __shfl_up(v, d);
      if (lane >= d) v += up;
    }
    return v;
  };
  int o, n, total = 0;
  for (int c = 0; c < a.ne; c += 64) total += __builtin_amdgcn_readlane(prefix(tiles(c, o, n)), 63);
  const uint64_t units = static_cast<uint64_t>(total) * nblk;
  const uint32_t x = blockIdx.x % 8;
  const uint32_t first = static_cast<uint32_t>(units * x / 8), last = static_cast<uint32_t>(units * (x + 1) / 8);
  uint32_t u = first + blockIdx.x / 8;
  if (u >= last) return false;
  for (int c = 0; c < a.ne; c += 64) {
    const int cnt = tiles(c, o, n);
    const int incl = prefix(cnt);
    const unsigned long long past = __ballot(static_cast<uint32_t>(incl) * nblk > u);
    if (past) {
      const int l = __ffsll(static_cast<long long>(past)) - 1;
      const int m = __builtin_amdgcn_readlane(cnt, l);
      uint32_t r = u - static_cast<uint32_t>(__builtin_amdgcn_readlane(incl, l) - m) * nblk;
      const uint32_t grp = r / (m * kGN);
      r -= grp * (m * kGN);
      const uint32_t gs = min(kGN, nblk - static_cast<int>(grp) * kGN);
      *nb = static_cast<int>(grp * kGN + r % gs);
      *m0 = static_cast<int>(r / gs) * TM;
      *e_out = a.e0 + c + l;
      *off_e = __builtin_amdgcn_readlane(o, l);
      *n_e = __builtin_amdgcn_readlane(n, l);
      return true;
    }
    u -= static_cast<uint32_t>(__builtin_amdgcn_readlane(incl, 63)) * nblk;
  }
  return false;
}

// silu(g) * u = g u / (1 + exp(-g)) in fp32. The library's expf and division
// are about 30 instructions an element, which no other work of the workgroup
// hides (a tile's 64 elements per lane took 4 of about 110 us); here exp(-g) is
// exp2 of -g log2(e) with that product's rounding error put back as a factor,
// and the quotient a reciprocal with one Newton step, each within an ulp or
// two. g enters the exponent held to +-90, beyond which exp(-g) is infinite
// (the quotient then g * 0) or below half an ulp of 1; g itself, infinite or
// not, enters the product.
__device__ __forceinline__ float swiglu(float g, float u) {
  const float x = __builtin_amdgcn_fmed3f(g, -90.0f, 90.0f);
  const float t = x * -1.44269504f;
  const float err = __builtin_fmaf(x, -1.44269504f, -t) + x * -1.92596303e-8f;
  const float e = __builtin_amdgcn_exp2f(t) * __builtin_fmaf(err, 0.693147182f, 1.0f);
  const float d = 1.0f + e;
  const float r = __builtin_amdgcn_rcpf(d);
  const float r1 = __builtin_fmaf(__builtin_fmaf(-d, r, 1.0f), r, r);
  return g * (d < 0x1p126f ? r1 : r) * u;
}

template <int ACT, int SDT, bool GATEUP, int TM>
__global__ __launch_bounds__(64 * kWaves) void k_tgemm(const GemmArgs a, int nblk) {
  typedef TileGeo<TM> Geo;
  __shared__ __attribute__((aligned(1024))) uint8_t lds[Geo::kLds];
  if (!GATEUP && static_cast<int>(blockIdx.y) * a.kb_per_split >= a.F / 128) return;   // an empty K split
  int e, off_e, n_e, m0, nb;
  if (!find_tile<TM>(a, nblk, &e, &off_e, &n_e, &m0, &nb)) return;

  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int lane = lane_id(), lc = lane & 15, lg = lane >> 4;
  const int wn = wave / Geo::WM, wm = wave % Geo::WM;
  const int K = GATEUP ? a.H : a.F;
  const int R = a.R;
  // this wave's 16 RT weight rows for the staging loads: the first half of
  // the gate/up waves takes the tile's gate rows, the second its up rows
  constexpr int kHalf = kWaves / 2, kRows = 16 * Geo::RT;
  const int proj = GATEUP ? wave / kHalf : PW_DOWN;
  const int grow = GATEUP ? nb * 128 + kRows * (wave % kHalf) : nb * 256 + kRows * wave;
  const int rb = grow / R, lr0 = grow - rb * R;
  const pw_page_entry ent = a.table[(static_cast<size_t>(e) * 3 + proj) * a.nrb_max + rb];
  const int bits = __builtin_amdgcn_readfirstlane(ent.bits);
  const int tbytes = bits == 16 ? 4096 : bits == 8 ? 2048 : 1024;
  const int nkb = K / 128;
  // the down projection may split K = F (grid y: the split; fp32 partials)
  const int split = GATEUP ? 0 : static_cast<int>(blockIdx.y);
  const int kb0 = GATEUP ? 0 : split * a.kb_per_split;
  const int kb1 = GATEUP ? nkb : min(nkb, kb0 + a.kb_per_split);
  const size_t tstride = static_cast<size_t>(nkb) * tbytes;
  const uint8_t* wbase = uniform_ptr(a.pool + ent.data_off + static_cast<size_t>(lr0 / 16) * tstride +
                                     static_cast<size_t>(kb0) * tbytes);
  const uint8_t* szbase = uniform_ptr(a.pool + ent.sz_off + static_cast<size_t>(lr0) * 4);
  const uint8_t* xbase =
      uniform_ptr(reinterpret_cast<const uint8_t*>(GATEUP ? a.x : a.h) + static_cast<size_t>(kb0) * 256);
  // activation rows (32-bit byte offsets: the host checks the ranges)
  uint32_t xoff[Geo::NX];
#pragma unroll
  for (int q = 0; q < Geo::NX; ++q) {
    const int i = (wave * Geo::NX + q) * 8 + (lane >> 3);
    const int m = clampi(m0 + i, 0, n_e - 1);
    const int row = GATEUP ? clampi(a.sorted_slot[off_e + m], 0, a.S - 1) / a.topk : off_e + m;
    xoff[q] = static_cast<uint32_t>(row) * static_cast<uint32_t>(K * 2) + 16u * ((lane & 7) ^ (i & 7));
  }
  // In an expert's ragged last tile, waves whose slots all lie past the
  // expert's slots still stage their share and pass every barrier, but read
  // no operands and issue no MFMAs (their LDS bandwidth goes to the others).
  const bool live = m0 + wm * (16 * Geo::NC) < n_e;
  const uint32_t lds0 =
      __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_u8_t)lds)));

  // Accumulator element r of tile (rt, ct) is row 16 rt + 4 lg + r, slot 16 ct + lc.
  auto finish = [&](auto& t) {
#pragma unroll
    for (int c = 0; c < Geo::NC; ++c) {
      const int m = m0 + (wm * Geo::NC + c) * 16 + lc;
      if (m >= n_e) continue;
      if constexpr (GATEUP) {
        uint16_t* dst = a.h + static_cast<size_t>(off_e + m) * a.F + nb * 128 + wn * (8 * Geo::NR) + 4 * lg;
#pragma unroll
        for (int r = 0; r < Geo::NR / 2; ++r) {
          const f32x4 g = t.acc[r][c], u = t.acc[r + Geo::NR / 2][c];
          u32x2 o;
          o[0] = pack2<ACT>(swiglu(g[0], u[0]), swiglu(g[1], u[1]));
          o[1] = pack2<ACT>(swiglu(g[2], u[2]), swiglu(g[3], u[3]));
          *reinterpret_cast<u32x2*>(dst + 16 * r) = o;
        }
      } else {
        float* dst = a.opart + (static_cast<size_t>(split) * a.S + off_e + m) * a.H + nb * 256 + wn * (16 * Geo::NR) +
                     4 * lg;
#pragma unroll
        for (int r = 0; r < Geo::NR; ++r) *reinterpret_cast<f32x4*>(dst + 16 * r) = t.acc[r][c];
      }
    }
  };
  // The host checks that every page is present, so bits is 16, 8 or 4 here; a
  // wave never leaves early (the loop's barriers need all eight).
  auto go = [&](auto& t) {
    t.lds = (lds_u8_t)lds;
    t.lds0 = lds0;
    t.xbase = xbase;
#pragma unroll
    for (int q = 0; q < Geo::NX; ++q) t.xoff[q] = xoff[q];
    t.wbase = wbase;
    t.tstride = tstride;
    t.szbase = szbase;
    // two groups of a 4-bit unit at G = 64, else one group twice
    t.szoff = 4u * (lane & 31) + (bits == 4 && a.G == 64 && lane >= 32 ? 4u * R : 0u);
    t.kstart = kb0 * 128;
    t.R = R;
    t.gshift = 31 - __builtin_clz(a.G);
    t.nstage = (kb1 - kb0) * 4;
    t.wave = wave;
    t.wn = wn;
    t.wm = wm;
    t.lane = lane;
    t.live = live;
    t.boff = 128 * lc + 16 * (lg ^ (lc & 7));
    t.run();
    if (live) finish(t);
  };
  if (bits == 16) {
    TileLoop<ACT, SDT, 16, GATEUP, TM> t;
    go(t);
  } else if (bits == 8) {
    TileLoop<ACT, SDT, 8, GATEUP, TM> t;
    go(t);
  } else {
    TileLoop<ACT, SDT, 4, GATEUP, TM> t;
    go(t);
  }
}

// ---------------------------------------------------------------------------
// Streaming paged GEMM for medium per-expert slot counts of few experts, and for
// bit-plane layers at any: HBM-bound, so the design goal is bytes in flight.
// A workgroup of 4 waves covers 128 weight rows (gate/up: 64 rows of gate and
// the same 64 rows of up; down: 128 rows) and MT slots of one expert. Each wave
// streams 32 rows of one page through a register ring of D stages (64 values
// of K each, about 8 KiB per wave for every format) and computes them against
// all MT slots itself, so weights never pass through LDS; the MT x 64 slice of
// activations is staged once per stage for the four waves. Quantized weights
// are dequantized in registers to fl32(z + c s) rounded to the activation
// dtype, as in the large-tile kernel.
// ---------------------------------------------------------------------------

template <int B> constexpr int sg_depth() { return B == 16 ? 2 : B == 8 || B == kApl8 ? 4 : 8; }
constexpr int kSgStagePad = 8;   // stage counts are padded to a multiple of every depth

template <int MT> constexpr int sg_xbuf() { return MT * kTK * 2; }            // one activation buffer
template <int MT> constexpr int sg_lds() { return 2 * sg_xbuf<MT>() + 4 * 1024; } // + a discard area

// The loop body has no branches (every load and store is unconditional, with
// clamped indices), so the compiler's wait counts stay static and the ring's
// D stages really are in flight.
// The wave's rows over 128-blocks [kb0, kb1) of the nkb blocks of a row.
template <int ACT, int SDT, int B, int MT>
__device__ __forceinline__ void sg_loop(uint8_t* lds, const uint8_t* tile0, const uint8_t* szrow,
                                        const uint8_t* xrow, int xf, int nkb, int kb0, int kb1, int R, int gshift,
                                        int wave, f32x4 (&acc)[2][MT / 16]) {
  constexpr int D = sg_depth<B>();
  constexpr int XF = MT >= 32 ? MT / 32 : 1;       // activation fragments per wave
  constexpr int XB = sg_xbuf<MT>();
  const int lane = lane_id(), lg = lane >> 4;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int u = 0; u < MT / 16; ++u) acc[t][u] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nstage = (kb1 - kb0) * 128 / kTK;
  const int st0 = kb0 * 128 / kTK;                 // first stage of the range within the row
  const int npad = (nstage + kSgStagePad - 1) / kSgStagePad * kSgStagePad;
  auto group_of = [&](int st) { return (st * kTK) >> gshift; };
  // waves past the tile's activation fragments write a discard area instead
  const int xoff = xf < MT / 8 ? 1024 * xf : 2 * XB + 1024 * wave - 1024 * xf;
  auto fetch_w = [&](WStage<B>& w, int st) {
    const int s = st0 + min(st, nstage - 1);
    w_fetch<B>(w, tile0, szrow, s >> 1, s & 1, group_of(s), nkb, R);
  };
  // activation fragment q of this wave: xf + q (slot tile (xf + q) / 2, k-step (xf + q) mod 2)
  auto fetch_x = [&](u32x4 (&xv)[XF], int st) {
    const int s = st0 + min(st, nstage - 1);
#pragma unroll
    for (int q = 0; q < XF; ++q)
      xv[q] = ld16(xrow + static_cast<size_t>(s * kTK + 32 * ((xf + q) & 1) + 8 * lg) * 2);
  };
  auto store_x = [&](const u32x4 (&xv)[XF], int b) {
    uint8_t* d = lds + (xf < MT / 8 ? b * XB : 0) + xoff + 16 * lane;
#pragma unroll
    for (int q = 0; q < XF; ++q) *reinterpret_cast<u32x4*>(d + 1024 * q) = xv[q];
  };
  WStage<B> ring[D];
  u32x4 xv[XF];
#pragma unroll
  for (int j = 0; j < D; ++j) fetch_w(ring[j], j);
  fetch_x(xv, 0);
  store_x(xv, 0);
  __syncthreads();
  for (int base = 0; base < npad; base += D) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
      const int st = base + j;
      const uint8_t* cur = lds + (st & 1) * XB + 16 * lane;
      fetch_x(xv, st + 1);
      __builtin_amdgcn_sched_barrier(0);   // issue the activation load first: its wait ends the stage
      const bool live = st < nstage;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        u32x4 bx[MT / 16];
#pragma unroll
        for (int u = 0; u < MT / 16; ++u) bx[u] = ld16(cur + 1024 * (2 * u + i));
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          u32x4 aw = w_piece<ACT, SDT, B>(ring[j], 2 * t + i);
          if (!live) aw = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
          for (int u = 0; u < MT / 16; ++u) acc[t][u] = mma<ACT>(aw, bx[u], acc[t][u]);
        }
      }
      fetch_w(ring[j], st + D);
      store_x(xv, (st + 1) & 1);
      __syncthreads();
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// LUT rows of the four waves (32 rows x 256 values each) for nested bit-plane pages
constexpr int kSgLutWave = 32 * 256 * 2;

template <int ACT, int SDT, bool GATEUP, int MT, bool APL>
__global__ __launch_bounds__(256) void k_sgemm(const GemmArgs a, int nblk, int mtmax) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[sg_lds<MT>() + (APL ? 4 * kSgLutWave : 0)];
  // the down projection may split K = F into a.nsplit ranges (fp32 partials,
  // summed by the combine); split-major block order
  const int nsplit = GATEUP ? 1 : a.nsplit;
  const int per_split = gridDim.x / nsplit;
  const int split = blockIdx.x / per_split, bid = blockIdx.x % per_split;
  const int per_xcd = per_split / 8;
  const int logical = (bid % 8) * per_xcd + bid / 8;
  const int band = logical / (kGN * mtmax), inb = logical % (kGN * mtmax);
  const int nb = band * kGN + inb % kGN, mt = inb / kGN;
  if (nb >= nblk) return;
  int e = 0, off_e = 0, n_e = 0, m0 = 0;
  {
    int rest = mt;
    bool found = false;
    for (int x = a.e0; x < a.e0 + a.ne && !found; ++x) {
      const int o = clampi(a.offsets[x], 0, a.S);
      const int n = clampi(a.offsets[x + 1], o, a.S) - o;
      const int cnt = (n + MT - 1) / MT;
      if (rest < cnt) {
        e = x;
        off_e = o;
        n_e = n;
        m0 = rest * MT;
        found = true;
      } else {
        rest -= cnt;
      }
    }
    if (!found) return;
  }
  const int wave = threadIdx.x >> 6, lane = lane_id(), lc = lane & 15, lg = lane >> 4;
  const int K = GATEUP ? a.H : a.F;
  const int R = a.R;
  int proj, grow;
  if (GATEUP) {
    proj = wave >> 1;                       // waves 0-1: gate; 2-3: up
    grow = nb * 64 + 32 * (wave & 1);
  } else {
    proj = PW_DOWN;
    grow = nb * 128 + 32 * wave;
  }
  const int rb = grow / R, lr0 = grow - rb * R;
  const pw_page_entry ent = a.table[(static_cast<size_t>(e) * 3 + proj) * a.nrb_max + rb];
  const int bits = ent.bits;
  const bool apl_page = APL && (ent.rsv & 0xFF) == PW_FMT_APL;
  const size_t tbytes = apl_page ? 256 : bits == 16 ? 4096 : bits == 8 ? 2048 : 1024;
  const uint8_t* tile0 = a.pool + ent.data_off + static_cast<size_t>(lr0 / 16) * (K / 128) * tbytes;
  const uint8_t* szrow = a.pool + ent.sz_off + static_cast<size_t>(lr0 + lc) * 4;
  if (APL && apl_page) {
    // the wave's 32 LUT rows of the committed precision go to its LDS area
    const int nl = bits == 8 ? 256 : 16;
    const size_t rk8 = static_cast<size_t>(R) * K / 8;
    const uint8_t* src = a.pool + ent.sz_off + (bits == 8 ? 32 * static_cast<size_t>(R) + 4 * rk8 : 0) +
                         static_cast<size_t>(lr0) * nl * 2;
    uint8_t* dst = lds + sg_lds<MT>() + wave * kSgLutWave;
    for (int o = 16 * lane; o < 32 * nl * 2; o += 16 * 64)
      *reinterpret_cast<u32x4*>(dst + o) = *reinterpret_cast<const u32x4*>(src + o);
    szrow = dst;
  }
  // this wave's activation fragments start at xf = wave * XF (slot tile xf / 2)
  constexpr int XF = MT >= 32 ? MT / 32 : 1;
  const int xf = wave * XF;
  const int m = clampi(m0 + (xf >> 1) * 16 + lc, 0, n_e - 1);
  const uint8_t* xrow;
  if (GATEUP) {
    const int slot = clampi(a.sorted_slot[off_e + m], 0, a.S - 1);
    xrow = reinterpret_cast<const uint8_t*>(a.x) + static_cast<size_t>(slot / a.topk) * a.H * 2;
  } else {
    xrow = reinterpret_cast<const uint8_t*>(a.h) + static_cast<size_t>(off_e + m) * a.F * 2;
  }
  // The host checks that every page is present, so bits is 16, 8 or 4 here; a
  // wave never leaves early (the loop's barriers need all four).
  f32x4 acc[2][MT / 16];
  const int nkb = K / 128;
  const int kb0 = GATEUP ? 0 : split * a.kb_per_split;
  const int kb1 = GATEUP ? nkb : min(nkb, kb0 + a.kb_per_split);
  if (kb0 >= kb1) return;                         // (whole workgroup: no barrier passed yet)
  const int gshift = 31 - __builtin_clz(a.G);     // G is a power of two, at least 64
  if constexpr (APL) {
    if (apl_page) {
      if (bits == 8) sg_loop<ACT, SDT, kApl8, MT>(lds, tile0, szrow, xrow, xf, nkb, kb0, kb1, R, gshift, wave, acc);
      else sg_loop<ACT, SDT, kApl4, MT>(lds, tile0, szrow, xrow, xf, nkb, kb0, kb1, R, gshift, wave, acc);
    } else if (bits == 16) {
      sg_loop<ACT, SDT, 16, MT>(lds, tile0, szrow, xrow, xf, nkb, kb0, kb1, R, gshift, wave, acc);
    } else if (bits == 8) {
      sg_loop<ACT, SDT, 8, MT>(lds, tile0, szrow, xrow, xf, nkb, kb0, kb1, R, gshift, wave, acc);
    } else {
      sg_loop<ACT, SDT, 4, MT>(lds, tile0, szrow, xrow, xf, nkb, kb0, kb1, R, gshift, wave, acc);
    }
  } else {
    if (bits == 16) sg_loop<ACT, SDT, 16, MT>(lds, tile0, szrow, xrow, xf, nkb, kb0, kb1, R, gshift, wave, acc);
    else if (bits == 8) sg_loop<ACT, SDT, 8, MT>(lds, tile0, szrow, xrow, xf, nkb, kb0, kb1, R, gshift, wave, acc);
    else sg_loop<ACT, SDT, 4, MT>(lds, tile0, szrow, xrow, xf, nkb, kb0, kb1, R, gshift, wave, acc);
  }

  const int wr = wave & 1;
  if (GATEUP) {
    // gate waves hand their 32 x MT accumulators to the up wave of the same rows
    float* xch = reinterpret_cast<float*>(lds) + wr * (2 * (MT / 16) * 64 * 4);
    if (proj == PW_GATE) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int u = 0; u < MT / 16; ++u)
          *reinterpret_cast<f32x4*>(xch + ((t * (MT / 16) + u) * 64 + lane) * 4) = acc[t][u];
    }
    __syncthreads();
    if (proj == PW_UP) {
#pragma unroll
      for (int u = 0; u < MT / 16; ++u) {
        const int mm = m0 + u * 16 + lc;
        if (mm < n_e) {
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const f32x4 g = *reinterpret_cast<const f32x4*>(xch + ((t * (MT / 16) + u) * 64 + lane) * 4);
            uint32_t hv[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) hv[r] = rne16(g[r] / (1.0f + expf(-g[r])) * acc[t][u][r], ACT);
            u32x2 o;
            o[0] = hv[0] | (hv[1] << 16);
            o[1] = hv[2] | (hv[3] << 16);
            *reinterpret_cast<u32x2*>(a.h + static_cast<size_t>(off_e + mm) * a.F + grow + t * 16 + 4 * lg) = o;
          }
        }
      }
    }
  } else {
#pragma unroll
    for (int u = 0; u < MT / 16; ++u) {
      const int mm = m0 + u * 16 + lc;
      if (mm < n_e) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
          *reinterpret_cast<f32x4*>(a.opart + (static_cast<size_t>(split) * a.S + off_e + mm) * a.H + grow + t * 16 +
                                    4 * lg) =
              acc[t][u];
      }
    }
  }
}

template <int ACT, int SDT, int MT>
void sgemm_go(const GemmArgs& a, bool gateup, hipStream_t st) {
  const int nblk = gateup ? a.F / 64 : a.H / 128;
  const int mtmax = (a.s_range + MT - 1) / MT + a.ne;
  const int n = ((nblk + kGN - 1) / kGN * kGN * mtmax + 7) / 8 * 8 * (gateup ? 1 : a.nsplit);
  if (a.apl) {
    if (gateup)
      hipLaunchKernelGGL((k_sgemm<ACT, SDT, true, MT, true>), dim3(n), dim3(256), 0, st, a, nblk, mtmax);
    else
      hipLaunchKernelGGL((k_sgemm<ACT, SDT, false, MT, true>), dim3(n), dim3(256), 0, st, a, nblk, mtmax);
  } else if (gateup) {
    hipLaunchKernelGGL((k_sgemm<ACT, SDT, true, MT, false>), dim3(n), dim3(256), 0, st, a, nblk, mtmax);
  } else {
    hipLaunchKernelGGL((k_sgemm<ACT, SDT, false, MT, false>), dim3(n), dim3(256), 0, st, a, nblk, mtmax);
  }
}

// Layers with nested bit-plane pages run this kernel at every batch size;
// at decode sizes (up to 24 expected slots per expert) 32-slot tiles halve
// the activation staging, and with the LUT rows the workgroup's LDS then fits
// twice per CU.
template <int ACT, int SDT>
void sgemm_mt(const GemmArgs& a, bool gateup, hipStream_t st) {
  const int expect = (a.s_range + a.ne - 1) / a.ne;
  if (a.apl && expect <= 24) sgemm_go<ACT, SDT, 32>(a, gateup, st);
  else sgemm_go<ACT, SDT, 64>(a, gateup, st);
}

template <int ACT, int SDT, int TM>
void tgemm_tm(const GemmArgs& a, bool gateup, hipStream_t st) {
  const int nblk = gateup ? a.F / 128 : a.H / 256;
  const int mtmax = (a.s_range + TM - 1) / TM + a.ne;   // an upper bound on slot tiles
  const int n = (nblk * mtmax + 7) / 8 * 8;
  if (gateup)
    hipLaunchKernelGGL((k_tgemm<ACT, SDT, true, TM>), dim3(n), dim3(64 * kWaves), 0, st, a, nblk);
  else
    hipLaunchKernelGGL((k_tgemm<ACT, SDT, false, TM>), dim3(n, a.nsplit), dim3(64 * kWaves), 0, st, a, nblk);
}

template <int ACT, int SDT>
void tgemm_go(const GemmArgs& a, bool gateup, hipStream_t st) {
  const int expect = (a.s_range + a.ne - 1) / a.ne;
  if (expect > kTileNarrow) tgemm_tm<ACT, SDT, 256>(a, gateup, st);
  else tgemm_tm<ACT, SDT, 128>(a, gateup, st);
}

}  // namespace

hipError_t launch_tgemm(const GemmArgs& a, bool gateup, hipStream_t st) {
  if (a.ne <= 0) return hipSuccess;
  if (a.act == PW_BF16) {
    if (a.sdt == PW_BF16) tgemm_go<PW_BF16, PW_BF16>(a, gateup, st);
    else tgemm_go<PW_BF16, PW_F16>(a, gateup, st);
  } else {
    if (a.sdt == PW_BF16) tgemm_go<PW_F16, PW_BF16>(a, gateup, st);
    else tgemm_go<PW_F16, PW_F16>(a, gateup, st);
  }
  return hipGetLastError();
}

// Streaming path (32- or 64-slot tiles): bit-plane layers, experts too few for
// the tiled kernel's tiles to fill the chip, and shapes that it does not take.
hipError_t launch_sgemm(const GemmArgs& a, bool gateup, hipStream_t st) {
  if (a.ne <= 0) return hipSuccess;
  if (a.act == PW_BF16) {
    if (a.sdt == PW_BF16) sgemm_mt<PW_BF16, PW_BF16>(a, gateup, st);
    else sgemm_mt<PW_BF16, PW_F16>(a, gateup, st);
  } else {
    if (a.sdt == PW_BF16) sgemm_mt<PW_F16, PW_BF16>(a, gateup, st);
    else sgemm_mt<PW_F16, PW_F16>(a, gateup, st);
  }
  return hipGetLastError();
}

}  // namespace pw
