// Device code shared by the HyperQuant codec kernels for gfx950 (MI355X).
//
// Lane layout (encode and decode): one wave64 owns one sub-stream of 512
// scalars = four 128-scalar tiles.  Lane l holds tile l / 16, coordinates
// 8 (l % 16) .. 8 (l % 16) + 7 (one 16-byte bf16 load), i.e. one E8 block,
// two D4 blocks, four A2 blocks or eight Z scalars; the symbol index of its
// j-th value inside the sub-stream is 8 l + j.  The Walsh-Hadamard stages
// h = 1, 2, 4 run in registers, h = 8, 16, 32, 64 across lanes l ^ 1, 2, 4, 8,
// in that order, so every fp32 value equals the reference stage order.
//
// Floating-point contraction is off for this file: each a * b + c that the
// method writes as two roundings stays two roundings.  The fused
// multiply-adds used below either have a multiplier of +-1 or +-2 (one
// rounding of a sum or difference, the same as the add or subtract they
// replace) or work on integer values (exact).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hq_internal.h"

#pragma clang fp contract(off)

namespace {

constexpr float kSqrt3 = 1.7320508075688772f;       // fp32 nearest sqrt(3)
constexpr float kInv2Sqrt3 = 0.28867513459481287f;  // fp32 nearest 1/(2 sqrt(3))
constexpr int kE8 = HQ_E8, kD4 = HQ_D4, kA2 = HQ_A2, kZ = HQ_Z;

// ------------------------------------------------------------------ helpers

__device__ __forceinline__ uint32_t readfirst(uint32_t v) {
  return __builtin_amdgcn_readfirstlane(v);
}

// DPP lane moves (data-parallel primitives of the gfx9 VALU): dst lane l reads
// src lane f(l) inside its 16-lane row; lanes whose row/bank is masked off
// keep `old`, lanes with no source read 0 when BC is set.
template <int CTRL, int RM = 0xF, int BM = 0xF, bool BC = false>
__device__ __forceinline__ uint32_t dpp(uint32_t old, uint32_t src) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)src, CTRL, RM, BM, BC);
}

constexpr int kDppQuadXor1 = 0xB1;  // quad_perm [1,0,3,2]
constexpr int kDppQuadXor2 = 0x4E;  // quad_perm [2,3,0,1]
constexpr int kDppRowShl4 = 0x104;  // lane l reads l + 4
constexpr int kDppRowShr1 = 0x111, kDppRowShr2 = 0x112, kDppRowShr4 = 0x114, kDppRowShr8 = 0x118;
constexpr int kDppRowRor8 = 0x128;  // lane l reads (l + 8) mod 16 = l ^ 8
constexpr int kDppRowBcast15 = 0x142, kDppRowBcast31 = 0x143;

// Value of lane l ^ M (M in 1, 2, 4, 8: inside the 16-lane row).
template <int M>
__device__ __forceinline__ uint32_t xor_lane(uint32_t v) {
  if constexpr (M == 1) {
    return dpp<kDppQuadXor1>(v, v);
  } else if constexpr (M == 2) {
    return dpp<kDppQuadXor2>(v, v);
  } else if constexpr (M == 4) {
    const uint32_t t = dpp<kDppRowShl4, 0xF, 0x5>(v, v);  // banks 0, 2 read l + 4
    return dpp<kDppRowShr4, 0xF, 0xA>(t, v);              // banks 1, 3 read l - 4
  } else {
    return dpp<kDppRowRor8>(v, v);
  }
}

template <int M>
__device__ __forceinline__ float xor_lane_f(float v) {
  return __uint_as_float(xor_lane<M>(__float_as_uint(v)));
}

// Value of lane (l & ~3) | I for every lane l (a quad broadcast).
template <int I>
__device__ __forceinline__ float quad_bcast(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), I * 0x55, 0xF, 0xF, true));
}

// Inclusive prefix sum over the 64 lanes (row shifts, then row broadcasts).
__device__ __forceinline__ uint32_t wave_scan_incl(uint32_t x) {
  x += dpp<kDppRowShr1, 0xF, 0xF, true>(0u, x);
  x += dpp<kDppRowShr2, 0xF, 0xF, true>(0u, x);
  x += dpp<kDppRowShr4, 0xF, 0xF, true>(0u, x);
  x += dpp<kDppRowShr8, 0xF, 0xF, true>(0u, x);
  x += dpp<kDppRowBcast15, 0xA, 0xF>(0u, x);
  x += dpp<kDppRowBcast31, 0xC, 0xF>(0u, x);
  return x;
}

// Two inclusive prefix sums over the 64 lanes at once (interleaved, so the
// two chains' latencies overlap).
__device__ __forceinline__ void wave_scan_incl2(uint32_t& a, uint32_t& b) {
  a += dpp<kDppRowShr1, 0xF, 0xF, true>(0u, a);
  b += dpp<kDppRowShr1, 0xF, 0xF, true>(0u, b);
  a += dpp<kDppRowShr2, 0xF, 0xF, true>(0u, a);
  b += dpp<kDppRowShr2, 0xF, 0xF, true>(0u, b);
  a += dpp<kDppRowShr4, 0xF, 0xF, true>(0u, a);
  b += dpp<kDppRowShr4, 0xF, 0xF, true>(0u, b);
  a += dpp<kDppRowShr8, 0xF, 0xF, true>(0u, a);
  b += dpp<kDppRowShr8, 0xF, 0xF, true>(0u, b);
  a += dpp<kDppRowBcast15, 0xA, 0xF>(0u, a);
  b += dpp<kDppRowBcast15, 0xA, 0xF>(0u, b);
  a += dpp<kDppRowBcast31, 0xC, 0xF>(0u, a);
  b += dpp<kDppRowBcast31, 0xC, 0xF>(0u, b);
}

// Sum over the 64 lanes, as a wave-uniform value.
__device__ __forceinline__ uint32_t wave_total(uint32_t x) {
  return __builtin_amdgcn_readlane(wave_scan_incl(x), 63);
}

// a ^ b ^ c in one instruction (gfx950 three-input bitwise op, truth table
// 0x96 over S0 = 0xF0, S1 = 0xCC, S2 = 0xAA).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t r;
  asm("v_bitop3_b32 %0, %1, %2, %3 bitop3:0x96" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// (a << sh) | c and (1 << sh) | c in one instruction each.
__device__ __forceinline__ uint32_t lshl_or(uint32_t a, uint32_t sh, uint32_t c) {
  uint32_t r;
  asm("v_lshl_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(sh), "v"(c));
  return r;
}
// (a << sh) | c with a wave-uniform shift below 32: the compiler's own, which
// may come right behind the instruction that writes the shift's scalar register
// (inline assembly would need its two wait states)
__device__ __forceinline__ uint32_t lshl_or_s(uint32_t a, uint32_t sh, uint32_t c) { return (a << sh) | c; }
__device__ __forceinline__ uint32_t bit_or(uint32_t sh, uint32_t c) {
  uint32_t r;
  asm("v_lshl_or_b32 %0, 1, %1, %2" : "=v"(r) : "v"(sh), "v"(c));
  return r;
}

// 2 v ^ (v >> 31); the doubling as an add, which gfx950 issues at the fast
// VALU rate (a left shift takes the slow one).
__device__ __forceinline__ uint32_t zigzag(int32_t v) {
  uint32_t d;
  asm("v_add_u32 %0, %1, %1" : "=v"(d) : "v"(v));
  return d ^ (uint32_t)(v >> 31);
}

__device__ __forceinline__ int32_t unzigzag(uint32_t m) {
  return (int32_t)(m >> 1) ^ -(int32_t)(m & 1u);
}

// In-byte select table: entry v packs, 4 bits per rank k = 0..7, the position
// of the k-th set bit of the byte value v (entries for ranks past popc(v)
// are unused); built at compile time, kernels copy it into LDS.
struct ByteSelectTable {
  uint32_t e[256];
  constexpr ByteSelectTable() : e() {
    for (uint32_t v = 0; v < 256; ++v) {
      uint32_t x = 0, k = 0;
      for (uint32_t b = 0; b < 8; ++b)
        if ((v >> b) & 1u) {
          x |= b << (4 * k);
          ++k;
        }
      e[v] = x;
    }
  }
};
__constant__ ByteSelectTable kByteSelect = ByteSelectTable();

// Position (0..31) of the r-th set bit (r from 0) of w.
__device__ __forceinline__ uint32_t select32(uint32_t w, uint32_t r) {
  uint32_t pos = 0, c;
  c = __popc(w & 0xFFFFu);
  if (r >= c) { r -= c; w >>= 16; pos += 16; }
  c = __popc(w & 0xFFu);
  if (r >= c) { r -= c; w >>= 8; pos += 8; }
  c = __popc(w & 0xFu);
  if (r >= c) { r -= c; w >>= 4; pos += 4; }
  c = __popc(w & 0x3u);
  if (r >= c) { r -= c; w >>= 2; pos += 2; }
  c = w & 1u;
  if (r >= c) { pos += 1; }
  return pos;
}

__device__ __forceinline__ float bf16_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

// Two fp32 -> bf16 (round to nearest even) in one word: lo in bits 0-15.
__device__ __forceinline__ uint32_t cvt_pk_bf16(float lo, float hi) {
  uint32_t r;
  asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r) : "v"(lo), "v"(hi));
  return r;
}

// IEEE round-to-nearest-even fp32 -> bf16 bits.
__device__ __forceinline__ uint32_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x40u;
  u += 0x7FFFu + ((u >> 16) & 1u);
  return u >> 16;
}

// ------------------------------------------------------------- Philox4x32-10
// Salmon, Moraes, Dror, Shaw (SC'11): ten rounds of two 32x32->64 products
// with the Weyl key schedule.
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t out[4]) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    // each 64-bit product is one v_mad_u64_u32 (both halves in one issue)
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
    const uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
    const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
  }
  out[0] = c0;
  out[1] = c1;
  out[2] = c2;
  out[3] = c3;
}

// ------------------------------------------------------ nearest-point decoders
// Conway & Sloane's closest-point algorithms on the integer realizations:
// 2E8 (two D8 cosets), D4 (round + parity fix), A2 (two rectangular cosets),
// Z (round).  rint is round-half-even; argmax ties take the lowest index.

template <int N>
__device__ __forceinline__ int argmax_abs(const float* e) {
  float best = __builtin_fabsf(e[0]);
  int j = 0;
#pragma unroll
  for (int i = 1; i < N; ++i) {
    const float a = __builtin_fabsf(e[i]);
    const bool gt = a > best;
    best = gt ? a : best;
    j = gt ? i : j;
  }
  return j;
}

__device__ __forceinline__ float tree8(const float* s) {
  return ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
}

__device__ __forceinline__ void quant_e8(const float* z, int32_t* c) {
  float ka[8], fb[8], ea[8], eb[8];
  int32_t sa = 0, sb = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float h = z[i] * 0.5f;
    ka[i] = __builtin_rintf(h);
    fb[i] = __builtin_floorf(h);
    ea[i] = __builtin_fmaf(-2.0f, ka[i], z[i]);        // z - 2k, one rounding
    eb[i] = z[i] - __builtin_fmaf(2.0f, fb[i], 1.0f);  // z - (2f + 1)
    sa += (int32_t)ka[i];
    sb += (int32_t)fb[i];
  }
  if (sa & 1) {
    const int j = argmax_abs<8>(ea);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (i == j) {
        ka[i] += (ea[i] >= 0.0f) ? 1.0f : -1.0f;
        ea[i] = __builtin_fmaf(-2.0f, ka[i], z[i]);
      }
  }
  if (sb & 1) {
    const int j = argmax_abs<8>(eb);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (i == j) {
        fb[i] += (eb[i] >= 0.0f) ? 1.0f : -1.0f;
        eb[i] = z[i] - __builtin_fmaf(2.0f, fb[i], 1.0f);
      }
  }
  float sqa[8], sqb[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    sqa[i] = ea[i] * ea[i];
    sqb[i] = eb[i] * eb[i];
  }
  const bool even = tree8(sqa) <= tree8(sqb);
#pragma unroll
  for (int i = 0; i < 8; ++i) c[i] = even ? 2 * (int32_t)ka[i] : 2 * (int32_t)fb[i] + 1;
}

__device__ __forceinline__ void quant_d4(const float* z, int32_t* c) {
  float k[4], e[4];
  int32_t s = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    k[i] = __builtin_rintf(z[i]);
    e[i] = z[i] - k[i];
    c[i] = (int32_t)k[i];
    s += c[i];
  }
  if (s & 1) {
    const int j = argmax_abs<4>(e);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i == j) c[i] += (e[i] >= 0.0f) ? 1 : -1;
  }
}

__device__ __forceinline__ void quant_a2(const float* z, int32_t* c) {
  const float y = z[0], x = z[1];
  const float a0 = __builtin_rintf(y * kInv2Sqrt3);
  const float b0 = __builtin_rintf(x * 0.5f);
  const float a1 = __builtin_rintf((y - kSqrt3) * kInv2Sqrt3);
  const float b1 = __builtin_rintf((x - 1.0f) * 0.5f);
  const int32_t ny0 = 2 * (int32_t)a0, nx0 = 2 * (int32_t)b0;
  const int32_t ny1 = 2 * (int32_t)a1 + 1, nx1 = 2 * (int32_t)b1 + 1;
  const float ey0 = y - kSqrt3 * (float)ny0, ex0 = x - (float)nx0;
  const float ey1 = y - kSqrt3 * (float)ny1, ex1 = x - (float)nx1;
  const float d0 = ey0 * ey0 + ex0 * ex0;
  const float d1 = ey1 * ey1 + ex1 * ex1;
  const bool first = d0 <= d1;
  c[0] = first ? ny0 : ny1;
  c[1] = first ? nx0 : nx1;
}

template <int LAT>
__device__ __forceinline__ void quantize8(const float* z, int32_t* c) {
  if constexpr (LAT == kE8) {
    quant_e8(z, c);
  } else if constexpr (LAT == kD4) {
    quant_d4(z, c);
    quant_d4(z + 4, c + 4);
  } else if constexpr (LAT == kA2) {
#pragma unroll
    for (int b = 0; b < 4; ++b) quant_a2(z + 2 * b, c + 2 * b);
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = (int32_t)__builtin_rintf(z[i]);
  }
}

// Lattice code -> coordinate in R (the A2 y axis carries sqrt(3)).
template <int LAT>
__device__ __forceinline__ float code_coord(int32_t c, int j) {
  if constexpr (LAT == kA2) {
    return (j & 1) ? (float)c : kSqrt3 * (float)c;
  } else {
    return (float)c;
  }
}

// E8's U = b - Q(b) for a box point b in [-2, 2)^8 whose coordinates are
// multiples of 2^-22: the point quant_e8 picks.  The even coset's error is
// ea = b - 2 rint(b / 2) (rint by the 1.5 * 2^23 shift, whose low bit is the
// rounded value's parity), the odd coset's b - sign(b); both are exact and
// never -0.  A coset whose parity is odd moves its first coordinate of largest
// error to the next point on the other side, which turns that error e into e -
// 2 sign(e); U is the nearer coset's error vector (the even one on a tie, the
// squared errors summed in quant_e8's fp32 tree).  This form carries both
// vectors out; it is the reference of dither_e8.
__device__ __forceinline__ void dither_e8_cosets(const float* b, float* u) {
  constexpr float kShift = 12582912.0f;  // 1.5 * 2^23
  float ea[8], eb[8];
  uint32_t pa = 0, pb = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float t = b[i] * 0.5f + kShift;
    ea[i] = __builtin_fmaf(-2.0f, t - kShift, b[i]);
    pa ^= __float_as_uint(t);
    const uint32_t sb = __float_as_uint(b[i]) & 0x80000000u;
    eb[i] = b[i] - __uint_as_float(sb | 0x3F800000u);
    pb ^= sb;
  }
  auto fix = [](float* e, bool odd) {
    float m = __builtin_fabsf(e[0]);
#pragma unroll
    for (int i = 1; i < 8; ++i) m = __builtin_fmaxf(m, __builtin_fabsf(e[i]));
    bool done = !odd;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const bool hit = !done && __builtin_fabsf(e[i]) == m;
      const float two = __uint_as_float((__float_as_uint(e[i]) & 0x80000000u) | 0x40000000u);
      e[i] = hit ? e[i] - two : e[i];
      done = done || hit;
    }
  };
  fix(ea, pa & 1u);
  fix(eb, pb >> 31);
  float sa[8], sq[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    sa[i] = ea[i] * ea[i];
    sq[i] = eb[i] * eb[i];
  }
  const bool even = tree8(sa) <= tree8(sq);
#pragma unroll
  for (int i = 0; i < 8; ++i) u[i] = even ? ea[i] : eb[i];
}

// The same point from the even coset's errors alone.  The odd one's are ea -
// sign(ea), so |eb| = 1 - |ea|: its largest is the smallest |ea|, and the two
// squared distances differ by
//   D = 8 - 2 sum |ea| + [odd coset's parity] 4 min |ea| - [even's] (4 - 4 max |ea|),
// whose sign is the decision wherever rounding cannot matter (the trees' and
// D's errors stay below 2^-15).  Then one pass adds the chosen coset's offset,
// 0 or -sign(ea), and at the moved coordinate -2 sign(ea) or +sign(ea).  A wave
// with a lane near a tie, or at the box's all-odd points (min |ea| = 1, where
// sign(eb) is not -sign(ea)), takes the two-coset form: about 0.3 % of them.
// Against it, half the passes over the 8 coordinates and no squares: KV decode
// of 32768 x 1024 rows 53.1 -> 49.1 us, 16 x 8192-token attention 465 -> 434.
__device__ __forceinline__ void dither_e8(const float* b, float* u) {
  constexpr float kShift = 12582912.0f;  // 1.5 * 2^23
  float ea[8];
  uint32_t tb[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float t = b[i] * 0.5f + kShift;
    ea[i] = __builtin_fmaf(-2.0f, t - kShift, b[i]);
    tb[i] = __float_as_uint(t);
  }
  const uint32_t pa = xor3(xor3(tb[0], tb[1], tb[2]), tb[3], tb[4]) ^ xor3(tb[5], tb[6], tb[7]);
  const uint32_t pb = xor3(xor3(__float_as_uint(b[0]), __float_as_uint(b[1]), __float_as_uint(b[2])),
                           __float_as_uint(b[3]), __float_as_uint(b[4])) ^
                      xor3(__float_as_uint(b[5]), __float_as_uint(b[6]), __float_as_uint(b[7]));
  float a[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = __builtin_fabsf(ea[i]);
  const float mx = fmaxf(fmaxf(fmaxf(a[0], a[1]), fmaxf(a[2], a[3])), fmaxf(fmaxf(a[4], a[5]), fmaxf(a[6], a[7])));
  const float mn = fminf(fminf(fminf(a[0], a[1]), fminf(a[2], a[3])), fminf(fminf(a[4], a[5]), fminf(a[6], a[7])));
  const bool oa = pa & 1u, ob = pb >> 31;
  const float D = __builtin_fmaf(-2.0f, tree8(a), 8.0f) + ((ob ? 4.0f * mn : 0.0f) - (oa ? 4.0f - 4.0f * mx : 0.0f));
  if (__ballot(__builtin_fabsf(D) < 0x1p-13f || mn >= 1.0f) != 0ull) {
    dither_e8_cosets(b, u);
    return;
  }
  const bool even = D > 0.0f;
  const float target = even ? (oa ? mx : 2.0f) : (ob ? mn : 2.0f);  // 2: no |ea| is, nothing moves
  const float base = even ? 0.0f : -1.0f, moved = even ? -2.0f : 1.0f;
  bool done = false;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const bool hit = !done && a[i] == target;
    done = done || hit;
    const float t = hit ? moved : base;
    u[i] = ea[i] + __uint_as_float(__float_as_uint(t) ^ (__float_as_uint(ea[i]) & 0x80000000u));
  }
}

// Dither U = b - Q(b) for the lane's 8 coordinates (columns col0 .. col0+7 of
// global row `row`, col0 a multiple of 8): b is a uniform point of a box that
// is a fundamental domain of a sublattice ([-2, 2)^m for 2E8, D4, Z;
// [-sqrt3, sqrt3) x [-1, 1) for A2), drawn from 24 bits of Philox word
// (col mod 4) at counter (col / 4, row_lo, row_hi, 0).  COSETS: E8's point from
// both cosets' errors.
template <int LAT, bool COSETS = false>
__device__ __forceinline__ void dither8(uint64_t seed, int64_t row, int64_t col0, float* u) {
  uint32_t r[8];
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  const uint32_t rl = (uint32_t)(uint64_t)row, rh = (uint32_t)((uint64_t)row >> 32);
  philox4x32_10((uint32_t)((uint64_t)col0 >> 2), rl, rh, 0u, k0, k1, r);
  philox4x32_10((uint32_t)((uint64_t)col0 >> 2) + 1u, rl, rh, 0u, k0, k1, r + 4);
  float b[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float centered = (float)((int32_t)(r[i] >> 8) - 8388608);
    if constexpr (LAT == kA2) {
      b[i] = (i & 1) ? centered * 0x1p-23f : (centered * 0x1p-23f) * kSqrt3;
    } else {
      b[i] = centered * 0x1p-22f;
    }
  }
  if constexpr (LAT == kE8) {
    if constexpr (COSETS)
      dither_e8_cosets(b, u);
    else
      dither_e8(b, u);
  } else {
    int32_t c[8];
    quantize8<LAT>(b, c);
#pragma unroll
    for (int i = 0; i < 8; ++i) u[i] = b[i] - code_coord<LAT>(c[i], i);
  }
}

// --------------------------------------------------------------- strip / unstrip

template <int LAT>
__device__ __forceinline__ void strip8(const int32_t* c, uint32_t* s) {
  if constexpr (LAT == kE8) {
    const int32_t cb = c[0] & 1;
    int32_t h[8], p = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) h[i] = (c[i] - cb) >> 1;
#pragma unroll
    for (int i = 0; i < 7; ++i) p += h[i];
    p &= 1;
    const int32_t t = (h[7] - p) >> 1;
#pragma unroll
    for (int i = 0; i < 7; ++i) s[i] = zigzag(h[i]);
    s[7] = 2u * zigzag(t) + (uint32_t)cb;
  } else if constexpr (LAT == kD4) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int32_t* cc = c + 4 * b;
      const int32_t p = (cc[0] + cc[1] + cc[2]) & 1;
      s[4 * b + 0] = zigzag(cc[0]);
      s[4 * b + 1] = zigzag(cc[1]);
      s[4 * b + 2] = zigzag(cc[2]);
      s[4 * b + 3] = zigzag((cc[3] - p) >> 1);
    }
  } else if constexpr (LAT == kA2) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int32_t p = c[2 * b + 1] & 1;
      s[2 * b] = zigzag((c[2 * b] - p) >> 1);
      s[2 * b + 1] = zigzag(c[2 * b + 1]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) s[i] = zigzag(c[i]);
  }
}

// E8 unstrip (Sec. 4.6) in closed form: 2 unzz(s) = s ^ -(s & 1), so
// c_i = 2 h_i + cb = (s_i ^ -(s_i & 1)) + cb for i < 7; h_i = unzz(s_i) has the
// parity of bit 1 ^ bit 0 of s_i, so p = bit 1 ^ bit 0 of the XOR of s_0..s_6;
// s_7 = 2 zz(t) + cb gives 2 t = z ^ -(z & 1) with z = s_7 >> 1, and
// c_7 = 2 (2 t + p) + cb.
__device__ __forceinline__ void e8_unstrip(const uint32_t* s, int32_t* c) {
  const uint32_t cb = s[7] & 1u;
#pragma unroll
  for (int i = 0; i < 7; ++i)
    c[i] = (int32_t)((s[i] ^ (uint32_t)__builtin_amdgcn_sbfe((int32_t)s[i], 0, 1)) + cb);
  const uint32_t X = xor3(xor3(s[0], s[1], s[2]), s[3], s[4]) ^ s[5] ^ s[6];
  const uint32_t p = ((X >> 1) ^ X) & 1u;
  const uint32_t t2 = (s[7] >> 1) ^ (uint32_t)__builtin_amdgcn_sbfe((int32_t)s[7], 1, 1);
  c[7] = (int32_t)((t2 << 1) + ((p << 1) | cb));
}

template <int LAT>
__device__ __forceinline__ void unstrip8(const uint32_t* s, int32_t* c) {
  if constexpr (LAT == kE8) {
    e8_unstrip(s, c);
  } else if constexpr (LAT == kD4) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      int32_t* cc = c + 4 * b;
      cc[0] = unzigzag(s[4 * b + 0]);
      cc[1] = unzigzag(s[4 * b + 1]);
      cc[2] = unzigzag(s[4 * b + 2]);
      cc[3] = 2 * unzigzag(s[4 * b + 3]) + ((cc[0] + cc[1] + cc[2]) & 1);
    }
  } else if constexpr (LAT == kA2) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      c[2 * b + 1] = unzigzag(s[2 * b + 1]);
      c[2 * b] = 2 * unzigzag(s[2 * b]) + (c[2 * b + 1] & 1);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = unzigzag(s[i]);
  }
}

// Rice class of the lane's j-th symbol: D4 codes its halved symbol and A2
// its n_x with a second parameter.
template <int LAT>
__device__ __forceinline__ constexpr int sym_class(int j) {
  return LAT == kD4 ? ((j & 3) == 3) : (LAT == kA2 ? (j & 1) : 0);
}

// Remainder bits of one lane (8 symbols) for parameters k0 (class 0), k1.
template <int LAT>
__device__ __forceinline__ uint32_t lane_rem_bits(uint32_t k0, uint32_t k1) {
  if constexpr (LAT == kD4) return 6 * k0 + 2 * k1;
  if constexpr (LAT == kA2) return 4 * k0 + 4 * k1;
  return 8 * k0;
}

// ----------------------------------------------------------- Walsh-Hadamard

__device__ __forceinline__ void fwht8_inlane(float* v) {
#pragma unroll
  for (int h = 1; h < 8; h <<= 1)
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if ((i & h) == 0) {
        const float a = v[i], b = v[i + h];
        v[i] = a + b;
        v[i + h] = a - b;
      }
}

// Butterfly with lane l ^ M: the lower lane keeps a + b, the upper a - b,
// with a the lower lane's value.  s = +1 (lower) or -1 (upper) makes it one
// exact-multiplier fma: fma(v, s, p) = round(p + s v).
template <int M>
__device__ __forceinline__ void fwht_xlane(float* v, float s) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float p = xor_lane_f<M>(v[j]);
    v[j] = __builtin_fmaf(v[j], s, p);
  }
}

// Per-lane butterfly signs for the cross-lane stages (h = 8, 16, 32, 64).
struct XSigns {
  float f[4];
  __device__ __forceinline__ explicit XSigns(int lane) {
#pragma unroll
    for (int b = 0; b < 4; ++b) f[b] = ((lane >> b) & 1) ? -1.0f : 1.0f;
  }
};

__device__ __forceinline__ void fwht128(float* v, const XSigns& sg) {
  fwht8_inlane(v);
  fwht_xlane<1>(v, sg.f[0]);
  fwht_xlane<2>(v, sg.f[1]);
  fwht_xlane<4>(v, sg.f[2]);
  fwht_xlane<8>(v, sg.f[3]);
}


// The 8 sign bits of columns col0 .. col0 + 7 (col0 a multiple of 8).
__device__ __forceinline__ uint32_t sign_bits8(const uint32_t* mask, int64_t col0) {
  return (mask[col0 >> 5] >> (uint32_t)(col0 & 31)) & 0xFFu;
}

__device__ __forceinline__ float flip(float v, uint32_t bits, int j) {
  return __uint_as_float(__float_as_uint(v) ^ (((bits >> j) & 1u) << 31));
}

// Four fp32 values as OCP E4M3 bytes (v_cvt_pk_fp8_f32: round to nearest
// even), the first in the low byte; the caller keeps them within +-448.
__device__ __forceinline__ uint32_t e4m3x4(float a, float b, float c, float d) {
  const int lo = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);
  return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(c, d, lo, true);
}

// Two values as OCP FP4 E2M1 codes of v / 2^X (magnitudes 0, .5, 1, 1.5, 2, 3,
// 4, 6 as codes 0 .. 7 with the sign in bit 3) in byte SEL of r, the first in
// the low nibble: the nearest value, ties to the even code, saturating at 6,
// the sign kept also when a value rounds to zero.  The instruction's scale
// operand is the float 2^X, of which it takes the exponent field (0 for the
// block exponent -127).  It gives NaN the code of 6: see e2m1_drop_nan.
template <int SEL>
__device__ __forceinline__ uint32_t e2m1_pair(uint32_t r, float a, float b, int32_t X) {
  return __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, a, b, __uint_as_float((uint32_t)(X + 127) << 23), SEL);
}

// Eight values in one word, the first in the lowest nibble.
__device__ __forceinline__ uint32_t e2m1_x8(const float* v, int32_t X) {
  uint32_t r = e2m1_pair<0>(0u, v[0], v[1], X);
  r = e2m1_pair<1>(r, v[2], v[3], X);
  r = e2m1_pair<2>(r, v[4], v[5], X);
  return e2m1_pair<3>(r, v[6], v[7], X);
}

// NaN is cast to a zero of its sign.
template <int N>
__device__ __forceinline__ void e2m1_drop_nan(float* v) {
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = v[i] != v[i] ? __builtin_copysignf(0.0f, v[i]) : v[i];
}

// The largest magnitude of a lane's N values, NaN where one of them is.
template <int N>
__device__ __forceinline__ float amax_or_nan(const float* v) {
  float am = 0.0f;
#pragma unroll
  for (int i = 0; i < N; ++i) am = __builtin_elementwise_maximum(am, __builtin_fabsf(v[i]));
  return am;
}

// The MX block exponent X = floor(log2 amax) - 2 of a block whose largest
// magnitude is amax (E8M0's range; -127 for an all-zero block).
__device__ __forceinline__ int32_t mx_exponent(float amax) {
  if (!(amax > 0.0f)) return -127;
  const int32_t e = __builtin_amdgcn_frexp_expf(amax);  // amax = m 2^e, m in [0.5, 1)
  return max(-127, min(127, e - 3));
}

// Lanes of one wave exchange values through LDS: every lane's earlier LDS
// writes are visible to the others' later reads.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// v <- M v for the tile of the lane's group of 16 (its coordinates
// 8 (lane % 16) + j): the qjl rotation of Sec. 4.2 with M = S (encode) or S^T
// (decode).  Mt is M^T row-major, so row k holds column k of M and a lane's 8
// outputs read 32 contiguous bytes of it per k.  Each output is the
// left-to-right fp32 sum of the rounded products from k = 0, the order the
// oracle defines; v passes through the group's 128 floats of `stage` (LDS).
__device__ __forceinline__ void qjl_tile(const float* __restrict__ Mt, float* stage, int lane,
                                         float* v) {
  float* t = stage + (lane >> 4) * HQ_TILE;
  const int c0 = (lane & 15) * 8;
  *(float4*)(t + c0) = make_float4(v[0], v[1], v[2], v[3]);
  *(float4*)(t + c0 + 4) = make_float4(v[4], v[5], v[6], v[7]);
  wave_lds_sync();
  float acc[8];
  {
    const float z = t[0];
    const float4 a = *(const float4*)(Mt + c0), b = *(const float4*)(Mt + c0 + 4);
    acc[0] = a.x * z; acc[1] = a.y * z; acc[2] = a.z * z; acc[3] = a.w * z;
    acc[4] = b.x * z; acc[5] = b.y * z; acc[6] = b.z * z; acc[7] = b.w * z;
  }
#pragma unroll 4
  for (int k = 1; k < HQ_TILE; ++k) {
    const float z = t[k];
    const float4 a = *(const float4*)(Mt + k * HQ_TILE + c0);
    const float4 b = *(const float4*)(Mt + k * HQ_TILE + c0 + 4);
    acc[0] = acc[0] + a.x * z; acc[1] = acc[1] + a.y * z;
    acc[2] = acc[2] + a.z * z; acc[3] = acc[3] + a.w * z;
    acc[4] = acc[4] + b.x * z; acc[5] = acc[5] + b.y * z;
    acc[6] = acc[6] + b.z * z; acc[7] = acc[7] + b.w * z;
  }
  wave_lds_sync();  // every lane has read the stage before it is written again
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = acc[i];
}

// The same rotation by a whole wave, its four tiles together: lane l forms
// outputs 2 l and 2 l + 1 of every tile, so a row of M^T (512 bytes over the
// wave) is read once for the four tiles and the tiles' k-th values come as one
// broadcast; the sums go back through `stage`.  Each output is the same
// left-to-right sum.  qjl_tile's lanes each load 32 bytes of M^T per k, the
// wave 2 KB, and the 64 bytes a clock at which a CU's cache returns data
// bound it: 2048 x 1024 rows appended in 41.4 us, 27.9 here.  `stage` is 16-byte
// aligned (a kernel's dynamic LDS is declared so): a misaligned b128 read takes
// about 64 cycles instead of 8 (70.6 us).
__device__ __forceinline__ void qjl_wave(const float* __restrict__ Mt, float* stage, int lane, float* v) {
  // z of tile t at stage[4 k + t]
  const int t0 = lane >> 4, c0 = (lane & 15) * 8;
#pragma unroll
  for (int i = 0; i < 8; ++i) stage[4 * (c0 + i) + t0] = v[i];
  wave_lds_sync();
  float acc[4][2];
  {
    const float2 m = *(const float2*)(Mt + 2 * lane);
    const float4 z = *(const float4*)stage;
    acc[0][0] = m.x * z.x; acc[0][1] = m.y * z.x;
    acc[1][0] = m.x * z.y; acc[1][1] = m.y * z.y;
    acc[2][0] = m.x * z.z; acc[2][1] = m.y * z.z;
    acc[3][0] = m.x * z.w; acc[3][1] = m.y * z.w;
  }
#pragma unroll 4  // eight take 22 more registers and cost the other rotations waves
  for (int k = 1; k < HQ_TILE; ++k) {
    const float2 m = *(const float2*)(Mt + k * HQ_TILE + 2 * lane);
    const float4 z = *(const float4*)(stage + 4 * k);
    acc[0][0] = acc[0][0] + m.x * z.x; acc[0][1] = acc[0][1] + m.y * z.x;
    acc[1][0] = acc[1][0] + m.x * z.y; acc[1][1] = acc[1][1] + m.y * z.y;
    acc[2][0] = acc[2][0] + m.x * z.z; acc[2][1] = acc[2][1] + m.y * z.z;
    acc[3][0] = acc[3][0] + m.x * z.w; acc[3][1] = acc[3][1] + m.y * z.w;
  }
  wave_lds_sync();
#pragma unroll
  for (int t = 0; t < 4; ++t) *(float2*)(stage + t * HQ_TILE + 2 * lane) = make_float2(acc[t][0], acc[t][1]);
  wave_lds_sync();
  const float4 a = *(const float4*)(stage + t0 * HQ_TILE + c0), b = *(const float4*)(stage + t0 * HQ_TILE + c0 + 4);
  wave_lds_sync();  // every lane has read the stage before it is written again
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// ------------------------------------------------------------ look-back scan
// Decoupled look-back (Merrill & Garland, 2016) over workgroups in index
// order.  Workgroups are dispatched in increasing index order, and a group
// only ever waits for lower indices, so every wait ends; each wait is also
// bounded, and a status that never arrives ends the wait with an error
// status instead of a hang.  The scan scratch starts with a 64-bit epoch word
// that the last workgroup of a launch advances after it has published its
// inclusive prefix (by then every group has read the epoch, since that prefix
// sums every group's published aggregate), so every launch -- also a
// replayed graph -- gets a fresh epoch without host help.  A status word
// packs the value (32 bits: words since the start of this launch), a flag
// (2 bits: 1 = aggregate, 2 = inclusive prefix) and the epoch (30 bits), so
// the array never needs clearing.

constexpr uint32_t kEpochMask = 0x3FFFFFFFu;
constexpr uint32_t kSpinLimit = 1u << 24;

__device__ __forceinline__ unsigned long long pack_status(uint32_t epoch, uint32_t flag,
                                                          uint32_t value) {
  return ((unsigned long long)(epoch & kEpochMask) << 34) | ((unsigned long long)flag << 32) |
         (unsigned long long)value;
}

// Relaxed is enough: a status word carries its own value, and no other data
// published by the workgroup is read through it.
__device__ __forceinline__ void store_status(unsigned long long* p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ unsigned long long load_status(unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------ bit assembly

// OR the 64 bits of v into the LDS bit array at bit position pos.
__device__ __forceinline__ void or_bits64(uint32_t* buf, uint32_t pos, uint64_t v) {
  if (v == 0) return;
  const uint32_t w = pos >> 5, sh = pos & 31u;
  const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  const uint32_t o0 = lo << sh;
  const uint32_t o1 = sh ? ((hi << sh) | (lo >> (32u - sh))) : hi;
  const uint32_t o2 = sh ? (hi >> (32u - sh)) : 0u;
  if (o0) atomicOr(&buf[w], o0);
  if (o1) atomicOr(&buf[w + 1], o1);
  if (o2) atomicOr(&buf[w + 2], o2);
}

// 64 bits of the LDS bit array starting at bit pos (words past nw read 0).
__device__ __forceinline__ uint64_t load_bits64(const uint32_t* buf, uint32_t pos, uint32_t nw) {
  const uint32_t w = pos >> 5, sh = pos & 31u;
  const uint32_t a = w < nw ? buf[w] : 0u;
  const uint32_t b = w + 1 < nw ? buf[w + 1] : 0u;
  const uint32_t c = w + 2 < nw ? buf[w + 2] : 0u;
  const uint32_t lo = sh ? ((a >> sh) | (b << (32u - sh))) : a;
  const uint32_t hi = sh ? ((b >> sh) | (c << (32u - sh))) : b;
  return ((uint64_t)hi << 32) | lo;
}

// Bit offset of field j inside a lane's remainder region.
template <int LAT>
__device__ __forceinline__ uint32_t rem_offset(int j, uint32_t k0, uint32_t k1) {
  if constexpr (LAT == kD4) {
    return (uint32_t)(j >> 2) * (3u * k0 + k1) + (uint32_t)(j & 3) * k0;
  } else if constexpr (LAT == kA2) {
    return (uint32_t)(j >> 1) * (k0 + k1) + (uint32_t)(j & 1) * k0;
  } else {
    return (uint32_t)j * k0;
  }
}

// ------------------------------------------------------------ twisted FWHT
// A cross-lane butterfly written as one multiply-add per value,
//   u <- u + s * u[l ^ M]      (s = +1 on the lower lane, -1 on the upper),
// leaves the lower lane a + b and the upper lane b - a = -(a - b): the
// butterfly output times s, rounded identically (round-to-nearest-even
// commutes with negation).  The partner lane of a stage shares the signs of
// every earlier stage, so earlier factors pull out of the butterfly and four
// chained stages leave each lane its outputs times sigma, the product of its
// four stage signs.  Callers fold sigma into the per-tile factor that
// follows.  The h = 8, 16, 64 stages are one DPP-fused v_fmac each
// (quad_perm and row_ror lane moves); the h = 32 stage (lane l ^ 4) reads
// its partner through ds_swizzle.

#define HQ_DPP_FULL "row_mask:0xf bank_mask:0xf bound_ctrl:1"
// v[j] += s * v[partner lane][j] for the 8 values of a lane; the s_nop pairs
// cover the two wait states between a VALU write and a DPP read of a VGPR.
#define HQ_FMAC_DPP8(CTRL, v, s)                                                            \
  asm("s_nop 1\n\t"                                                                         \
      "v_fmac_f32_dpp %0, %0, %8 " CTRL " " HQ_DPP_FULL "\n\t"                              \
      "v_fmac_f32_dpp %1, %1, %8 " CTRL " " HQ_DPP_FULL "\n\t"                              \
      "v_fmac_f32_dpp %2, %2, %8 " CTRL " " HQ_DPP_FULL "\n\t"                              \
      "v_fmac_f32_dpp %3, %3, %8 " CTRL " " HQ_DPP_FULL "\n\t"                              \
      "v_fmac_f32_dpp %4, %4, %8 " CTRL " " HQ_DPP_FULL "\n\t"                              \
      "v_fmac_f32_dpp %5, %5, %8 " CTRL " " HQ_DPP_FULL "\n\t"                              \
      "v_fmac_f32_dpp %6, %6, %8 " CTRL " " HQ_DPP_FULL "\n\t"                              \
      "v_fmac_f32_dpp %7, %7, %8 " CTRL " " HQ_DPP_FULL "\n\t"                              \
      "s_nop 1"                                                                             \
      : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), \
        "+v"(v[7])                                                                          \
      : "v"(s))

// Value of lane l ^ 4 (ds_swizzle bit-mask mode: and 0x1F, or 0, xor 4).
__device__ __forceinline__ float swz_xor4(float v) {
  return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x101F));
}

// Value of lane l ^ 16 (the same mode with xor 16) and of lane l ^ 32.
__device__ __forceinline__ float swz_xor16(float v) {
  return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x401F));
}
__device__ __forceinline__ float lane_xor32(float v) {
  return __int_as_float(__shfl_xor(__float_as_int(v), 32, 64));
}



// Value of lane l ^ M for M = 1, 2, 8 (bound_ctrl DPP moves, which fold into
// the consuming VOP2 instruction).
template <int M>
__device__ __forceinline__ float dpp_xor(float v) {
  constexpr int ctrl = M == 1 ? kDppQuadXor1 : (M == 2 ? kDppQuadXor2 : kDppRowRor8);
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), ctrl, 0xF, 0xF, true));
}

// MXFP4 of a wave's values, eight a lane, 32-blocks of four neighbouring lanes:
// the lane's word of codes and its block's X.  The test for NaN stands behind
// the cast, which it repeats without it: before it, or once behind all blocks
// of a row, it cost the prep of some row lengths 7 to 11 %.
__device__ __forceinline__ uint32_t mxfp4_x8(float* v, int32_t& X) {
  const float am0 = amax_or_nan<8>(v);
  auto cast = [&](float am) {
    am = __builtin_fmaxf(am, dpp_xor<1>(am));
    am = __builtin_fmaxf(am, dpp_xor<2>(am));
    X = mx_exponent(am);
    return e2m1_x8(v, X);
  };
  uint32_t r = cast(am0);
  if (__builtin_expect(__ballot(am0 != am0) != 0ull, 0)) {
    e2m1_drop_nan<8>(v);
    r = cast(amax_or_nan<8>(v));
  }
  return r;
}

// Stage signs of a lane (h = 8, 16, 32, 64 <-> lane bits 0..3) and sigma's
// sign bit.
struct TwSigns {
  float f[4];
  uint32_t sigma;  // 0 or 0x80000000
  __device__ __forceinline__ explicit TwSigns(int lane) {
#pragma unroll
    for (int b = 0; b < 4; ++b) f[b] = ((lane >> b) & 1) ? -1.0f : 1.0f;
    sigma = (uint32_t)(__popc((uint32_t)lane & 15u) & 1) << 31;
    // kept in registers for the whole kernel rather than recomputed from
    // the lane index before every transform
#pragma unroll
    for (int b = 0; b < 4; ++b) asm volatile("" : "+v"(f[b]));
    asm volatile("" : "+v"(sigma));
  }
};

// v = sigma * (H v) over the tile (in-lane stages h = 1, 2, 4 first).
__device__ __forceinline__ void fwht128_tw(float* v, const TwSigns& sg) {
  fwht8_inlane(v);
  HQ_FMAC_DPP8("quad_perm:[1,0,3,2]", v, sg.f[0]);
  HQ_FMAC_DPP8("quad_perm:[2,3,0,1]", v, sg.f[1]);
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = __builtin_fmaf(swz_xor4(v[j]), sg.f[2], v[j]);
  HQ_FMAC_DPP8("row_ror:8", v, sg.f[3]);
}

// ------------------------------------------------------------ transform on the matrix cores
// A plain weight plan's codes are integers, so its inverse transform is exact
// in any order, and 32 of a tile's 128 points fit one matrix-core step: with
// lane l holding block (l & 3) | (l >> 4) << 2 of tile (l >> 2) & 3, the lane's 8
// coordinates and the lanes l, l + 16, l + 32, l + 48 make the K index
// 8 (l / 16) + j of v_mfma_f32_16x16x32_f16's B operand, column l % 16.  The A
// operand is H32 with its rows in the order that returns every sum to the
// lane layout it came from (row 4 g' + r of product h is coordinate 4 h + r
// of lane group g'), and the blocks' two low index bits remain, as two DPP
// butterflies.  The codes enter as 1536 + c in fp16 (exact for |c| < 512: one
// shift-and-add per pair); the bias shows only in the all-ones row, where the
// C operand takes 32 * 1536 away.  All values are integers below 2^24: exact.
// Against the seven-stage transform on the VALU (integer conversions, 24 adds,
// 32 cross-lane multiply-adds) it leaves 16 cross-lane ones.
typedef _Float16 v8h_t __attribute__((ext_vector_type(8)));
typedef float v4f_t __attribute__((ext_vector_type(4)));
typedef uint32_t v4u_t __attribute__((ext_vector_type(4)));
constexpr uint32_t kCodeBias = 0x66006600u;  // 1536 in each fp16 half

struct MfmaRht {
  v4u_t a0, a1;  // the two products' A rows, fp16 +-1 pairs
  v4f_t c0;      // C of product 0
  float f[2];    // stage signs of the lane's block bits 0 and 1
  uint32_t sigma;
  __device__ __forceinline__ explicit MfmaRht(int lane) {
    const uint32_t r = lane & 3, go = (lane >> 2) & 3, gi = (uint32_t)lane >> 4;
    const uint32_t s = __popc(gi & go) & 1u;
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // K values j = 2 i and 2 i + 1: sign (-1)^(popc(j & r) + s)
      const uint32_t lo = (__popc((2 * i) & r) + s) & 1u, hi = (__popc((2 * i + 1) & r) + s) & 1u;
      w[i] = 0x3C003C00u ^ (lo << 15) ^ (hi << 31);
    }
    a0 = (v4u_t){w[0], w[1], w[2], w[3]};
    a1 = (v4u_t){w[0], w[1], w[2] ^ 0x80008000u, w[3] ^ 0x80008000u};  // coordinate bit 2 set
    c0 = (v4f_t){lane < 16 ? -32.0f * 1536.0f : 0.0f, 0.0f, 0.0f, 0.0f};
    f[0] = (lane & 1) ? -1.0f : 1.0f;
    f[1] = (lane & 2) ? -1.0f : 1.0f;
    sigma = (uint32_t)(__popc((uint32_t)lane & 3u) & 1) << 31;
    // kept in registers for the whole kernel
    asm volatile("" : "+v"(a0), "+v"(a1), "+v"(c0), "+v"(f[0]), "+v"(f[1]), "+v"(sigma));
  }
  // y = sigma * (H c) for |c| < 512, c given as biased fp16 pairs.
  __device__ __forceinline__ void small(const uint32_t (&pair)[4], float* y) const {
    const v8h_t b = __builtin_bit_cast(v8h_t, (v4u_t){pair[0], pair[1], pair[2], pair[3]});
    v4f_t lo = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h_t, a0), b, c0, 0, 0, 0);
    v4f_t hi = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h_t, a1), b, (v4f_t){}, 0, 0, 0);
    // stages() reads the results in inline assembly, and the compiler does not
    // look into assembly for the 8 wait states behind a matrix instruction of
    // four passes: they stand here
    asm volatile("s_nop 7" : "+v"(lo), "+v"(hi));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      y[j] = lo[j];
      y[4 + j] = hi[j];
    }
    stages(y);
  }
  // The same for any code, on the VALU.
  __device__ __forceinline__ void any(float* y, int lane) const {
    fwht8_inlane(y);
    const float s4 = (lane & 16) ? -1.0f : 1.0f, s5 = (lane & 32) ? -1.0f : 1.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) y[j] = __builtin_fmaf(y[j], s4, swz_xor16(y[j]));
#pragma unroll
    for (int j = 0; j < 8; ++j) y[j] = __builtin_fmaf(y[j], s5, lane_xor32(y[j]));
    stages(y);
  }
  __device__ __forceinline__ void stages(float* y) const {
    HQ_FMAC_DPP8("quad_perm:[1,0,3,2]", y, f[0]);
    HQ_FMAC_DPP8("quad_perm:[2,3,0,1]", y, f[1]);
  }
};

// Tiles longer than 128 (Sec. 7.2 sweeps 128 .. 2048).  A wave holds four
// consecutive sub-streams of 512 scalars, lane l coordinates 8 l .. 8 l + 7
// of each, so a tile of n <= 512 spans n / 8 lanes of one sub-stream and a
// longer one spans n / 512 whole sub-streams of the wave.  The transform's
// stages h = 128 and 256 pair lanes l ^ 16 and l ^ 32 (twisted as the
// h = 8 .. 64 stages, which multiplies sigma by the two lane signs); the
// stages h = 512 and 1024 pair sub-streams i ^ 1 and i ^ 2 of the same lane,
// plain butterflies (both operands carry the lane's sigma).  Returns the
// sign bit of the lane's sigma.
__device__ __forceinline__ uint32_t fwht_tiled(float (*x)[8], int lane, uint32_t tile,
                                               const TwSigns& sg) {
  uint32_t sigma = sg.sigma;
#pragma unroll
  for (int i = 0; i < 4; ++i) fwht128_tw(x[i], sg);
  if (tile >= 256u) {
    const float s4 = (lane & 16) ? -1.0f : 1.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 8; ++j) x[i][j] = __builtin_fmaf(swz_xor16(x[i][j]), s4, x[i][j]);
    sigma ^= (uint32_t)(lane & 16) << 27;
  }
  if (tile >= 512u) {
    const float s5 = (lane & 32) ? -1.0f : 1.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 8; ++j) x[i][j] = __builtin_fmaf(lane_xor32(x[i][j]), s5, x[i][j]);
    sigma ^= (uint32_t)(lane & 32) << 26;
  }
  if (tile >= 1024u) {
#pragma unroll
    for (int i = 0; i < 4; i += 2)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float a = x[i][j], b = x[i + 1][j];
        x[i][j] = a + b;
        x[i + 1][j] = a - b;
      }
  }
  if (tile >= 2048u) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float a = x[i][j], b = x[i + 2][j];
        x[i][j] = a + b;
        x[i + 2][j] = a - b;
      }
  }
  return sigma;
}

__device__ __forceinline__ float xor_sign(float v, uint32_t bit) {
  return __uint_as_float(__float_as_uint(v) ^ bit);
}

// --------------------------------------------------- E8 decision in closed form
// The decision works on w = z / 2 (the encoder's scale carries the factor
// 1/2, which is exact), where the two classes of the 2E8 realization are the
// integer points with even sum (D8 / 2) and that set shifted by 1/2.  With
// k_i = rint(w_i), ea_i = w_i - k_i (exact, |ea_i| <= 1/2), the nearest
// point of the shifted class takes floor(w_i) + 1/2 per coordinate, at
// distance 1/2 - |ea_i|.  Before the parity fixes
// sum(ea^2) - sum(eb^2) = sum(|ea_i| - 1/4); a fix moves one coordinate by 1,
// adding 1 - 2 max|ea| (first class) or 2 min|ea| (second) to its distance.
// In quarters of the full-scale difference:
//   D = sum|ea_i| - 2 + [odd_a] (1 - 2 max|ea|) - [odd_b] 2 min|ea|,
// odd_a the parity of sum k_i and odd_b that of sum floor(w_i), which differs
// from odd_a by the number of negative ea_i (the parity of the XOR of their
// sign bits).  Rounding moves the fp32 sums by far less than kE8Tie / 4, so
// a lane outside the band takes the same class as the two-sum comparison; a
// wave with any lane inside it runs quant_e8 step by step on z = 2 w.
//
// The chosen point, as h = (c - cb) / 2 (the stripped coordinates), is
// k_i for the first class and floor(w_i) = k_i - [ea_i < 0] for the second,
// plus the parity fix: +-1 on the first coordinate of largest error.  That
// error is |ea_i| in the first class and fl(1/2 - |ea_i|) in the second
// (fp32 w - (floor(w) + 1/2) has that magnitude with the reference's
// rounding), and the fix moves towards w: +1 when ea_j >= 0 (first class),
// +1 when ea_j < 0 (second; a coordinate with ea_j = +1/2 would move +1 too,
// so min|ea| = 1/2 also takes the step-by-step path).  Every +-1 is a lane
// mask folded into an add or subtract with carry.

constexpr float kE8Tie = 1.0e-3f;  // band on the full-scale distance difference

// x + carry-in / x - borrow-in, the carry a lane mask (bit l for lane l) that
// scalar logic made: straight from a vector compare it would need two wait
// states, which the compiler does not keep before inline assembly.
__device__ __forceinline__ int32_t add_lanemask(int32_t x, uint64_t m) {
  int32_t r;
  uint64_t co;
  asm("v_addc_co_u32_e64 %0, %1, %2, 0, %3" : "=v"(r), "=s"(co) : "v"(x), "s"(m));
  return r;
}
__device__ __forceinline__ int32_t sub_lanemask(int32_t x, uint64_t m) {
  int32_t r;
  uint64_t co;
  asm("v_subb_co_u32_e64 %0, %1, %2, 0, %3" : "=v"(r), "=s"(co) : "v"(x), "s"(m));
  return r;
}


// The class decision of a block inside the tie band, exactly as the
// step-by-step procedure takes it: the two classes' squared distances in
// fp32 (z units, z = 2 w), each error rebuilt exactly from ea = w - rint(w).
// The first class's error on coordinate i is 2 ea_i, and its parity fix
// (the first coordinate of largest |ea|) leaves 2 (1 - |ea_j|) in magnitude;
// the second class's is 2 (1/2 - |ea_i|), and its fix (the first coordinate
// of largest 1/2 - |ea|) leaves 2 (|ea_j| + 1/2).  Every doubling is exact,
// so each value is the procedure's own rounding; the squares are summed in
// its tree order, and the first class wins ties.
__device__ __forceinline__ bool e8_even_exact(const float* ea, float mx, float mn, bool odd_a,
                                              bool odd_b) {
  const float topb = 0.5f - mn;
  bool fixa = odd_a, fixb = odd_b;
  float sa[8], sb[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float a = __builtin_fabsf(ea[i]);
    float ua = a, ub = 0.5f - a;
    if (fixa && a == mx) {
      ua = 1.0f - a;
      fixa = false;
    }
    if (fixb && ub == topb) {
      ub = a + 0.5f;
      fixb = false;
    }
    ua = ua + ua;
    ub = ub + ub;
    sa[i] = ua * ua;
    sb[i] = ub * ub;
  }
  return tree8(sa) <= tree8(sb);
}

__device__ __forceinline__ void e8_nearest(const float* w, int32_t* h, int32_t& cb) {
  float ea[8];
  int32_t K[8];
  uint32_t eb[8];
  // rint(w) by the shift 1.5 * 2^23: for |w| < 2^22 (the scale bounds |w| by
  // alpha sqrt(128) / 2) the sum lies in [2^23, 2^24), where the fp32
  // spacing is 1, so it rounds w to the nearest integer, ties to even (the
  // shift is even); the integer is the sum's bit pattern less the shift's.
  // Four fast-rate adds instead of a rounding and a conversion.
  // ea = w + (shift - t) = w - rint(w), exact; written as a sum so that it is
  // never -0 (w = -0, which the signed scale makes of an exact zero, gives
  // -0 + +0 = +0, where w - rint(w) would give -0): the parity below reads
  // the sign bits of ea, the rounding the sign of its value, and the two
  // must agree.
  constexpr float kShift = 12582912.0f;  // 1.5 * 2^23, bits 0x4B400000
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float t = w[i] + kShift;
    const float nk = kShift - t;
    ea[i] = w[i] + nk;
    K[i] = (int32_t)(__float_as_uint(t) - 0x4B400000u);
    eb[i] = __float_as_uint(ea[i]);
  }
  float Sabs = __builtin_fabsf(ea[0]) + __builtin_fabsf(ea[1]);
#pragma unroll
  for (int i = 2; i < 8; ++i) Sabs += __builtin_fabsf(ea[i]);
  float mx = __builtin_fabsf(ea[0]), mn = mx;
#pragma unroll
  for (int i = 1; i < 8; ++i) {
    mx = __builtin_fmaxf(mx, __builtin_fabsf(ea[i]));
    mn = __builtin_fminf(mn, __builtin_fabsf(ea[i]));
  }
  // parities: sum k_i (low bits of the XOR) and the count of negative ea_i
  const uint32_t kp = xor3(xor3(xor3((uint32_t)K[0], (uint32_t)K[1], (uint32_t)K[2]), (uint32_t)K[3],
                                (uint32_t)K[4]),
                           (uint32_t)K[5], (uint32_t)K[6]) ^ (uint32_t)K[7];
  const uint32_t sx = xor3(xor3(xor3(eb[0], eb[1], eb[2]), eb[3], eb[4]), eb[5], eb[6]) ^ eb[7];
  const bool odd_a = kp & 1u;
  const bool odd_b = ((kp << 31) ^ sx) >> 31;
  const float D0 = Sabs - 2.0f;
  const float D1 = odd_a ? __builtin_fmaf(-2.0f, mx, Sabs - 1.0f) : D0;
  const float D = odd_b ? __builtin_fmaf(-2.0f, mn, D1) : D1;
  bool even = D < 0.0f;
  // Inside the tie band (or with every |ea_i| = 1/2, where the second
  // class's fix moves up from ea_j = +1/2 too) the lane takes the exact
  // decision; a wave with no such lane skips it.
  const bool tie = __builtin_fabsf(D) <= 0.25f * kE8Tie || mn >= 0.5f;
  const bool any_tie = __ballot(tie) != 0ull;
  if (any_tie && tie) even = e8_even_exact(ea, mx, mn, odd_a, odd_b);
  // lane masks: the class, whether its parity needs the fix, and per
  // coordinate the largest-error hits and the sign of ea.  The error of
  // coordinate i in the lane's class is key_i = fma(|ea_i|, +-1, 0 or 1/2):
  // |ea_i| (exact) in the first class, fl(1/2 - |ea_i|) (one rounding, as
  // the subtraction) in the second; its largest value is mx or fl(1/2 - mn).
  const uint64_t E = __ballot(even);
  const uint64_t need = (E & __ballot(odd_a)) | (~E & __ballot(odd_b));
  const float ks = even ? 1.0f : -1.0f, kc = even ? 0.0f : 0.5f;
  const float top = even ? mx : 0.5f - mn;
  uint64_t done = ~need;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint64_t hit = __ballot(__builtin_fmaf(__builtin_fabsf(ea[i]), ks, kc) == top);
    const uint64_t fix = hit & ~done;
    done |= hit;
    const uint64_t neg = __ballot(ea[i] < 0.0f);
    // up by the fix where the class and the sign agree to move up; down by
    // the fix otherwise, or by the odd class's floor (never both)
    const uint64_t t = E ^ neg;
    const uint64_t up = fix & t;
    const uint64_t down = (fix & ~t) | (neg & ~E);
    h[i] = sub_lanemask(add_lanemask(K[i], up), down);
  }
  // every |ea_i| = 1/2: the second class wins and its fix (coordinate 0)
  // moves up also from ea_0 = +1/2, where the masks above moved it down
  if (any_tie && mn >= 0.5f && !even && odd_b && ea[0] > 0.0f) h[0] += 2;
  cb = even ? 0 : 1;
}

// E8 strip (Sec. 4.6) from h = (c - cb) / 2: s_i = zz(h_i) for i < 7,
// s_7 = 2 zz(t) + cb with t = (h_7 - p) / 2 and p the parity of
// h_0 + .. + h_6.
__device__ __forceinline__ void e8_strip(const int32_t* h, int32_t cb, uint32_t* s) {
#pragma unroll
  for (int i = 0; i < 7; ++i) s[i] = zigzag(h[i]);
  const uint32_t p = xor3(xor3((uint32_t)h[0], (uint32_t)h[1], (uint32_t)h[2]), (uint32_t)h[3],
                          (uint32_t)h[4]) ^ (uint32_t)h[5] ^ (uint32_t)h[6];
  const int32_t t = (h[7] - (int32_t)(p & 1u)) >> 1;
  s[7] = 2u * zigzag(t) + (uint32_t)cb;
}

// ------------------------------------------------------------ decode kernel
// Rice decode of one sub-stream per wave: the remainder fields are at fixed
// positions; the unary terminators are located by per-word popcounts, a
// wave prefix sum and a select inside the word that holds terminator 8 l - 1.
// Lane l then reads its 8 codes from a 32-bit window at that position (the
// common case: its codes span at most 32 bits), clearing one terminator per
// code; a lane whose codes run past the window walks a 64-bit window that
// slides along the bit array.  Each wave only touches its own LDS region.
// MODE 0: fp32 out, 1: bf16 out, 2: int8 lattice codes and per-tile g (no
// inverse RHT).

__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Bits [pos, pos + 32) of the LDS bit array (the word after the last one
// read must exist).
__device__ __forceinline__ uint32_t bits32_at(const uint32_t* buf, uint32_t pos) {
  const uint32_t w = pos >> 5;
  return __builtin_amdgcn_alignbit(buf[w + 1], buf[w], pos & 31u);
}

// One sub-stream's table entry, checked against the buffers, and its first
// 128 payload words (two per lane): loaded one sub-stream ahead of its decode.
struct DecHead {
  uint32_t start, kb, W, R;  // wave-uniform
  bool ok;                   // entry within bounds (wave-uniform)
  uint32_t w0, w1;           // payload words lane and lane + 64
};

template <int LAT>
__device__ __forceinline__ DecHead dec_head(const hq_decode_args& A, bool active, uint32_t start,
                                            uint32_t end, uint32_t kb, int lane) {
  DecHead h;
  const uint32_t k0 = (LAT == kA2) ? (kb & 15u) : kb;
  const uint32_t k1 = (LAT == kA2) ? (kb >> 4) : (LAT == kD4 ? (k0 > 0 ? k0 - 1 : 0) : k0);
  h.start = start;
  h.kb = kb;
  h.W = end - start;
  h.R = 64 * lane_rem_bits<LAT>(k0, k1);
  h.ok = active && end >= start && (int64_t)end <= A.cap_words && h.W <= A.lds_words &&
         k0 <= HQ_KMAX && h.R <= 32u * h.W;
  // a raw buffer of the sub-stream's words: lanes past its end read zero, with
  // no per-lane branch
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(A.payload + start), (short)0, h.ok ? (int)(4u * h.W) : 0, 0x00020000);
  h.w0 = __builtin_amdgcn_raw_buffer_load_b32(rs, lane * 4, 0, 0);
  h.w1 = __builtin_amdgcn_raw_buffer_load_b32(rs, lane * 4 + 256, 0, 0);
  return h;
}

// Position (0..31) of the r-th set bit (r from 0, r < popc(w)) of w: the byte
// by halving, the bit from the table.
__device__ __forceinline__ uint32_t select32_half(uint32_t w, uint32_t r, const uint32_t* tbl) {
  const uint32_t c = __popc(w & 0xFFFFu);
  const bool hi = r >= c;
  const uint32_t v = hi ? w >> 16 : w & 0xFFFFu;
  r = hi ? r - c : r;
  const uint32_t c8 = __popc(v & 0xFFu);
  const bool up = r >= c8;
  const uint32_t byte = up ? v >> 8 : v & 0xFFu;
  r = up ? r - c8 : r;
  return (hi ? 16u : 0u) + (up ? 8u : 0u) + __builtin_amdgcn_ubfe(tbl[byte & 0xFFu], 4 * r, 3);
}

// decode_symbols' general path, for group `grp` of a sub-stream of Wl words
// already in `buf`: any code length, corrupt sub-streams too.  `known` (wave-
// uniform): the group's codes start at `pos`, else it is searched.  A corrupt
// sub-stream (any lane's parse failed) decodes as all-zero symbols in every
// lane; callers drop its factor too.
template <int LAT>
__device__ __forceinline__ bool decode_symbols_general(bool ok, uint32_t Wl, uint32_t R, uint32_t k0,
                                                       uint32_t k1, int lane, uint32_t grp, bool known,
                                                       uint32_t pos, const uint32_t* buf, uint32_t* starts,
                                                       uint32_t* sym) {
  const uint32_t lrem = lane_rem_bits<LAT>(k0, k1);
  if (!known) {
    wave_sync_lds();
    starts[lane] = (lane == 0) ? R : 0xFFFFFFFFu;
    wave_sync_lds();
    // unary terminators: popcount prefix over the unary words, then the start
    // of each group's codes (just past terminator 8 j - 1)
    const uint32_t uw0 = R >> 5;
    const uint32_t nuw = ok ? Wl - uw0 : 0u;
    uint32_t carry = 0;
    for (uint32_t base = 0; base < nuw; base += 64) {
      const uint32_t wi = base + lane;
      const uint32_t v = (wi < nuw) ? buf[uw0 + wi] : 0u;
      const uint32_t cnt = __popc(v);
      const uint32_t incl = wave_scan_incl(cnt);
      const uint32_t P = carry + incl - cnt;
      for (uint32_t t = (P & ~7u) + 7u; t < P + cnt; t += 8u) {
        const uint32_t j = (t + 1u) >> 3;
        if (j < 64u) starts[j] = (uw0 + wi) * 32u + select32(v, t - P) + 1u;
      }
      carry += __builtin_amdgcn_readlane(incl, 63);
    }
    wave_sync_lds();
    pos = starts[grp];
  }

  // lane's 8 quotients
  const uint32_t nbits = 32u * Wl;
  ok = ok && pos < nbits;
  uint32_t qv[8];
  bool fast = false;
  if (ok) {
    // q_j = the zeros before the next terminator: shift the window past
    // each code (all 8 terminators lie inside it on this path, so every
    // shift is below 32; otherwise the values are discarded below)
    const uint32_t win = bits32_at(buf, pos);
    fast = __popc(win) >= 8;
    uint32_t sh = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      qv[j] = (uint32_t)__builtin_ctz(win >> sh);
      sh += qv[j] + 1u;
    }
  }
  if (ok && !fast) {
    // the codes run past 32 bits: a 64-bit window sliding along the array
    uint64_t win = load_bits64(buf, pos, Wl);
    uint32_t valid = 64;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      uint32_t q = 0;
      while (ok && win == 0ull) {
        q += valid;
        pos += valid;
        if (pos >= nbits) {
          ok = false;
          break;
        }
        win = load_bits64(buf, pos, Wl);
        valid = 64;
      }
      const uint32_t lo = (uint32_t)win, hi = (uint32_t)(win >> 32);
      const uint32_t tz =
          lo ? (uint32_t)__builtin_ctz(lo) : 32u + (uint32_t)__builtin_ctz(hi | (hi == 0u));
      q += tz;
      pos += tz + 1;
      valid -= tz + 1;
      win = (tz >= 63u) ? 0ull : (win >> (tz + 1));
      qv[j] = q;
    }
  }
  // lane's 8 remainders (fields at fixed positions)
  const uint32_t rpos = __umul24(grp, lrem);  // lrem < 2^24
  if (lrem <= 32) {
    const uint32_t acc = (ok && lrem) ? bits32_at(buf, rpos) : 0u;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t kk = sym_class<LAT>(j) ? k1 : k0;
      sym[j] = (qv[j] << kk) | __builtin_amdgcn_ubfe(acc, rem_offset<LAT>(j, k0, k1), kk);
    }
  } else if (lrem <= 64) {
    const uint64_t acc = ok ? ((uint64_t)bits32_at(buf, rpos + 32) << 32) | bits32_at(buf, rpos) : 0ull;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t kk = sym_class<LAT>(j) ? k1 : k0;
      const uint32_t r = (uint32_t)(acc >> rem_offset<LAT>(j, k0, k1)) & ((1u << kk) - 1u);
      sym[j] = (qv[j] << kk) | r;
    }
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t kk = sym_class<LAT>(j) ? k1 : k0;
      const uint32_t r = ok ? (uint32_t)load_bits64(buf, rpos + rem_offset<LAT>(j, k0, k1), Wl) : 0u;
      sym[j] = (qv[j] << kk) | (r & ((1u << kk) - 1u));
    }
  }
  // a corrupt sub-stream (any lane's parse failed) decodes as all-zero
  // symbols in every lane; callers drop its factor too
  if (__ballot(!ok) != 0ull) {
#pragma unroll
    for (int j = 0; j < 8; ++j) sym[j] = 0u;
  }
  return ok;
}

// LDS byte address of a pointer into shared memory.
__device__ __forceinline__ uint32_t lds_addr(const uint32_t* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint32_t*)p;
}

// a[OFF / 4] = v in the lanes where n > N, without a branch around the store.
template <int N>
__device__ __forceinline__ void store_slot(uint32_t a, uint32_t v, int32_t n) {
  uint64_t saved;
  asm volatile(
      "v_cmp_lt_i32 vcc, %4, %3\n\t"
      "s_and_saveexec_b64 %0, vcc\n\t"
      "ds_write_b32 %1, %2 offset:%5\n\t"
      "s_mov_b64 exec, %0"
      : "=&s"(saved)
      : "v"(a), "v"(v), "v"(n), "n"(N), "n"(4 * N)
      : "vcc", "scc", "memory");
}

// The 8 symbols of group `grp` (0 .. 63, a permutation of the lanes) of a
// sub-stream, into sym; returns the lanes whose parse failed (wave-uniform;
// any: the sub-stream is corrupt and every symbol is zero).  Almost every
// sub-stream takes a path with no per-lane branch: it fits the 128 words of
// its head, its unary codes at most 64, at least 512 terminators are there
// (so every group's codes exist and end), every group's 8 codes lie in 32
// bits and its remainders too.  `small` (wave-uniform) then says that every
// symbol is below 25 2^k with k <= 4.  The others, corrupt ones among them, go
// through decode_symbols_general.
template <int LAT>
__device__ __forceinline__ unsigned long long decode_symbols(const hq_decode_args& A, const DecHead& h, int lane,
                                                             uint32_t grp, uint32_t* buf, uint32_t* starts,
                                                             const uint32_t* seltbl, uint32_t* sym, bool& small) {
  const uint32_t kb = h.kb;
  const uint32_t k0 = (LAT == kA2) ? (kb & 15u) : kb;
  const uint32_t k1 = (LAT == kA2) ? (kb >> 4) : (LAT == kD4 ? (k0 > 0 ? k0 - 1 : 0) : k0);
  const uint32_t lrem = lane_rem_bits<LAT>(k0, k1);
  const uint32_t R = h.R;
  const uint32_t Wl = h.ok ? h.W : 0u;
  const uint32_t uw0 = R >> 5;
  small = false;
  bool known = false;
  uint32_t pos = 0;
  // lds_words >= 62: the wave's region holds 128 words (66 follow its buffer)
  if (h.ok && Wl <= 126u && A.lds_words >= 62u && lrem <= 32u && Wl - uw0 <= 64u) {
    buf[lane] = h.w0;  // zeros past the end
    buf[lane + 64] = h.w1;
    wave_sync_lds();
    // one unary word per lane (uw0 <= 64): word w holds terminators excl ..
    // incl - 1, and group j >= 1 starts just past terminator 8 j - 1, so word w
    // is the start word of groups j in [(excl + 8) / 8, incl / 8] (at most
    // four).  Each word's lane writes its index and the group's rank among its
    // terminators into those groups' slots; each lane then reads its group's
    // and selects inside that word.
    const uint32_t cnt = __popc(buf[uw0 + lane]);
    const uint32_t incl = wave_scan_incl(cnt);
    if (__builtin_amdgcn_readlane(incl, 63) >= 512u) {
      const uint32_t excl = incl - cnt;
      const uint32_t e8 = excl + 8u, llo = e8 >> 3;
      const int32_t m = (int32_t)(min(incl >> 3, 63u) - llo);  // last slot less the first; 64 and beyond are no groups
      const uint32_t entry = ((uint32_t)lane << 5) + ((e8 & ~7u) - 1u - excl);
      // the slots lie behind the words that are still read
      const uint32_t slot = lds_addr(starts) + 4u * llo;
      store_slot<0>(slot, entry, m + 1);
      store_slot<1>(slot, entry + 8u, m + 1);
      store_slot<2>(slot, entry + 16u, m + 1);
      store_slot<3>(slot, entry + 24u, m + 1);
      wave_sync_lds();
      // group 0 begins at bit R and has no slot: its lane reads word 0 and drops the result
      const uint32_t slot_g = starts[grp];
      const uint32_t e = grp != 0u ? slot_g : 0u;
      const uint32_t uw = uw0 + (e >> 5);
      pos = uw * 32u + select32_half(buf[uw], e & 31u, seltbl) + 1u;
      pos = grp != 0u ? pos : R;
      const uint32_t win = bits32_at(buf, pos);
      if (__ballot(__popc(win) < 8) == 0ull) {
        // (__umul24 becomes the slow 32-bit product; the two wait states a vector
        // instruction needs behind one that wrote its scalar operand stand here)
        uint32_t rpos;
        asm("s_nop 1\n\tv_mul_u32_u24 %0, %1, %2" : "=v"(rpos) : "v"(grp), "s"(lrem));
        const uint32_t acc = bits32_at(buf, rpos);
        uint32_t sh = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const uint32_t kk = sym_class<LAT>(j) ? k1 : k0;
          const uint32_t q = (uint32_t)__builtin_ctz(win >> sh);
          sh += q + 1u;
          sym[j] = (q << kk) | __builtin_amdgcn_ubfe(acc, rem_offset<LAT>(j, k0, k1), kk);
        }
        small = k0 <= 4u && k1 <= 4u;
        return 0ull;
      }
      known = true;
    }
  } else {
    if ((uint32_t)lane < Wl) buf[lane] = h.w0;
    if ((uint32_t)lane + 64u < Wl) buf[lane + 64] = h.w1;
    for (uint32_t w = 128u + lane; w < Wl; w += 64) buf[w] = A.payload[(uint64_t)h.start + w];
    if (lane < 2) buf[Wl + lane] = 0u;  // two zero words past the end
  }
  return __ballot(!decode_symbols_general<LAT>(h.ok, Wl, R, k0, k1, lane, grp, known, pos, buf, starts, sym));
}

inline bool kv_variant(const hq_plan_s* p) { return p->rotation || p->dither || p->norm_fp16; }

}  // namespace
