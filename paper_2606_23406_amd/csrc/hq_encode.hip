// HyperQuant encode kernels for gfx950 (MI355X); the lane layout is in hq_device.h.
#include <mutex>

#include "hq_device.h"
#include "hq_lds.h"

#pragma clang fp contract(off)

namespace {

// ------------------------------------------------------------ encode kernel
// One workgroup encodes HQ_ENC_SUBS_PER_WG consecutive sub-streams (four
// waves with four each, one at a time, or sixteen waves with one each) and
// keeps their bits in LDS; then its first wave alone publishes the group's
// word count, looks back for the group's absolute word offset and writes
// payload and offsets.  KV = false is the weight path (no rotation, no
// dither, fp32 norms) compiled without those branches; KV = true reads the
// three options at run time.

// Number of k in 1..KMAX with sum >= thr[k] (thresholds clamped below 2^30
// on the host, sums below 2^26), on scalar registers.
__device__ __forceinline__ uint32_t kstar_count(uint32_t sum, const uint32_t* thr) {
  // thr[1..15] is nondecreasing, so the count is the largest t with
  // sum >= thr[t]: a binary search, each level's threshold picked by selects
  uint32_t a = sum >= thr[8] ? 8u : 0u;
  const uint32_t t4 = a ? thr[12] : thr[4];
  a += sum >= t4 ? 4u : 0u;
  const uint32_t t2 = a < 8u ? (a ? thr[6] : thr[2]) : (a == 8u ? thr[10] : thr[14]);
  a += sum >= t2 ? 2u : 0u;
  const uint32_t t1 = a < 8u ? (a < 4u ? (a ? thr[3] : thr[1]) : (a == 4u ? thr[5] : thr[7]))
                             : (a < 12u ? (a == 8u ? thr[9] : thr[11]) : (a == 12u ? thr[13] : thr[15]));
  a += sum >= t1 ? 1u : 0u;
  return a;
}

// One look-back round over the NR * 64 workgroups hi, hi - 1, ... (lane l
// takes distances r * 64 + l below hi + 1, r < NR): waits until each has
// published, then adds their values down to the nearest inclusive prefix
// into `prefix`.  Returns true when that prefix was among them (or the wait
// timed out: then `timed_out` is set).
template <int NR>
__device__ __forceinline__ bool lookback_round(unsigned long long* status, int64_t hi,
                                               uint32_t epoch, int lane, uint32_t& prefix,
                                               bool& timed_out) {
  unsigned long long st[NR];
  bool ready[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    st[r] = 0ull;
    ready[r] = hi - (r * 64 + lane) < 0;
  }
  uint32_t spins = 0;
  for (;;) {
    bool all = true;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      if (!ready[r]) {
        st[r] = load_status(&status[hi - (r * 64 + lane)]);
        ready[r] = (uint32_t)(st[r] >> 34) == epoch && ((st[r] >> 32) & 3u) != 0u;
      }
      all = all && ready[r];
    }
    if (__ballot(!all) == 0ull) break;
    if (++spins > kSpinLimit) {
      timed_out = true;
      return true;
    }
    __builtin_amdgcn_s_sleep(1);
  }
  // nearest inclusive prefix: the first r with one, then its lowest lane
  uint32_t stop = 64u * NR;
#pragma unroll
  for (int r = NR - 1; r >= 0; --r) {
    const bool incl = hi - (r * 64 + lane) >= 0 && ((st[r] >> 32) & 3u) == 2u;
    const unsigned long long m = __ballot(incl);
    if (m) stop = (uint32_t)(r * 64) + (uint32_t)__builtin_ctzll(m);
  }
  uint32_t v = 0;
#pragma unroll
  for (int r = 0; r < NR; ++r)
    if (hi - (r * 64 + lane) >= 0 && (uint32_t)(r * 64 + lane) <= stop) v += (uint32_t)st[r];
  prefix += wave_total(v);
  return stop < 64u * NR;
}

// Position of one wave's sub-stream: wave-uniform row and first column.
struct SubPos {
  bool active;
  uint32_t lrow, col0;
};

// The 16 (bf16) or 32 (fp32) input bytes of one lane and its RHT signs:
// bf16 XOR words (bit 15 / bit 31 of each column pair) or fp32 sign bits.
struct LaneInput {
  uint4 a, b, sw;
};

// An inactive sub-stream (past the last row; its results are discarded) has
// lrow = col0 = 0 and reads the first row, so no lane is zero-filled.
template <int XT>
__device__ __forceinline__ LaneInput load_lane_input(const hq_encode_args& A, const SubPos& P,
                                                     int lane) {
  // uniform row base plus a 32-bit per-lane byte offset (columns < 2^28)
  LaneInput in;
  const uint32_t col = P.col0 + 8u * (uint32_t)lane;
  if constexpr (XT == HQ_BF16) {
    const char* row = (const char*)((const uint16_t*)A.x + (int64_t)P.lrow * A.ld);
    in.a = *(const uint4*)(row + (col << 1));
    in.b = make_uint4(0u, 0u, 0u, 0u);
    in.sw = *(const uint4*)((const char*)A.dsign16 + (col << 1));
  } else {
    const char* row = (const char*)((const float*)A.x + (int64_t)P.lrow * A.ld);
    const uint4* p = (const uint4*)(row + (col << 2));
    in.a = p[0];
    in.b = p[1];
    in.sw = make_uint4(sign_bits8(A.dmask, col), 0u, 0u, 0u);
  }
  return in;
}

// OR the low 32 + sh bits of v << sh into buf at bit pos (two words).
__device__ __forceinline__ void or_word(uint32_t* buf, uint32_t pos, uint32_t v) {
  const uint64_t t = (uint64_t)v << (pos & 31u);
  atomicOr(&buf[pos >> 5], (uint32_t)t);
  atomicOr(&buf[(pos >> 5) + 1], (uint32_t)(t >> 32));
}

// The lane's 8 input values with the RHT signs D applied, kept in their
// loaded form until the transform needs them: four bf16 pairs or eight fp32
// words.  A wave holding several sub-streams keeps the pending ones at half
// the registers of their fp32 values (bf16), which is what lets the encoder
// run eight waves per SIMD.
template <int XT>
struct Packed {
  uint32_t w[XT == HQ_BF16 ? 4 : 8];
};

template <int XT>
__device__ __forceinline__ Packed<XT> pack_signed(const LaneInput& in) {
  Packed<XT> p;
  if constexpr (XT == HQ_BF16) {
    p.w[0] = in.a.x ^ in.sw.x;
    p.w[1] = in.a.y ^ in.sw.y;
    p.w[2] = in.a.z ^ in.sw.z;
    p.w[3] = in.a.w ^ in.sw.w;
  } else {
    const uint32_t w8[8] = {in.a.x, in.a.y, in.a.z, in.a.w, in.b.x, in.b.y, in.b.z, in.b.w};
#pragma unroll
    for (int i = 0; i < 8; ++i) p.w[i] = w8[i] ^ (((in.sw.x >> i) & 1u) << 31);
  }
  return p;
}

template <int XT>
__device__ __forceinline__ void unpack(const Packed<XT>& p, float* x) {
  if constexpr (XT == HQ_BF16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[2 * i] = __uint_as_float(p.w[i] << 16);
      x[2 * i + 1] = __uint_as_float(p.w[i] & 0xFFFF0000u);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = __uint_as_float(p.w[i]);
  }
}

// The tile's sum of squares: a pairwise tree in index order (the lane
// butterflies 1, 2, 4, 8 add the same pairs in the same order).
template <int XT>
__device__ __forceinline__ float tile_sumsq(const Packed<XT>& p) {
  float x[8], sq[8];
  unpack<XT>(p, x);
#pragma unroll
  for (int i = 0; i < 8; ++i) sq[i] = x[i] * x[i];
  float ss = tree8(sq);
  ss = ss + dpp_xor<1>(ss);
  ss = ss + dpp_xor<2>(ss);
  ss = ss + swz_xor4(ss);
  ss = ss + dpp_xor<8>(ss);
  return ss;
}

// The lane's 8 remainder fields (k0 / k1 bits by class, packed in symbol
// order), ORed into the buffer at bit rpos.
template <int LAT>
__device__ __forceinline__ void put_remainders(uint32_t* buf, uint32_t rpos, const uint32_t (&sym)[8],
                                               uint32_t k0, uint32_t k1, uint32_t lrem) {
  if (lrem <= 32) {
    uint32_t acc = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t kk = sym_class<LAT>(j) ? k1 : k0;
      acc = lshl_or_s(sym[j] & ((1u << kk) - 1u), readfirst(rem_offset<LAT>(j, k0, k1)), acc);
    }
    or_word(buf, rpos, acc);
  } else if (lrem <= 64) {
    uint64_t acc = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t kk = sym_class<LAT>(j) ? k1 : k0;
      acc |= (uint64_t)(sym[j] & ((1u << kk) - 1u)) << rem_offset<LAT>(j, k0, k1);
    }
    or_bits64(buf, rpos, acc);
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t kk = sym_class<LAT>(j) ? k1 : k0;
      or_bits64(buf, rpos + rem_offset<LAT>(j, k0, k1), sym[j] & ((1u << kk) - 1u));
    }
  }
}

// The lane's 8 unary codes (q zeros and a one each, ulen bits in all),
// ORed into the buffer from bit upos.
__device__ __forceinline__ void put_unary(uint32_t* buf, uint32_t upos, const uint32_t (&qv)[8],
                                          uint32_t ulen) {
  if (ulen <= 32) {
    uint32_t m = 0, t = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      t += qv[j];
      m = bit_or(t, m);
      t += 1;
    }
    or_word(buf, upos, m);
  } else if (ulen <= 64) {
    uint64_t m = 0;
    uint32_t t = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      t += qv[j];
      m |= 1ull << t;
      t += 1;
    }
    or_bits64(buf, upos, m);
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      upos += qv[j];
      or_bits64(buf, upos, 1ull);
      upos += 1;
    }
  }
}

template <int LAT, int XT, bool KV>
__device__ __forceinline__ void encode_substream(const hq_encode_args& A, const hq_rice_thr& T,
                                                 const SubPos& P, int lane, float* x, float scale_tw,
                                                 uint32_t* buf, float* stage, uint32_t& W_out,
                                                 uint32_t& kb_out, uint32_t& bits_out,
                                                 bool& overflow_out) {
  const bool active = P.active;  // wave-uniform
  const uint32_t col = P.col0 + 8u * (uint32_t)lane;  // tile lane/16, coordinates 8 (lane % 16) + j
  const int64_t grow = A.first_row + P.lrow;
  const bool use_rot = KV && A.rotation == HQ_ROT_SIGNS;
  const bool use_dither = KV && A.dither;

  // ---- z = (sigma H D x) * (sigma alpha / r): the scale carries the sign sigma
#pragma unroll
  for (int i = 0; i < 8; ++i) x[i] = x[i] * scale_tw;
  if (use_rot) {
    const uint32_t sbits = sign_bits8(A.smask, (lane & 15) * 8);
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = flip(x[i], sbits, i);
  }
  // z <- S z, S^T read from global memory (a workgroup copy in LDS was tried only
  // while LDS reads were misaligned, 64 cycles each: 3x slower then)
  if (KV && A.rotation == HQ_ROT_QJL) qjl_wave(A.qjlt, stage, lane, x);
  if (use_dither) {
    float u[8];
    dither8<LAT>(A.dither_seed, grow, col, u);
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = x[i] + (LAT == kE8 ? 0.5f * u[i] : u[i]);
  }

  // ---- quantize + strip
  uint32_t sym[8];
  bool huge = false;
  if constexpr (LAT == kE8) {
    int32_t h[8], cb;  // c = 2 h + cb
    e8_nearest(x, h, cb);  // an inactive sub-stream's symbols are never written
    e8_strip(h, cb, sym);
  } else {
    int32_t c[8];
    quantize8<LAT>(x, c);
#pragma unroll
    for (int i = 0; i < 8; ++i) huge = huge || (c[i] > 65536 || c[i] < -65536);
    if (huge || !active) {
#pragma unroll
      for (int i = 0; i < 8; ++i) c[i] = 0;
    }
    strip8<LAT>(c, sym);
  }

  // ---- Rice parameters (wave-uniform), quotients and the unary-length scan
  uint32_t k0, k1, qv[8], ulen, uincl = 0;  // uincl: set by the k* scan or below
  bool scanned = false;
  if constexpr (LAT == kE8 || LAT == kZ) {
    uint32_t s0 = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) s0 += sym[j];
    if (A.rice_k >= 0) {
      k0 = (uint32_t)A.rice_k;
      ulen = 8;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        qv[j] = sym[j] >> k0;
        ulen += qv[j];
      }
    } else {
      const uint32_t a0 = kstar_count(wave_total(s0), T.thr0);
      // the better of k* and k* + 1: k* + 1 saves sum((m >> k) - (m >> (k+1)))
      // unary bits and costs one remainder bit per symbol.  Both candidates'
      // unary-length scans run in one pass; their totals give that saving,
      // and the chosen one's scan places the codes.
      uint32_t ga = 0, gb = 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        qv[j] = sym[j] >> a0;
        ga += qv[j];
        gb += qv[j] >> 1;
      }
      uint32_t ia = 8 + ga, ib = 8 + gb;
      wave_scan_incl2(ia, ib);
      const uint32_t Ua = __builtin_amdgcn_readlane(ia, 63), Ub = __builtin_amdgcn_readlane(ib, 63);
      const uint32_t d = (a0 < HQ_KMAX && Ua - Ub > (uint32_t)HQ_SUB) ? 1u : 0u;
      k0 = a0 + d;
#pragma unroll
      for (int j = 0; j < 8; ++j) qv[j] >>= d;
      ulen = 8 + (d ? gb : ga);
      uincl = d ? ib : ia;
      scanned = true;
    }
    k1 = k0;
  } else {
    if (A.rice_k >= 0) {
      k0 = (uint32_t)A.rice_k;
      k1 = (LAT == kD4) ? (k0 > 0 ? k0 - 1 : 0) : k0;
    } else {
      uint32_t s0 = 0, s1 = 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if (sym_class<LAT>(j)) s1 += sym[j]; else s0 += sym[j];
      }
      const uint32_t a0 = kstar_count(wave_total(s0), T.thr0);
      const uint32_t a1 = (LAT == kA2) ? kstar_count(wave_total(s1), T.thr1) : 0u;
      const uint32_t b0 = a0 < HQ_KMAX ? a0 + 1 : a0;
      const uint32_t b1 = a1 < HQ_KMAX ? a1 + 1 : a1;
      uint32_t g0 = 0, g1 = 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if (LAT == kD4) {
          const uint32_t ka = sym_class<LAT>(j) ? (a0 > 0 ? a0 - 1 : 0) : a0;
          const uint32_t kb = sym_class<LAT>(j) ? (b0 > 0 ? b0 - 1 : 0) : b0;
          g0 += (sym[j] >> ka) - (sym[j] >> kb);
        } else if (sym_class<LAT>(j)) {
          g1 += (sym[j] >> a1) - (sym[j] >> b1);
        } else {
          g0 += (sym[j] >> a0) - (sym[j] >> b0);
        }
      }
      const uint32_t gain0 = wave_total(g0);
      uint32_t cost0;
      if (LAT == kD4) {
        cost0 = (b0 - a0) * (3u * HQ_SUB / 4u) +
                ((b0 > 0 ? b0 - 1 : 0) - (a0 > 0 ? a0 - 1 : 0)) * (HQ_SUB / 4u);
      } else {
        cost0 = (b0 - a0) * (HQ_SUB / 2u);
      }
      k0 = gain0 > cost0 ? b0 : a0;
      if (LAT == kA2) {
        const uint32_t gain1 = wave_total(g1);
        k1 = gain1 > (b1 - a1) * (HQ_SUB / 2u) ? b1 : a1;
      } else {
        k1 = k0 > 0 ? k0 - 1 : 0;
      }
    }
    ulen = 8;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      qv[j] = sym[j] >> (sym_class<LAT>(j) ? k1 : k0);
      ulen += qv[j];
    }
  }

  // ---- code lengths: remainder region then unary region
  const uint32_t lrem = lane_rem_bits<LAT>(k0, k1);
  const uint32_t R = 64 * lrem;
  if (!scanned) uincl = wave_scan_incl(ulen);
  const uint32_t U = __builtin_amdgcn_readlane(uincl, 63);
  const uint32_t uoff = uincl - ulen;
  uint32_t W = (R + U + 31) >> 5;
  // A sub-stream that does not fit the plan's bound (only non-finite or
  // out-of-range input can do that) is written as all-zero symbols with
  // k = 0: 512 unary terminators, 16 words.
  const bool overflow = active && W > A.lds_words;
  if (!active) W = 0;
  if (overflow) W = HQ_SUB / 32;

  // ---- assemble in this sub-stream's LDS buffer (two spare words past W
  //      take the zero high halves of the ORs)
  for (uint32_t w = lane; w < W; w += 64) buf[w] = overflow ? 0xFFFFFFFFu : 0u;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  if (active && !overflow) {
    // remainder fields, packed per lane
    put_remainders<LAT>(buf, __umul24((uint32_t)lane, lrem), sym, k0, k1, lrem);  // lrem < 2^24
    // unary codes
    put_unary(buf, R + uoff, qv, ulen);
  }
  W_out = W;
  kb_out = overflow ? 0u : (LAT == kA2 ? (k0 | (k1 << 4)) : k0);
  bits_out = overflow ? (uint32_t)HQ_SUB : R + U;
  overflow_out = overflow;
}

// One sub-stream of B consecutive 512-symbol blocks (S = 512 B, weight
// plans): x[b] holds block b's transformed values and scl[b] its tile scale.
// Every block is quantized and stripped first; the Rice parameters then
// follow from the whole sub-stream's symbols (the sums and the k* / k* + 1
// decision taken over all S symbols), and the split layout places the S
// remainder fields (block b's at bit b 64 lrem) before the S unary codes
// (block b's after the unary bits of blocks 0 .. b - 1).
template <int LAT, int B>
__device__ __forceinline__ void encode_multiblock(const hq_encode_args& A, const hq_rice_thr& T,
                                                  bool active, int lane, float (*x)[8],
                                                  const float* scl, uint32_t tsig, uint32_t* buf,
                                                  uint32_t& W_out, uint32_t& kb_out,
                                                  uint32_t& bits_out, bool& overflow_out) {
  constexpr uint32_t S = (uint32_t)HQ_SUB * B;
  uint32_t sym[B][8];
#pragma unroll
  for (int b = 0; b < B; ++b) {
    float z[8];
    const float sc = xor_sign(scl[b], tsig);
#pragma unroll
    for (int i = 0; i < 8; ++i) z[i] = x[b][i] * sc;
    if constexpr (LAT == kE8) {
      int32_t h[8], cb;
      e8_nearest(z, h, cb);
      e8_strip(h, cb, sym[b]);
    } else {
      int32_t c[8];
      quantize8<LAT>(z, c);
      bool huge = false;
#pragma unroll
      for (int i = 0; i < 8; ++i) huge = huge || (c[i] > 65536 || c[i] < -65536);
      if (huge || !active) {
#pragma unroll
        for (int i = 0; i < 8; ++i) c[i] = 0;
      }
      strip8<LAT>(c, sym[b]);
    }
  }
  // ---- Rice parameters over the whole sub-stream (wave-uniform)
  uint32_t k0, k1;
  if (A.rice_k >= 0) {
    k0 = (uint32_t)A.rice_k;
    k1 = (LAT == kD4) ? (k0 > 0 ? k0 - 1 : 0) : k0;
  } else if constexpr (LAT == kE8 || LAT == kZ) {
    uint32_t s0 = 0;
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
      for (int j = 0; j < 8; ++j) s0 += sym[b][j];
    const uint32_t a0 = kstar_count(wave_total(s0), T.thr0);
    // k* + 1 saves sum((m >> k*) - (m >> (k* + 1))) unary bits for S remainder bits
    uint32_t g = 0;
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint32_t q = sym[b][j] >> a0;
        g += q - (q >> 1);
      }
    k0 = (a0 < HQ_KMAX && wave_total(g) > S) ? a0 + 1 : a0;
    k1 = k0;
  } else {
    uint32_t s0 = 0, s1 = 0;
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if (sym_class<LAT>(j)) s1 += sym[b][j]; else s0 += sym[b][j];
      }
    const uint32_t a0 = kstar_count(wave_total(s0), T.thr0);
    const uint32_t a1 = (LAT == kA2) ? kstar_count(wave_total(s1), T.thr1) : 0u;
    const uint32_t b0 = a0 < HQ_KMAX ? a0 + 1 : a0;
    const uint32_t b1 = a1 < HQ_KMAX ? a1 + 1 : a1;
    uint32_t g0 = 0, g1 = 0;
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint32_t m = sym[b][j];
        if (LAT == kD4) {
          const uint32_t ka = sym_class<LAT>(j) ? (a0 > 0 ? a0 - 1 : 0) : a0;
          const uint32_t kb = sym_class<LAT>(j) ? (b0 > 0 ? b0 - 1 : 0) : b0;
          g0 += (m >> ka) - (m >> kb);
        } else if (sym_class<LAT>(j)) {
          g1 += (m >> a1) - (m >> b1);
        } else {
          g0 += (m >> a0) - (m >> b0);
        }
      }
    const uint32_t gain0 = wave_total(g0);
    // one more remainder bit on each symbol of the class (D4: 3 S / 4 of
    // class 0, S / 4 of class 1; A2: S / 2 each)
    const uint32_t cost0 = (LAT == kD4)
                               ? (b0 - a0) * (3u * S / 4u) +
                                     ((b0 > 0 ? b0 - 1 : 0) - (a0 > 0 ? a0 - 1 : 0)) * (S / 4u)
                               : (b0 - a0) * (S / 2u);
    k0 = gain0 > cost0 ? b0 : a0;
    if (LAT == kA2) {
      const uint32_t gain1 = wave_total(g1);
      k1 = gain1 > (b1 - a1) * (S / 2u) ? b1 : a1;
    } else {
      k1 = k0 > 0 ? k0 - 1 : 0;
    }
  }
  // ---- code lengths: the B remainder regions, then the B unary regions
  const uint32_t lrem = lane_rem_bits<LAT>(k0, k1);
  const uint32_t Rb = 64 * lrem, Rt = (uint32_t)B * Rb;
  uint32_t ulen[B], uincl[B], U = 0;
#pragma unroll
  for (int b = 0; b < B; ++b) {
    ulen[b] = 8;
#pragma unroll
    for (int j = 0; j < 8; ++j) ulen[b] += sym[b][j] >> (sym_class<LAT>(j) ? k1 : k0);
    uincl[b] = wave_scan_incl(ulen[b]);
    U += __builtin_amdgcn_readlane(uincl[b], 63);
  }
  uint32_t W = (Rt + U + 31) >> 5;
  // a sub-stream past the plan's bound is written as S zero symbols with k = 0
  const bool overflow = active && W > A.lds_words;
  if (!active) W = 0;
  if (overflow) W = S / 32;
  for (uint32_t w = lane; w < W; w += 64) buf[w] = overflow ? 0xFFFFFFFFu : 0u;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  if (active && !overflow) {
    uint32_t ubase = Rt;  // where block b's unary codes begin
#pragma unroll
    for (int b = 0; b < B; ++b) {
      uint32_t qv[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) qv[j] = sym[b][j] >> (sym_class<LAT>(j) ? k1 : k0);
      put_remainders<LAT>(buf, (uint32_t)b * Rb + __umul24((uint32_t)lane, lrem), sym[b], k0, k1, lrem);
      put_unary(buf, ubase + uincl[b] - ulen[b], qv, ulen[b]);
      ubase += __builtin_amdgcn_readlane(uincl[b], 63);
    }
  }
  W_out = W;
  kb_out = overflow ? 0u : (LAT == kA2 ? (k0 | (k1 << 4)) : k0);
  bits_out = overflow ? S : Rt + U;
  overflow_out = overflow;
}

// TILED: a plan whose tile is not 128 (weights only: no rotation or
// dither); the wave takes four consecutive sub-streams, so that every tile
// of up to 2048 scalars lies inside one wave.
template <int LAT, int XT, bool KV, int SPW, bool TILED = false, int MB = 1>
__device__ __forceinline__ void encode_wg(const hq_encode_args& A, const hq_rice_thr& T,
                                          const uint32_t wg) {
  static_assert(SPW == 1 || SPW == 4, "one or four sub-streams per wave");
  static_assert(!TILED || (SPW == 4 && !KV), "long tiles: four sub-streams per wave, weights");
  static_assert(MB == 1 || (TILED && (MB == 2 || MB == 4)), "multi-block sub-streams: long-tile front end");
  constexpr int NSUB = HQ_ENC_SUBS_PER_WG;  // sub-streams per workgroup
  constexpr int WAVES = NSUB / SPW;         // wave64s per workgroup
  extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
  __shared__ uint32_t s_epoch;
  __shared__ uint32_t s_words[NSUB];
  __shared__ uint32_t s_pad[WAVES];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = (int)readfirst((uint32_t)(tid >> 6));
  const uint32_t stride = A.lds_words + 2;  // words per sub-stream buffer
  if (tid == 0)
    s_epoch = (uint32_t)__hip_atomic_load(A.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) &
              kEpochMask;
  const TwSigns sg(lane);
  // sub-streams of MB > 1 consecutive 512-symbol blocks (the long-tile
  // front end, any tile): positions below count blocks
  constexpr uint32_t mb = (uint32_t)MB;
  const uint32_t nblk = (uint32_t)A.nsub * mb;

  // ---- this wave's sub-streams: wg * NSUB + i * WAVES + wave, i < SPW (row and
  //      column advanced on scalar registers)
  SubPos pos[SPW];
  {
    const uint32_t spr = (uint32_t)A.spr * mb;
    const uint32_t step = TILED ? 1u : (uint32_t)WAVES;
    const uint32_t sub0 = wg * NSUB + (uint32_t)wave * (TILED ? (uint32_t)SPW : 1u);
    uint32_t row = sub0 / spr, c = sub0 - row * spr;
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
      pos[i].active = sub0 + (uint32_t)i * step < nblk;
      pos[i].lrow = pos[i].active ? row : 0u;
      pos[i].col0 = pos[i].active ? c * HQ_SUB : 0u;
      c += step;
      while (c >= spr) {
        c -= spr;
        ++row;
      }
    }
  }
  Packed<XT> pk[SPW];
  float ss[SPW];
  bool nonfinite = false;
  float xt[TILED ? SPW : 1][8];  // long tiles: the transformed values of the wave
  uint32_t tsig = 0;             // long tiles: the sign bit of the lane's sigma
  if constexpr (TILED) {
    // ---- long tiles: every load first, then each 128-block's sum of squares
    //      (tree8 and the lane butterflies 1, 2, 4, 8), widened to the tile
    //      by lanes l ^ 16, l ^ 32 and then across sub-streams, in the
    //      pairwise tree's order
    const uint32_t n = (uint32_t)A.tile;
#pragma unroll
    for (int i = 0; i < SPW; ++i) unpack<XT>(pack_signed<XT>(load_lane_input<XT>(A, pos[i], lane)), xt[i]);
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
      float sq[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) sq[j] = xt[i][j] * xt[i][j];
      float v = tree8(sq);
      v = v + dpp_xor<1>(v);
      v = v + dpp_xor<2>(v);
      v = v + swz_xor4(v);
      v = v + dpp_xor<8>(v);
      if (n >= 256u) v = v + swz_xor16(v);
      if (n >= 512u) v = v + lane_xor32(v);
      ss[i] = v;
    }
    if (n >= 1024u) {
      const float a = ss[0] + ss[1], b = ss[2] + ss[3];
      ss[0] = a; ss[1] = a; ss[2] = b; ss[3] = b;
    }
    if (n >= 2048u) {
      const float a = ss[0] + ss[2];
      ss[0] = a; ss[1] = a; ss[2] = a; ss[3] = a;
    }
    // ---- norms and scales: every lane its own tile's; the lane holding a
    //      tile's first coordinate stores the norm
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
      const float r = __builtin_sqrtf(ss[i]);
      const bool bad = !(r <= 3.0e38f);  // an infinite or NaN input
      nonfinite = nonfinite || bad;
      ss[i] = (r == 0.0f || bad) ? 0.0f : (LAT == kE8 ? A.alpha_half : A.alpha) / r;
      const uint32_t sub = wg * NSUB + (uint32_t)(wave * SPW + i);
      const uint64_t flat = (uint64_t)sub * HQ_SUB + 8u * (uint32_t)lane;
      if (pos[i].active && (flat & (n - 1u)) == 0u) {
        ((float*)A.norms)[A.first_row * A.tpr + (int64_t)(flat / n)] = r;
        if (bad && A.stats) {
          atomicAdd(&A.stats->overflow_tiles, 1u);
          atomicCAS(&A.stats->status, 0u, (uint32_t)HQ_ERR_OVERFLOW);
        }
      }
    }
    if (__ballot(nonfinite) != 0ull) {
#pragma unroll
      for (int i = 0; i < SPW; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) xt[i][j] = ss[i] == 0.0f ? 0.0f : xt[i][j];
    }
    tsig = fwht_tiled(xt, lane, n, sg);
  } else {
  // ---- every input load of the wave's sub-streams is issued first; each is
  //      kept packed with its signs applied, and its tile sums of squares
  //      taken (the transforms wait until each sub-stream is coded)
#pragma unroll
  for (int i = 0; i < SPW; ++i) pk[i] = pack_signed<XT>(load_lane_input<XT>(A, pos[i], lane));
#pragma unroll
  for (int i = 0; i < SPW; ++i) ss[i] = tile_sumsq<XT>(pk[i]);

  // ---- tile norms and scales, once for the wave's tiles: with four
  //      sub-streams lane l takes sub-stream i = l & 3, tile t = l >> 4 (each
  //      tile's 16 lanes hold its sum of squares, so the merged value repeats
  //      in every quad); with one, every lane takes its own tile l >> 4
  {
    const int qi = SPW == 4 ? (lane & 3) : 0;
    float ssm = ss[0];
    if constexpr (SPW == 4) ssm = qi == 0 ? ss[0] : (qi == 1 ? ss[1] : (qi == 2 ? ss[2] : ss[3]));
    const bool fp16_norm = KV && A.norm_fp16;
    const float r = __builtin_sqrtf(ssm);
    float rs = r;
    nonfinite = !(r <= 3.0e38f);  // an infinite or NaN input (r is at most 2^64 otherwise)
    bool bad_tile = nonfinite;
    if (fp16_norm) {
      rs = (float)(_Float16)r;
      bad_tile = bad_tile || !(rs <= 65504.0f);
    }
    // E8 decides on z / 2: its scale is (alpha / 2) / r_s, exactly half of alpha / r_s
    const float scale =
        (rs == 0.0f || bad_tile) ? 0.0f : (LAT == kE8 ? A.alpha_half : A.alpha) / rs;
    const uint32_t sub_l = wg * NSUB + (uint32_t)(qi * WAVES + wave);
    const bool writer = SPW == 4 ? ((lane >> 2) & 3) == 0 : (lane & 15) == 0;
    if (writer && sub_l < (uint32_t)A.nsub) {
      // tile (lane >> 4) of sub-stream sub_l: 4 tiles per sub-stream, rows contiguous
      const int64_t t = A.first_row * A.tpr + 4 * (int64_t)sub_l + (lane >> 4);
      if (fp16_norm) {
        ((_Float16*)A.norms)[t] = (_Float16)r;
      } else {
        ((float*)A.norms)[t] = r;
      }
      if (bad_tile && A.stats) {
        atomicAdd(&A.stats->overflow_tiles, 1u);
        atomicCAS(&A.stats->status, 0u, (uint32_t)HQ_ERR_OVERFLOW);
      }
    }
    if constexpr (SPW == 4) {
      ss[0] = quad_bcast<0>(scale);
      ss[1] = quad_bcast<1>(scale);
      ss[2] = quad_bcast<2>(scale);
      ss[3] = quad_bcast<3>(scale);
    } else {
      ss[0] = scale;
    }
  }
  // A non-finite tile has scale 0 and is coded as if its transform were
  // zero (its values would turn the product into NaN); zero tiles, the other
  // tiles with scale 0, hold zeros already.
  if (__ballot(nonfinite) != 0ull) {
#pragma unroll
    for (int i = 0; i < SPW; ++i)
#pragma unroll
      for (int j = 0; j < (XT == HQ_BF16 ? 4 : 8); ++j) pk[i].w[j] = ss[i] == 0.0f ? 0u : pk[i].w[j];
  }
  }  // 128-tiles

  // ---- quantize and Rice-code each sub-stream into its LDS buffer
  uint32_t padsum = 0;
  if constexpr (MB > 1) {
    // sub-streams of MB blocks: the wave's four blocks are 4 / MB of them,
    // sub-stream ls of the group in buffer ls (s_words past the group's
    // 16 / MB sub-streams stay 0)
    constexpr uint32_t ns = (uint32_t)NSUB / MB;
    if (lane == 0 && wave == 0)
      for (uint32_t q = ns; q < (uint32_t)NSUB; ++q) s_words[q] = 0;
#pragma unroll
    for (int j = 0; j < SPW / MB; ++j) {
      const uint32_t ls = (uint32_t)wave * (uint32_t)(SPW / MB) + (uint32_t)j;
      const uint32_t gs = wg * ns + ls;
      const bool act = pos[j * MB].active;
      uint32_t W, kb, bits;
      bool ovf;
      encode_multiblock<LAT, MB>(A, T, act, lane, xt + j * MB, ss + j * MB, tsig, smem + ls * stride,
                                 W, kb, bits, ovf);
      if (act) {
        if (lane == 0) {
          A.kparam[A.first_sub + gs] = (uint8_t)kb;
          s_words[ls] = W;
          if (ovf && A.stats) atomicCAS(&A.stats->status, 0u, (uint32_t)HQ_ERR_OVERFLOW);
        }
        padsum += W * 32u - bits;
      } else if (lane == 0) {
        s_words[ls] = 0;
      }
    }
  } else
#pragma unroll
  for (int i = 0; i < SPW; ++i) {
    // 128-tiles: neighbouring waves take neighbouring sub-streams
    const int li = TILED ? wave * SPW + i : i * WAVES + wave;
    const uint32_t sub = wg * NSUB + (uint32_t)li;
    uint32_t W, kb, bits;
    bool ovf;
    float x[8];  // x <- sigma H D x
    if constexpr (TILED) {
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = xt[i][j];
    } else {
      unpack<XT>(pk[i], x);
      fwht128_tw(x, sg);
    }
    encode_substream<LAT, XT, KV>(A, T, pos[i], lane, x, xor_sign(ss[i], TILED ? tsig : sg.sigma),
                                  smem + li * stride,
                                  (float*)(smem + NSUB * stride) + wave * HQ_QJL_STAGE, W, kb,
                                  bits, ovf);
    if (pos[i].active) {
      if (lane == 0) {
        A.kparam[A.first_sub + sub] = (uint8_t)kb;
        s_words[li] = W;
        if (ovf && A.stats) atomicCAS(&A.stats->status, 0u, (uint32_t)HQ_ERR_OVERFLOW);
      }
      padsum += W * 32u - bits;
    } else if (lane == 0) {
      s_words[li] = 0;
    }
  }
  if (lane == 0) {
    s_pad[wave] = padsum;
  }
  __syncthreads();
  // The other waves are done: their slots go to the next workgroups while wave 0
  // alone waits for the group's offset and writes every sub-stream out.
  // (No workgroup barrier follows.)
  if (wave != 0) return;

  const uint32_t epoch = readfirst(s_epoch);
  // ---- publish this group's word count at once, so successors can pass it;
  //      the group's pad bits go to its stats word first (packed as
  //      words << 11 | pad: at most 2^19 words and 64 * 31 pad bits)
  static_assert(NSUB <= 64, "one sub-stream word count per lane");
  const uint32_t agg = wave_total(lane < NSUB ? s_words[lane] : 0u);
  if (lane == 0) {
    if (A.stats) {
      uint32_t gp = 0;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) gp += s_pad[w];
      store_status(&A.wgstat[wg], pack_status(epoch, 1u, (agg << 11) | gp));
    }
    if (wg > 0) store_status(&A.status[wg], pack_status(epoch, 1u, agg));
  }

  // ---- look-back: 256 predecessors per round trip, until the nearest
  //      published inclusive prefix
  uint32_t prefix = 0;
  bool timed_out = false;
  for (int64_t hi = (int64_t)wg - 1; hi >= 0; hi -= 256)
    if (lookback_round<4>(A.status, hi, epoch, lane, prefix, timed_out)) break;
  // an append to an empty stream starts at word 0, like a fresh encode
  const unsigned long long base =
      (A.first_sub > 0 ? (unsigned long long)readfirst(A.offsets[A.first_sub]) : 0ull) + prefix;
  if (lane == 0) {
    store_status(&A.status[wg], pack_status(epoch, 2u, prefix + agg));
    // the last group: every group has read this launch's epoch; advance it
    if (wg == A.nwg - 1)
      __hip_atomic_store(A.epoch, (unsigned long long)((epoch + 1u) & kEpochMask), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    if (timed_out && A.stats) atomicCAS(&A.stats->status, 0u, (uint32_t)HQ_ERR_HIP);
  }

  // ---- write payload and offsets of all of the group's sub-streams: lane
  //      l < NSUB takes sub-stream l's word count (0 when inactive) and its
  //      prefix inside the group; then 16 lanes per sub-stream copy four
  //      sub-streams at a time, every load of a lane issued before its stores
  static_assert(NSUB <= 16, "one row of lanes holds the group's word counts");
  {
    const uint32_t wl = lane < NSUB ? s_words[lane] : 0u;
    uint32_t il = wl;  // inclusive prefix inside the first row of 16 lanes
    il += dpp<kDppRowShr1, 0xF, 0xF, true>(0u, il);
    il += dpp<kDppRowShr2, 0xF, 0xF, true>(0u, il);
    il += dpp<kDppRowShr4, 0xF, 0xF, true>(0u, il);
    il += dpp<kDppRowShr8, 0xF, 0xF, true>(0u, il);
    const uint32_t xl = il - wl;
    const uint32_t ns = (uint32_t)NSUB / mb;  // sub-streams per group
    const uint32_t sub_l = wg * ns + (uint32_t)lane;
    if ((uint32_t)lane < ns && sub_l < (uint32_t)A.nsub) {
      const unsigned long long end = base + il;
      if (sub_l == 0 && A.first_sub == 0) A.offsets[0] = 0u;
      A.offsets[A.first_sub + sub_l + 1] = (uint32_t)end;
      if (end > (unsigned long long)A.cap_words && A.stats)
        atomicCAS(&A.stats->status, 0u, (uint32_t)HQ_ERR_CAPACITY);
    }
#pragma unroll
    for (int r = 0; r < NSUB / 4; ++r) {
      const int li = 4 * r + (lane >> 4);
      const uint32_t W = (uint32_t)__shfl((int)wl, li);
      const unsigned long long st = base + (uint32_t)__shfl((int)xl, li);
      if (st + W > (unsigned long long)A.cap_words) continue;  // reported above
      const uint32_t* buf = smem + li * stride;
      for (uint32_t j = (uint32_t)(lane & 15); j < W; j += 64) {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = j + 16u * u < W ? buf[j + 16u * u] : 0u;
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (j + 16u * u < W) A.payload[st + j + 16u * u] = v[u];
      }
    }
  }
  // ---- bit counts: the last group of every 256 adds up their stats words
  //      (all of them were stored before their owners' aggregates, which this
  //      group's look-back has passed), so the stats block takes one atomic
  //      per 256 groups instead of one per group
  if (A.stats && ((wg & 255u) == 255u || wg == A.nwg - 1)) {
    uint32_t gw = 0, gp = 0;  // words, pad bits
    bool late = false;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t idx = (wg & ~255u) + (uint32_t)(r * 64 + lane);
      if (idx > wg) continue;
      uint32_t spins = 0;
      for (;;) {
        const unsigned long long st = load_status(&A.wgstat[idx]);
        if ((uint32_t)(st >> 34) == epoch && ((st >> 32) & 3u) != 0u) {
          gw += (uint32_t)st >> 11;
          gp += (uint32_t)st & 2047u;
          break;
        }
        if (++spins > kSpinLimit) {
          late = true;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
    }
    const uint32_t tw = wave_total(gw), tp = wave_total(gp);  // < 2^27 words, < 2^19 pad bits
    if (late) atomicCAS(&A.stats->status, 0u, (uint32_t)HQ_ERR_HIP);
    if (lane == 0) {
      atomicAdd(&A.stats->payload_bits, 32ull * tw - tp);
      atomicAdd(&A.stats->pad_bits, (unsigned long long)tp);
    }
  }
}

// The E8 KV encode of bf16 rows, four sub-streams per wave, needs 81 registers
// of its own accord, one too many for six waves per SIMD; held to 80 it moves
// two outside the loops to scratch: 32768 x 1024 rows 86.6 -> 80 us (fp32 rows
// would spill 15).
template <int LAT, int XT, bool KV, int SPW>
__global__ __launch_bounds__(64 * HQ_ENC_SUBS_PER_WG / SPW) __attribute__((amdgpu_waves_per_eu(
    KV && LAT == kE8 && XT == HQ_BF16 && SPW == HQ_ENC_SUBS_PER_WAVE ? 6 : 1))) void hq_encode_kernel(hq_encode_args A, hq_rice_thr T) {
  encode_wg<LAT, XT, KV, SPW>(A, T, blockIdx.x);
}

// MB: 512-symbol blocks per sub-stream (1, or 2 / 4 for S = 1024 / 2048)
template <int LAT, int XT, int MB>
__global__ __launch_bounds__(64 * HQ_ENC_WAVES) void hq_encode_tiled_kernel(hq_encode_args A,
                                                                           hq_rice_thr T) {
  encode_wg<LAT, XT, false, HQ_ENC_SUBS_PER_WAVE, true, MB>(A, T, blockIdx.x);
}

// Several matrices in one launch: workgroups wg_begin[i] .. wg_begin[i+1]-1
// encode member i (its own stream, scan scratch and epoch), so small
// matrices share the machine instead of each filling only part of it.
template <int LAT, int XT, bool KV>
__global__ __launch_bounds__(64 * HQ_ENC_WAVES) __attribute__((amdgpu_waves_per_eu(
    KV && LAT == kE8 && XT == HQ_BF16 ? 6 : 1))) void hq_encode_group_kernel(hq_encode_group_args G) {
  int mi = 0;
  for (int i = 1; i < G.count; ++i) mi = blockIdx.x >= G.wg_begin[i] ? i : mi;
  encode_wg<LAT, XT, KV, HQ_ENC_SUBS_PER_WAVE>(G.m[mi], G.thr, blockIdx.x - G.wg_begin[mi]);
}

__global__ void hq_zero_kernel(uint32_t* p, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// One encode launch: a single matrix (hq_encode_args + thresholds; four or
// one sub-streams per wave) or a group (four per wave).
template <int LAT, int XT, bool KV>
void launch_encode_kernel(const hq_encode_args& a, const hq_rice_thr& t, uint32_t nwg,
                          uint32_t lds_words, hipStream_t st) {
  const size_t per_sub = (size_t)(lds_words + 2) * sizeof(uint32_t);
  const size_t lds = per_sub * HQ_ENC_SUBS_PER_WG;
  // the qjl rotation stages four tiles per wave after the sub-stream buffers
  const size_t stage = a.qjlt ? (size_t)HQ_QJL_STAGE * sizeof(float) : 0;
  if (a.spw == 1)
    hipLaunchKernelGGL((hq_encode_kernel<LAT, XT, KV, 1>), dim3(nwg), dim3(64 * HQ_ENC_SUBS_PER_WG),
                       lds + stage * HQ_ENC_SUBS_PER_WG, st, a, t);
  else
    hipLaunchKernelGGL((hq_encode_kernel<LAT, XT, KV, HQ_ENC_SUBS_PER_WAVE>), dim3(nwg),
                       dim3(64 * HQ_ENC_WAVES), lds + stage * HQ_ENC_WAVES, st, a, t);
}

template <int LAT, int XT, bool KV>
void launch_encode_kernel(const hq_encode_group_args& g, const hq_rice_thr&, uint32_t nwg,
                          uint32_t lds_words, hipStream_t st) {
  const size_t lds = (size_t)(lds_words + 2) * HQ_ENC_SUBS_PER_WG * sizeof(uint32_t);
  hipLaunchKernelGGL((hq_encode_group_kernel<LAT, XT, KV>), dim3(nwg), dim3(64 * HQ_ENC_WAVES), lds, st, g);
}

template <int LAT, typename Args>
int launch_encode_lat(const Args& a, const hq_rice_thr& t, uint32_t nwg, uint32_t lds_words, int xt,
                      bool kv, hipStream_t st) {
  if (xt == HQ_BF16) {
    if (kv)
      launch_encode_kernel<LAT, HQ_BF16, true>(a, t, nwg, lds_words, st);
    else
      launch_encode_kernel<LAT, HQ_BF16, false>(a, t, nwg, lds_words, st);
  } else {
    if (kv)
      launch_encode_kernel<LAT, HQ_FP32, true>(a, t, nwg, lds_words, st);
    else
      launch_encode_kernel<LAT, HQ_FP32, false>(a, t, nwg, lds_words, st);
  }
  return (int)hipGetLastError();
}

// Long tiles, or sub-streams of several blocks (weight plans): four
// consecutive 512-symbol blocks per wave.
template <int LAT, int XT, int MB>
int launch_encode_tiled_mb(const hq_encode_args& a, const hq_rice_thr& t, hipStream_t st) {
  const size_t lds = (size_t)(a.lds_words + 2) * HQ_ENC_SUBS_PER_WG * sizeof(uint32_t);
  static hq_lds_granted granted;
  hq_allow_lds((const void*)hq_encode_tiled_kernel<LAT, XT, MB>, lds, granted);
  hipLaunchKernelGGL((hq_encode_tiled_kernel<LAT, XT, MB>), dim3(a.nwg), dim3(64 * HQ_ENC_WAVES), lds, st,
                     a, t);
  return (int)hipGetLastError();
}

template <int LAT>
int launch_encode_tiled(const hq_encode_args& a, const hq_rice_thr& t, int xt, hipStream_t st) {
  if (xt == HQ_BF16) {
    if (a.mb == 4) return launch_encode_tiled_mb<LAT, HQ_BF16, 4>(a, t, st);
    if (a.mb == 2) return launch_encode_tiled_mb<LAT, HQ_BF16, 2>(a, t, st);
    return launch_encode_tiled_mb<LAT, HQ_BF16, 1>(a, t, st);
  }
  if (a.mb == 4) return launch_encode_tiled_mb<LAT, HQ_FP32, 4>(a, t, st);
  if (a.mb == 2) return launch_encode_tiled_mb<LAT, HQ_FP32, 2>(a, t, st);
  return launch_encode_tiled_mb<LAT, HQ_FP32, 1>(a, t, st);
}

}  // namespace

int hq_launch_encode(const hq_plan_s* p, const hq_encode_args& a, const hq_rice_thr& t, int xt,
                     void* stream) {
  hipStream_t st = (hipStream_t)stream;
  if (p->tile != HQ_TILE || p->substream != HQ_SUB) {  // long tiles, or sub-streams of 2 or 4 blocks
    switch (p->lattice) {
      case HQ_E8: return launch_encode_tiled<kE8>(a, t, xt, st);
      case HQ_D4: return launch_encode_tiled<kD4>(a, t, xt, st);
      case HQ_A2: return launch_encode_tiled<kA2>(a, t, xt, st);
      default: return launch_encode_tiled<kZ>(a, t, xt, st);
    }
  }
  const bool kv = kv_variant(p);
  const uint32_t lw = a.lds_words;
  switch (p->lattice) {
    case HQ_E8: return launch_encode_lat<kE8>(a, t, a.nwg, lw, xt, kv, st);
    case HQ_D4: return launch_encode_lat<kD4>(a, t, a.nwg, lw, xt, kv, st);
    case HQ_A2: return launch_encode_lat<kA2>(a, t, a.nwg, lw, xt, kv, st);
    default: return launch_encode_lat<kZ>(a, t, a.nwg, lw, xt, kv, st);
  }
}

int hq_launch_encode_group(const hq_plan_s* p, const hq_encode_group_args& g, uint32_t nwg,
                           uint32_t lds_words, int xt, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  const bool kv = kv_variant(p);
  switch (p->lattice) {
    case HQ_E8: return launch_encode_lat<kE8>(g, g.thr, nwg, lds_words, xt, kv, st);
    case HQ_D4: return launch_encode_lat<kD4>(g, g.thr, nwg, lds_words, xt, kv, st);
    case HQ_A2: return launch_encode_lat<kA2>(g, g.thr, nwg, lds_words, xt, kv, st);
    default: return launch_encode_lat<kZ>(g, g.thr, nwg, lds_words, xt, kv, st);
  }
}

int hq_launch_zero(void* ptr, size_t bytes, void* stream) {
  const size_t n = bytes / 4;
  if (n == 0) return 0;
  hipLaunchKernelGGL(hq_zero_kernel, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0,
                     (hipStream_t)stream, (uint32_t*)ptr, n);
  return (int)hipGetLastError();
}

// ------------------------------------------------------------ fixed scratch
// The look-back scratch of hq_encode_noalloc, for callers that cannot
// allocate: one array per device, alive until the process ends.  Host code
// never passes the array's name to a kernel (on the host it is a stand-in,
// not a device address); it uses the address hipGetSymbolAddress returns for
// the current device, looked up once per device.
static __device__ __align__(256) unsigned char scratch[HQ_NOALLOC_SCAN_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];
}  // namespace

int hq_noalloc_scan(void** ptr, void* stream) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return -1;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return -1;
    // the epoch word and every status word start at zero (a fill kernel, so
    // a first call under graph capture records no memset node)
    if (hq_launch_zero(p, HQ_NOALLOC_SCAN_BYTES, stream) != 0) return -1;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return 0;
}

