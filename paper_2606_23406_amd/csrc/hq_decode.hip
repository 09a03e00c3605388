// HyperQuant decode kernels for gfx950 (MI355X); the lane layout is in hq_device.h.
#include <algorithm>
#include <type_traits>

#include "hq_device.h"
#include "hq_lds.h"

#pragma clang fp contract(off)

namespace {

// 16 output bytes that this kernel does not read again: past the caches, which
// keep the payload.  A layer of seven E8@4 matrices takes 176 us with plain stores
// and 168 so (178 and 148 where the same streams are decoded again), 32768 x 1024
// KV rows 50.8 and 48.9.  A product of 16 rows that reads the matrix next finds
// less of it in the caches: with its decode, 14336 x 4096 takes 67 and 73 us,
// 2048 x 4096 28.8 and 27.3.
__device__ __forceinline__ void store_stream(void* p, uint4 v) {
  __builtin_nontemporal_store((v4u_t){v.x, v.y, v.z, v.w}, (v4u_t*)p);
}

// SPW consecutive sub-streams per wave: 4, or 1 for launches too small to
// fill the chip with four per wave.
template <int LAT, int MODE, bool KV, int SPW = HQ_DEC_SUBS_PER_WAVE>
__device__ __forceinline__ void decode_wg(const hq_decode_args& A, const uint32_t wgi) {
  extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
  __shared__ uint32_t s_sel[256];
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t wave = readfirst((uint32_t)(tid >> 6));
  uint32_t* buf = smem + wave * (A.lds_words + 66);
  uint32_t* starts = buf + A.lds_words + 2;
  const bool use_rot = KV && A.rotation == HQ_ROT_SIGNS;
  const bool use_dither = KV && A.dither;
  const bool fp16_norm = KV && A.norm_fp16;
  s_sel[tid] = kByteSelect.e[tid];  // 256 threads, one entry each
  __syncthreads();

  // this wave's sub-streams: SPW consecutive ones; their table entries are
  // read at once, each one's payload one sub-stream ahead
  const uint32_t sub0 = (wgi * HQ_WAVES_PER_WG + wave) * SPW;
  const uint32_t nsub = (uint32_t)A.nsub;
  uint32_t off[SPW + 1], kbs[SPW];
#pragma unroll
  for (int i = 0; i <= SPW; ++i) {
    const uint32_t sub = sub0 + (uint32_t)i;
    off[i] = sub <= nsub ? readfirst(A.offsets[(uint32_t)A.first_sub + sub]) : 0u;
    if (i < SPW)
      kbs[i] = sub < nsub ? readfirst(A.kparam[(uint32_t)A.first_sub + sub]) : 0u;
  }
  DecHead head = dec_head<LAT>(A, sub0 < nsub, off[0], off[1], kbs[0], lane);
  const uint32_t spr = (uint32_t)A.spr;
  // plain weight plans transform their integer codes on the matrix cores, in
  // that layout's lane order; group grp is block grp % 16 of tile grp / 16
  constexpr bool PI = MODE <= 1 && !KV && LAT != kA2;
  const uint32_t ltile = PI ? (uint32_t)(lane >> 2) & 3u : (uint32_t)lane >> 4;
  const uint32_t grp = PI ? ltile * 16u + ((uint32_t)(lane & 3) | (uint32_t)(lane >> 4) << 2) : (uint32_t)lane;
  const typename std::conditional<PI, MfmaRht, TwSigns>::type sg(lane);
  const uint32_t sbits = use_rot ? sign_bits8(A.smask, (lane & 15) * 8) : 0u;
  // tile factors g = r_s / (alpha n), once for the wave's tiles: lane l
  // takes sub-stream l & 3 (SPW = 4) or the one sub-stream, and its tile
  // (rows are contiguous, 4 tiles per sub-stream; a quad shares its tile);
  // with four, sub-stream i reads them back by a quad broadcast
  static_assert(SPW == 4 || SPW == 1, "one sub-stream per lane of a quad, or one per wave");
  float gm = 0.0f;
  {
    const uint32_t subq = sub0 + (SPW == 4 ? (uint32_t)(lane & 3) : 0u);
    if (subq < nsub) {
      // the casts (MODE >= 2) also serve long-tile weight plans: tile of the
      // 128 columns at flat position subq * 512 + 128 (lane >> 4)
      const int64_t t =
          MODE >= 2 ? A.first_row * A.tpr + (int64_t)((((uint64_t)subq << 9) + (uint64_t)((lane >> 4) << 7)) >>
                                                       __builtin_ctz((uint32_t)A.tile))
                    : A.first_row * A.tpr + 4 * (int64_t)subq + ltile;
      const float rs = fp16_norm ? (float)((const _Float16*)A.norms)[t] : ((const float*)A.norms)[t];
      gm = rs / A.alpha_n;
    }
  }

  uint32_t lrow = sub0 / spr, csub = sub0 - lrow * spr;  // row and sub-stream in it, advanced below
#pragma unroll
  for (int i = 0; i < SPW; ++i) {
    const uint32_t sub = sub0 + (uint32_t)i;
    if (sub >= nsub) break;
    DecHead next;
    if (i + 1 < SPW)
      next = dec_head<LAT>(A, sub + 1 < nsub, off[i + 1], off[i + 2], kbs[i + 1], lane);
    const uint32_t col = csub * HQ_SUB + 8u * grp;
    const int64_t grow = A.first_row + lrow;
    // output signs, loaded before the bit walk
    uint4 sw = make_uint4(0u, 0u, 0u, 0u);
    if (MODE == 1) sw = *(const uint4*)(A.dsign16 + (col >> 1));

    uint32_t sym[8];
    bool small;
    const unsigned long long bad = decode_symbols<LAT>(A, head, lane, grp, buf, starts, s_sel, sym, small);
    if (bad && A.stats) {
      // count the sub-stream once (its first failing lane reports)
      if ((unsigned)lane == (unsigned)__builtin_ctzll(bad)) {
        atomicAdd(&A.stats->corrupt_substreams, 1u);
        atomicCAS(&A.stats->status, 0u, (uint32_t)HQ_ERR_CORRUPT);
      }
    }
    int32_t c[8];
    unstrip8<LAT>(sym, c);
    float g = SPW == 1 ? gm
                       : (i == 0 ? quad_bcast<0>(gm)
                                 : (i == 1 ? quad_bcast<1>(gm) : (i == 2 ? quad_bcast<2>(gm) : quad_bcast<3>(gm))));
    if (bad) g = 0.0f;  // a corrupt sub-stream decodes as zeros, dither included

    if constexpr (MODE == 2) {
      uint32_t clamps = 0;
      const int32_t hi = max(max(max(c[0], c[1]), max(c[2], c[3])), max(max(c[4], c[5]), max(c[6], c[7])));
      const int32_t lo = min(min(min(c[0], c[1]), min(c[2], c[3])), min(min(c[4], c[5]), min(c[6], c[7])));
      if (__ballot(hi > 127 || lo < -127) != 0ull) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          clamps += c[j] > 127 || c[j] < -127;
          c[j] = max(min(c[j], 127), -127);
        }
      }
      uint32_t packed[2];
#pragma unroll
      for (int j = 0; j < 2; ++j)  // the low bytes of four codes
        packed[j] = __builtin_amdgcn_perm((uint32_t)c[4 * j + 1], (uint32_t)c[4 * j], 0x0C0C0400u) |
                    __builtin_amdgcn_perm((uint32_t)c[4 * j + 3], (uint32_t)c[4 * j + 2], 0x04000C0Cu);
      int8_t* out = (int8_t*)A.y + (int64_t)lrow * A.ld + col;
      *(uint2*)out = make_uint2(packed[0], packed[1]);
      if ((col & (uint32_t)(A.tile - 1)) == 0)
        A.g[(int64_t)lrow * A.tpr + (col >> __builtin_ctz((uint32_t)A.tile))] = g;
      if (clamps && A.stats) atomicAdd(&A.stats->clamps, clamps);
    } else if constexpr (MODE == 4) {
      // the MXFP4 cast of the reconstruction (Sec. 4.8, Sec. 6.4): v = g c in
      // the rotated coordinates (one fp32 product); blocks of 32 values (four
      // lanes, inside one tile) share X = floor(log2 amax) - 2, and each value
      // becomes E2M1(v / 2^X), two per byte (the even k in the low nibble),
      // the scale byte X + 127
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = (float)c[j] * g;
      int32_t X;
      const uint32_t packed = mxfp4_x8(v, X);
      uint8_t* out = (uint8_t*)A.y + (int64_t)lrow * A.ld + (col >> 1);
      *(uint32_t*)out = packed;
      if ((lane & 3) == 0) A.mxs[(int64_t)lrow * (A.spr * (HQ_SUB / 32)) + (col >> 5)] = (uint8_t)(X + 127);
    } else if constexpr (MODE == 3) {
      // the fp8 cast (Sec. 4.8): E4M3 of each code, round to nearest even,
      // magnitudes beyond 448 saturated and counted
      float v[8];
      uint32_t clamps = 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        v[j] = (float)c[j];
        if (v[j] > 448.0f) { v[j] = 448.0f; ++clamps; }
        if (v[j] < -448.0f) { v[j] = -448.0f; ++clamps; }
      }
      const uint32_t w0 = e4m3x4(v[0], v[1], v[2], v[3]), w1 = e4m3x4(v[4], v[5], v[6], v[7]);
      uint8_t* out = (uint8_t*)A.y + (int64_t)lrow * A.ld + col;
      *(uint2*)out = make_uint2(w0, w1);
      if ((col & (uint32_t)(A.tile - 1)) == 0)
        A.g[(int64_t)lrow * A.tpr + (col >> __builtin_ctz((uint32_t)A.tile))] = g;
      if (clamps && A.stats) atomicAdd(&A.stats->clamps, clamps);
    } else {
      // y = D H^T (S) (code - U) * r / (alpha n); the integer codes make the
      // transform exact in fp32 (|sum| <= 128 * 65536 < 2^24) whenever there
      // is no dither
      float y[8];
      if constexpr (PI) {
        if (small) {
          uint32_t pair[4];
#pragma unroll
          for (int j = 0; j < 4; ++j)
            pair[j] = ((uint32_t)c[2 * j + 1] << 16) + ((uint32_t)c[2 * j] + kCodeBias);
          sg.small(pair, y);
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j) y[j] = (float)c[j];
          sg.any(y, lane);
        }
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) y[j] = code_coord<LAT>(c[j], j);
        if (use_dither) {
          float u[8];
          dither8<LAT>(A.dither_seed, grow, col, u);
#pragma unroll
          for (int j = 0; j < 8; ++j) y[j] = y[j] - u[j];
        }
        if (use_rot) {
#pragma unroll
          for (int j = 0; j < 8; ++j) y[j] = flip(y[j], sbits, j);
        }
        fwht128_tw(y, sg);
      }
      const float g_tw = xor_sign(g, sg.sigma);
#pragma unroll
      for (int j = 0; j < 8; ++j) y[j] = y[j] * g_tw;
      if constexpr (MODE == 0) {
        const uint32_t dbits = sign_bits8(A.dmask, col);
#pragma unroll
        for (int j = 0; j < 8; ++j) y[j] = flip(y[j], dbits, j);
        float4* out = (float4*)((float*)A.y + (int64_t)lrow * A.ld + col);
        out[0] = make_float4(y[0], y[1], y[2], y[3]);
        out[1] = make_float4(y[4], y[5], y[6], y[7]);
      } else {
        uint4 o;
        o.x = cvt_pk_bf16(y[0], y[1]) ^ sw.x;
        o.y = cvt_pk_bf16(y[2], y[3]) ^ sw.y;
        o.z = cvt_pk_bf16(y[4], y[5]) ^ sw.z;
        o.w = cvt_pk_bf16(y[6], y[7]) ^ sw.w;
        store_stream((uint16_t*)A.y + (int64_t)lrow * A.ld + col, o);
      }
    }
    if (i + 1 < SPW) head = next;
    if (++csub == spr) {
      csub = 0;
      ++lrow;
    }
  }
}

// Block b of a sub-stream of B 512-symbol blocks (already in `buf`, Wl
// words): its remainder fields sit at bit b 64 lrem, its unary codes begin
// at bit ustart (anywhere in a word: the bits below it belong to block
// b - 1).  Lane l's codes start just past this block's terminator 8 l - 1,
// found by a popcount scan from ustart that stops once all 64 starts are
// known.  Returns false (in every lane) for a parse that runs out of words;
// `uend` becomes the bit past the block's last code.
template <int LAT>
__device__ __forceinline__ bool decode_block_mb(const uint32_t* buf, uint32_t Wl, uint32_t* starts,
                                                uint32_t ustart, uint32_t rem_base, uint32_t k0,
                                                uint32_t k1, int lane, bool ok, uint32_t* sym,
                                                uint32_t& uend) {
  const uint32_t lrem = lane_rem_bits<LAT>(k0, k1);
  const uint32_t nbits = 32u * Wl;
  starts[lane] = (lane == 0) ? ustart : 0xFFFFFFFFu;
  wave_sync_lds();
  const uint32_t uw0 = ustart >> 5;
  const uint32_t nuw = (ok && Wl > uw0) ? Wl - uw0 : 0u;
  const uint32_t lowmask = ~((1u << (ustart & 31u)) - 1u);
  uint32_t carry = 0;
  for (uint32_t base = 0; base < nuw && carry < 504u; base += 64) {
    const uint32_t wi = base + lane;
    uint32_t v = (wi < nuw) ? buf[uw0 + wi] : 0u;
    if (wi == 0u) v &= lowmask;
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
  uint32_t pos = starts[lane];
  ok = ok && pos < nbits;
  uint32_t qv[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) qv[j] = 0;
  if (ok) {
    // the q_j: zeros before each of the lane's 8 terminators, a 64-bit
    // window sliding along the buffer
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
  uend = __builtin_amdgcn_readlane(pos, 63);
  // the lane's 8 remainders
  const uint32_t rpos = rem_base + __umul24((uint32_t)lane, lrem);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const uint32_t kk = sym_class<LAT>(j) ? k1 : k0;
    const uint32_t r = (ok && kk) ? (uint32_t)load_bits64(buf, rpos + rem_offset<LAT>(j, k0, k1), Wl) : 0u;
    sym[j] = (qv[j] << kk) | (r & ((1u << kk) - 1u));
  }
  return __ballot(!ok) == 0ull;
}

// Long tiles (weights, bf16 or fp32 out): the wave's four consecutive
// sub-streams are decoded first and kept as lattice coordinates, then the
// tiles they form are transformed together (fwht_tiled) and denormalized.
// A corrupt sub-stream's codes count as zeros in its tile.
template <int LAT, int MODE>
__device__ __forceinline__ void decode_wg_tiled(const hq_decode_args& A, const uint32_t wgi) {
  extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
  __shared__ uint32_t s_sel[256];
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t wave = readfirst((uint32_t)(tid >> 6));
  uint32_t* buf = smem + wave * (A.lds_words + 66);
  uint32_t* starts = buf + A.lds_words + 2;
  s_sel[tid] = kByteSelect.e[tid];  // 256 threads, one entry each
  __syncthreads();

  const uint32_t n = (uint32_t)A.tile;
  const uint32_t mb = (uint32_t)A.mb;
  float y[HQ_DEC_SUBS_PER_WAVE][8];
  // the wave's four consecutive 512-symbol blocks (sub-streams when mb = 1)
  const uint32_t sub0 = (wgi * HQ_WAVES_PER_WG + wave) * HQ_DEC_SUBS_PER_WAVE;
  const uint32_t nsub = (uint32_t)A.nsub * mb;  // blocks
  const uint32_t spr = (uint32_t)A.spr * mb;
  const TwSigns sg(lane);
  if (mb > 1u) {
    // sub-streams of mb blocks: the whole sub-stream goes to the wave's
    // buffer, then its blocks are parsed in order (each block's unary codes
    // start where the previous block's end); a corrupt sub-stream decodes
    // as zeros in all of its blocks
    for (uint32_t j = 0; j < HQ_DEC_SUBS_PER_WAVE / mb; ++j) {
      const uint32_t s = sub0 / mb + j;  // sub-stream
      const bool act = s < (uint32_t)A.nsub;
      uint32_t start = 0, end = 0, kb = 0;
      if (act) {
        start = readfirst(A.offsets[(uint32_t)A.first_sub + s]);
        end = readfirst(A.offsets[(uint32_t)A.first_sub + s + 1]);
        kb = readfirst(A.kparam[(uint32_t)A.first_sub + s]);
      }
      const uint32_t k0 = (LAT == kA2) ? (kb & 15u) : kb;
      const uint32_t k1 = (LAT == kA2) ? (kb >> 4) : (LAT == kD4 ? (k0 > 0 ? k0 - 1 : 0) : k0);
      const uint32_t Rb = 64u * lane_rem_bits<LAT>(k0, k1);
      const uint32_t W = end - start;
      bool ok = act && end >= start && (int64_t)end <= A.cap_words && W <= A.lds_words &&
                k0 <= HQ_KMAX && mb * Rb <= 32u * W;
      const uint32_t Wl = ok ? W : 0u;
      for (uint32_t w = lane; w < Wl; w += 64) buf[w] = A.payload[(uint64_t)start + w];
      if (lane < 2) buf[Wl + lane] = 0u;  // two zero words past the end
      wave_sync_lds();
      uint32_t ustart = mb * Rb;
      for (uint32_t b = 0; b < mb; ++b) {
        uint32_t sym[8], uend;
        ok = decode_block_mb<LAT>(buf, Wl, starts, ustart, b * Rb, k0, k1, lane, ok, sym, uend);
        ustart = uend;
        int32_t c[8];
        unstrip8<LAT>(sym, c);
        const uint32_t i = j * mb + b;
#pragma unroll
        for (int q = 0; q < HQ_DEC_SUBS_PER_WAVE; ++q)
          if ((uint32_t)q == i)
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) y[q][jj] = act ? code_coord<LAT>(c[jj], jj) : 0.0f;
      }
      if (act && !ok) {
#pragma unroll
        for (int q = 0; q < HQ_DEC_SUBS_PER_WAVE; ++q)
          if ((uint32_t)q / mb == j)
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) y[q][jj] = 0.0f;
        if (A.stats && lane == 0) {
          atomicAdd(&A.stats->corrupt_substreams, 1u);
          atomicCAS(&A.stats->status, 0u, (uint32_t)HQ_ERR_CORRUPT);
        }
      }
    }
  } else {
  uint32_t off[HQ_DEC_SUBS_PER_WAVE + 1], kbs[HQ_DEC_SUBS_PER_WAVE];
#pragma unroll
  for (int i = 0; i <= HQ_DEC_SUBS_PER_WAVE; ++i) {
    const uint32_t sub = sub0 + (uint32_t)i;
    off[i] = sub <= nsub ? readfirst(A.offsets[(uint32_t)A.first_sub + sub]) : 0u;
    if (i < HQ_DEC_SUBS_PER_WAVE)
      kbs[i] = sub < nsub ? readfirst(A.kparam[(uint32_t)A.first_sub + sub]) : 0u;
  }
  DecHead head = dec_head<LAT>(A, sub0 < nsub, off[0], off[1], kbs[0], lane);
#pragma unroll
  for (int i = 0; i < HQ_DEC_SUBS_PER_WAVE; ++i) {
    const uint32_t sub = sub0 + (uint32_t)i;
    DecHead next;
    if (i + 1 < HQ_DEC_SUBS_PER_WAVE)
      next = dec_head<LAT>(A, sub + 1 < nsub, off[i + 1], off[i + 2], kbs[i + 1], lane);
    if (sub < nsub) {
      uint32_t sym[8];
      bool small;
      const unsigned long long bad =
          decode_symbols<LAT>(A, head, lane, (uint32_t)lane, buf, starts, s_sel, sym, small);
      if (bad && A.stats && (unsigned)lane == (unsigned)__builtin_ctzll(bad)) {
        atomicAdd(&A.stats->corrupt_substreams, 1u);
        atomicCAS(&A.stats->status, 0u, (uint32_t)HQ_ERR_CORRUPT);
      }
      int32_t c[8];
      unstrip8<LAT>(sym, c);
#pragma unroll
      for (int j = 0; j < 8; ++j) y[i][j] = code_coord<LAT>(c[j], j);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) y[i][j] = 0.0f;
    }
    if (i + 1 < HQ_DEC_SUBS_PER_WAVE) head = next;
  }
  }  // one block per sub-stream
  // y = D H^T code * r / (alpha n): the tiles' transforms, then each lane
  // its own tile's factor
  const uint32_t sigma = fwht_tiled(y, lane, n, sg);
#pragma unroll
  for (int i = 0; i < HQ_DEC_SUBS_PER_WAVE; ++i) {
    const uint32_t sub = sub0 + (uint32_t)i;
    if (sub >= nsub) break;
    const uint32_t lrow = sub / spr;
    const uint32_t col = (sub - lrow * spr) * HQ_SUB + 8u * (uint32_t)lane;
    const uint64_t flat = (uint64_t)sub * HQ_SUB + 8u * (uint32_t)lane;
    const float rs = ((const float*)A.norms)[A.first_row * A.tpr + (int64_t)(flat / n)];
    const float g_tw = xor_sign(rs / A.alpha_n, sigma);
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = y[i][j] * g_tw;
    if constexpr (MODE == 0) {
      const uint32_t dbits = sign_bits8(A.dmask, col);
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = flip(v[j], dbits, j);
      float4* out = (float4*)((float*)A.y + (int64_t)lrow * A.ld + col);
      out[0] = make_float4(v[0], v[1], v[2], v[3]);
      out[1] = make_float4(v[4], v[5], v[6], v[7]);
    } else {
      const uint4 sw = *(const uint4*)(A.dsign16 + (col >> 1));
      uint4 o;
      o.x = cvt_pk_bf16(v[0], v[1]) ^ sw.x;
      o.y = cvt_pk_bf16(v[2], v[3]) ^ sw.y;
      o.z = cvt_pk_bf16(v[4], v[5]) ^ sw.z;
      o.w = cvt_pk_bf16(v[6], v[7]) ^ sw.w;
      *(uint4*)((uint16_t*)A.y + (int64_t)lrow * A.ld + col) = o;
    }
  }
}

template <int LAT, int MODE>
__global__ __launch_bounds__(256) void hq_decode_tiled_kernel(hq_decode_args A) {
  decode_wg_tiled<LAT, MODE>(A, blockIdx.x);
}

// ------------------------------------------------------------ qjl decode on the matrix cores
// KV streams with the qjl rotation, decoded to fp32 or bf16.  S^T y is a
// dense 128 x 128 contraction per tile, so it runs on the fp32 matrix cores
// (v_mfma_f32_16x16x4_f32) instead of the VALU with S streamed from LDS.
// A workgroup takes 16 consecutive sub-streams (64 tiles) per pass:
//  1. each wave decodes its four sub-streams, undithers them and writes
//     y = code - U into the workgroup's tile array Y in LDS (tile rows of
//     kQjlRow floats: the 16 rows one operand load reads fall in distinct
//     banks);
//  2. wave w forms columns 32 w .. 32 w + 31 of Z = Y S for all 64 tiles
//     (row z of Z is (S^T y)^T) with its 32 columns of S held in registers,
//     then, once every wave has read Y, writes them over it;
//  3. each wave finishes its own tiles from Z: inverse RHT, scale, signs,
//     store.
// The contraction sums in the matrix cores' order, so the output equals
// the oracle's left-to-right fp32 sums to rounding, not bit for bit.
constexpr int kQjlRow = 130;            // floats per tile row of Y
constexpr int kQjlTiles = 64;           // tiles per workgroup pass (16 sub-streams)

// Held to three waves per SIMD (168 registers): E8 takes 172 of its own accord,
// and 20000 x 1024 dithered rows then 106 us instead of 92.
template <int LAT, int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void hq_decode_qjl_kernel(hq_decode_args A) {
  extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
  __shared__ uint32_t s_sel[256];
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t wave = readfirst((uint32_t)(tid >> 6));
  uint32_t* buf = smem + wave * (A.lds_words + 66);
  uint32_t* starts = buf + A.lds_words + 2;
  float* const Y = (float*)(smem + HQ_WAVES_PER_WG * (A.lds_words + 66));
  s_sel[tid] = kByteSelect.e[tid];
  // B operands: step s covers k = 4 s .. 4 s + 3 (lane / 16 picks k), block
  // cb the columns n = 32 wave + 16 cb + lane % 16
  float sb[32][2];
#pragma unroll
  for (int s = 0; s < 32; ++s) {
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
      sb[s][cb] = A.qjl[(4 * s + (lane >> 4)) * HQ_TILE + 32 * (int)wave + 16 * cb + (lane & 15)];
  }
  __syncthreads();
  const TwSigns sg(lane);
  const uint32_t nsub = (uint32_t)A.nsub, spr = (uint32_t)A.spr;
  const uint32_t ngroups = (nsub + 15u) / 16u;
  for (uint32_t grp = blockIdx.x; grp < ngroups; grp += gridDim.x) {
    const uint32_t sub0 = grp * 16u + wave * 4u;
    // ---- 1. decode into Y rows wave * 16 + 4 i + lane / 16
    float gi[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t sub = sub0 + (uint32_t)i;
      gi[i] = 0.0f;
      if (sub >= nsub) continue;  // wave-uniform; the row's Z is never stored
      const uint32_t o0 = readfirst(A.offsets[(uint32_t)A.first_sub + sub]);
      const uint32_t o1 = readfirst(A.offsets[(uint32_t)A.first_sub + sub + 1]);
      const uint32_t kb = readfirst(A.kparam[(uint32_t)A.first_sub + sub]);
      const DecHead head = dec_head<LAT>(A, true, o0, o1, kb, lane);
      const int64_t t = A.first_row * A.tpr + 4 * (int64_t)sub + (lane >> 4);
      const float rs = A.norm_fp16 ? (float)((const _Float16*)A.norms)[t] : ((const float*)A.norms)[t];
      const uint32_t lrow = sub / spr;
      const uint32_t col = (sub - lrow * spr) * HQ_SUB + 8u * (uint32_t)lane;
      uint32_t sym[8];
      bool small;
      const unsigned long long bad =
          decode_symbols<LAT>(A, head, lane, (uint32_t)lane, buf, starts, s_sel, sym, small);
      if (bad && A.stats && (unsigned)lane == (unsigned)__builtin_ctzll(bad)) {
        atomicAdd(&A.stats->corrupt_substreams, 1u);
        atomicCAS(&A.stats->status, 0u, (uint32_t)HQ_ERR_CORRUPT);
      }
      gi[i] = bad ? 0.0f : rs / A.alpha_n;  // a corrupt sub-stream decodes as zeros
      int32_t c[8];
      unstrip8<LAT>(sym, c);
      float y[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) y[j] = code_coord<LAT>(c[j], j);
      if (A.dither) {
        float u[8];
        // (the one-coset form takes 12 registers more beside S's 64)
        dither8<LAT, true>(A.dither_seed, A.first_row + lrow, col, u);
#pragma unroll
        for (int j = 0; j < 8; ++j) y[j] = y[j] - u[j];
      }
      float* row = Y + (wave * 16u + 4u * (uint32_t)i + (uint32_t)(lane >> 4)) * kQjlRow + (lane & 15) * 8;
#pragma unroll
      for (int j = 0; j < 8; j += 2) *(float2*)(row + j) = make_float2(y[j], y[j + 1]);
    }
    __syncthreads();
    // ---- 2. Z[:, 32 wave .. +31] = Y S
    v4f_t acc[4][2];
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) {
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) acc[rb][cb] = v4f_t{0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll  // sb is indexed by s: only a full unroll keeps it in registers
    for (int s = 0; s < 32; ++s) {
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) {
        const float a = Y[(rb * 16 + (lane & 15)) * kQjlRow + 4 * s + (lane >> 4)];
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
          acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, sb[s][cb], acc[rb][cb], 0, 0, 0);
      }
    }
    __syncthreads();  // every wave has read Y
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) {
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          Y[(rb * 16 + 4 * (lane >> 4) + r) * kQjlRow + 32 * (int)wave + 16 * cb + (lane & 15)] = acc[rb][cb][r];
      }
    }
    __syncthreads();
    // ---- 3. this wave's tiles: inverse RHT, scale, signs, store
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t sub = sub0 + (uint32_t)i;
      if (sub >= nsub) break;
      const uint32_t lrow = sub / spr;
      const uint32_t col = (sub - lrow * spr) * HQ_SUB + 8u * (uint32_t)lane;
      const float* row = Y + (wave * 16u + 4u * (uint32_t)i + (uint32_t)(lane >> 4)) * kQjlRow + (lane & 15) * 8;
      float y[8];
#pragma unroll
      for (int j = 0; j < 8; j += 2) {
        const float2 v = *(const float2*)(row + j);
        y[j] = v.x;
        y[j + 1] = v.y;
      }
      fwht128_tw(y, sg);
      const float g_tw = xor_sign(gi[i], sg.sigma);
#pragma unroll
      for (int j = 0; j < 8; ++j) y[j] = y[j] * g_tw;
      if constexpr (MODE == 0) {
        const uint32_t dbits = sign_bits8(A.dmask, col);
#pragma unroll
        for (int j = 0; j < 8; ++j) y[j] = flip(y[j], dbits, j);
        float4* out = (float4*)((float*)A.y + (int64_t)lrow * A.ld + col);
        out[0] = make_float4(y[0], y[1], y[2], y[3]);
        out[1] = make_float4(y[4], y[5], y[6], y[7]);
      } else {
        const uint4 sw = *(const uint4*)(A.dsign16 + (col >> 1));
        uint4 o;
        o.x = cvt_pk_bf16(y[0], y[1]) ^ sw.x;
        o.y = cvt_pk_bf16(y[2], y[3]) ^ sw.y;
        o.z = cvt_pk_bf16(y[4], y[5]) ^ sw.z;
        o.w = cvt_pk_bf16(y[6], y[7]) ^ sw.w;
        *(uint4*)((uint16_t*)A.y + (int64_t)lrow * A.ld + col) = o;
      }
    }
  }
}

// (256, 2): at most 256 registers, so that the matrix cores' results go to
// plain ones (otherwise four copies to and eight from accumulation registers
// per sub-stream).
template <int LAT, int MODE, bool KV>
__global__ __launch_bounds__(256, 2) void hq_decode_kernel(hq_decode_args A) {
  decode_wg<LAT, MODE, KV>(A, blockIdx.x);
}

// Single matrices of fewer than HQ_DEC_SMALL sub-streams: one per wave.
template <int LAT, int MODE, bool KV>
__global__ __launch_bounds__(256, 2) void hq_decode_small_kernel(hq_decode_args A) {
  decode_wg<LAT, MODE, KV, 1>(A, blockIdx.x);
}

template <int LAT, int MODE, bool KV>
__global__ __launch_bounds__(256, 2) void hq_decode_group_kernel(hq_decode_group_args G) {
  int mi = 0;
  for (int i = 1; i < G.count; ++i) mi = blockIdx.x >= G.wg_begin[i] ? i : mi;
  decode_wg<LAT, MODE, KV>(G.m[mi], blockIdx.x - G.wg_begin[mi]);
}

// One decode launch: a single matrix (hq_decode_args) or a group.
template <int LAT, int MODE, bool KV, typename Args>
void launch_decode_kernel(const Args& a, uint32_t nwg, size_t lds, hipStream_t st) {
  static hq_lds_granted granted;
  hq_allow_lds(sizeof(Args) == sizeof(hq_decode_args) ? (const void*)hq_decode_kernel<LAT, MODE, KV>
                                                      : (const void*)hq_decode_group_kernel<LAT, MODE, KV>,
               lds, granted);
  if constexpr (sizeof(Args) == sizeof(hq_decode_args))
    hipLaunchKernelGGL((hq_decode_kernel<LAT, MODE, KV>), dim3(nwg), dim3(256), lds, st, a);
  else
    hipLaunchKernelGGL((hq_decode_group_kernel<LAT, MODE, KV>), dim3(nwg), dim3(256), lds, st, a);
}

template <int LAT, typename Args>
int launch_decode_lat(const Args& a, uint32_t nwg, uint32_t lds_words, int mode, bool kv,
                      hipStream_t st) {
  const size_t lds = (size_t)(lds_words + 66) * HQ_WAVES_PER_WG * sizeof(uint32_t);
  if (mode == 0) {
    if (kv) launch_decode_kernel<LAT, 0, true>(a, nwg, lds, st);
    else launch_decode_kernel<LAT, 0, false>(a, nwg, lds, st);
  } else if (mode == 1) {
    if (kv) launch_decode_kernel<LAT, 1, true>(a, nwg, lds, st);
    else launch_decode_kernel<LAT, 1, false>(a, nwg, lds, st);
  } else {
    if (kv) launch_decode_kernel<LAT, 2, true>(a, nwg, lds, st);
    else launch_decode_kernel<LAT, 2, false>(a, nwg, lds, st);
  }
  return (int)hipGetLastError();
}

template <int LAT>
int launch_decode_tiled(const hq_decode_args& a, uint32_t nwg, int mode, hipStream_t st) {
  const size_t lds = (size_t)(a.lds_words + 66) * HQ_WAVES_PER_WG * sizeof(uint32_t);
  static hq_lds_granted granted_0, granted_1;
  if (mode == 0) {
    hq_allow_lds((const void*)hq_decode_tiled_kernel<LAT, 0>, lds, granted_0);
    hipLaunchKernelGGL((hq_decode_tiled_kernel<LAT, 0>), dim3(nwg), dim3(256), lds, st, a);
  } else {
    hq_allow_lds((const void*)hq_decode_tiled_kernel<LAT, 1>, lds, granted_1);
    hipLaunchKernelGGL((hq_decode_tiled_kernel<LAT, 1>), dim3(nwg), dim3(256), lds, st, a);
  }
  return (int)hipGetLastError();
}

}  // namespace

static uint32_t decode_wgs(int64_t nsub) {
  constexpr int per_wg = HQ_WAVES_PER_WG * HQ_DEC_SUBS_PER_WAVE;
  return (uint32_t)((nsub + per_wg - 1) / per_wg);
}

// qjl streams of tile 128: the matrix-core decode, a grid of workgroups
// that each take every gridDim-th pass of 16 sub-streams.
template <int LAT>
int launch_decode_qjl(const hq_decode_args& a, int mode, hipStream_t st) {
  const int64_t ngroups = (a.nsub + 15) / 16;
  if (ngroups == 0) return 0;
  const uint32_t nwg = (uint32_t)std::min<int64_t>(ngroups, 2048);
  const size_t lds = (size_t)(a.lds_words + 66) * HQ_WAVES_PER_WG * sizeof(uint32_t) +
                     (size_t)kQjlTiles * kQjlRow * sizeof(float);
  static hq_lds_granted granted0, granted1;
  if (mode == 0) {
    hq_allow_lds((const void*)hq_decode_qjl_kernel<LAT, 0>, lds, granted0);
    hipLaunchKernelGGL((hq_decode_qjl_kernel<LAT, 0>), dim3(nwg), dim3(256), lds, st, a);
  } else {
    hq_allow_lds((const void*)hq_decode_qjl_kernel<LAT, 1>, lds, granted1);
    hipLaunchKernelGGL((hq_decode_qjl_kernel<LAT, 1>), dim3(nwg), dim3(256), lds, st, a);
  }
  return (int)hipGetLastError();
}

// A single matrix of fewer than HQ_DEC_SMALL sub-streams, fp32 or bf16 out:
// one sub-stream per wave, so that its workgroups spread over more of the
// chip than four per wave would.
template <int LAT>
int launch_decode_small(const hq_decode_args& a, int mode, bool kv, hipStream_t st) {
  const uint32_t nwg = (uint32_t)((a.nsub + HQ_WAVES_PER_WG - 1) / HQ_WAVES_PER_WG);
  const size_t lds = (size_t)(a.lds_words + 66) * HQ_WAVES_PER_WG * sizeof(uint32_t);
  static hq_lds_granted granted[4];
#define HQ_SMALL_CASE(M, K, I)                                                             \
  hq_allow_lds((const void*)hq_decode_small_kernel<LAT, M, K>, lds, granted[I]);           \
  hipLaunchKernelGGL((hq_decode_small_kernel<LAT, M, K>), dim3(nwg), dim3(256), lds, st, a)
  if (mode == 0) {
    if (kv) { HQ_SMALL_CASE(0, true, 0); } else { HQ_SMALL_CASE(0, false, 1); }
  } else {
    if (kv) { HQ_SMALL_CASE(1, true, 2); } else { HQ_SMALL_CASE(1, false, 3); }
  }
#undef HQ_SMALL_CASE
  return (int)hipGetLastError();
}

int hq_launch_decode(const hq_plan_s* p, const hq_decode_args& a, int yt, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  const int mode = (yt == HQ_FP32) ? 0 : 1;
  const bool kv = kv_variant(p);
  const uint32_t nwg = decode_wgs(a.nsub * a.mb), lw = a.lds_words;
  if (a.qjl && p->tile == HQ_TILE && p->substream == HQ_SUB) {
    switch (p->lattice) {
      case HQ_E8: return launch_decode_qjl<kE8>(a, mode, st);
      case HQ_D4: return launch_decode_qjl<kD4>(a, mode, st);
      case HQ_A2: return launch_decode_qjl<kA2>(a, mode, st);
      default: return launch_decode_qjl<kZ>(a, mode, st);
    }
  }
  if (!a.qjl && a.nsub < HQ_DEC_SMALL && p->tile == HQ_TILE && p->substream == HQ_SUB) {
    if (a.nsub == 0) return 0;
    switch (p->lattice) {
      case HQ_E8: return launch_decode_small<kE8>(a, mode, kv, st);
      case HQ_D4: return launch_decode_small<kD4>(a, mode, kv, st);
      case HQ_A2: return launch_decode_small<kA2>(a, mode, kv, st);
      default: return launch_decode_small<kZ>(a, mode, kv, st);
    }
  }
  if (p->tile != HQ_TILE || p->substream != HQ_SUB) {
    switch (p->lattice) {
      case HQ_E8: return launch_decode_tiled<kE8>(a, nwg, mode, st);
      case HQ_D4: return launch_decode_tiled<kD4>(a, nwg, mode, st);
      case HQ_A2: return launch_decode_tiled<kA2>(a, nwg, mode, st);
      default: return launch_decode_tiled<kZ>(a, nwg, mode, st);
    }
  }
  switch (p->lattice) {
    case HQ_E8: return launch_decode_lat<kE8>(a, nwg, lw, mode, kv, st);
    case HQ_D4: return launch_decode_lat<kD4>(a, nwg, lw, mode, kv, st);
    case HQ_A2: return launch_decode_lat<kA2>(a, nwg, lw, mode, kv, st);
    default: return launch_decode_lat<kZ>(a, nwg, lw, mode, kv, st);
  }
}

int hq_launch_decode_group(const hq_plan_s* p, const hq_decode_group_args& g, uint32_t nwg,
                           uint32_t lds_words, int yt, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  const int mode = (yt == HQ_FP32) ? 0 : 1;
  const bool kv = kv_variant(p);
  switch (p->lattice) {
    case HQ_E8: return launch_decode_lat<kE8>(g, nwg, lds_words, mode, kv, st);
    case HQ_D4: return launch_decode_lat<kD4>(g, nwg, lds_words, mode, kv, st);
    case HQ_A2: return launch_decode_lat<kA2>(g, nwg, lds_words, mode, kv, st);
    default: return launch_decode_lat<kZ>(g, nwg, lds_words, mode, kv, st);
  }
}

uint32_t hq_decode_workgroups(int64_t nsub) { return decode_wgs(nsub); }

int hq_launch_decode_int8(const hq_plan_s* p, const hq_decode_args& a, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  const bool kv = kv_variant(p);
  switch (p->lattice) {
    case HQ_E8: return launch_decode_lat<kE8>(a, decode_wgs(a.nsub), a.lds_words, 2, kv, st);
    case HQ_D4: return launch_decode_lat<kD4>(a, decode_wgs(a.nsub), a.lds_words, 2, kv, st);
    default: return launch_decode_lat<kZ>(a, decode_wgs(a.nsub), a.lds_words, 2, kv, st);
  }
}

// The fp8 (mode 3) and MXFP4 (mode 4) casts; a plan of fp16 norms takes the KV
// form, which reads them as such.
template <int MODE>
static int launch_decode_cast(const hq_plan_s* p, const hq_decode_args& a, hipStream_t st) {
  const size_t lds = (size_t)(a.lds_words + 66) * HQ_WAVES_PER_WG * sizeof(uint32_t);
  const uint32_t nwg = decode_wgs(a.nsub);
  const bool kv = kv_variant(p);
  switch (p->lattice) {
    case HQ_E8:
      if (kv) launch_decode_kernel<kE8, MODE, true>(a, nwg, lds, st);
      else launch_decode_kernel<kE8, MODE, false>(a, nwg, lds, st);
      break;
    case HQ_D4:
      if (kv) launch_decode_kernel<kD4, MODE, true>(a, nwg, lds, st);
      else launch_decode_kernel<kD4, MODE, false>(a, nwg, lds, st);
      break;
    default:
      if (kv) launch_decode_kernel<kZ, MODE, true>(a, nwg, lds, st);
      else launch_decode_kernel<kZ, MODE, false>(a, nwg, lds, st);
  }
  return (int)hipGetLastError();
}

int hq_launch_decode_mxfp4(const hq_plan_s* p, const hq_decode_args& a, void* stream) {
  return launch_decode_cast<4>(p, a, (hipStream_t)stream);
}

int hq_launch_decode_fp8(const hq_plan_s* p, const hq_decode_args& a, void* stream) {
  return launch_decode_cast<3>(p, a, (hipStream_t)stream);
}
