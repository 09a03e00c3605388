// Fused decode + GEMV, fused decode + attention and the GEMM activation prep for gfx950 (MI355X);
// the lane layout is in hq_device.h.
#include <type_traits>

#include "hq_device.h"

#pragma clang fp contract(off)

namespace {

// ------------------------------------------------------------ fused decode + GEMV
// y[r] = sum_k W^[r, k] x[k] for one token: the decode fused with a
// matrix-vector product (the fused decode-GEMV kernel of Sec. 6.6).  On a
// weight plan, tile t of decoded row r is
// g_t D_t H coord(c_t) with H the symmetric unnormalized Walsh-Hadamard
// matrix (the RHT absorbed into the product, Sec. 4.1), so its product with
// x_t is g_t coord(c_t) . (H D_t x_t): the transform moves from every row
// onto x, once per call (hq_gemv_prep_kernel), and a row costs its Rice
// decode, the unstrip and one dot product per lattice block.  One workgroup
// per row: each wave walks a fixed share of the row's sub-streams with a
// per-lane partial sum, a fixed butterfly over the wave and a fixed order
// over the four waves follow, so the result does not depend on scheduling.

// xt = H D x per 128-column tile, fp32; one wave per 512 columns.
__global__ __launch_bounds__(256) void hq_gemv_prep_kernel(const void* x, int x_bf16, int64_t K,
                                                           const uint32_t* dmask, float* xt) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int64_t base = ((int64_t)blockIdx.x * 4 + (tid >> 6)) * HQ_SUB;
  if (base >= K) return;  // K is a multiple of 512
  const int64_t col = base + (lane >> 4) * HQ_TILE + (lane & 15) * 8;
  float v[8];
  if (x_bf16) {
    const uint4 raw = *(const uint4*)((const uint16_t*)x + col);
    const uint32_t w4[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = bf16_to_f32(w4[i] & 0xFFFFu);
      v[2 * i + 1] = bf16_to_f32(w4[i] >> 16);
    }
  } else {
    const float4 a = *(const float4*)((const float*)x + col);
    const float4 b = *(const float4*)((const float*)x + col + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
  const uint32_t dbits = sign_bits8(dmask, col);
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = flip(v[i], dbits, i);
  const XSigns sg(lane);
  fwht128(v, sg);
  *(float4*)(xt + col) = make_float4(v[0], v[1], v[2], v[3]);
  *(float4*)(xt + col + 4) = make_float4(v[4], v[5], v[6], v[7]);
}

template <int LAT>
__global__ __launch_bounds__(256) void hq_decode_gemv_kernel(hq_decode_args A, const float* xt,
                                                             void* y, int y_bf16) {
  extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
  __shared__ uint32_t s_sel[256];
  __shared__ float s_part[HQ_WAVES_PER_WG];
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t wave = readfirst((uint32_t)(tid >> 6));
  uint32_t* buf = smem + wave * (A.lds_words + 66);
  uint32_t* starts = buf + A.lds_words + 2;
  s_sel[tid] = kByteSelect.e[tid];  // 256 threads, one entry each
  __syncthreads();
  // one row per workgroup: wave w takes the row's sub-streams w, w + 4, ...,
  // each one's table entry and first payload words loaded a step ahead
  const uint32_t spr = (uint32_t)A.spr;
  const int64_t row = blockIdx.x;  // within the call's rows
  const uint32_t sub0 = (uint32_t)A.first_sub + (uint32_t)row * spr;
  const bool fp16_norm = A.norm_fp16;
  auto head_of = [&](uint32_t j) {
    const uint32_t start = readfirst(A.offsets[sub0 + j]), end = readfirst(A.offsets[sub0 + j + 1]);
    return dec_head<LAT>(A, true, start, end, readfirst(A.kparam[sub0 + j]), lane);
  };
  float acc = 0.0f;
  DecHead head;
  if (wave < spr) head = head_of(wave);
  for (uint32_t j = wave; j < spr; j += HQ_WAVES_PER_WG) {
    DecHead next;
    if (j + HQ_WAVES_PER_WG < spr) next = head_of(j + HQ_WAVES_PER_WG);
    uint32_t sym[8];
    bool small;
    const unsigned long long bad =
        decode_symbols<LAT>(A, head, lane, (uint32_t)lane, buf, starts, s_sel, sym, small);
    if (bad && A.stats) {
      if ((unsigned)lane == (unsigned)__builtin_ctzll(bad)) {
        atomicAdd(&A.stats->corrupt_substreams, 1u);
        atomicCAS(&A.stats->status, 0u, (uint32_t)HQ_ERR_CORRUPT);
      }
    }
    int32_t c[8];
    unstrip8<LAT>(sym, c);
    const int64_t col = (int64_t)j * HQ_SUB + 8 * lane;
    const float4 xa = *(const float4*)(xt + col);
    const float4 xb = *(const float4*)(xt + col + 4);
    const float xv[8] = {xa.x, xa.y, xa.z, xa.w, xb.x, xb.y, xb.z, xb.w};
    float d = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) d = __builtin_fmaf(code_coord<LAT>(c[i], i), xv[i], d);
    const int64_t t = (A.first_row + row) * A.tpr + 4 * (int64_t)j + (lane >> 4);
    const float rs = fp16_norm ? (float)((const _Float16*)A.norms)[t] : ((const float*)A.norms)[t];
    acc = __builtin_fmaf(rs, d, acc);  // the common 1 / (alpha n) once per row
    head = next;
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) acc += __shfl_xor(acc, m, 64);
  if (lane == 0) s_part[wave] = acc;
  __syncthreads();
  if (tid == 0) {
    const float v = (((s_part[0] + s_part[1]) + s_part[2]) + s_part[3]) / A.alpha_n;
    if (y_bf16)
      ((uint16_t*)y)[row] = (uint16_t)f32_to_bf16(v);
    else
      ((float*)y)[row] = v;
  }
}

// The same product with one wave per row (rows >= HQ_GEMV_WAVE_ROWS): the
// wave walks all of its row's sub-streams, each one's table entry and first
// payload words a step ahead, and a butterfly over the wave ends the sum; no
// barrier after the table copy.
template <int LAT>
__global__ __launch_bounds__(256) void hq_decode_gemv_rows_kernel(hq_decode_args A, const float* xt,
                                                                  void* y, int y_bf16, int64_t rows) {
  extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
  __shared__ uint32_t s_sel[256];
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t wave = readfirst((uint32_t)(tid >> 6));
  s_sel[tid] = kByteSelect.e[tid];  // 256 threads, one entry each
  __syncthreads();
  const int64_t row = (int64_t)blockIdx.x * HQ_WAVES_PER_WG + wave;  // within the call's rows
  if (row >= rows) return;  // whole waves; no barrier follows
  uint32_t* buf = smem + wave * (A.lds_words + 66);
  uint32_t* starts = buf + A.lds_words + 2;
  const uint32_t spr = (uint32_t)A.spr;
  const uint32_t sub0 = (uint32_t)A.first_sub + (uint32_t)row * spr;
  const bool fp16_norm = A.norm_fp16;
  auto head_of = [&](uint32_t j) {
    const uint32_t start = readfirst(A.offsets[sub0 + j]), end = readfirst(A.offsets[sub0 + j + 1]);
    return dec_head<LAT>(A, true, start, end, readfirst(A.kparam[sub0 + j]), lane);
  };
  const int64_t t0 = (A.first_row + row) * A.tpr + (lane >> 4);
  float acc = 0.0f;
  DecHead head = head_of(0);
  float rs = fp16_norm ? (float)((const _Float16*)A.norms)[t0] : ((const float*)A.norms)[t0];
  unsigned long long bad = 0;
  for (uint32_t j = 0; j < spr; ++j) {
    DecHead next;
    float rs_next = 0.0f;
    if (j + 1 < spr) {
      next = head_of(j + 1);
      const int64_t t = t0 + 4 * (int64_t)(j + 1);
      rs_next = fp16_norm ? (float)((const _Float16*)A.norms)[t] : ((const float*)A.norms)[t];
    }
    uint32_t sym[8];
    bool small;
    bad |= decode_symbols<LAT>(A, head, lane, (uint32_t)lane, buf, starts, s_sel, sym, small);
    int32_t c[8];
    unstrip8<LAT>(sym, c);
    const int64_t col = (int64_t)j * HQ_SUB + 8 * lane;
    const float4 xa = *(const float4*)(xt + col);
    const float4 xb = *(const float4*)(xt + col + 4);
    const float xv[8] = {xa.x, xa.y, xa.z, xa.w, xb.x, xb.y, xb.z, xb.w};
    float d = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) d = __builtin_fmaf(code_coord<LAT>(c[i], i), xv[i], d);
    acc = __builtin_fmaf(rs, d, acc);  // the common 1 / (alpha n) once per row
    head = next;
    rs = rs_next;
  }
  if (bad && A.stats) {
    if ((unsigned)lane == (unsigned)__builtin_ctzll(bad)) {
      atomicAdd(&A.stats->corrupt_substreams, 1u);
      atomicCAS(&A.stats->status, 0u, (uint32_t)HQ_ERR_CORRUPT);
    }
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) acc += __shfl_xor(acc, m, 64);
  if (lane == 0) {
    const float v = acc / A.alpha_n;
    if (y_bf16)
      ((uint16_t*)y)[row] = (uint16_t)f32_to_bf16(v);
    else
      ((float*)y)[row] = v;
  }
}

// ------------------------------------------------------------ fused decode + attention
// One query token per sequence attending over its coded KV cache (the KV
// path of Sec. 5.2, read back as in Sec. 5.3, for the one-token decoding of
// Sec. 6.6).  A decoded key tile is k^ = g D H S (code - U), H the symmetric
// unnormalized Walsh-Hadamard matrix (Sec. 4.1, 4.2, 4.4), so
// q . k^ = g (S H D q) . (code - U): the query moves into the coded
// coordinates once per call (hq_attn_prep_kernel) and a key then costs its
// Rice decode, the unstrip, its dither and one dot product.  The values are
// summed in the same coordinates, sum_t p_t v^_t = D H S sum_t p_t g_t
// (code_t - U_t), and transformed back once per head (hq_attn_combine_kernel).
// The softmax runs online in base 2 (the query carries scale * log2 e).
// Work: one workgroup per (sequence, sub-stream column j, split of 4 * chunk
// tokens); wave w walks its chunk of tokens, its lane group of 16 holding one
// KV head's tile and the G query heads that read it.  Every sum has a fixed
// order, so results depend on the call's shape only, not on scheduling.

// Sum over the 16 lanes of a row; every lane gets the same bits.
__device__ __forceinline__ float row16_sum(float v) {
  v += xor_lane_f<8>(v);
  v += xor_lane_f<4>(v);
  v += xor_lane_f<2>(v);
  v += xor_lane_f<1>(v);
  return v;
}

// One step of a transposed row sum over lane bit M: of the N values a lane
// holds, the lanes with that bit set keep the upper half and the others the
// lower half, each adding its partner's copy of the half it keeps (N = 1:
// a plain butterfly step).
template <int M, int N>
__device__ __forceinline__ void tsum_step(float* d, int lane) {
  if constexpr (N > 1) {
    const bool up = (lane & M) != 0;
#pragma unroll
    for (int h = 0; h < N / 2; ++h) {
      const float keep = up ? d[h + N / 2] : d[h];
      const float send = up ? d[h] : d[h + N / 2];
      d[h] = keep + xor_lane_f<M>(send);
    }
  } else {
    d[0] += xor_lane_f<M>(d[0]);
  }
}

// Sums over the 16 lanes of a row of G per-lane values at once: lane l
// returns the sum of value (l mod 16) / (16 / G), every lane of a run of
// 16 / G the same bits.
template <int G>
__device__ __forceinline__ float row16_sums(float* d, int lane) {
  tsum_step<8, G>(d, lane);
  tsum_step<4, (G > 1 ? G / 2 : 1)>(d, lane);
  tsum_step<2, (G > 3 ? G / 4 : 1)>(d, lane);
  tsum_step<1, (G > 7 ? G / 8 : 1)>(d, lane);
  return d[0];
}

// Value of lane N of the lane's 16-lane row (DPP row_newbcast).
template <int N>
__device__ __forceinline__ float row_bcast(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x150 + N, 0xF, 0xF, false));
}

// v of each of the row's G head runs (lane g (16 / G) for head g).
template <int G>
__device__ __forceinline__ void bcast_heads(float v, float* out) {
  out[0] = row_bcast<0>(v);
  if constexpr (G > 1) out[1] = row_bcast<16 / G>(v);
  if constexpr (G > 2) {
    out[2] = row_bcast<2 * (16 / G)>(v);
    out[3] = row_bcast<3 * (16 / G)>(v);
  }
  if constexpr (G > 4) {
    out[4] = row_bcast<8>(v);
    out[5] = row_bcast<10>(v);
    out[6] = row_bcast<12>(v);
    out[7] = row_bcast<14>(v);
  }
}

// Token count of sequence b, clamped to what its table row can hold; a bad
// value is reported in the key stream's counters.
__device__ __forceinline__ int64_t attn_seq_len(const hq_attn_args& A, int64_t b, bool report) {
  const int64_t cap = (int64_t)A.max_blocks * A.block_tokens;
  int64_t len = A.seq_lens[b];
  if (len < 0 || len > cap) {
    if (report && A.K.stats) atomicCAS(&A.K.stats->status, 0u, (uint32_t)HQ_ERR_INVALID_ARG);
    len = len < 0 ? 0 : cap;
  }
  return len;
}

// Tokens of a sequence read from the coded streams: all but the residual
// window's last min(window, len).
__device__ __forceinline__ int64_t attn_coded_len(const hq_attn_args& A, int64_t len) {
  return len - (len < A.window ? len : (int64_t)A.window);
}

// 8 consecutive values (16-byte aligned) of a bf16 or fp32 array as fp32.
__device__ __forceinline__ void load8(const void* p, int64_t i, bool bf16, float* v) {
  if (bf16) {
    const uint4 raw = *(const uint4*)((const uint16_t*)p + i);
    const uint32_t w4[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[2 * k] = bf16_to_f32(w4[k] & 0xFFFFu);
      v[2 * k + 1] = bf16_to_f32(w4[k] >> 16);
    }
  } else {
    const float4 a = *(const float4*)((const float*)p + i);
    const float4 b = *(const float4*)((const float*)p + i + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
}

// qt = (S H D q) * scale * log2(e) per query head, with the key plan's signs
// (D of the head's own columns); one lane group of 16 per head.
__global__ __launch_bounds__(256) void hq_attn_prep_kernel(hq_attn_args A) {
  __shared__ float s_stage[HQ_WAVES_PER_WG * HQ_QJL_STAGE];  // qjl keys only
  const int tid = threadIdx.x, lane = tid & 63;
  const int64_t pair = ((int64_t)blockIdx.x * HQ_WAVES_PER_WG + (tid >> 6)) * 4 + (lane >> 4);
  if (pair >= A.batch * A.heads_q) return;  // whole lane groups
  const int32_t kvh = (int32_t)(pair % A.heads_q) / A.group;
  const int c0 = (lane & 15) * 8;
  float v[8];
  load8(A.q, pair * HQ_TILE + c0, A.q_bf16, v);
  const uint32_t dbits = sign_bits8(A.K.dmask, (int64_t)kvh * HQ_TILE + c0);
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = flip(v[i], dbits, i);
  const XSigns sg(lane);
  fwht128(v, sg);
  if (A.K.rotation == HQ_ROT_QJL) qjl_tile(A.K.qjlt, s_stage + (tid >> 6) * HQ_QJL_STAGE, lane, v);
  const uint32_t sbits = A.K.rotation == HQ_ROT_SIGNS ? sign_bits8(A.K.smask, c0) : 0u;
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = flip(v[i], sbits, i) * A.qscale;
  float* o = A.qt + pair * HQ_TILE + c0;
  *(float4*)o = make_float4(v[0], v[1], v[2], v[3]);
  *(float4*)(o + 4) = make_float4(v[4], v[5], v[6], v[7]);
}

// The lane's 8 coordinates of one coded tile, code - U (U the stream's
// dither at that row).
template <int LAT>
__device__ __forceinline__ unsigned long long attn_tile(const hq_decode_args& S, const DecHead& head, int lane,
                                                        uint32_t* buf, uint32_t* starts, const uint32_t* sel,
                                                        uint32_t row, uint32_t j, float* y) {
  uint32_t sym[8];
  bool small;
  const unsigned long long bad = decode_symbols<LAT>(S, head, lane, (uint32_t)lane, buf, starts, sel, sym, small);
  int32_t c[8];
  unstrip8<LAT>(sym, c);
#pragma unroll
  for (int i = 0; i < 8; ++i) y[i] = code_coord<LAT>(c[i], i);
  if (S.dither) {
    float u[8];
    dither8<LAT>(S.dither_seed, row, (int64_t)j * HQ_SUB + 8 * lane, u);
#pragma unroll
    for (int i = 0; i < 8; ++i) y[i] = y[i] - u[i];
  }
  if (bad) {  // a corrupt sub-stream contributes zeros
#pragma unroll
    for (int i = 0; i < 8; ++i) y[i] = 0.0f;
  }
  return bad;
}

// Stored tile norm r of the lane's tile in `row` (fp32 or fp16).
__device__ __forceinline__ float attn_norm(const hq_decode_args& S, uint32_t row, uint32_t j,
                                           int lane) {
  const int64_t t = (int64_t)row * S.tpr + 4 * (int64_t)j + (lane >> 4);
  return S.norm_fp16 ? (float)((const _Float16*)S.norms)[t] : ((const float*)S.norms)[t];
}

// Table entry (start, end, k) of one token's sub-stream, fetched earlier by
// lane i of the wave for the i-th token of a run of 64.
struct AttnMeta {
  uint32_t s, e, k;
};

__device__ __forceinline__ uint32_t lane_val(uint32_t v, uint32_t i) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)i);
}

// Two passes over the same grid and token chunks.  The key pass (VAL =
// false) decodes each key tile and stores its G scores per KV head, base 2,
// at scores[(b, j, t), 4 G] plus every wave's largest score per head.  The
// value pass (VAL = true) decodes each value tile and adds p g (code - U)
// with p = 2^(s - m), m that wave's largest score, so no sum is ever
// rescaled inside the token loop; the four waves then rescale to their
// common maximum and write one partial per workgroup.  Each pass holds one
// stream's decode state: the single-pass form held both plus the value sums
// (163 registers, three waves per SIMD).  Scores, maxima and weights are
// per lane: lane l of a row of 16 handles query head hl = (l mod 16) /
// (16 / G) of the row's G, and the value pass broadcasts each head's weight
// p across the row.
// The value pass at G <= 4 is held to 128 registers (four waves per SIMD);
// what that moves to scratch is saved before the token loop and restored
// after it.
template <int LAT, int G, bool VAL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(VAL && G <= 4 ? 4 : 1)))
void hq_attn_kernel(hq_attn_args A) {
  extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
  __shared__ uint32_t s_sel[256];
  __shared__ float s_m[HQ_WAVES_PER_WG][4 * G];
  __shared__ float s_l[HQ_WAVES_PER_WG][4 * G];
  __shared__ float4 s_q[VAL ? 1 : 4 * G * 32];  // key pass: the query tiles, coded coordinates
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t wave = readfirst((uint32_t)(tid >> 6));
  const uint32_t spr = (uint32_t)A.K.spr;
  const uint32_t x = blockIdx.x % (uint32_t)A.nx;
  const uint32_t bj = blockIdx.x / (uint32_t)A.nx;
  const uint32_t b = bj / spr, j = bj - b * spr;
  const int64_t len =
      attn_coded_len(A, attn_seq_len(A, b, !VAL && tid == 0 && x == 0 && j == 0));
  const int64_t wg_t0 = (int64_t)x * HQ_WAVES_PER_WG * A.chunk;
  if (wg_t0 >= len) return;  // the whole workgroup, before any barrier
  const hq_decode_args& S = VAL ? A.V : A.K;
  s_sel[tid] = kByteSelect.e[tid];
  // KV heads 4j .. 4j+3 read query heads (4j) G .. (4j + 4) G - 1: one block
  const int64_t hq0 = (int64_t)b * A.heads_q + (int64_t)j * 4 * G;
  if constexpr (!VAL) {
    for (int i = tid; i < 4 * G * 32; i += 256) s_q[i] = ((const float4*)(A.qt + hq0 * HQ_TILE))[i];
  }
  __syncthreads();
  uint32_t* buf = smem + wave * (A.lds_words + 66);
  uint32_t* starts = buf + A.lds_words + 2;
  float* comb = (float*)(smem + HQ_WAVES_PER_WG * (A.lds_words + 66));

  const int q4 = lane >> 4, c0 = (lane & 15) * 8;
  const int hl = (lane & 15) / (16 / G);
  const bool lead = (lane & (16 / G - 1)) == 0;  // first lane of its head's run
  const float4* qrow = s_q + (q4 * G) * 32 + (lane & 15) * 2;  // head g: + 32 g
  // scores of (b, j): token t's 4 G heads at + 4 G t, this lane group's at + G q4
  float* srow =
      A.scores + (int64_t)bj * ((int64_t)A.max_blocks * A.block_tokens) * (4 * G) + q4 * G + hl;
  float* wmax = A.wmax + ((int64_t)blockIdx.x * HQ_WAVES_PER_WG + wave) * (4 * G) + q4 * G + hl;
  float acc[VAL ? G : 1][8];
  float m = -__builtin_inff(), l = 0.0f;  // head hl's
  if constexpr (VAL) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[g][i] = 0.0f;
    }
  }

  const int64_t t0 = wg_t0 + (int64_t)wave * A.chunk;
  const int64_t t1 = t0 + A.chunk < len ? t0 + A.chunk : len;
  if (VAL && t0 < t1) m = *wmax;  // written by the key pass for these tokens
  const uint32_t bt = (uint32_t)A.block_tokens;
  const int32_t* trow = A.table + (int64_t)b * A.max_blocks;
  unsigned long long bad = 0;
  for (int64_t tb = t0; tb < t1; tb += 64) {
    // lane i fetches token tb + i's row and table entry (rows past the
    // streams or a negative block id: row ~0u, the token is skipped)
    const uint32_t n = (uint32_t)(t1 - tb < 64 ? t1 - tb : 64);
    uint32_t rv = ~0u;
    AttnMeta me = {0u, 0u, 0u};
    if ((uint32_t)lane < n) {
      const uint32_t t = (uint32_t)(tb + lane);
      const uint32_t bi = t / bt;
      const int32_t blk = trow[bi];
      const int64_t r = (int64_t)blk * bt + (t - bi * bt);
      if (blk >= 0 && r < A.rows) {
        rv = (uint32_t)r;
        const int64_t sub = r * spr + j;
        me = {S.offsets[sub], S.offsets[sub + 1], S.kparam[sub]};
      }
    }
    if (!VAL && __ballot(rv == ~0u && (uint32_t)lane < n) && lane == 0 && A.K.stats)
      atomicCAS(&A.K.stats->status, 0u, (uint32_t)HQ_ERR_INVALID_ARG);  // block id out of range
    // token i's head, norm and (value pass) scores, each loaded one token ahead
    auto fetch = [&](uint32_t i, uint32_t& row, DecHead& h, float& nr, float& sc) {
      row = lane_val(rv, i);
      if (row != ~0u) {
        h = dec_head<LAT>(S, true, lane_val(me.s, i), lane_val(me.e, i), lane_val(me.k, i), lane);
        nr = attn_norm(S, row, j, lane);
        if constexpr (VAL) sc = srow[(tb + i) * (4 * G)];
      }
    };
    uint32_t row;
    DecHead hd;
    float nr = 0.0f, sc = 0.0f;
    fetch(0, row, hd, nr, sc);
    for (uint32_t i = 0; i < n; ++i) {
      uint32_t nrow = ~0u;
      DecHead nhd;
      float nnr = 0.0f, nsc = 0.0f;
      if (i + 1 < n) fetch(i + 1, nrow, nhd, nnr, nsc);
      if (row != ~0u) {
        float y[8];
        bad |= attn_tile<LAT>(S, hd, lane, buf, starts, s_sel, row, j, y);
        const float gs = nr / S.alpha_n;
        if constexpr (!VAL) {
          float d[G];
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const float4 qa = qrow[32 * g], qb = qrow[32 * g + 1];
            float e = qa.x * y[0];
            e = __builtin_fmaf(qa.y, y[1], e);
            e = __builtin_fmaf(qa.z, y[2], e);
            e = __builtin_fmaf(qa.w, y[3], e);
            e = __builtin_fmaf(qb.x, y[4], e);
            e = __builtin_fmaf(qb.y, y[5], e);
            e = __builtin_fmaf(qb.z, y[6], e);
            e = __builtin_fmaf(qb.w, y[7], e);
            d[g] = e;
          }
          const float sl = gs * row16_sums<G>(d, lane);
          m = __builtin_fmaxf(m, sl);
          if (lead) srow[(tb + i) * (4 * G)] = sl;
        } else {
          const float p = exp2f(sc - m);
          l += p;
          float pg[G];
          bcast_heads<G>(p * gs, pg);
#pragma unroll
          for (int g = 0; g < G; ++g) {
#pragma unroll
            for (int i2 = 0; i2 < 8; ++i2) acc[g][i2] = __builtin_fmaf(pg[g], y[i2], acc[g][i2]);
          }
        }
      }
      row = nrow;
      hd = nhd;
      nr = nnr;
      sc = nsc;
    }
  }
  if (bad && A.K.stats) {
    if ((unsigned)lane == (unsigned)__builtin_ctzll(bad)) {
      atomicAdd(&A.K.stats->corrupt_substreams, 1u);
      atomicCAS(&A.K.stats->status, 0u, (uint32_t)HQ_ERR_CORRUPT);
    }
  }
  if constexpr (!VAL) {
    if (t0 < t1 && lead) *wmax = m;
    return;
  } else {
    // the four waves' sums, rescaled to their common maximum, in wave order
    if (lead) s_m[wave][q4 * G + hl] = m;
    __syncthreads();
    float M = s_m[0][q4 * G + hl];
#pragma unroll
    for (int w = 1; w < HQ_WAVES_PER_WG; ++w) M = __builtin_fmaxf(M, s_m[w][q4 * G + hl]);
    const float f = m == -__builtin_inff() ? 0.0f : exp2f(m - M);
    l *= f;
    m = M;
    float fg[G];
    bcast_heads<G>(f, fg);
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[g][i] *= fg[g];
    }
    if (wave > 0) {
      float* cw = comb + ((wave - 1) * 64 + lane) * 8 * G;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        *(float4*)(cw + 8 * g) = make_float4(acc[g][0], acc[g][1], acc[g][2], acc[g][3]);
        *(float4*)(cw + 8 * g + 4) = make_float4(acc[g][4], acc[g][5], acc[g][6], acc[g][7]);
      }
      if (lead) s_l[wave][q4 * G + hl] = l;
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int w = 1; w < HQ_WAVES_PER_WG; ++w) {
        const float* cw = comb + ((w - 1) * 64 + lane) * 8 * G;
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const float4 a = *(const float4*)(cw + 8 * g);
          const float4 c = *(const float4*)(cw + 8 * g + 4);
          acc[g][0] += a.x; acc[g][1] += a.y; acc[g][2] += a.z; acc[g][3] += a.w;
          acc[g][4] += c.x; acc[g][5] += c.y; acc[g][6] += c.z; acc[g][7] += c.w;
        }
        l += s_l[w][q4 * G + hl];
      }
      const int64_t h0 = hq0 + (int64_t)q4 * G;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int64_t pi = (h0 + g) * A.nx + x;
        float* o = A.part_acc + pi * HQ_TILE + c0;
        *(float4*)o = make_float4(acc[g][0], acc[g][1], acc[g][2], acc[g][3]);
        *(float4*)(o + 4) = make_float4(acc[g][4], acc[g][5], acc[g][6], acc[g][7]);
      }
      if (lead) {
        const int64_t pi = (h0 + hl) * A.nx + x;
        A.part_m[pi] = m;
        A.part_l[pi] = l;
      }
    }
  }
}

// out = (D H S sum_x f_x acc_x + sum_i p_i v_i) / (sum_x f_x l_x + sum_i p_i):
// the coded splits that hold tokens (f_x = 2^(m_x - M)) with the value
// plan's signs, plus the residual window's exact tokens i (p_i = 2^(s_i - M),
// s_i = q . k_i scaled in natural coordinates), M the maximum over both; an
// empty sequence gives zeros.  One workgroup per query head: lane group k of
// 16 takes splits k, k + 16, ... and window tokens k, k + 16, ..., and the 16
// groups' sums meet in LDS in group order.
__global__ __launch_bounds__(256) void hq_attn_combine_kernel(hq_attn_args A) {
  __shared__ float s_red[16];
  __shared__ float s_win[HQ_ATTN_WINDOW_MAX];
  __shared__ float4 s_acc[16][32];
  __shared__ float4 s_nat[16][32];
  const int tid = threadIdx.x, lane = tid & 63, grp = tid >> 4;
  const int64_t pair = blockIdx.x;
  const int64_t b = pair / A.heads_q;
  const int32_t kvh = (int32_t)(pair - b * A.heads_q) / A.group;
  const int c0 = (lane & 15) * 8;
  const int64_t len = attn_seq_len(A, b, false);
  const int64_t clen = attn_coded_len(A, len);
  const int32_t w = (int32_t)(len - clen);
  const int64_t per = (int64_t)HQ_WAVES_PER_WG * A.chunk;
  const int32_t n = (int32_t)((clen + per - 1) / per);
  const float* pm = A.part_m + pair * A.nx;
  const float* pl = A.part_l + pair * A.nx;
  const int64_t hkv = (int64_t)A.heads_q / A.group;
  float M = -__builtin_inff();
  if (w > 0) {
    float q[8];
    load8(A.q, pair * HQ_TILE + c0, A.q_bf16, q);
    for (int32_t i = grp; i < w; i += 16) {
      const int64_t slot = (clen + i) % A.window;
      float k[8];
      load8(A.win_k, ((b * A.window + slot) * hkv + kvh) * HQ_TILE + c0, A.win_bf16, k);
      float d = q[0] * k[0];
#pragma unroll
      for (int e = 1; e < 8; ++e) d = __builtin_fmaf(q[e], k[e], d);
      const float si = row16_sum(d) * A.qscale;
      if ((tid & 15) == 0) s_win[i] = si;
      M = __builtin_fmaxf(M, si);
    }
  }
  for (int32_t x = grp; x < n; x += 16) M = __builtin_fmaxf(M, pm[x]);
  if ((tid & 15) == 0) s_red[grp] = M;
  __syncthreads();
  M = s_red[0];
#pragma unroll
  for (int k = 1; k < 16; ++k) M = __builtin_fmaxf(M, s_red[k]);
  float L = 0.0f, v[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
  float vn[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
  if (M != -__builtin_inff()) {
    for (int32_t x = grp; x < n; x += 16) {
      const float mx = pm[x];
      const float f = mx == -__builtin_inff() ? 0.0f : exp2f(mx - M);
      L = __builtin_fmaf(f, pl[x], L);
      const float* a = A.part_acc + (pair * A.nx + x) * HQ_TILE + c0;
      const float4 a0 = *(const float4*)a;
      const float4 a1 = *(const float4*)(a + 4);
      v[0] = __builtin_fmaf(f, a0.x, v[0]); v[1] = __builtin_fmaf(f, a0.y, v[1]);
      v[2] = __builtin_fmaf(f, a0.z, v[2]); v[3] = __builtin_fmaf(f, a0.w, v[3]);
      v[4] = __builtin_fmaf(f, a1.x, v[4]); v[5] = __builtin_fmaf(f, a1.y, v[5]);
      v[6] = __builtin_fmaf(f, a1.z, v[6]); v[7] = __builtin_fmaf(f, a1.w, v[7]);
    }
    for (int32_t i = grp; i < w; i += 16) {
      const int64_t slot = (clen + i) % A.window;
      const float p = exp2f(s_win[i] - M);
      L += p;
      float val[8];
      load8(A.win_v, ((b * A.window + slot) * hkv + kvh) * HQ_TILE + c0, A.win_bf16, val);
#pragma unroll
      for (int e = 0; e < 8; ++e) vn[e] = __builtin_fmaf(p, val[e], vn[e]);
    }
  }
  __syncthreads();  // every group has read s_red
  s_acc[grp][(lane & 15) * 2] = make_float4(v[0], v[1], v[2], v[3]);
  s_acc[grp][(lane & 15) * 2 + 1] = make_float4(v[4], v[5], v[6], v[7]);
  s_nat[grp][(lane & 15) * 2] = make_float4(vn[0], vn[1], vn[2], vn[3]);
  s_nat[grp][(lane & 15) * 2 + 1] = make_float4(vn[4], vn[5], vn[6], vn[7]);
  if ((tid & 15) == 0) s_red[grp] = L;
  __syncthreads();
  if (tid >= 16) return;  // group 0 finishes: no barrier follows
  L = 0.0f;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const float4 a0 = s_acc[k][tid * 2], a1 = s_acc[k][tid * 2 + 1];
    const float4 n0 = s_nat[k][tid * 2], n1 = s_nat[k][tid * 2 + 1];
    if (k == 0) {
      v[0] = a0.x; v[1] = a0.y; v[2] = a0.z; v[3] = a0.w;
      v[4] = a1.x; v[5] = a1.y; v[6] = a1.z; v[7] = a1.w;
      vn[0] = n0.x; vn[1] = n0.y; vn[2] = n0.z; vn[3] = n0.w;
      vn[4] = n1.x; vn[5] = n1.y; vn[6] = n1.z; vn[7] = n1.w;
    } else {
      v[0] += a0.x; v[1] += a0.y; v[2] += a0.z; v[3] += a0.w;
      v[4] += a1.x; v[5] += a1.y; v[6] += a1.z; v[7] += a1.w;
      vn[0] += n0.x; vn[1] += n0.y; vn[2] += n0.z; vn[3] += n0.w;
      vn[4] += n1.x; vn[5] += n1.y; vn[6] += n1.z; vn[7] += n1.w;
    }
    L += s_red[k];
  }
  const float inv = L > 0.0f ? 1.0f / L : 0.0f;
  const uint32_t sbits = A.V.rotation == HQ_ROT_SIGNS ? sign_bits8(A.V.smask, c0) : 0u;
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = flip(v[i] * inv, sbits, i);
  if (A.V.rotation == HQ_ROT_QJL) qjl_tile(A.V.qjl, (float*)s_acc, lane, v);  // v <- S^T v
  const XSigns sg(lane);
  fwht128(v, sg);
  const uint32_t dbits = sign_bits8(A.V.dmask, (int64_t)kvh * HQ_TILE + c0);
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = __builtin_fmaf(vn[i], inv, flip(v[i], dbits, i));
  if (A.out_bf16) {
    uint4 o;
    o.x = cvt_pk_bf16(v[0], v[1]);
    o.y = cvt_pk_bf16(v[2], v[3]);
    o.z = cvt_pk_bf16(v[4], v[5]);
    o.w = cvt_pk_bf16(v[6], v[7]);
    *(uint4*)((uint16_t*)A.out + pair * HQ_TILE + c0) = o;
  } else {
    float* o = (float*)A.out + pair * HQ_TILE + c0;
    *(float4*)o = make_float4(v[0], v[1], v[2], v[3]);
    *(float4*)(o + 4) = make_float4(v[4], v[5], v[6], v[7]);
  }
}

// ------------------------------------------------------------ activation prep
// y = H D a per tile (canonical stage order, the weights' signs), amax over the
// row, then the cast.

// Tile 128, at most 2048 NIT columns: one workgroup per token row, every value
// in registers from its load to its code (wave w holds columns 512 (4 i + w)
// ..), so a row is read once and written once and only the row's maximum goes
// through LDS (MXFP4's blocks are four lanes: nothing does).  CAST 0 int8, 1
// E4M3, 2 MXFP4.  int8's values carry the twisted transform's lane sign, which
// the scale takes back (rounding is symmetric); the other two codes keep the
// sign of a zero, so they take the plain transform.  4096 x 4096 to int8: 17.0 -> 13.9
// us (3.6 TB/s), 1000 x 14336 to E4M3 21.3 -> 16.0, 2048 x 4096 to MXFP4 12.3 ->
// 10.8 against the LDS form below.
template <int NIT, int CAST>
__global__ __launch_bounds__(256) void hq_act_prep_regs_kernel(hq_actprep_args A) {
  __shared__ float s_max[4];
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t wave = readfirst((uint32_t)(tid >> 6));
  const int64_t row = blockIdx.x;
  const uint16_t* arow = (const uint16_t*)A.a + row * A.lda;
  const uint32_t K = (uint32_t)A.K;
  const typename std::conditional<CAST == 0, TwSigns, XSigns>::type sg(lane);
  uint4 raw[NIT];
#pragma unroll
  for (int i = 0; i < NIT; ++i) {
    const uint32_t base = (4u * i + wave) * HQ_SUB;
    if (base < K) raw[i] = *(const uint4*)(arow + base + 8 * lane);
  }
  float v[NIT][8], amax = 0.0f;
#pragma unroll
  for (int i = 0; i < NIT; ++i) {
    const uint32_t base = (4u * i + wave) * HQ_SUB;
    if (base >= K) break;
    const uint4 sw = *(const uint4*)(A.dsign16 + ((base + 8 * lane) >> 1));
    const uint32_t w4[4] = {raw[i].x ^ sw.x, raw[i].y ^ sw.y, raw[i].z ^ sw.z, raw[i].w ^ sw.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[i][2 * e] = bf16_to_f32(w4[e] & 0xFFFFu);
      v[i][2 * e + 1] = __uint_as_float(w4[e] & 0xFFFF0000u);
    }
    if constexpr (CAST == 0)
      fwht128_tw(v[i], sg);
    else
      fwht128(v[i], sg);
    if constexpr (CAST == 2) {
      int32_t X;
      const uint32_t packed = mxfp4_x8(v[i], X);
      const int64_t col = base + 8 * lane;
      *(uint32_t*)((uint8_t*)A.xq + row * (A.K / 2) + col / 2) = packed;
      if ((lane & 3) == 0) A.mxs[row * (A.K / 32) + col / 32] = (uint8_t)(X + 127);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) amax = __builtin_fmaxf(amax, __builtin_fabsf(v[i][e]));
    }
  }
  if constexpr (CAST == 2) return;
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) amax = __builtin_fmaxf(amax, __shfl_xor(amax, m, 64));
  if (lane == 0) s_max[wave] = amax;
  __syncthreads();
  amax = __builtin_fmaxf(__builtin_fmaxf(s_max[0], s_max[1]), __builtin_fmaxf(s_max[2], s_max[3]));
  const float top = CAST == 1 ? 448.0f : 127.0f;  // E4M3's largest magnitude, or int8's
  float inv = (amax == 0.0f) ? 0.0f : top / amax;
  if constexpr (CAST == 0) inv = xor_sign(inv, sg.sigma);
#pragma unroll
  for (int i = 0; i < NIT; ++i) {
    const uint32_t base = (4u * i + wave) * HQ_SUB;
    if (base >= K) break;
    uint32_t packed[2] = {0u, 0u};
    float q[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      q[e] = v[i][e] * inv;
      if (CAST == 0) q[e] = __builtin_rintf(q[e]);
      q[e] = __builtin_fminf(__builtin_fmaxf(q[e], -top), top);
    }
    if constexpr (CAST == 1) {
      packed[0] = e4m3x4(q[0], q[1], q[2], q[3]);
      packed[1] = e4m3x4(q[4], q[5], q[6], q[7]);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) packed[e >> 2] |= ((uint32_t)(int32_t)q[e] & 0xFFu) << (8 * (e & 3));
    }
    *(uint2*)(A.xq + row * A.K + base + 8 * lane) = make_uint2(packed[0], packed[1]);
  }
  if (tid == 0) A.sx[row] = amax / top;
}

// Any tile and row length: one workgroup per token row, stages h = 1 .. 64 in
// registers per 128 columns, then for a longer tile h = 128 .. tile / 2 in LDS.
__global__ __launch_bounds__(256) void hq_act_prep_kernel(hq_actprep_args A) {
  extern __shared__ __attribute__((aligned(16))) float ybuf[];
  __shared__ float s_max[4];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int64_t row = blockIdx.x;
  const uint16_t* arow = (const uint16_t*)A.a + row * A.lda;
  const XSigns sg(lane);
  float amax = 0.0f;
  for (int64_t base = (int64_t)wave * HQ_SUB; base < A.K; base += 4 * HQ_SUB) {
    const int64_t col = base + (lane >> 4) * HQ_TILE + (lane & 15) * 8;
    float v[8];
    const uint4 raw = *(const uint4*)(arow + col);
    const uint32_t w4[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = bf16_to_f32(w4[i] & 0xFFFFu);
      v[2 * i + 1] = bf16_to_f32(w4[i] >> 16);
    }
    const uint32_t dbits = sign_bits8(A.dmask, col);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = flip(v[i], dbits, i);
    fwht128(v, sg);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      amax = __builtin_fmaxf(amax, __builtin_fabsf(v[i]));
    }
    *(float4*)(ybuf + col) = make_float4(v[0], v[1], v[2], v[3]);
    *(float4*)(ybuf + col + 4) = make_float4(v[4], v[5], v[6], v[7]);
  }
  if (A.tile > HQ_TILE) {
    // the remaining butterflies of a long tile, one stage at a time over the
    // row: pair p of stage h, a power of two, is (j, j + h) with j = (p / h) 2h +
    // p % h = p + (p & -h).  With 64-bit divisions by h 16 x 14336 to E4M3 at
    // tile 512 took 18.7 us instead of 13.4, 4096 x 4096 28.5 instead of 20.7.
    for (uint32_t h = HQ_TILE; h < (uint32_t)A.tile; h <<= 1) {
      __syncthreads();
      for (uint32_t p = (uint32_t)tid; p < (uint32_t)A.K / 2; p += 256) {
        const uint32_t j = p + (p & (0u - h));
        const float a = ybuf[j], b = ybuf[j + h];
        ybuf[j] = a + b;
        ybuf[j + h] = a - b;
      }
    }
    __syncthreads();
    amax = 0.0f;
    for (int64_t c = tid; c < A.K; c += 256) amax = __builtin_fmaxf(amax, __builtin_fabsf(ybuf[c]));
  }
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) amax = __builtin_fmaxf(amax, __shfl_xor(amax, m, 64));
  if (lane == 0) s_max[wave] = amax;
  __syncthreads();
  if (A.fp8 == 2) {
    // MXFP4: blocks of 32 (eight threads of four values each) share
    // X = floor(log2 amax) - 2 and hold E2M1(y / 2^X); no per-token factor
    for (int64_t base = 0; base < A.K; base += 1024) {
      const int64_t col = base + (int64_t)tid * 4;
      const bool in = col < A.K;  // whole 32-blocks are in or out (K is a multiple of 512)
      float q[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) q[i] = in ? ybuf[col + i] : 0.0f;
      int32_t X;
      auto cast = [&](float am) {
        am = __builtin_fmaxf(am, __shfl_xor(am, 1, 64));
        am = __builtin_fmaxf(am, __shfl_xor(am, 2, 64));
        am = __builtin_fmaxf(am, __shfl_xor(am, 4, 64));
        X = mx_exponent(am);
        return e2m1_pair<1>(e2m1_pair<0>(0u, q[0], q[1], X), q[2], q[3], X);
      };
      const float am0 = amax_or_nan<4>(q);
      uint32_t packed = cast(am0);
      if (__builtin_expect(__ballot(am0 != am0) != 0ull, 0)) {
        e2m1_drop_nan<4>(q);
        packed = cast(amax_or_nan<4>(q));
      }
      if (in) {
        *(uint16_t*)((uint8_t*)A.xq + row * (A.K / 2) + col / 2) = (uint16_t)packed;
        if ((tid & 7) == 0) A.mxs[row * (A.K / 32) + col / 32] = (uint8_t)(X + 127);
      }
    }
    return;
  }
  amax = __builtin_fmaxf(__builtin_fmaxf(s_max[0], s_max[1]), __builtin_fmaxf(s_max[2], s_max[3]));
  const float top = A.fp8 ? 448.0f : 127.0f;  // E4M3's largest magnitude, or int8's
  const float inv = (amax == 0.0f) ? 0.0f : top / amax;
  int8_t* xrow = A.xq + row * A.K;
  for (int64_t col = (int64_t)tid * 4; col < A.K; col += 1024) {
    uint32_t packed = 0;
    if (A.fp8) {
      float q[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) q[i] = __builtin_fminf(__builtin_fmaxf(ybuf[col + i] * inv, -448.0f), 448.0f);
      packed = e4m3x4(q[0], q[1], q[2], q[3]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float qv = __builtin_rintf(ybuf[col + i] * inv);
        qv = __builtin_fminf(__builtin_fmaxf(qv, -127.0f), 127.0f);
        packed |= ((uint32_t)(int32_t)qv & 0xFFu) << (8 * i);
      }
    }
    *(uint32_t*)(xrow + col) = packed;
  }
  if (tid == 0) A.sx[row] = amax / top;
}


}  // namespace

template <int CAST>
static void launch_act_prep_regs(const hq_actprep_args& a, hipStream_t st) {
  const dim3 grid((uint32_t)a.M), wg(256);
  if (a.K <= 2048)
    hipLaunchKernelGGL((hq_act_prep_regs_kernel<1, CAST>), grid, wg, 0, st, a);
  else if (a.K <= 4096)
    hipLaunchKernelGGL((hq_act_prep_regs_kernel<2, CAST>), grid, wg, 0, st, a);
  else if (a.K <= 8192)
    hipLaunchKernelGGL((hq_act_prep_regs_kernel<4, CAST>), grid, wg, 0, st, a);
  else
    hipLaunchKernelGGL((hq_act_prep_regs_kernel<8, CAST>), grid, wg, 0, st, a);
}

int hq_launch_act_prep(const hq_actprep_args& a, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  // values of up to 16384 columns fit the registers of four waves; the outputs
  // go out 8 (MXFP4: 4) bytes a lane
  if (a.tile == HQ_TILE && a.K <= 16384 && (uintptr_t)a.xq % (a.fp8 == 2 ? 4 : 8) == 0) {
    if (a.fp8 == 2)
      launch_act_prep_regs<2>(a, st);
    else if (a.fp8)
      launch_act_prep_regs<1>(a, st);
    else
      launch_act_prep_regs<0>(a, st);
    return (int)hipGetLastError();
  }
  const size_t lds = (size_t)a.K * sizeof(float);
  hipLaunchKernelGGL(hq_act_prep_kernel, dim3((uint32_t)a.M), dim3(256), lds, st, a);
  return (int)hipGetLastError();
}

int hq_launch_decode_gemv(const hq_plan_s* p, const hq_decode_args& a, const void* x, int xt,
                          float* xtr, void* y, int yt, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  const int64_t K = p->cols;
  hipLaunchKernelGGL(hq_gemv_prep_kernel, dim3((uint32_t)((K + 4 * HQ_SUB - 1) / (4 * HQ_SUB))),
                     dim3(256), 0, st, x, xt == HQ_BF16 ? 1 : 0, K, a.dmask, xtr);
  const int64_t rows = a.nsub / a.spr;
  const size_t lds = (size_t)(a.lds_words + 66) * HQ_WAVES_PER_WG * sizeof(uint32_t);
  const int yb = yt == HQ_BF16 ? 1 : 0;
  if (rows >= HQ_GEMV_WAVE_ROWS) {  // enough rows to fill the chip one wave each
    const uint32_t nwr = (uint32_t)((rows + HQ_WAVES_PER_WG - 1) / HQ_WAVES_PER_WG);
    switch (p->lattice) {
      case HQ_E8:
        hipLaunchKernelGGL(hq_decode_gemv_rows_kernel<kE8>, dim3(nwr), dim3(256), lds, st, a, xtr, y, yb, rows);
        break;
      case HQ_D4:
        hipLaunchKernelGGL(hq_decode_gemv_rows_kernel<kD4>, dim3(nwr), dim3(256), lds, st, a, xtr, y, yb, rows);
        break;
      case HQ_A2:
        hipLaunchKernelGGL(hq_decode_gemv_rows_kernel<kA2>, dim3(nwr), dim3(256), lds, st, a, xtr, y, yb, rows);
        break;
      default:
        hipLaunchKernelGGL(hq_decode_gemv_rows_kernel<kZ>, dim3(nwr), dim3(256), lds, st, a, xtr, y, yb, rows);
    }
    return (int)hipGetLastError();
  }
  const uint32_t nwg = (uint32_t)rows;  // one workgroup per row
  switch (p->lattice) {
    case HQ_E8:
      hipLaunchKernelGGL(hq_decode_gemv_kernel<kE8>, dim3(nwg), dim3(256), lds, st, a, xtr, y, yb);
      break;
    case HQ_D4:
      hipLaunchKernelGGL(hq_decode_gemv_kernel<kD4>, dim3(nwg), dim3(256), lds, st, a, xtr, y, yb);
      break;
    case HQ_A2:
      hipLaunchKernelGGL(hq_decode_gemv_kernel<kA2>, dim3(nwg), dim3(256), lds, st, a, xtr, y, yb);
      break;
    default:
      hipLaunchKernelGGL(hq_decode_gemv_kernel<kZ>, dim3(nwg), dim3(256), lds, st, a, xtr, y, yb);
  }
  return (int)hipGetLastError();
}

int hq_launch_decode_attention(const hq_attn_args& a, int lattice, void* stream) {
  const hipStream_t st = (hipStream_t)stream;
  const uint32_t heads = (uint32_t)((a.batch * a.heads_q + 15) / 16);
  hipLaunchKernelGGL(hq_attn_prep_kernel, dim3(heads), dim3(256), 0, st, a);
  const uint32_t nwg = (uint32_t)(a.batch * a.K.spr * a.nx);
  const size_t lds_k = (size_t)HQ_WAVES_PER_WG * (a.lds_words + 66) * 4;
  const size_t lds_v = lds_k + (size_t)(HQ_WAVES_PER_WG - 1) * 64 * 8 * a.group * 4;
#define HQ_ATTN_CASE(L, GG)                                                                  \
  hipLaunchKernelGGL((hq_attn_kernel<L, GG, false>), dim3(nwg), dim3(256), lds_k, st, a); \
  hipLaunchKernelGGL((hq_attn_kernel<L, GG, true>), dim3(nwg), dim3(256), lds_v, st, a)
#define HQ_ATTN_GROUPS(L)           \
  switch (a.group) {                \
    case 1: HQ_ATTN_CASE(L, 1); break; \
    case 2: HQ_ATTN_CASE(L, 2); break; \
    case 4: HQ_ATTN_CASE(L, 4); break; \
    default: HQ_ATTN_CASE(L, 8);    \
  }
  switch (lattice) {
    case HQ_E8: HQ_ATTN_GROUPS(kE8); break;
    case HQ_D4: HQ_ATTN_GROUPS(kD4); break;
    case HQ_A2: HQ_ATTN_GROUPS(kA2); break;
    default: HQ_ATTN_GROUPS(kZ);
  }
#undef HQ_ATTN_GROUPS
#undef HQ_ATTN_CASE
  hipLaunchKernelGGL(hq_attn_combine_kernel, dim3((uint32_t)(a.batch * a.heads_q)), dim3(256), 0,
                     st, a);
  return (int)hipGetLastError();
}
