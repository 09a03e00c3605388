// Block-scaled GEMM kernels for gfx950 (MI355X): int8, E4M3 and MXFP4.
//
// int8 and E4M3: out[m, n] = s_x[m] * sum_t g[n, t] * P_t[m, n], P_t the sum
// over one factor tile of K: exact int32 on the int8 matrix cores
// (v_mfma_i32_32x32x32_i8), fp32 on the f8f6f4 ones for E4M3
// (v_mfma_scale_f32_32x32x64_f8f6f4 with unit scales).  MXFP4: out[m, n] =
// sum_k X[m, k] W[n, k] over the element-times-block-scale values on the
// same instruction, whose E8M0 scales carry every factor.
//
// Both operands are K-contiguous rows and every lane reads the same k range
// of A and B, so the contraction pairs identical k whatever order the
// instruction assigns inside a step.  Output lane l of a 32 x 32 block holds
// column l % 32 and rows 8 (r / 4) + 4 (l / 32) + r % 4.
//
// The rescale is a floating-point accumulation (contraction of its product
// and sum is written out as an fma); results are held to a tolerance.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hq_internal.h"
#include "hq_lds.h"

#pragma clang fp contract(off)

namespace {

typedef uint32_t v2u_t __attribute__((ext_vector_type(2)));
typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef int v8i_t __attribute__((ext_vector_type(8)));
typedef int v16i_t __attribute__((ext_vector_type(16)));
typedef float v16f_t __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void lds_void_t;

template <bool C, class T, class F> struct gemm_pick { using type = T; };
template <class T, class F> struct gemm_pick<false, T, F> { using type = F; };

// A kernel's shape: MODE 0 int8, 1 E4M3, 2 MXFP4; workgroup tile BM tokens x
// BN weight rows by WM x WN waves; LONG: factor tiles of several stages
// (their partial sums stay in registers until the tile ends); R LDS stages.
// A stage is 128 bytes of every A and B row (128 k of int8 / E4M3, 256 of
// MXFP4) and its side data: the weight rows' factors, or the 8 scale bytes of
// every A and B row.
template <int MODE_, int BM_, int BN_, int WM_, int WN_, bool LONG_, int R_>
struct GemmCfg {
  static constexpr int MODE = MODE_, BM = BM_, BN = BN_, WM = WM_, WN = WN_, R = R_;
  static constexpr bool LONG = LONG_;
  static constexpr bool RESCALE = MODE != 2;
  static constexpr int W = WM * WN;                    // waves
  static constexpr int NA = BM / WM / 32, NB = BN / WN / 32;  // a wave's 32 x 32 blocks
  static constexpr int NBLK = NA * NB;
  static constexpr int U = MODE == 2 ? 2 : 1;          // 128-deep K units per stage
  static constexpr int NS = MODE == 1 ? 2 : 4;         // MFMA steps per stage
  static constexpr int FW = MODE == 1 ? 2 : 1;         // 16-byte chunks per fragment
  static constexpr int LA = BM / 8 / W, LB = BN / 8 / W;  // 1 KB row loads per wave
  static constexpr int SX = (BM / 32 + W - 1) / W, SW = (BN / 32 + W - 1) / W;  // scale loads
  static constexpr int NL = LA + LB + (MODE == 2 ? SX + SW : 1);
  static constexpr int SIDE = (BM + BN) * 128;         // side data offset in a stage
  static constexpr int SIDE_WS = BM * 8;               // MXFP4: B's scales after A's
  static constexpr int STAGE = SIDE + (MODE == 2 ? (BM + BN) * 8 : BN * 4);
  static constexpr int OUT_ROW = 272;                  // epilogue: 64 fp32 (or bf16) and 16 bytes
  static constexpr int LDS = R * STAGE;
  using acc_t = typename gemm_pick<MODE == 0, v16i_t, v16f_t>::type;
  static_assert(LA * 8 * W == BM && LB * 8 * W == BN, "whole row loads per wave");
  static_assert(NA % 2 == 0 && NB == 2, "the fragment pipeline alternates two A buffers");
  static_assert(LDS <= 160 * 1024, "the ring fits one CU");
  static_assert(W * 32 * OUT_ROW + BM * 4 <= LDS, "the epilogue's staging fits the ring");
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t gemm_rsrc(const void* base, int64_t bytes) {
  // raw buffer (stride 0); the third descriptor word of gfx9 data buffers.
  // The operands are workgroup-uniform: read them into scalar registers.
  const uint64_t p = (uint64_t)base;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)p);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32));
  const int n = __builtin_amdgcn_readfirstlane((int)bytes);
  return __builtin_amdgcn_make_buffer_rsrc((void*)(((uint64_t)hi << 32) | lo), (short)0, n, 0x00020000);
}

// The direct-to-LDS loads go through buffer resources based at the
// workgroup's first A row, B row, factor row and scale rows: a lane's 32-bit
// offset within them is fixed for the whole K loop and the stage's offset is
// a scalar.  LDS rows are 128 bytes with the 16-byte chunk c of row r at
// position c ^ ((r / 2) % 8): a wave's 1 KB load fills rows 8q .. 8q + 7 (lane
// l at row 8q + l / 8, position l % 8), and the 16 lanes of one LDS cycle
// reading one chunk of 16 consecutive rows cover the 64 banks exactly once.
// Rows past M or N read the last valid row: they only feed outputs that are
// never stored, and every access stays inside its resource.  Side loads are 4
// bytes a lane; waves past the side data's end repeat others' loads, so every
// wave issues the same number and the loop has no branch.
template <class C>
struct GemmLoads {
  __amdgpu_buffer_rsrc_t ra, rb, rg, rxs, rws;
  uint32_t a[C::LA], b[C::LB], g, xs[C::SX], ws[C::SW];
  int lm;  // log2 of the 128-deep K units per factor tile

  __device__ __forceinline__ GemmLoads(const hq_gemm_args& A, int64_t m0, int64_t n0, int wave, int lane) {
    const int64_t rb_ = C::MODE == 2 ? A.K / 2 : A.K;  // row bytes
    const int64_t T = A.K / A.tile, ks = A.K / 32;     // factors and MX scale bytes per row
    const int64_t ma = min<int64_t>(A.M - m0, C::BM), nb = min<int64_t>(A.N - n0, C::BN);
    ra = gemm_rsrc(A.xq + m0 * rb_, ma * rb_);
    rb = gemm_rsrc(A.w + n0 * rb_, nb * rb_);
    rg = gemm_rsrc(C::RESCALE ? A.g + n0 * T : nullptr, C::RESCALE ? nb * T * 4 : 0);
    rxs = gemm_rsrc(C::RESCALE ? nullptr : A.xs + m0 * ks, C::RESCALE ? 0 : ma * ks);
    rws = gemm_rsrc(C::RESCALE ? nullptr : A.ws + n0 * ks, C::RESCALE ? 0 : nb * ks);
    // row 8q + l / 8 holds chunk (l % 8) ^ ((4q + l / 16) % 8) at position l % 8
    auto off = [&](int q, int64_t rows) {
      return (uint32_t)(min<int64_t>(8 * q + (lane >> 3), rows - 1) * rb_) +
             (uint32_t)(((lane & 7) ^ ((4 * q + (lane >> 4)) & 7)) << 4);
    };
#pragma unroll
    for (int i = 0; i < C::LA; ++i) a[i] = off(wave * C::LA + i, ma);
#pragma unroll
    for (int i = 0; i < C::LB; ++i) b[i] = off(wave * C::LB + i, nb);
    lm = __builtin_ctz((uint32_t)(A.tile / HQ_TILE));
    g = (uint32_t)(min<int64_t>((wave % (C::BN / 64)) * 64 + lane, nb - 1) * T * 4);
    // scale dword d of a side array: row d / 2, half d % 2
#pragma unroll
    for (int i = 0; i < C::SX; ++i) {
      const int d = (wave + i * C::W) % (C::BM / 32) * 64 + lane;
      xs[i] = (uint32_t)(min<int64_t>(d >> 1, ma - 1) * ks + (d & 1) * 4);
    }
#pragma unroll
    for (int i = 0; i < C::SW; ++i) {
      const int d = (wave + i * C::W) % (C::BN / 32) * 64 + lane;
      ws[i] = (uint32_t)(min<int64_t>(d >> 1, nb - 1) * ks + (d & 1) * 4);
    }
  }

  // Direct-to-LDS loads of stage t into `stage` (wave is wave-uniform): B row
  // load i, and load n of the others (A rows, then the side data).
  __device__ __forceinline__ void fetch_b(int t, int wave, int8_t* stage, int i) const {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        rb, (lds_void_t*)(stage + C::BM * 128 + (wave * C::LB + i) * 1024), 16, b[i], (uint32_t)t * 128, 0, 0);
  }
  __device__ __forceinline__ void fetch_a(int t, int wave, int8_t* stage, int n) const {
    int8_t* const side = stage + C::SIDE;
    if (n < C::LA) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void_t*)(stage + (wave * C::LA + n) * 1024), 16,
                                               a[n < C::LA ? n : 0], (uint32_t)t * 128, 0, 0);
    } else if constexpr (C::RESCALE) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rg, (lds_void_t*)(side + (wave % (C::BN / 64)) * 256), 4, g,
                                               (uint32_t)((t >> lm) * 4), 0, 0);
    } else if (n < C::LA + C::SX) {
      const int i = n - C::LA;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rxs, (lds_void_t*)(side + (wave + i * C::W) % (C::BM / 32) * 256), 4, xs[i], (uint32_t)(t * 8), 0, 0);
    } else {
      const int i = n - C::LA - C::SX;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rws, (lds_void_t*)(side + C::SIDE_WS + (wave + i * C::W) % (C::BN / 32) * 256), 4, ws[i],
          (uint32_t)(t * 8), 0, 0);
    }
  }
};

// One 32-row operand block of a stage in registers: its fragments, and for
// MXFP4 the lane's scale words (the 8 scale bytes of its row, shifted so that
// byte 0 / byte 2 of the low word are the lane's blocks of the stage's first /
// second 64-deep step and those of the high word its third / fourth; the
// lane's half of step s is block 2 s + l / 32).
template <class C>
struct GemmFrag {
  v4i_t f[C::NS][C::FW];
  uint2 sc;

  __device__ __forceinline__ void set_scales(v2u_t v, int lane) {
    const int h = lane >> 5;
    sc = make_uint2(v.x >> (8 * h), v.y >> (8 * h));
  }
};

template <class T>
__device__ __forceinline__ const __attribute__((address_space(3))) T* lds_at(uint32_t addr) {
  return (const __attribute__((address_space(3))) T*)addr;
}

// The lane's part of a fragment's LDS address: its row inside a 32-row block
// and chunk c = s * FW * 2 + h * FW + w (int8: 32-deep step s, chunk 2 s + h;
// E4M3: 64-deep step s, chunks 4 s + 2 h and the next; MXFP4: 64-deep step s,
// chunk 2 s + h, one MX block), which row r holds at c ^ ((r / 2) % 8).
template <class C>
__device__ __forceinline__ uint32_t gemm_lane_addr(int s, int w, int lane) {
  const int r = lane & 31, h = lane >> 5;
  return (uint32_t)(r * 128 + (((s * C::FW * 2 + h * C::FW + w) ^ ((r >> 1) & 7)) << 4));
}

template <int OPSEL>
__device__ __forceinline__ v16f_t mfma_mxfp4(v4i_t a, v4i_t b, v16f_t c, uint32_t sa, uint32_t sb) {
  const v8i_t a8 = {a[0], a[1], a[2], a[3], 0, 0, 0, 0};
  const v8i_t b8 = {b[0], b[1], b[2], b[3], 0, 0, 0, 0};
  // cbsz = blgp = 4: both operands E2M1; the scales are E8M0 bytes
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8, b8, c, 4, 4, OPSEL, (int)sa, OPSEL, (int)sb);
}

// MFMA step s of one stage's block.
template <class C>
__device__ __forceinline__ typename C::acc_t gemm_step(const GemmFrag<C>& a, const GemmFrag<C>& b, int s,
                                                       typename C::acc_t c) {
  if constexpr (C::MODE == 0) {
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(a.f[s][0], b.f[s][0], c, 0, 0, 0);
  } else if constexpr (C::MODE == 1) {
    const v8i_t x = {a.f[s][0][0], a.f[s][0][1], a.f[s][0][2], a.f[s][0][3],
                     a.f[s][1][0], a.f[s][1][1], a.f[s][1][2], a.f[s][1][3]};
    const v8i_t y = {b.f[s][0][0], b.f[s][0][1], b.f[s][0][2], b.f[s][0][3],
                     b.f[s][1][0], b.f[s][1][1], b.f[s][1][2], b.f[s][1][3]};
    // cbsz = blgp = 0: both operands E4M3; scale bytes 127 (2^0)
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(x, y, c, 0, 0, 0, 127, 0, 127);
  } else {
    // step s of the stage is K unit s / 2: its scale word, byte 2 (s % 2)
    const uint32_t xa = s < 2 ? a.sc.x : a.sc.y, wb = s < 2 ? b.sc.x : b.sc.y;
    return (s & 1) ? mfma_mxfp4<2>(a.f[s][0], b.f[s][0], c, xa, wb) : mfma_mxfp4<0>(a.f[s][0], b.f[s][0], c, xa, wb);
  }
}

template <class C, int R0 = 0, int R1 = 16>
__device__ __forceinline__ void gemm_rescale(const typename C::acc_t& p, float g, float (&acc)[16]) {
#pragma unroll
  for (int r = R0; r < R1; ++r) acc[r] = __builtin_fmaf((float)p[r], g, acc[r]);
}

// fp32 -> bf16, round to nearest even (v_cvt_pk_bf16_f32).  Not by inline
// assembly: the value may be a matrix core's result, and the compiler does not
// look into assembly for the wait states before it.
__device__ __forceinline__ uint16_t gemm_bf16(float v) {
  return __builtin_bit_cast(uint16_t, (__bf16)v);
}

// One 32-row by 64-column slab of a wave's outputs: into the wave's LDS
// region in the MFMA layout (rows padded by 16 bytes, so that the two lane
// halves' rows fall in different banks), then to memory 16 bytes a lane
// along whole rows (element stores at a ragged right edge).
template <bool BF16>
__device__ __forceinline__ void gemm_store_slab(const hq_gemm_args& A, int8_t* tile, const float (&v)[2][16],
                                                int64_t r0, int64_t c0, int lane) {
  constexpr int ES = BF16 ? 2 : 4;  // bytes per value
  constexpr int RS = 64 * ES + 16;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      int8_t* const p = tile + (8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * RS + (b * 32 + (lane & 31)) * ES;
      if constexpr (BF16)
        *(uint16_t*)p = gemm_bf16(v[b][r]);
      else
        *(float*)p = v[b][r];
    }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  constexpr int VPL = 16 / ES, LPR = 64 / VPL, ROWS = 64 / LPR;  // values, lanes, rows per pass
#pragma unroll
  for (int i = 0; i < 32 / ROWS; ++i) {
    const int row = i * ROWS + lane / LPR, col = (lane % LPR) * VPL;
    const int64_t m = r0 + row, n = c0 + col;
    if (m >= A.M || n >= A.N) continue;
    const uint4 q = *(const uint4*)(tile + row * RS + col * ES);
    char* const dst = (char*)A.out + (m * A.N + n) * ES;
    if (n + VPL <= A.N && (uint64_t)dst % 16 == 0) {
      *(uint4*)dst = q;
    } else {
      const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int e = 0; e < VPL; ++e)
        if (n + e < A.N) {
          if constexpr (BF16)
            ((uint16_t*)dst)[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
          else
            ((uint32_t*)dst)[e] = w[e];
        }
    }
  }
}

// The output tile of workgroup `id`: workgroup i runs on XCD i % 8, so each
// XCD takes a contiguous run of the tile order, and the order walks groups of
// eight tile rows column by column: the tiles an XCD works on at one time
// share their operand rows in its L2.
__device__ __forceinline__ void gemm_tile_of(uint32_t id, uint32_t gm, uint32_t gn, uint32_t& tm, uint32_t& tn) {
  const uint32_t n = gm * gn, q = n / 8, r = n % 8, x = id % 8;
  const uint32_t s = x * q + min(x, r) + id / 8;
  const uint32_t grp = s / (8 * gn), first = grp * 8, rows = min(8u, gm - first), in = s - first * gn;
  tn = in / rows;
  tm = first + in - tn * rows;
}

// The product.  A wave walks its NA x NB blocks (a-major) once per stage:
// block j's MFMAs (one chain over the stage's K) are issued between parts of
// the previous block's rescale into the fp32 accumulators (an MFMA runs 32 or
// 64 cycles and takes one issue slot, so most of the rescale's VALU work runs
// under it), and each step's A fragment is replaced by the next block's as soon as
// its last MFMA is issued; scheduling barriers keep that order.  Before the
// stage's last block every fragment of the stage is in registers: there the
// wave waits for its own loads of the next stage, one workgroup barrier
// follows (the next stage is complete in LDS, and no wave still reads this
// one's A rows), A's loads of stage t + R begin into this stage's slot, and
// the next stage's first fragments are read under the last block's MFMAs.
//
// What bounds it: no one unit.  The matrix cores are busy 0.46 (int8), 0.52 (E4M3)
// and 0.47 (MXFP4) of the SIMD cycles at 256 x 256; a stage's fragment reads and
// row loads keep LDS for about as many cycles as its MFMAs take; and the rescale
// under them still costs int8 a quarter (4096 x 14336 x 4096 at tile 512, one
// rescale per four stages and 256 x 128 tiles: 256 us against 340).  With every CU busy
// the clock falls too: a stage takes 1.43 us on 8 CUs and 2.4 us on 256 (int8, tile
// 128), its MFMAs alone 0.87 us on constant and 1.24 us on random operands.  4096
// x 14336 x 4096, random operands: int8 288 us, E4M3 242 us, MXFP4 141 us, against
// 370, 318 and 230 us with 256 x 128 tiles whose eight waves alternated a load-and-
// rescale phase with an MFMA phase (64 x 64 outputs a wave: half as many products
// per LDS byte, and the two phases' times added up).
template <class C>
__device__ __forceinline__ void gemm_body(const hq_gemm_args& A) {
  using acc_t = typename C::acc_t;
  constexpr int J = C::NBLK - 1;
  constexpr bool KEEP = !C::RESCALE || C::LONG;  // a block's sums stay across stages
  extern __shared__ __attribute__((aligned(128))) int8_t gsm[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / C::WN, wn = wave % C::WN;
  uint32_t tm, tn;
  gemm_tile_of(blockIdx.x, (uint32_t)((A.M + C::BM - 1) / C::BM), (uint32_t)((A.N + C::BN - 1) / C::BN), tm, tn);
  const int64_t m0 = (int64_t)tm * C::BM, n0 = (int64_t)tn * C::BN;
  const int TS = (int)(A.K / HQ_TILE / C::U);                // stages
  const uint32_t tmask = (uint32_t)(A.tile / HQ_TILE) - 1u;  // LONG: stages per factor tile, less one

  float acc[C::RESCALE ? C::NBLK : 1][16];
  acc_t p[KEEP ? C::NBLK : 2];
  float g[2] = {0.0f, 0.0f}, gn[2] = {0.0f, 0.0f};
  if constexpr (C::RESCALE) {
#pragma unroll
    for (int j = 0; j < C::NBLK; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][r] = 0.0f;
  }
#pragma unroll
  for (int j = 0; j < (KEEP ? C::NBLK : 2); ++j) p[j] = (acc_t){};

  const GemmLoads<C> gl(A, m0, n0, wave, lane);
#pragma unroll
  for (int i = 0; i < C::R; ++i) {
#pragma unroll
    for (int n = 0; n < C::NL - C::LB; ++n) gl.fetch_a(min(i, TS - 1), wave, gsm + i * C::STAGE, n);
#pragma unroll
    for (int n = 0; n < C::LB; ++n) gl.fetch_b(min(i, TS - 1), wave, gsm + i * C::STAGE, n);
  }
  GemmFrag<C> fa, fb[2];
  // LDS addresses: of the lane's A fragments in the stage being read, less the
  // block; B's lie a wave-uniform distance behind, the side data's at `sv`
  const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int8_t*)gsm;
  const uint32_t b_off = (uint32_t)(C::BM * 128 + wn * 8192 - wm * (C::BM / C::WM) * 128);
  uint32_t av[C::NS][C::FW];
#pragma unroll
  for (int s = 0; s < C::NS; ++s)
#pragma unroll
    for (int w = 0; w < C::FW; ++w)
      av[s][w] = base + gemm_lane_addr<C>(s, w, lane) + (uint32_t)(wm * (C::BM / C::WM) * 128);
  const uint32_t sv = base + C::SIDE + (uint32_t)(lane & 31) * (C::RESCALE ? 4 : 8);
  const uint32_t sa = (uint32_t)(wm * (C::BM / C::WM) * 8);                       // MXFP4 scale rows
  const uint32_t sb = (uint32_t)(C::RESCALE ? wn * 256 : C::SIDE_WS + wn * 512);  // factors, or scale rows
  auto read_a = [&](uint32_t st, int a, int s) {
#pragma unroll
    for (int w = 0; w < C::FW; ++w) fa.f[s][w] = *lds_at<v4i_t>(av[s][w] + a * 4096);
    if (!C::RESCALE && s == C::NS - 1) fa.set_scales(*lds_at<v2u_t>(sv + (st + sa) + a * 256), lane);
  };
  auto read_b = [&](uint32_t st, int b) {
#pragma unroll
    for (int s = 0; s < C::NS; ++s)
#pragma unroll
      for (int w = 0; w < C::FW; ++w) fb[b].f[s][w] = *lds_at<v4i_t>((av[s][w] + b_off) + b * 4096);
    if (!C::RESCALE) fb[b].set_scales(*lds_at<v2u_t>(sv + (st + sb) + b * 256), lane);
  };
  auto read_g = [&](uint32_t st) {
    if constexpr (C::RESCALE)
#pragma unroll
      for (int b = 0; b < 2; ++b) gn[b] = *lds_at<float>(sv + (st + sb) + b * 128);
  };
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((C::R - 1) * C::NL) : "memory");
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = 0; s < C::NS; ++s) read_a(0, 0, s);
  read_b(0, 0);
  read_g(0);

  // The loads of stage t + R are spread over the blocks: B's rows from block 2
  // on (every wave has read its B fragments by then, a second barrier says
  // so), the others from the last block on.  Waves wait at a load until the
  // CU's address unit takes it (about 17 cycles for 1 KB), and a stage's loads
  // need most of a stage's time to land.
  constexpr int NLA = C::NL - C::LB;
  constexpr int PA = (NLA + 2) / 3, PB = (C::LB + J - 3) / (J - 2);  // loads per block
  uint32_t st = 0, stp = 0;  // this stage's slot, the previous one's
  for (int t = 0; t < TS; ++t) {
    const uint32_t stn = st + C::STAGE == C::R * C::STAGE ? 0 : st + C::STAGE;
    if constexpr (C::RESCALE && C::LONG) {
      if (((uint32_t)t & tmask) == 0u) {  // wave-uniform: a factor tile begins
#pragma unroll
        for (int j = 0; j < C::NBLK; ++j) {
          gemm_rescale<C>(p[j], g[j & 1], acc[j]);
          p[j] = (acc_t){};
        }
        g[0] = gn[0];
        g[1] = gn[1];
      }
    }
#pragma unroll
    for (int j = 0; j < C::NBLK; ++j) {
      const int a = j >> 1, b = j & 1;
      if (j == 0) read_b(st, 1);
      if (j == J) {
        // this wave's loads of the next stage: all but the newest R - 2 stages'
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((C::R - 2) * C::NL + C::LB) : "memory");
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < C::NS; ++s)
#pragma unroll
          for (int w = 0; w < C::FW; ++w) av[s][w] += stn - st;
        read_b(stn, 0);
        read_g(stn);
      }
      if (j == 2) asm volatile("s_barrier" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      acc_t c = {};
      if constexpr (KEEP) c = p[j];
      const int jp = j == 0 ? J : j - 1;
#pragma unroll
      for (int s = 0; s < C::NS; ++s) {
        // an MFMA, the read that replaces its A fragment, and a part of the
        // previous block's rescale, in this order
        c = gemm_step<C>(fa, fb[b], s, c);
        if (b == 1) read_a(j == J ? stn : st, j == J ? 0 : a + 1, s);
        if (j >= 2 && j < J) {
#pragma unroll
          for (int n = (j - 2) * PB + s * PB / C::NS; n < (j - 2) * PB + (s + 1) * PB / C::NS; ++n)
            if (n < C::LB) gl.fetch_b(min(t + C::R, TS - 1), wave, gsm + st, n);
        } else if (j == J || t > 0) {
          const int k = j == J ? 0 : j + 1, tf = j == J ? t + C::R : t - 1 + C::R;
#pragma unroll
          for (int n = k * PA + s * PA / C::NS; n < k * PA + (s + 1) * PA / C::NS; ++n)
            if (n < NLA) gl.fetch_a(min(tf, TS - 1), wave, gsm + (j == J ? st : stp), n);
        }
        if constexpr (!KEEP) {
          constexpr int E = 16 / C::NS;
#pragma unroll
          for (int r = 0; r < E; ++r)
            acc[jp][s * E + r] = __builtin_fmaf((float)p[jp & 1][s * E + r], g[jp & 1], acc[jp][s * E + r]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (KEEP) {
        p[j] = c;
      } else {
        p[j & 1] = c;
        if (j == 0) {
          g[0] = gn[0];
          g[1] = gn[1];
        }
      }
    }
    stp = st;
    st = stn;
  }
  // the loads that the last barrier's stage did not issue are left out: they
  // would only refill a slot that nothing reads
  if constexpr (C::RESCALE) {
    if constexpr (C::LONG) {
#pragma unroll
      for (int j = 0; j < C::NBLK; ++j) gemm_rescale<C>(p[j], g[j & 1], acc[j]);
    } else {
      gemm_rescale<C>(p[J & 1], g[1], acc[J]);
    }
  }
  // every wave's re-fetches of the last stage have landed: the ring is free
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  float* const s_sx = (float*)(gsm + C::W * 32 * C::OUT_ROW);
  if constexpr (C::RESCALE) {
    for (int i = tid; i < C::BM; i += C::W * 64) s_sx[i] = A.sx[min<int64_t>(m0 + i, A.M - 1)];
    __syncthreads();
  }
  int8_t* const tile = gsm + wave * 32 * C::OUT_ROW;
#pragma unroll
  for (int a = 0; a < C::NA; ++a) {
    const int row0 = wm * (C::BM / C::WM) + a * 32;
    float v[2][16];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if constexpr (C::RESCALE)
          v[b][r] = s_sx[row0 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)] * acc[2 * a + b][r];
        else
          v[b][r] = p[2 * a + b][r];
      }
    if (A.out_bf16)
      gemm_store_slab<true>(A, tile, v, m0 + row0, n0 + wn * 64, lane);
    else
      gemm_store_slab<false>(A, tile, v, m0 + row0, n0 + wn * 64, lane);
  }
}

// At most 256 registers (two waves per SIMD), also where a workgroup's LDS
// leaves room for one wave: beyond them the compiler puts the products in
// accumulation registers, which the rescale cannot read, and copies them (104
// copies in 248 vector instructions of an E4M3 stage at 128 x 128).  Measured
// with and without: 768 x 6144 x 14336 in E4M3 155 -> 131 us, in int8 171 -> 151.
template <class C>
__global__ __launch_bounds__(C::W * 64, 2) void hq_gemm_kernel(hq_gemm_args A) {
  gemm_body<C>(A);
}

template <class C>
int gemm_launch(const hq_gemm_args& a, hipStream_t st) {
  static hq_lds_granted granted;
  if (const int e = hq_allow_lds((const void*)hq_gemm_kernel<C>, C::LDS, granted)) return e;
  const int64_t wgs = ((a.M + C::BM - 1) / C::BM) * ((a.N + C::BN - 1) / C::BN);
  hipLaunchKernelGGL(hq_gemm_kernel<C>, dim3((uint32_t)wgs), dim3(C::W * 64), C::LDS, st, a);
  return (int)hipGetLastError();
}

template <int MODE>
int gemm_dispatch(const hq_gemm_args& a, hipStream_t st) {
  const bool lng = MODE != 2 && a.tile > HQ_TILE;
  const hq_gemm_tile t = hq_gemm_tile_of(MODE, lng, a.M, a.N);
  if constexpr (MODE != 2) {
    if (lng) {
      if (t == HQ_GEMM_64x64) return gemm_launch<GemmCfg<MODE, 64, 64, 1, 1, true, 4>>(a, st);
      if (t == HQ_GEMM_128x128) return gemm_launch<GemmCfg<MODE, 128, 128, 2, 2, true, 4>>(a, st);
      return gemm_launch<GemmCfg<MODE, 256, 128, 4, 2, true, 3>>(a, st);
    }
  }
  if (t == HQ_GEMM_64x64) return gemm_launch<GemmCfg<MODE, 64, 64, 1, 1, false, 4>>(a, st);
  if (t == HQ_GEMM_128x128) return gemm_launch<GemmCfg<MODE, 128, 128, 2, 2, false, 4>>(a, st);
  if (t == HQ_GEMM_256x128) return gemm_launch<GemmCfg<MODE, 256, 128, 4, 2, false, 3>>(a, st);
  return gemm_launch<GemmCfg<MODE, 256, 256, 2, 4, false, 2>>(a, st);
}

}  // namespace

int hq_launch_gemm(const hq_gemm_args& a, void* stream) {
  if (a.K % 256 != 0) return -1;  // an even number of 128-deep K tiles
  hipStream_t st = (hipStream_t)stream;
  if (a.fp8 == 2) return gemm_dispatch<2>(a, st);
  return a.fp8 ? gemm_dispatch<1>(a, st) : gemm_dispatch<0>(a, st);
}
