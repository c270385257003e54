// Softmax attention on the matrix cores (v_mfma_f32_32x32x16_bf16) for head dimensions 32 and 64 and
// bf16 storage: forward, and the backward pass split into a query-major and a key-major kernel.
// Operands are quantizer codes (Section 3.1: Q, K, V and the softmax probabilities are quantized
// before their products), so Q*K^T and P*V are exact integer products in fp32.
//
// Layout trick used throughout: the score tile is computed transposed,
// D[key][query] = K_tile * Q_tile^T, so that in the 32x32 accumulator layout a lane
// owns ONE query (lane % 32) and 16 of the 32 keys of the tile; the other 16 keys sit
// in lane ^ 32.  Row-wise softmax statistics then need a single cross-lane exchange,
// and the accumulator registers already have the layout of the B operand of the next
// product (contraction over keys), with the key order fixed by `key_of`.  The key-major
// kernel mirrors it: D[query][key] = Q_tile * K_tile^T, a lane owns one key.
//
// All tiles (K, V, Q, dC) sit row-major in LDS as they do in memory; where a product
// needs an operand with the contraction index along the rows, the fragment is gathered
// with the transposing LDS read (ds_read_tr16_b64), see `ld_frag_tr`.
//
// A block is up to 128 rows (32 per wavefront) of one (batch, head).  The other side of the
// product passes through LDS in chunks of 128 rows, so a block takes 37 KB (20 KB for head
// dimension 32) and registers, not LDS, say how many share a compute unit.  Up to 128 keys (one
// chunk) the scores and probabilities stay in registers between the pass that forms the row
// statistics and the pass that uses them.  Longer rows are shared out among the wavefronts of a block of 32
// queries (attn_fwd_row_k, attn_bwd_q_row_k), with three exceptions: the query-major kernel of the FAST
// arithmetic forms its tiles again for each pass; the key-major kernels, whose rows are keys, take 128 of
// them a block and the queries in chunks; and the forward on real-valued operands (REAL) keeps a row of up
// to 512 keys in one wavefront, since its products are chains.  The scores, the exponentials and the
// quantizer are vector-ALU work, which is what bounds these kernels, and a whole row in one wavefront's
// registers leaves one wavefront per SIMD.  Wavefronts per SIMD (head dimension 64, not REAL): forward 3 to 4;
// query-major backward 2 to 3 (160 to 256 registers).  Chunks beyond the valid keys of a sequence are skipped.
#include "mrem_common.h"
#include "mrem_kernels.h"

#include <type_traits>

namespace mrem {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

constexpr int kChunk = 128;  // rows of the other operand in LDS at a time
// elements per row of a row-major LDS tile (144 or 80 bytes: 16-byte stores and reads without bank conflicts)
template <int D>
struct Tile { static constexpr int kStride = D + 8; };

// key (row of the transposed score tile) held in accumulator register i of a lane in half h
__device__ __forceinline__ int key_of(int t, int i, int h) { return 32 * t + 8 * (i >> 2) + 4 * h + (i & 3); }

struct FwdScales {
  float qk, sp, sv, p_qp;
  float rsp;  // correctly rounded 1 / sp
};
// x / d from rd = fl(1 / d): t = fl(x * rd), then t + fl(x - d * t) * rd with fused multiply-adds.
// The residual is exact and, rd being correctly rounded, the result is the correctly rounded
// quotient (the residual-correction step of FMA division), so this matches an IEEE division while
// one reciprocal serves a whole row (softmax sums) or tensor (step sizes).
__device__ __forceinline__ float div_by(float x, float d, float rd) {
  const float t = __fmul_rn(x, rd);
  return __fmaf_rn(__fmaf_rn(-d, t, x), rd, t);
}
// Two arithmetics.  Which one serves a shape is part of its results: a probability that rounds the other way flips a code,
// and flips multiply from layer to layer, so the bits of a forward pass are kept.
//   FAST (head dimension 64, 64 to 384 tokens): the hardware's 2^t with t rounded to fp32 (up to 20 ulp for the smallest
//     probabilities), a row's exponentials added one after the other by each half wavefront.
//   otherwise: expf, and the order of a row that is spread over 64 lanes, lane l adding keys l, l + 64, ... and the lanes
//     meeting in a binary tree; products of operands that are not integer codes are fp32 fused multiply-adds with the
//     contraction index ascending where the caller asks for it (see Epilogue::chain).  These are the results of the
//     scalar kernels (mrem_attn.hip), bit for bit.
template <bool FAST>
__device__ __forceinline__ float exp_neg(float x) {
  if constexpr (FAST) return __expf(x);
  else return expf(x);
}
__device__ __forceinline__ FwdScales load_fwd_scales(const AttnQ& a, int d) {
  FwdScales s;
  const float sq = a.q.on ? *a.q.s : 1.f, sk = a.k.on ? *a.k.s : 1.f;
  s.sp = a.p.on ? *a.p.s : 1.f;
  s.sv = a.v.on ? *a.v.s : 1.f;
  s.qk = sq * sk / sqrtf((float)d);
  s.p_qp = a.p.qp;
  s.rsp = __fdiv_rn(1.0f, s.sp);
  return s;
}

// a - b, an operation of its own: never half of a fused multiply-add, whatever the compiler finds in front of it
__device__ __forceinline__ float sub_apart(float a, float b) {
#pragma clang fp contract(off)
  return a - b;
}
// scores of 32 keys from accumulators, first key `key0`; -inf beyond the valid keys (a tile without such keys skips the tests,
// two of the six instructions a score costs a forward pass ahead of its exponential)
__device__ __forceinline__ void mask_scores(f32x16_t& a, int key0, int half, int len) {
  if (key0 + 32 <= len) return;
#pragma unroll
  for (int r = 0; r < 16; ++r)
    if (key_of(0, r, half) + key0 >= len) a[r] = -INFINITY;
}
__device__ __forceinline__ void scale_scores(f32x16_t& a, const FwdScales& sc, int key0, int half, int len) {
#pragma unroll
  for (int r = 0; r < 16; ++r) a[r] = __fmul_rn(a[r], sc.qk);
  mask_scores(a, key0, half, len);
}
// the same plus `c`, in one rounding: how the backward pass takes a score less the row's maximum
__device__ __forceinline__ void scale_scores(f32x16_t& a, const FwdScales& sc, int key0, int half, int len, float c) {
#pragma unroll
  for (int r = 0; r < 16; ++r) a[r] = __fmaf_rn(a[r], sc.qk, c);
  mask_scores(a, key0, half, len);
}
// what the exponentials of a row are taken against: with a row of -inf only, 0, so that each of them is 0 and not NaN
__device__ __forceinline__ float finite_max(float mx) { return mx == -INFINITY ? 0.f : mx; }
// code of a probability (NaN gives code 0; PQ: its quantizer is on), or the probability itself.  PQ is an argument of every
// kernel: a test on each element made each a basic block of its own, so that a lane's sixteen chains of dependent operations
// ran one after the other instead of side by side.
template <bool PQ>
__device__ __forceinline__ float prob_code(float p, const FwdScales& sc) {
  return PQ ? rintf(__builtin_amdgcn_fmed3f(div_by(p, sc.sp, sc.rsp), 0.f, sc.p_qp)) : p;
}

// Rows [0, S) of a [S, D] slice (row stride ld elements) on their way to LDS, row-major, zero rows up to s_pad.  A block of w
// wavefronts takes at most 32 w rows, D / 16 pieces of 16 bytes a thread; all of them are in flight at once, and those of a
// second slice with them.  With that, PQ, and accumulators in ordinary registers (a bound of two wavefronts a SIMD: without
// one the compiler moved them to accumulation registers and back for every tile), alone, us: forward over 512 heads of 128
// keys 16.1 -> 14.4 (mean of both passes), query-major backward 26.3 -> 23.1; key-major backward over 256 heads of 384 70 ->
// 46, over 96 heads of 512 65 -> 50.  All are bound by vector-ALU instructions now (40 to 70 percent of the cycles).
template <int D>
struct Rows {
  u32x4_t v[D / 16];
  __device__ __forceinline__ void load(const bf16_t* __restrict__ src, int ld, int S) {
#pragma unroll
    for (int i = 0; i < D / 16; ++i) {
      const int q = threadIdx.x + i * blockDim.x, row = max(min(q / (D / 8), S - 1), 0);
      v[i] = *reinterpret_cast<const u32x4_t*>(src + (size_t)row * ld + q % (D / 8) * 8);
    }
  }
  __device__ __forceinline__ void store(bf16_t* dst, int S, int s_pad) const {
#pragma unroll
    for (int i = 0; i < D / 16; ++i) {
      const int q = threadIdx.x + i * blockDim.x, row = q / (D / 8);
      if (row < s_pad) *reinterpret_cast<u32x4_t*>(dst + row * Tile<D>::kStride + q % (D / 8) * 8) = row < S ? v[i] : u32x4_t{0u, 0u, 0u, 0u};
    }
  }
};
__device__ __forceinline__ bf16x8_t ld_frag(const bf16_t* p) { return *reinterpret_cast<const bf16x8_t*>(p); }

// MFMA operand fragment gathered down the rows of a row-major LDS tile with the
// transposing LDS read (ds_read_b64_tr_b16): lane l receives, for column c0 + l%32, rows
// r_first + 0..3 and r_second + 0..3 (the caller picks the two row bases for its half l/32).  In a
// group of 16 lanes, lane s supplies the 8-byte chunk of row s/4, columns 4*(s%4)..+3, and receives
// column s of the four rows.  Lets K, V, Q and dC stay row-major in LDS (16-byte conflict-free stores)
// where the products contract over their row index.
typedef short s16x4_t __attribute__((ext_vector_type(4)));
template <int D>
__device__ __forceinline__ bf16x8_t ld_frag_tr(const bf16_t* tile, int c0, int r_first, int r_second, int lane) {
  const int g = lane >> 4, s = lane & 15;
  const bf16_t* p = tile + (s >> 2) * Tile<D>::kStride + c0 + 16 * (g & 1) + 4 * (s & 3);
  union { bf16x8_t v; s16x4_t h[2]; } u;
  u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(p + r_first * Tile<D>::kStride));
  u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(p + r_second * Tile<D>::kStride));
  return u.v;
}

__device__ __forceinline__ void store4(bf16_t* p, float a, float b, float c, float d) {
  bf16x4_t v = {static_cast<bf16_t>(a), static_cast<bf16_t>(b), static_cast<bf16_t>(c), static_cast<bf16_t>(d)};
  *reinterpret_cast<bf16x4_t*>(p) = v;
}

__device__ __forceinline__ f32x16_t zero16() {
  f32x16_t z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}
// a 32 x 32 tile: rows [row0, row0 + 32) of the LDS tile times the transposed 32 rows held as fragments (one per 16 columns)
template <int D>
__device__ __forceinline__ f32x16_t tile_product(const bf16_t* tile, int row0, int lane, const bf16x8_t (&frag)[D / 16]) {
  f32x16_t acc = zero16();
  const bf16_t* p = tile + (row0 + (lane & 31)) * Tile<D>::kStride + (lane >> 5) * 8;
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ld_frag(p + kk * 16), frag[kk], acc, 0, 0, 0);
  return acc;
}
// acc[e][lane's row] += sum over the tile's 32 rows (LDS rows [row0, row0 + 32)) of tile[row][e] * w[row], with w in
// accumulator order (key_of): the contraction over what the accumulator registers of a tile enumerate
template <int D>
__device__ __forceinline__ void accumulate_rows(f32x16_t (&acc)[D / 32], const bf16_t* tile, int row0, int lane, const float* w) {
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    bf16x8_t f;
#pragma unroll
    for (int i = 0; i < 8; ++i) f[i] = static_cast<bf16_t>(w[8 * s + i]);
    const int k0 = row0 + 16 * s + 4 * (lane >> 5);
#pragma unroll
    for (int et = 0; et < D / 32; ++et)
      acc[et] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ld_frag_tr<D>(tile, 32 * et, k0, k0 + 8, lane), f, acc[et], 0, 0, 0);
  }
}

// accumulate_rows with the rows in natural order along the contraction (8 consecutive ones a half wavefront), which is the
// order of sums that the key gradients of FAST shapes keep: the halves exchange every other four rows
template <int D>
__device__ __forceinline__ void accumulate_rows_natural(f32x16_t (&acc)[D / 32], const bf16_t* tile, int row0, int lane, const float* w) {
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    union { bf16x8_t v; unsigned u[4]; } f;
#pragma unroll
    for (int i = 0; i < 8; ++i) f.v[i] = static_cast<bf16_t>(w[8 * s + i]);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const auto x = __builtin_amdgcn_permlane32_swap(f.u[i], f.u[i + 2], false, false);
      f.u[i] = x[0];
      f.u[i + 2] = x[1];
    }
    const int k0 = row0 + 16 * s + 8 * (lane >> 5);
#pragma unroll
    for (int et = 0; et < D / 32; ++et)
      acc[et] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ld_frag_tr<D>(tile, 32 * et, k0, k0 + 4, lane), f.v, acc[et], 0, 0, 0);
  }
}
// The same two products for operands that are not integer codes, as chains of fp32 fused multiply-adds:
// v_mfma_f32_32x32x2_f32 adds its two products with k ascending and rounds after each (16 times the cycles of the bf16 form).
// Values 2 j (lower half of the wavefront) and 2 j + 1 (upper half) of 8 consecutive ones:
__device__ __forceinline__ float pick(unsigned pair, int half) { return __uint_as_float(half ? pair & 0xffff0000u : pair << 16); }
template <int D>
__device__ __forceinline__ f32x16_t tile_product_chain(const bf16_t* tile, int row0, int lane, const float (&frag)[D / 2]) {
  f32x16_t acc = zero16();
  const bf16_t* p = tile + (row0 + (lane & 31)) * Tile<D>::kStride;
#pragma unroll
  for (int c = 0; c < D / 8; ++c) {
    const u32x4_t v = *reinterpret_cast<const u32x4_t*>(p + 8 * c);
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(pick(v[j], lane >> 5), frag[4 * c + j], acc, 0, 0, 0);
  }
  return acc;
}
template <int D>
__device__ __forceinline__ void accumulate_rows_chain(f32x16_t (&acc)[D / 32], const bf16_t* tile, int row0, int lane, const float* w) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    // registers 4 g .. 4 g + 3 hold rows 8 g + 0..3 in the lower half of the wavefront and 8 g + 4..7 in the upper one;
    // exchanging halves gives pairs (row, row + 1) of the two halves: 0 1, 4 5 from the first two registers, 2 3, 6 7
    float b[4];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(w[4 * g + 2 * i]), __float_as_uint(w[4 * g + 2 * i + 1]), false, false);
      b[i] = __uint_as_float(x[0]);
      b[2 + i] = __uint_as_float(x[1]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bf16_t* row = tile + (row0 + 8 * g + 2 * i + (lane >> 5)) * Tile<D>::kStride + (lane & 31);
#pragma unroll
      for (int et = 0; et < D / 32; ++et)
        acc[et] = __builtin_amdgcn_mfma_f32_32x32x2f32(static_cast<float>(row[32 * et]), b[i], acc[et], 0, 0, 0);
    }
  }
}
// accumulate_rows with weights of 24 bits, in three bf16 parts that add up to them (the gradient of a score where it is
// held in 32 bits: the sum over a row is zero, and 16 bits leave 2^-9 of its terms)
template <int D>
__device__ __forceinline__ void accumulate_rows_wide(f32x16_t (&acc)[D / 32], const bf16_t* tile, int row0, int lane, const float* w) {
  float rest[16], part[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) rest[r] = w[r];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      part[r] = round_to<bf16_t>(rest[r]);
      rest[r] = __fsub_rn(rest[r], part[r]);
    }
    accumulate_rows<D>(acc, tile, row0, lane, part);
  }
}

// sum of a lane's 16 partial sums and those of the other half of the wavefront, in the order of the binary tree
__device__ __forceinline__ float sum_of_parts(const float (&part)[16]) {
  float x[4];  // keys 8 g .. 8 g + 7: bits 0 and 1 of the key, then bit 2, which is the half of the wavefront
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    x[g] = (part[4 * g] + part[4 * g + 1]) + (part[4 * g + 2] + part[4 * g + 3]);
    x[g] += __shfl_xor(x[g], 32, 64);
  }
  return (x[0] + x[1]) + (x[2] + x[3]);
}
// a wavefront's partial ranges: of its rows' largest probabilities, and behind all of those of its part of the context
__device__ __forceinline__ void store_ranges(float* __restrict__ ranges, int part, int nparts, const MinMax& pmax, const MinMax& ctx, int lane) {
  const MinMax p = pmax.wave(), c = ctx.wave();
  if (lane == 0) {
    p.store(ranges + (size_t)part * 3);
    c.rounded<bf16_t>().store(ranges + ((size_t)nparts + part) * 3);
  }
}
// 32 columns of the context of a lane's query (16 of them here, from element `o` on) and their codes
template <bool FAST>
__device__ __forceinline__ void store_context(const f32x16_t& acc, const AttnQ& aq, const FwdScales& sc, int len, size_t o, bf16_t* __restrict__ ctx,
                                              bf16_t* __restrict__ ctx_codes, int8_t* __restrict__ ctx_codes8, MinMax& range) {
  const float os = sc.sp * sc.sv;
  QuantParam qc5 = {aq.c.on ? *aq.c.s : 1.f, 0.f, aq.c.qn, aq.c.qp, aq.c.on, 0.f};
  qc5.rs = quant_reciprocal(qc5.s);
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float a = acc[4 * g + i];
      // a sequence without a valid key has no softmax
      v[i] = len <= 0 ? NAN : FAST ? __fmul_rn(a, os) : __fmul_rn(__fmul_rn(a, sc.sp), sc.sv);
    }
    store4(ctx + o + 8 * g, v[0], v[1], v[2], v[3]);
#pragma unroll
    for (int i = 0; i < 4; ++i) range.add(v[i]);  // (dead where nobody asks)
    if (ctx_codes || ctx_codes8) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float r = round_to<bf16_t>(v[i]);
        v[i] = qc5.on ? q_code(q_ratio_fma(r, qc5), qc5) : r;
      }
      if (ctx_codes) store4(ctx_codes + o + 8 * g, v[0], v[1], v[2], v[3]);
      if (ctx_codes8) {
        const unsigned pk = ((unsigned)(int)v[0] & 0xffu) | (((unsigned)(int)v[1] & 0xffu) << 8) | (((unsigned)(int)v[2] & 0xffu) << 16) |
                            (((unsigned)(int)v[3] & 0xffu) << 24);
        *reinterpret_cast<unsigned*>(ctx_codes8 + o + 8 * g) = pk;
      }
    }
  }
}

// ------------------------------------------------------------------------------
// forward: one block = up to 128 queries of one (batch, head); one wavefront = 32 queries
// ONE: at most 128 keys.  REAL: the operands are not integer codes and their products are chains (not FAST).
// ------------------------------------------------------------------------------
template <int D, bool ONE, bool FAST, bool REAL, bool PQ>
__global__ __launch_bounds__(256, ONE ? 2 : 1) void attn_fwd_mfma_k(const bf16_t* __restrict__ codes, bf16_t* __restrict__ ctx,
                                                       bf16_t* __restrict__ ctx_codes, AttnQ aq, const int32_t* __restrict__ seqlens,
                                                       int S, int H, float* __restrict__ ranges, float* __restrict__ stat_m,
                                                       float* __restrict__ stat_l, int8_t* __restrict__ ctx_codes8) {
  __shared__ __attribute__((aligned(16))) bf16_t Ks[kChunk * Tile<D>::kStride];
  __shared__ __attribute__((aligned(16))) bf16_t Vs[kChunk * Tile<D>::kStride];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5;
  const int h = blockIdx.y, b = blockIdx.z, nh = gridDim.y;
  const int ld = 3 * H;
  const bf16_t* base = codes + (size_t)b * S * ld + h * D;
  const int len = seqlens ? min(seqlens[b], S) : S;
  const int rows = FAST ? S : len;  // keys that are staged: those beyond are zero rows
  const FwdScales sc = load_fwd_scales(aq, D);

  const int q0 = blockIdx.x * 128 + wave * 32;
  const int waves = blockDim.x >> 6, nparts = gridDim.x * nh * gridDim.z * waves, part_idx = ((b * nh + h) * gridDim.x + blockIdx.x) * waves + wave;
  const bool active = q0 < S;
  const int q = q0 + (lane & 31);
  const int qc = q < S ? q : S - 1;
  bf16x8_t qf[D / 16];
  float qr[D / 2];
  if constexpr (REAL) {
#pragma unroll
    for (int c = 0; c < D / 8; ++c) {
      const u32x4_t v = *reinterpret_cast<const u32x4_t*>(base + (size_t)qc * ld + 8 * c);
#pragma unroll
      for (int j = 0; j < 4; ++j) qr[4 * c + j] = pick(v[j], half);
    }
  } else {
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) qf[kk] = ld_frag(base + (size_t)qc * ld + (kk * 2 + half) * 8);
  }

  // scores of 32 keys (chunk rows [32 t, 32 t + 32), first key j0), -inf beyond the valid keys
  auto scores = [&](int t, int j0) {
    f32x16_t a;
    if constexpr (REAL) a = tile_product_chain<D>(Ks, 32 * t, lane, qr);
    else a = tile_product<D>(Ks, 32 * t, lane, qf);
    scale_scores(a, sc, j0 + 32 * t, half, len);
    return a;
  };
  f32x16_t oacc[D / 32];
#pragma unroll
  for (int et = 0; et < D / 32; ++et) oacc[et] = zero16();
  float mx = -INFINITY, sum = 0.f;
  // probabilities from exponentials, quantized, times V
  auto weigh = [&](const f32x16_t& e, int t, float rsum) {
    float w[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float p = div_by(e[r], sum, rsum);
      w[r] = REAL ? round_to<bf16_t>(p) : prob_code<PQ>(p, sc);
    }
    if constexpr (REAL) accumulate_rows_chain<D>(oacc, Vs, 32 * t, lane, w);
    else accumulate_rows<D>(oacc, Vs, 32 * t, lane, w);
  };
  auto exps = [&](const f32x16_t& a) {
    f32x16_t e;
    const float top = finite_max(mx);
#pragma unroll
    for (int r = 0; r < 16; ++r) e[r] = exp_neg<FAST>(sub_apart(a[r], top));
    return e;
  };
  auto raise_max = [&](const f32x16_t& a) {
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, a[r]);
  };
  // the row sum in the order of the arithmetic; `odd`: parity of the tile (keys l and l + 64 are two tiles apart)
  float part[2][16];
  if constexpr (!FAST) {
#pragma unroll
    for (int r = 0; r < 16; ++r) part[0][r] = part[1][r] = 0.f;
  }
  auto add_exps = [&](const f32x16_t& e, auto odd) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if constexpr (FAST) sum += e[r];
      else part[decltype(odd)::value][r] += e[r];
    }
  };
  auto finish_sum = [&]() {
    if constexpr (FAST) {
      sum += __shfl_xor(sum, 32, 64);
    } else {
      const float y = sum_of_parts(part[0]);
      sum = y + sum_of_parts(part[1]);
    }
  };
  constexpr std::integral_constant<int, 0> even{};
  constexpr std::integral_constant<int, 1> odd{};
  if constexpr (ONE) {
    const int nt = (len + 31) / 32;
    Rows<D> kr, vr;
    kr.load(base + H, ld, rows);
    vr.load(base + 2 * H, ld, rows);
    kr.store(Ks, rows, 32 * nt);
    vr.store(Vs, rows, 32 * nt);
    __syncthreads();
    if (!active) {
      if (ranges) store_ranges(ranges, part_idx, nparts, MinMax(), MinMax(), lane);
      return;
    }
    f32x16_t sacc[kChunk / 32];
#pragma unroll
    for (int t = 0; t < kChunk / 32; ++t)
      if (t < nt) {
        sacc[t] = scores(t, 0);
        raise_max(sacc[t]);
      }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
#pragma unroll
    for (int t = 0; t < kChunk / 32; ++t)
      if (t < nt) {
        sacc[t] = exps(sacc[t]);
        if (t & 1) add_exps(sacc[t], odd);
        else add_exps(sacc[t], even);
      }
    finish_sum();
    const float rsum = __fdiv_rn(1.0f, sum);
#pragma unroll
    for (int t = 0; t < kChunk / 32; ++t)
      if (t < nt) weigh(sacc[t], t, rsum);
  } else {
    static_assert(REAL, "rows of more than one chunk: attn_fwd_row_k");
    // a chain of products is formed once: the whole row (up to 512 keys) stays in registers
    constexpr int C = 512 / kChunk, N = kChunk / 32;
    f32x16_t sacc[C * N];
    Rows<D> rr;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int left = len - c * kChunk;
      if (left <= 0) break;
      rr.load(base + (size_t)c * kChunk * ld + H, ld, left);
      __syncthreads();
      rr.store(Ks, left, min((left + 31) / 32 * 32, kChunk));
      __syncthreads();
      if (active)
#pragma unroll
        for (int t = 0; t < N; ++t)
          if (32 * t < left) {
            sacc[N * c + t] = scores(t, c * kChunk);
            raise_max(sacc[N * c + t]);
          }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
#pragma unroll
    for (int t = 0; t < C * N; ++t)
      if (32 * t < len) {
        sacc[t] = exps(sacc[t]);
        if (t & 1) add_exps(sacc[t], odd);
        else add_exps(sacc[t], even);
      }
    finish_sum();
    const float rsum = __fdiv_rn(1.0f, sum);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int left = len - c * kChunk;
      if (left <= 0) break;
      rr.load(base + (size_t)c * kChunk * ld + 2 * H, ld, left);
      __syncthreads();
      rr.store(Vs, left, min((left + 31) / 32 * 32, kChunk));
      __syncthreads();
      if (active)
#pragma unroll
        for (int t = 0; t < N; ++t)
          if (32 * t < left) weigh(sacc[N * c + t], t, rsum);
    }
    if (!active) {
      if (ranges) store_ranges(ranges, part_idx, nparts, MinMax(), MinMax(), lane);
      return;
    }
  }
  const size_t stat_idx = ((size_t)b * nh + h) * S + q;
  MinMax pmax, range;
  if (half == 0 && q < S) {
    if (stat_m) { stat_m[stat_idx] = mx; stat_l[stat_idx] = sum; }
    pmax.add(1.0f / sum);  // the largest exponential of a row is exp(0) = 1
  }
  if (q < S) {
    const size_t orow = ((size_t)b * S + q) * H + h * D;
#pragma unroll
    for (int et = 0; et < D / 32; ++et) store_context<FAST>(oacc[et], aq, sc, len, orow + 32 * et + 4 * half, ctx, ctx_codes, ctx_codes8, range);
  }
  if (ranges) store_ranges(ranges, part_idx, nparts, pmax, range, lane);
}

// ------------------------------------------------------------------------------
// Rows of more than 128 keys: a block is 32 queries, its four wavefronts share out the keys, so that a wavefront's scores (up
// to four tiles) stay in registers from the product to the probabilities.  A sum rescaled whenever the maximum rises would be
// another sum; this way every exponential is still formed once and not twice, every score once and not three times.  Maximum
// and row sum pass through LDS, the sum from wavefront to wavefront, since its order is part of the result.  The probabilities
// go to LDS as the fragments of their product with V, which one wavefront per 32 columns forms, in the order of the keys.
// K comes straight from memory (no two wavefronts read the same rows), V through LDS in chunks of 128 rows.
// Vector-ALU instructions bound it; 3 or 4 blocks a compute unit.  Inside a step, against 128 queries a block, every tile
// formed three times: 8 x 512 tokens, 12 heads: 99 -> 53 us; 16 x 384 tokens, 16 heads: 87 -> 69 us.
// ------------------------------------------------------------------------------

// Which head and which of the nq blocks of its rows a block takes: the blocks of a head run on one XCD, whose L2 then holds the
// other side of its products.  Blocks are dealt out to the eight XCDs in turn; heads beyond a multiple of eight go in order.
__device__ __forceinline__ void row_of_block(int nq, int heads, int& head, int& blk) {
  const int id = blockIdx.x, dealt = heads / 8 * 8 * nq;
  if (id < dealt) {
    head = id / 8 / nq * 8 + id % 8;
    blk = id / 8 % nq;
  } else {
    head = heads / 8 * 8 + (id - dealt) / nq;
    blk = (id - dealt) % nq;
  }
}

template <int D, bool FAST, bool PQ>
__global__ __launch_bounds__(256, FAST ? 4 : 3) void attn_fwd_row_k(const bf16_t* __restrict__ codes, bf16_t* __restrict__ ctx, bf16_t* __restrict__ ctx_codes,
                                                         AttnQ aq, const int32_t* __restrict__ seqlens, int S, int B, int nh,
                                                         float* __restrict__ ranges, float* __restrict__ stat_m, float* __restrict__ stat_l,
                                                         int8_t* __restrict__ ctx_codes8) {
  // tiles of a wavefront (up to 384 or 512 keys); rows of V in LDS at a time (FAST: four blocks a compute unit); 16-byte pieces of those per thread
  constexpr int TW = FAST ? 3 : 4, RC = 32 * TW, CH = RC * (D / 8) / 256;
  static_assert(RC * (D / 8) % 256 == 0, "whole pieces");
  __shared__ __attribute__((aligned(16))) bf16_t Vs[RC * Tile<D>::kStride];
  // the sums on their way from wavefront to wavefront, then the fragments of the probabilities
  __shared__ __attribute__((aligned(16))) union { float sums[32][64]; u32x4_t p[4 * TW][2][64]; } x;
  __shared__ float row_max[4][32], row_sum[32];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  int head, blk;
  row_of_block((S + 31) / 32, B * nh, head, blk);
  const int b = head / nh, h = head % nh, H = nh * D, ld = 3 * H;
  const bf16_t* base = codes + (size_t)b * S * ld + h * D;
  const int len = seqlens ? min(seqlens[b], S) : S;
  const int rows = FAST ? S : len;  // rows of V that are staged: those beyond are zero rows
  const FwdScales sc = load_fwd_scales(aq, D);
  const int nt = max(len + 31, 0) / 32, tw = (nt + 3) / 4;  // tiles of the row, of a wavefront
  const int t0 = wave * tw, n = max(min(nt - t0, tw), 0);
  const int q = blk * 32 + (lane & 31), qc = min(q, S - 1);

  u32x4_t vreg[CH];
  auto load_v = [&](int j0) {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = threadIdx.x + 256 * i, row = j0 + c / (D / 8);
      vreg[i] = u32x4_t{0u, 0u, 0u, 0u};
      if (row < rows) vreg[i] = *reinterpret_cast<const u32x4_t*>(base + 2 * H + (size_t)row * ld + c % (D / 8) * 8);
    }
  };
  auto store_v = [&]() {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = threadIdx.x + 256 * i;
      *reinterpret_cast<u32x4_t*>(Vs + c / (D / 8) * Tile<D>::kStride + c % (D / 8) * 8) = vreg[i];
    }
  };
  bf16x8_t qf[D / 16], kf[TW][D / 16];
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) qf[kk] = ld_frag(base + (size_t)qc * ld + (kk * 2 + half) * 8);
#pragma unroll
  for (int t = 0; t < TW; ++t)
    if (t < n) {
      const bf16_t* p = base + H + (size_t)min(32 * (t0 + t) + (lane & 31), S - 1) * ld + half * 8;
#pragma unroll
      for (int kk = 0; kk < D / 16; ++kk) kf[t][kk] = ld_frag(p + kk * 16);
    }
  load_v(0);
  f32x16_t e[TW];
  float mx = -INFINITY;
#pragma unroll
  for (int t = 0; t < TW; ++t)
    if (t < n) {
      e[t] = zero16();
#pragma unroll
      for (int kk = 0; kk < D / 16; ++kk) e[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t][kk], qf[kk], e[t], 0, 0, 0);
      scale_scores(e[t], sc, 32 * (t0 + t), half, len);
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, e[t][r]);
    }
  mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
  if (half == 0) row_max[wave][lane] = mx;
  store_v();
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 4; ++w) mx = fmaxf(mx, row_max[w][lane & 31]);
  const float top = finite_max(mx);
#pragma unroll
  for (int t = 0; t < TW; ++t)
    if (t < n)
#pragma unroll
      for (int r = 0; r < 16; ++r) e[t][r] = exp_neg<FAST>(sub_apart(e[t][r], top));
  // the row sum in the order of the arithmetic (see exp_neg)
#pragma unroll 1
  for (int w = 0; w < 4; ++w) {
    if (wave == w) {
      if constexpr (FAST) {
        float sum = w ? x.sums[0][lane] : 0.f;
#pragma unroll
        for (int t = 0; t < TW; ++t)
          if (t < n)
#pragma unroll
            for (int r = 0; r < 16; ++r) sum += e[t][r];
        if (w < 3) {
          x.sums[0][lane] = sum;
        } else {
          sum += __shfl_xor(sum, 32, 64);
          if (half == 0) row_sum[lane] = sum;
        }
      } else {
        float y[2];
#pragma unroll
        for (int o = 0; o < 2; ++o) {  // tiles of either parity (keys l and l + 64 are two tiles apart)
          float part[16];
#pragma unroll
          for (int r = 0; r < 16; ++r) part[r] = w ? x.sums[16 * o + r][lane] : 0.f;
#pragma unroll
          for (int t = 0; t < TW; ++t)
            if (t < n && ((t0 + t) & 1) == o)
#pragma unroll
              for (int r = 0; r < 16; ++r) part[r] += e[t][r];
          if (w < 3) {
#pragma unroll
            for (int r = 0; r < 16; ++r) x.sums[16 * o + r][lane] = part[r];
          } else {
            y[o] = sum_of_parts(part);
          }
        }
        if (w == 3 && half == 0) row_sum[lane] = y[0] + y[1];
      }
    }
    __syncthreads();
  }
  const float sum = row_sum[lane & 31], rsum = __fdiv_rn(1.0f, sum);
#pragma unroll
  for (int t = 0; t < TW; ++t)
    if (t < n)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        bf16x8_t f;
#pragma unroll
        for (int i = 0; i < 8; ++i) f[i] = static_cast<bf16_t>(prob_code<PQ>(div_by(e[t][8 * s + i], sum, rsum), sc));
        x.p[t0 + t][s][lane] = __builtin_bit_cast(u32x4_t, f);
      }
  f32x16_t oacc = zero16();
  for (int j0 = 0; j0 < len; j0 += RC) {
    const bool more = j0 + RC < len;
    if (more) load_v(j0 + RC);
    __syncthreads();
    if (wave < D / 32)
#pragma unroll
      for (int t = 0; t < TW; ++t)
        if (j0 + 32 * t < len)
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            const int k0 = 32 * t + 16 * s + 4 * half;
            const bf16x8_t f = __builtin_bit_cast(bf16x8_t, x.p[j0 / 32 + t][s][lane]);
            oacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ld_frag_tr<D>(Vs, 32 * wave, k0, k0 + 8, lane), f, oacc, 0, 0, 0);
          }
    if (more) {
      __syncthreads();
      store_v();
    }
  }
  if (wave >= D / 32) return;
  const size_t stat_idx = (size_t)head * S + q;
  MinMax pmax, range;
  if (q < S) {
    if (wave == 0 && half == 0 && stat_m) { stat_m[stat_idx] = mx; stat_l[stat_idx] = sum; }
    pmax.add(1.0f / sum);  // the largest exponential of a row is exp(0) = 1
    store_context<FAST>(oacc, aq, sc, len, ((size_t)b * S + q) * H + h * D + 32 * wave + 4 * half, ctx, ctx_codes, ctx_codes8, range);
  }
  if (ranges) store_ranges(ranges, (int)blockIdx.x * (D / 32) + wave, (int)gridDim.x * (D / 32), pmax, range, lane);
}

// ------------------------------------------------------------------------------
// backward: P recomputed from the saved row statistics, with the rounding steps of the forward but for one: a score less the
// row's maximum is one fused multiply-add, in every kernel of the pass (the forward rounds the score first, so a probability
// may differ from the forward's by the rounding of its score).  dP^ = dC * V^T, the straight-through rule of the probability
// quantizer and the softmax backward dA = P * (dP - rowdot), rowdot = sum_j dP[q][j] * P[q][j].  Up to 128 keys the
// query-major kernel leaves P^T and dA^T (bf16) for the key-major one, which is then a pure product (512 heads of 128
// tokens, inside a step: 17 us against 40 us for forming them again); beyond that the 4 bytes per query-key pair each way
// cost more than the arithmetic, and the key-major kernel forms them itself (256 heads of 384 tokens, both kernels: 164 us
// against 215 us).
// Tiles without masked keys skip the mask's tests (256 heads of 384 tokens, query-major: 89 -> 73 us inside a step), and the
// tiles of P^T and dA^T are transposed in LDS on their way out, 16 bytes a lane instead of 2 (512 heads of 128: 37 -> 34 us).
// ------------------------------------------------------------------------------

// one probability (x: its score less the row's maximum) and its gradient through the quantizer
struct ProbGrad { float p, code, dp; };
template <bool FAST, bool PQ>
__device__ __forceinline__ ProbGrad prob_grad(float x, float dacc, bool valid, float l, float rl, const FwdScales& sc, float& dsp) {
  ProbGrad g;
  g.p = valid ? div_by(exp_neg<FAST>(x), l, rl) : 0.f;
  const float dph = dacc * sc.sv;
  g.code = g.p;
  g.dp = dph;
  if constexpr (PQ) {
    const float v = div_by(g.p, sc.sp, sc.rsp);
    const bool in = v <= sc.p_qp;
    g.code = rintf(fminf(v, sc.p_qp));
    dsp += dph * (g.code - (in ? v : 0.f));
    g.dp = in ? dph : 0.f;
  }
  return g;
}

// query-major part: rowdot (ONE: P^T and dA^T; kept for the key-major kernel), the step-size gradient of the probability quantizer, dQ^ = dA * K^
template <int D, bool ONE, bool PQ>
__global__ __launch_bounds__(256, 2) void attn_bwd_q_mfma_k(const bf16_t* __restrict__ codes, const bf16_t* __restrict__ dctx,
                                                         bf16_t* __restrict__ d_qkvh, AttnQ aq, const int32_t* __restrict__ seqlens, int S,
                                                         int H, const float* __restrict__ stat_m, const float* __restrict__ stat_l,
                                                         float* __restrict__ rowdot_out, bf16_t* __restrict__ pt_out,
                                                         bf16_t* __restrict__ dat_out, float* __restrict__ ds_parts) {
  __shared__ __attribute__((aligned(16))) bf16_t Ks[kChunk * Tile<D>::kStride];
  __shared__ __attribute__((aligned(16))) bf16_t Vs[kChunk * Tile<D>::kStride];
  __shared__ __attribute__((aligned(16))) bf16_t Ts[ONE ? 4 : 1][2][ONE ? 32 * Tile<32>::kStride : 8];  // ONE: a tile of P and dA per wavefront
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5, waves = blockDim.x >> 6;
  const int h = blockIdx.y, b = blockIdx.z, nh = gridDim.y;
  const int ld = 3 * H;
  const bf16_t* base = codes + (size_t)b * S * ld + h * D;
  const int len = seqlens ? min(seqlens[b], S) : S;
  const FwdScales sc = load_fwd_scales(aq, D);
  const float sk = aq.k.on ? *aq.k.s : 1.f;

  const int q0 = blockIdx.x * 128 + wave * 32;
  const int part_idx = (((b * nh + h) * gridDim.x) + blockIdx.x) * waves + wave;
  const bool active = q0 < S;
  const int q = q0 + (lane & 31);
  const bool qvalid = q < S;
  const int qc = qvalid ? q : S - 1;
  bf16x8_t qf[D / 16], cf[D / 16];
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) {
    qf[kk] = ld_frag(base + (size_t)qc * ld + (kk * 2 + half) * 8);
    cf[kk] = ld_frag(dctx + ((size_t)b * S + qc) * H + h * D + (kk * 2 + half) * 8);
  }
  const size_t stat_idx = ((size_t)b * nh + h) * S + qc;
  const float mx = stat_m[stat_idx], l = stat_l[stat_idx];  // row maximum and row sum of the forward
  const float rl = __fdiv_rn(1.0f, l);

  float rowdot = 0.f, dsp = 0.f, unused = 0.f;
  f32x16_t dqacc[D / 32];
#pragma unroll
  for (int et = 0; et < D / 32; ++et) dqacc[et] = zero16();
  // P and dP of one tile of 32 keys
  auto probs = [&](int t, int j0, float* p, float* dp, float& ds) {
    f32x16_t sacc = tile_product<D>(Ks, 32 * t, lane, qf);
    const f32x16_t dacc = tile_product<D>(Vs, 32 * t, lane, cf);
    scale_scores(sacc, sc, j0 + 32 * t, half, len, -mx);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const ProbGrad g = prob_grad<true, PQ>(sacc[r], dacc[r], true, l, rl, sc, ds);
      p[r] = g.p;
      dp[r] = g.dp;
    }
  };
  auto consume = [&](int t, const float* p, const float* dp) {
    float da[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) da[r] = p[r] * (dp[r] - rowdot);
    accumulate_rows<D>(dqacc, Ks, 32 * t, lane, da);
  };
  if constexpr (ONE) {
    const int nt = (len + 31) / 32;
    Rows<D> kr, vr;
    kr.load(base + H, ld, S);
    vr.load(base + 2 * H, ld, S);
    kr.store(Ks, S, 32 * nt);
    vr.store(Vs, S, 32 * nt);
    __syncthreads();
    if (!active) {
      if (lane == 0) ds_parts[part_idx] = 0.f;
      return;
    }
    float p[kChunk / 32][16], dp[kChunk / 32][16];
#pragma unroll
    for (int t = 0; t < kChunk / 32; ++t)
      if (t < nt) {
        probs(t, 0, p[t], dp[t], dsp);
#pragma unroll
        for (int r = 0; r < 16; ++r) rowdot += dp[t][r] * p[t][r];
      }
    rowdot += __shfl_xor(rowdot, 32, 64);
    const int s_pad = (S + 31) / 32 * 32;
    const size_t tbase = ((size_t)b * nh + h) * s_pad * s_pad;
#pragma unroll
    for (int t = 0; t < kChunk / 32; ++t)
      if (t < nt) {
        float da[16], code[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          da[r] = qvalid ? p[t][r] * (dp[t][r] - rowdot) : 0.f;
          const float c = PQ ? rintf(fminf(div_by(p[t][r], sc.sp, sc.rsp), sc.p_qp)) : p[t][r];
          code[r] = qvalid ? c : 0.f;
        }
        accumulate_rows<D>(dqacc, Ks, 32 * t, lane, da);
        // transposed on the way: a lane holds a query, a row in memory is a key
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int o = (lane & 31) * Tile<32>::kStride + 8 * g + 4 * half;
          store4(Ts[wave][0] + o, code[4 * g], code[4 * g + 1], code[4 * g + 2], code[4 * g + 3]);
          store4(Ts[wave][1] + o, da[4 * g], da[4 * g + 1], da[4 * g + 2], da[4 * g + 3]);
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const int k0 = 16 * s + 8 * half;
          const size_t o = tbase + (size_t)(32 * t + (lane & 31)) * s_pad + q0 + k0;
          *reinterpret_cast<bf16x8_t*>(pt_out + o) = ld_frag_tr<32>(Ts[wave][0], 0, k0, k0 + 4, lane);
          *reinterpret_cast<bf16x8_t*>(dat_out + o) = ld_frag_tr<32>(Ts[wave][1], 0, k0, k0 + 4, lane);
        }
      }
  } else {
    Rows<D> kr, vr;  // the next chunk, on its way while this one is multiplied
    auto fetch = [&](int j0) {
      kr.load(base + (size_t)j0 * ld + H, ld, S - j0);
      vr.load(base + (size_t)j0 * ld + 2 * H, ld, S - j0);
    };
    fetch(0);
    for (int pass = 0; pass < 2; ++pass) {
      for (int j0 = 0; j0 < len; j0 += kChunk) {
        const int nt = (min(len - j0, kChunk) + 31) / 32;
        __syncthreads();
        kr.store(Ks, S - j0, 32 * nt);
        vr.store(Vs, S - j0, 32 * nt);
        __syncthreads();
        if (j0 + kChunk < len || pass == 0) fetch(j0 + kChunk < len ? j0 + kChunk : 0);
        if (!active) continue;
        float p[16], dp[16];
        if (pass == 0) {
#pragma unroll 1
          for (int t = 0; t < nt; ++t) {
            probs(t, j0, p, dp, dsp);
#pragma unroll
            for (int r = 0; r < 16; ++r) rowdot += dp[r] * p[r];
          }
        } else {
#pragma unroll 1
          for (int t = 0; t < nt; ++t) {
            probs(t, j0, p, dp, unused);
            consume(t, p, dp);
          }
        }
      }
      if (pass == 0) rowdot += __shfl_xor(rowdot, 32, 64);
    }
    if (!active) {
      if (lane == 0) ds_parts[part_idx] = 0.f;
      return;
    }
  }
  // step-size gradient terms of the probability quantizer (padded query rows excluded)
  dsp = wave_sum(qvalid ? dsp : 0.f);
  if (lane == 0) ds_parts[part_idx] = dsp;
  if (qvalid) {
    if (!ONE && half == 0) rowdot_out[stat_idx] = rowdot;
    const float f = sk / sqrtf((float)D);
    const size_t orow = ((size_t)b * S + q) * ld + h * D;
#pragma unroll
    for (int et = 0; et < D / 32; ++et)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        store4(d_qkvh + orow + 32 * et + 8 * g + 4 * half, dqacc[et][4 * g] * f, dqacc[et][4 * g + 1] * f, dqacc[et][4 * g + 2] * f,
               dqacc[et][4 * g + 3] * f);
  }
}

// The query-major part of the other arithmetic (not FAST): 32 queries a block, the keys shared out among its wavefronts as in
// attn_fwd_row_k, so that probabilities and their gradients are formed once and stay in registers until the row's sum over
// them is known, instead of being formed again.  Every sum over keys is one chain with the keys ascending, as in a wavefront
// that holds the whole row: rowdot, the step gradient's sum and the accumulators of dQ^ go from wavefront to wavefront
// through LDS.  Inside a step, 8 x 512 tokens, 12 heads: 101 -> 72 us against 128 queries a block and two passes over the keys
// (60 us with parts summed apart and the row maximum subtracted on its own, which moved a step's results by up to 0.5%).
template <int D, bool PQ>
__global__ __launch_bounds__(256, 2) void attn_bwd_q_row_k(const bf16_t* __restrict__ codes, const bf16_t* __restrict__ dctx,
                                                           bf16_t* __restrict__ d_qkvh, AttnQ aq, const int32_t* __restrict__ seqlens, int S, int B,
                                                           int nh, const float* __restrict__ stat_m, const float* __restrict__ stat_l,
                                                           float* __restrict__ rowdot_out, float* __restrict__ ds_parts) {
  constexpr int TW = 4;  // tiles of a wavefront (up to 512 keys)
  // per wavefront: what a unit of dP^ adds to the step gradient, then 32 columns of a tile of K
  __shared__ __attribute__((aligned(16))) union { float4 term[TW][4][64]; bf16_t k[32 * Tile<32>::kStride]; } x[4];
  __shared__ float dq_sums[D / 32][16][64], dots[64], dsps[64];  // from wavefront to wavefront
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5, waves = blockDim.x >> 6;
  const int nq = (S + 127) / 128 * waves;  // one partial sum for each 32 queries of whole groups of 128
  int head, blk;
  row_of_block(nq, B * nh, head, blk);
  if (32 * blk >= S) {
    if (threadIdx.x == 0) ds_parts[(size_t)head * nq + blk] = 0.f;
    return;
  }
  const int b = head / nh, h = head % nh, H = nh * D, ld = 3 * H;
  const bf16_t* base = codes + (size_t)b * S * ld + h * D;
  const int len = seqlens ? min(seqlens[b], S) : S;
  const FwdScales sc = load_fwd_scales(aq, D);
  const float sk = aq.k.on ? *aq.k.s : 1.f;
  const int nt = max(len + 31, 0) / 32, tw = (nt + waves - 1) / waves;  // tiles of the row, of a wavefront
  const int t0 = wave * tw, n = max(min(nt - t0, tw), 0);
  const int q = blk * 32 + (lane & 31), qc = min(q, S - 1);
  const bool qvalid = q < S;
  // a lane's part of rows 32 (t0 + t) .. + 31 of K or V as an operand; rows beyond the sequence repeat its last one (their
  // probabilities are 0)
  auto row_at = [&](int column, int t) { return base + column + (size_t)min(32 * (t0 + t) + (lane & 31), S - 1) * ld + half * 8; };
  auto load_rows = [&](bf16x8_t (&f)[D / 16], int column, int t) {
    const bf16_t* p = row_at(column, t);
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) f[kk] = ld_frag(p + kk * 16);
  };
  bf16x8_t qf[D / 16], cf[D / 16], kf[D / 16], vf[D / 16];
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) {
    qf[kk] = ld_frag(base + (size_t)qc * ld + (kk * 2 + half) * 8);
    cf[kk] = ld_frag(dctx + ((size_t)b * S + qc) * H + h * D + (kk * 2 + half) * 8);
  }
  if (n > 0) {
    load_rows(kf, H, 0);
    load_rows(vf, 2 * H, 0);
  }
  const size_t stat_idx = (size_t)head * S + qc;
  const float mx = stat_m[stat_idx], l = stat_l[stat_idx];  // row maximum and row sum of the forward
  const float rl = __fdiv_rn(1.0f, l);

  // the probability, negative where the quantizer clips it, and the gradient of its code
  float p[TW][16], dph[TW][16];
#pragma unroll
  for (int t = 0; t < TW; ++t)
    if (t < n) {
      f32x16_t sacc = zero16(), dacc = zero16();
#pragma unroll
      for (int kk = 0; kk < D / 16; ++kk) {
        sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk], qf[kk], sacc, 0, 0, 0);
        dacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[kk], cf[kk], dacc, 0, 0, 0);
      }
      if (t + 1 < TW && t + 1 < n) {
        load_rows(kf, H, t + 1);
        load_rows(vf, 2 * H, t + 1);
      }
      scale_scores(sacc, sc, 32 * (t0 + t), half, len, -mx);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float term[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float pr = div_by(exp_neg<false>(sacc[4 * g + i]), l, rl);
          const float v = div_by(pr, sc.sp, sc.rsp);
          const bool in = v <= sc.p_qp;
          term[i] = rintf(fminf(v, sc.p_qp)) - (in ? v : 0.f);
          p[t][4 * g + i] = in || !PQ ? pr : -pr;
          dph[t][4 * g + i] = dacc[4 * g + i] * sc.sv;
        }
        x[wave].term[t][g][lane] = make_float4(term[0], term[1], term[2], term[3]);
      }
    }
  auto dp_of = [&](int t, int r) { return signbit(p[t][r]) ? 0.f : dph[t][r]; };
#pragma unroll 1
  for (int w = 0; w < waves; ++w) {
    if (wave == w) {
      float rowdot = w ? dots[lane] : 0.f, dsp = w ? dsps[lane] : 0.f;
#pragma unroll
      for (int t = 0; t < TW; ++t)
        if (t < n)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const float4 term = x[wave].term[t][g][lane];
            const float e[4] = {term.x, term.y, term.z, term.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              rowdot = __fmaf_rn(dp_of(t, 4 * g + i), fabsf(p[t][4 * g + i]), rowdot);
              if constexpr (PQ) dsp = __fmaf_rn(dph[t][4 * g + i], e[i], dsp);
            }
          }
      if (w == waves - 1) {
        rowdot += __shfl_xor(rowdot, 32, 64);
        dsp = wave_sum(qvalid ? dsp : 0.f);  // step-size gradient terms of the probability quantizer (padded query rows excluded)
        if (lane == 0) ds_parts[(size_t)head * nq + blk] = dsp;
        if (half == 0 && qvalid) rowdot_out[stat_idx] = rowdot;
      }
      dots[lane] = rowdot;
      dsps[lane] = dsp;
    }
    __syncthreads();
  }
  const float rowdot = dots[lane];

  // the gradient of a score in three bf16 parts that add up to it (see accumulate_rows_wide)
  bf16x8_t da[TW][3][2];
#pragma unroll
  for (int t = 0; t < TW; ++t)
    if (t < n)
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          float rest = fabsf(p[t][8 * s + i]) * (dp_of(t, 8 * s + i) - rowdot);
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            da[t][k][s][i] = static_cast<bf16_t>(rest);
            rest = __fsub_rn(rest, static_cast<float>(da[t][k][s][i]));
          }
        }
  // 32 columns at a time: while a wavefront adds to the second ones, the next adds to the first
  auto load_columns = [&](bf16x8_t (&f)[2], int et, int t) {
    const bf16_t* r = row_at(H + 32 * et, t);
    f[0] = ld_frag(r);
    f[1] = ld_frag(r + 16);
  };
  bf16x8_t kc[2];
  if (n > 0) load_columns(kc, 0, 0);
#pragma unroll 1
  for (int s = 0; s < waves + D / 32 - 1; ++s) {
    const int et = s - wave;
    if (et >= 0 && et < D / 32 && (n > 0 || wave == 0)) {
      f32x16_t acc = zero16();
      if (wave)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = dq_sums[et][r][lane];
#pragma unroll
      for (int t = 0; t < TW; ++t)
        if (t < n) {
#pragma unroll
          for (int c = 0; c < 2; ++c)
            *reinterpret_cast<bf16x8_t*>(&x[wave].k[(lane & 31) * Tile<32>::kStride + (c * 2 + half) * 8]) = kc[c];
          if (t + 1 < TW && t + 1 < n) load_columns(kc, et, t + 1);
          else if (et + 1 < D / 32) load_columns(kc, et + 1, 0);
#pragma unroll
          for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              const int k0 = 16 * j + 4 * half;
              acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ld_frag_tr<32>(x[wave].k, 0, k0, k0 + 8, lane), da[t][k][j], acc, 0, 0, 0);
            }
        }
#pragma unroll
      for (int r = 0; r < 16; ++r) dq_sums[et][r][lane] = acc[r];
    }
    __syncthreads();
  }
  if (!qvalid) return;
  const float f = sk / sqrtf((float)D);
  const size_t orow = ((size_t)b * S + q) * ld + h * D;
  for (int i = wave; i < D / 8; i += waves) {  // 8 columns, 4 of them here
    const float(&v)[16][64] = dq_sums[i / 4];
    const int r = 4 * (i % 4);
    store4(d_qkvh + orow + 8 * i + 4 * half, v[r][lane] * f, v[r + 1][lane] * f, v[r + 2][lane] * f, v[r + 3][lane] * f);
  }
}

// key-major part for at most 128 tokens: dV^ = P^T dC, dK^ = dA^T Q^ / sqrt(d) from the tiles the query-major kernel left.
// One wavefront = 32 keys.
template <int D>
__global__ __launch_bounds__(256, 2) void attn_bwd_k_one_mfma_k(const bf16_t* __restrict__ codes, const bf16_t* __restrict__ dctx,
                                                             bf16_t* __restrict__ d_qkvh, AttnQ aq, const int32_t* __restrict__ seqlens, int S,
                                                             int H, const bf16_t* __restrict__ pt_in, const bf16_t* __restrict__ dat_in) {
  __shared__ __attribute__((aligned(16))) bf16_t Qs[kChunk * Tile<D>::kStride];
  __shared__ __attribute__((aligned(16))) bf16_t Cs[kChunk * Tile<D>::kStride];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5;
  const int h = blockIdx.y, b = blockIdx.z, nh = gridDim.y;
  const int ld = 3 * H, s_pad = (S + 31) / 32 * 32;
  const bf16_t* base = codes + (size_t)b * S * ld + h * D;
  const int len = seqlens ? min(seqlens[b], S) : S;
  Rows<D> qr, cr;
  qr.load(base, ld, S);
  cr.load(dctx + (size_t)b * S * H + h * D, H, S);
  qr.store(Qs, S, s_pad);
  cr.store(Cs, S, s_pad);
  __syncthreads();
  f32x16_t vacc[D / 32], kacc[D / 32];
#pragma unroll
  for (int et = 0; et < D / 32; ++et) vacc[et] = kacc[et] = zero16();
  if (32 * wave < len) {  // keys beyond the valid ones have P = 0, and no tile
    const size_t row = (((size_t)b * nh + h) * s_pad + 32 * wave + (lane & 31)) * s_pad + 8 * half;
    for (int s = 0; s < s_pad / 16; ++s) {
      const bf16x8_t pf = ld_frag(pt_in + row + 16 * s), af = ld_frag(dat_in + row + 16 * s);
      const int q0 = 16 * s + 8 * half;  // queries of this lane's k-slots, in natural order
#pragma unroll
      for (int et = 0; et < D / 32; ++et) {
        vacc[et] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pf, ld_frag_tr<D>(Cs, 32 * et, q0, q0 + 4, lane), vacc[et], 0, 0, 0);
        kacc[et] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, ld_frag_tr<D>(Qs, 32 * et, q0, q0 + 4, lane), kacc[et], 0, 0, 0);
      }
    }
  }
  const float sp = aq.p.on ? *aq.p.s : 1.f;
  const float fq = (aq.q.on ? *aq.q.s : 1.f) / sqrtf((float)D);
#pragma unroll
  for (int et = 0; et < D / 32; ++et)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int j = key_of(wave, r, half);
      if (j < S) {
        const size_t o = ((size_t)b * S + j) * ld + h * D + 32 * et + (lane & 31);
        d_qkvh[o + H] = static_cast<bf16_t>(kacc[et][r] * fq);
        d_qkvh[o + 2 * H] = static_cast<bf16_t>(vacc[et][r] * sp);
      }
    }
}

// key-major part: dV^[j] = sum_q P^[q][j] dC[q], dK^[j] = sum_q dA[q][j] Q^[q] / sqrt(d).  One wavefront = 32 keys (a lane
// owns one key, the accumulator registers enumerate queries); queries pass through LDS in chunks of 128 with their statistics.
template <int D, bool FAST, bool PQ>
__global__ __launch_bounds__(256, 2) void attn_bwd_k_mfma_k(const bf16_t* __restrict__ codes, const bf16_t* __restrict__ dctx,
                                                         bf16_t* __restrict__ d_qkvh, AttnQ aq, const int32_t* __restrict__ seqlens, int S,
                                                         int H, const float* __restrict__ stat_m, const float* __restrict__ stat_l,
                                                         const float* __restrict__ rowdot_in) {
  __shared__ __attribute__((aligned(16))) bf16_t Qs[kChunk * Tile<D>::kStride];
  __shared__ __attribute__((aligned(16))) bf16_t Cs[kChunk * Tile<D>::kStride];
  __shared__ __attribute__((aligned(16))) float stats[4][kChunk];  // row maximum, row sum, its reciprocal, rowdot
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5;
  const int h = blockIdx.y, b = blockIdx.z, nh = gridDim.y;
  const int ld = 3 * H;
  const bf16_t* base = codes + (size_t)b * S * ld + h * D;
  const bf16_t* cbase = dctx + (size_t)b * S * H + h * D;
  const size_t sbase = ((size_t)b * nh + h) * S;
  const int len = seqlens ? min(seqlens[b], S) : S;
  const FwdScales sc = load_fwd_scales(aq, D);
  const int j0 = blockIdx.x * 128 + wave * 32;
  const int j = j0 + (lane & 31);
  const int jc = j < S ? j : S - 1;
  const bool active = j0 < len;  // keys beyond the valid ones have P = 0
  bf16x8_t kf[D / 16], vf[D / 16];
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) {
    kf[kk] = ld_frag(base + (size_t)jc * ld + H + (kk * 2 + half) * 8);
    vf[kk] = ld_frag(base + (size_t)jc * ld + 2 * H + (kk * 2 + half) * 8);
  }
  f32x16_t vacc[D / 32], kacc[D / 32];
#pragma unroll
  for (int et = 0; et < D / 32; ++et) vacc[et] = kacc[et] = zero16();
  float unused = 0.f;

  // a chunk of queries and their statistics, on their way while the one before is multiplied; a thread's row of the chunk:
  Rows<D> qr, cr;
  const int si = threadIdx.x;
  float st_m = 0.f, st_l = 1.f, st_d = 0.f;
  auto fetch = [&](int c0) {
    qr.load(base + (size_t)c0 * ld, ld, S - c0);
    cr.load(cbase + (size_t)c0 * H, H, S - c0);
    // rows beyond the sequence: their Q and dC are zero, so any finite statistics will do
    const bool v = si < kChunk && c0 + si < S;
    st_m = v ? stat_m[sbase + c0 + si] : 0.f;
    st_l = v ? stat_l[sbase + c0 + si] : 1.f;
    st_d = v ? rowdot_in[sbase + c0 + si] : 0.f;
  };
  if ((int)blockIdx.x * 128 < len) {
    fetch(0);
    for (int c0 = 0; c0 < S; c0 += kChunk) {
      const int cn = (min(S - c0, kChunk) + 31) / 32;  // 32-query tiles
      __syncthreads();
      qr.store(Qs, S - c0, 32 * cn);
      cr.store(Cs, S - c0, 32 * cn);
      if (si < 32 * cn) {
        stats[0][si] = st_m;
        stats[1][si] = st_l;
        stats[2][si] = __fdiv_rn(1.0f, st_l);
        stats[3][si] = st_d;
      }
      __syncthreads();
      if (c0 + kChunk < S) fetch(c0 + kChunk);
      if (!active) continue;
#pragma unroll 1
      for (int t = 0; t < cn; ++t) {
        const f32x16_t sacc = tile_product<D>(Qs, 32 * t, lane, kf), dacc = tile_product<D>(Cs, 32 * t, lane, vf);
        float code[16], da[16];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int qi = 32 * t + 8 * g + 4 * half;  // registers 4 g .. 4 g + 3 hold queries qi .. qi + 3
          float st[4][4];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float4 x = *reinterpret_cast<const float4*>(&stats[k][qi]);
            st[k][0] = x.x; st[k][1] = x.y; st[k][2] = x.z; st[k][3] = x.w;
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const ProbGrad pg = prob_grad<FAST, PQ>(__fmaf_rn(sacc[4 * g + i], sc.qk, -st[0][i]), dacc[4 * g + i], j < len, st[1][i], st[2][i], sc, unused);
            code[4 * g + i] = pg.code;
            da[4 * g + i] = pg.p * (pg.dp - st[3][i]);
          }
        }
        if constexpr (FAST) {
          accumulate_rows_natural<D>(vacc, Cs, 32 * t, lane, code);
          accumulate_rows_natural<D>(kacc, Qs, 32 * t, lane, da);
        } else {
          accumulate_rows<D>(vacc, Cs, 32 * t, lane, code);
          accumulate_rows_wide<D>(kacc, Qs, 32 * t, lane, da);
        }
      }
    }
  }
  if (j >= S) return;
  const float sp = sc.sp;
  const float fq = (aq.q.on ? *aq.q.s : 1.f) / sqrtf((float)D);
  const size_t orow = ((size_t)b * S + j) * ld + h * D;
#pragma unroll
  for (int et = 0; et < D / 32; ++et)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const size_t o = orow + 32 * et + 8 * g + 4 * half;
      store4(d_qkvh + o + H, kacc[et][4 * g] * fq, kacc[et][4 * g + 1] * fq, kacc[et][4 * g + 2] * fq, kacc[et][4 * g + 3] * fq);
      store4(d_qkvh + o + 2 * H, vacc[et][4 * g] * sp, vacc[et][4 * g + 1] * sp, vacc[et][4 * g + 2] * sp, vacc[et][4 * g + 3] * sp);
    }
}

// ------------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------------
bool attn_mfma_ok(int dt, int d) { return dt == DT_BF16 && (d == 32 || d == 64); }

static int block_waves(int S) { return S >= 128 ? 4 : (S + 31) / 32; }

static bool fast(int S, int d) { return d == 64 && S >= 64 && S <= 384; }

// partial ranges that the forward leaves (at most: rows of more than 128 keys may have fewer)
int attn_fwd_mfma_parts(int B, int S, int nh, int d) { return max((S + 127) / 128 * block_waves(S), (S + 31) / 32 * (d / 32)) * nh * B; }

int attn_fwd_mfma(const void* codes, void* ctx, void* ctx_codes, const AttnQ& aq, const int32_t* seqlens, int B, int S, int nh, int d,
                  float* ranges, float* stat_m, float* stat_l, hipStream_t st, bool chain, int8_t* ctx_codes8) {
  auto launch = [&](auto dim, auto one, auto is_fast, auto real, auto pq) {
    constexpr int D = decltype(dim)::value;
    hipLaunchKernelGGL((attn_fwd_mfma_k<D, decltype(one)::value, decltype(is_fast)::value, decltype(real)::value, decltype(pq)::value>),
                       dim3((S + 127) / 128, nh, B), dim3(64 * block_waves(S)), 0, st, (const bf16_t*)codes, (bf16_t*)ctx, (bf16_t*)ctx_codes, aq, seqlens,
                       S, nh * D, ranges, stat_m, stat_l, ctx_codes8);
    return (S + 127) / 128 * nh * B * block_waves(S);
  };
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  constexpr std::integral_constant<int, 32> d32{};
  constexpr std::integral_constant<int, 64> d64{};
  auto launch_row = [&](auto dim, auto is_fast, auto pq) {
    constexpr int D = decltype(dim)::value;
    hipLaunchKernelGGL((attn_fwd_row_k<D, decltype(is_fast)::value, decltype(pq)::value>), dim3((S + 31) / 32 * nh * B), dim3(256), 0, st,
                       (const bf16_t*)codes, (bf16_t*)ctx, (bf16_t*)ctx_codes, aq, seqlens, S, B, nh, ranges, stat_m, stat_l, ctx_codes8);
    return (S + 31) / 32 * nh * B * (D / 32);
  };
  const bool one = S <= kChunk, real = !aq.p.on && chain;
  auto with = [&](auto pq) -> int {
    if (fast(S, d)) return one ? launch(d64, yes, yes, no, pq) : launch_row(d64, yes, pq);
    if (d == 64) return one ? launch(d64, yes, no, no, pq) : launch_row(d64, no, pq);
    return one ? launch(d32, yes, no, no, pq) : launch_row(d32, no, pq);
  };
  if (aq.p.on) return with(yes);
  if (!real || fast(S, d)) return with(no);
  if (d == 64) return one ? launch(d64, yes, no, yes, no) : launch(d64, no, no, yes, no);
  return one ? launch(d32, yes, no, yes, no) : launch(d32, no, no, yes, no);
}

// returns the number of partial sums written to ds_parts
int attn_bwd_mfma(const void* codes, const void* dctx, void* d_qkvh, const AttnQ& aq, const int32_t* seqlens, int B, int S, int nh, int d,
                  const float* stat_m, const float* stat_l, void* scratch0, void* scratch1, float* ds_parts, hipStream_t st) {
  const int waves = block_waves(S);
  const dim3 g((S + 127) / 128, nh, B), blk(64 * waves);
  const bf16_t *c = (const bf16_t*)codes, *dc = (const bf16_t*)dctx;
  bf16_t* out = (bf16_t*)d_qkvh;
  const int H = nh * d, parts = (int)(g.x * g.y * g.z) * waves;
  auto launch = [&](auto dim, auto is_fast, auto pq) {
    constexpr int D = decltype(dim)::value;
    constexpr bool FAST = decltype(is_fast)::value, PQ = decltype(pq)::value;
    if constexpr (FAST) {
      hipLaunchKernelGGL((attn_bwd_q_mfma_k<D, false, PQ>), g, blk, 0, st, c, dc, out, aq, seqlens, S, H, stat_m, stat_l, (float*)scratch0,
                         (bf16_t*)nullptr, (bf16_t*)nullptr, ds_parts);
    } else {
      hipLaunchKernelGGL((attn_bwd_q_row_k<D, PQ>), dim3(parts), dim3(64 * waves), 0, st, c, dc, out, aq, seqlens, S, B, nh, stat_m, stat_l,
                         (float*)scratch0, ds_parts);
    }
    hipLaunchKernelGGL((attn_bwd_k_mfma_k<D, FAST, PQ>), g, blk, 0, st, c, dc, out, aq, seqlens, S, H, stat_m, stat_l, (const float*)scratch0);
  };
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  constexpr std::integral_constant<int, 32> d32{};
  constexpr std::integral_constant<int, 64> d64{};
  auto with = [&](auto pq) {
    if (!fast(S, d)) return d == 64 ? launch(d64, no, pq) : launch(d32, no, pq);
    if (S > kChunk) return launch(d64, yes, pq);
    hipLaunchKernelGGL((attn_bwd_q_mfma_k<64, true, decltype(pq)::value>), g, blk, 0, st, c, dc, out, aq, seqlens, S, H, stat_m, stat_l, (float*)nullptr,
                       (bf16_t*)scratch0, (bf16_t*)scratch1, ds_parts);
    hipLaunchKernelGGL((attn_bwd_k_one_mfma_k<64>), g, blk, 0, st, c, dc, out, aq, seqlens, S, H, (const bf16_t*)scratch0, (const bf16_t*)scratch1);
  };
  aq.p.on ? with(yes) : with(no);
  return parts;
}

}  // namespace mrem
