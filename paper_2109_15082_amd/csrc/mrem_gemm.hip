// C[M,N] = A[M,K] * B[N,K]^T with a fused epilogue: the products of the four linear
// layers of an encoder layer in the quantized module (integer codes as operands,
// step sizes applied to the accumulator -- Section 3.1, Eq. 1), of the
// full-precision module, and of the backward pass (input and weight gradients).
#include "mrem_common.h"
#include "mrem_kernels.h"

#include <hip/hip_ext.h>

#include <algorithm>
#include <atomic>
#include <string>
#include <cstdlib>
#include <type_traits>

#include <vector>

// Compiled as a whole, or in five parts: 1 to 4 hold the tiles of one operand form each, 0 the rest.
#if !defined(MREM_GEMM_PART)
#define MREM_GEMM_REST 1
#elif MREM_GEMM_PART == 0
#define MREM_GEMM_REST 1
#else
#define MREM_GEMM_REST 0
#endif

namespace mrem {

// ---- optional timing of every product launch with HIP events (measurement aid) ----
// The records live in a GemmProfile that the caller (a context) owns.  Return codes of event calls are
// not looked at here: the runtime keeps the last error, and every entry point of the library ends by
// reading it (hipGetLastError).
#if MREM_GEMM_REST
thread_local LaunchEvents tl_launch_events;

void gemm_profile_begin(GemmProfile* p) {
  for (auto& r : p->recs) { (void)hipEventDestroy(r.e0); (void)hipEventDestroy(r.e1); }
  p->recs.clear();
  p->stats.clear();
  p->on = true;
}
int gemm_profile_end(GemmProfile* p, double ms[2], double flops[2], int64_t launches[2]) {
  p->on = false;
  ms[0] = ms[1] = flops[0] = flops[1] = 0.0;
  launches[0] = launches[1] = 0;
  int rc = 0;
  for (auto& r : p->recs) {
    float e = 0.f;
    if (hipEventSynchronize(r.e1) != hipSuccess || hipEventElapsedTime(&e, r.e0, r.e1) != hipSuccess) rc = -1;
    if (r.cls < 2) {
      ms[r.cls] += e;
      flops[r.cls] += r.flops;
      launches[r.cls] += 1;
    } else {
      KernelStat* ks = nullptr;
      for (auto& k : p->stats)
        if (k.label == r.label || std::string(k.label) == r.label) ks = &k;
      if (!ks) { p->stats.push_back(KernelStat{r.label, 0.0, 0.0, 0}); ks = &p->stats.back(); }
      ks->ms += e;
      ks->bytes += r.flops;
      ks->launches += 1;
    }
    (void)hipEventDestroy(r.e0);
    (void)hipEventDestroy(r.e1);
  }
  p->recs.clear();
  return rc;
}

#endif

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

struct EpiVals {
  float alpha, beta;
};

// the epilogue's value with every operation rounded (see Epilogue::apart): cs = alpha * col_scale[n], t = col_vec[n] +
// row_vec[m]
__device__ __forceinline__ float epilogue_apart(float acc, float cs, bool has_beta, float beta, float t, bool has_bias, float bias) {
#pragma clang fp contract(off)
  float v = acc * cs;
  if (has_beta) v = __builtin_fmaf(beta, t, v);
  if (has_bias) v = v + bias;
  return v;
}
// Epilogue::post: the block's output tile, as it is stored, lies in LDS (rows of post_stride values), and goes out in whole
// 16-byte pieces beside those of post_in.  The accumulators are dead by then: with the other tensors' values and addresses beside
// them the kernel of 256 x 256 tiles spilled 99 registers.
template <int BN>
constexpr int post_stride = BN + 8;
__device__ __forceinline__ QuantParam post_quantizer(const QArg& a) {
  QuantParam q = {*a.s, a.z ? *a.z : 0.f, a.qn, a.qp, 1, 0.f};
  q.rs = quant_reciprocal(q.s);
  return q;
}
// what quantizes column n (POST_QKV: by sections)
template <int POST>
__device__ __forceinline__ QuantParam post_quantizer(const Epilogue& e, int n) {
  if constexpr (POST == POST_QKV) {
    const int section = n / e.post_cols;
    const QuantParam q0 = post_quantizer(e.post_q), q1 = post_quantizer(e.post_q1), q2 = post_quantizer(e.post_q2);
    return section == 0 ? q0 : section == 1 ? q1 : q2;
  } else {
    return post_quantizer(e.post_q);
  }
}
// POST_GELU and POST_QKV straight from a lane's value v (stored as o) at element `at`
template <int POST>
__device__ __forceinline__ void post_code(const Epilogue& e, const QuantParam& q, size_t at, float v) {
  const float o = round_to<bf16_t>(v), c = q_code(q_ratio_fma(POST == POST_GELU ? gelu_t<bf16_t>(o) : o, q), q);
  if (e.post_out) stf(static_cast<bf16_t*>(e.post_out), at, c);
  if constexpr (POST == POST_GELU) {
    if (e.post_out8) e.post_out8[at] = (int8_t)((int)c - e.post_shift);
  }
}

// GELU and its quantizer for stored values: bf16 values between 2^-14 and 8 of either sign are 4352, whose codes a block forms once
// and then looks up (8 vector instructions a value, 29 when each is formed by itself, which are 13 us for 4096 x 4096 values).
struct GeluCodes {
  static constexpr unsigned LOW = 113u << 7, N = 17u * 128u;  // bits of 2^-14; values of one sign
  unsigned char code[2 * N];
  static __device__ __forceinline__ unsigned form(unsigned bits, const QuantParam& q) {
    return (unsigned)q_code(q_ratio_fma(gelu_t<bf16_t>(__uint_as_float(bits << 16)), q), q);
  }
  __device__ __forceinline__ void fill(const QuantParam& q) {
    for (unsigned i = threadIdx.x; i < 2 * N; i += blockDim.x) code[i] = (unsigned char)form((i < N ? LOW : 0x8000u + LOW - N) + i, q);
  }
};
template <int BM, int BN, int THREADS>
__device__ __forceinline__ void gelu_tile(unsigned char* lds, const Epilogue& e, bf16_t* __restrict__ C, int ldc, int m0, int n0) {
  constexpr int ROWS = THREADS / (BN / 8);
  const bf16_t* tile = reinterpret_cast<const bf16_t*>(lds);
  GeluCodes* table = reinterpret_cast<GeluCodes*>(lds + BM * post_stride<BN> * sizeof(bf16_t));
  const QuantParam q = post_quantizer(e.post_q);
  table->fill(q);
  __syncthreads();
  const int row0 = threadIdx.x / (BN / 8), col = threadIdx.x % (BN / 8) * 8;
  const size_t at0 = (size_t)(m0 + row0) * ldc + n0 + col;
  const unsigned shift = 0x01010101u * (unsigned)e.post_shift;
#pragma unroll 4
  for (int p = 0; p < BM; p += ROWS) {
    const u32x4_t o = *reinterpret_cast<const u32x4_t*>(tile + (row0 + p) * post_stride<BN> + col);
    unsigned code[8], low = ~0u, high = 0u;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const unsigned bits = (j & 1) ? o[j >> 1] >> 16 : o[j >> 1] & 0xffffu, i = (bits & 0x7fffu) - GeluCodes::LOW;
      low = min(low, bits & 0x7fffu);
      high = max(high, bits & 0x7fffu);
      code[j] = table->code[min(i, GeluCodes::N - 1) + (bits >> 15) * GeluCodes::N];
    }
    if (low < GeluCodes::LOW || high >= GeluCodes::LOW + GeluCodes::N) {
#pragma unroll 1
      for (int j = 0; j < 8; ++j) {
        const unsigned bits = (unsigned)(o[j >> 1] >> (16 * (j & 1))) & 0xffffu, c = GeluCodes::form(bits, q);
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (k == j) code[k] = c;
      }
    }
    const size_t at = at0 + (size_t)p * ldc;
    if (C) *reinterpret_cast<u32x4_t*>(C + at) = o;
    if (e.post_out) {
      bf16x8_t c;
#pragma unroll
      for (int j = 0; j < 8; ++j) c[j] = static_cast<bf16_t>((float)code[j]);
      *reinterpret_cast<bf16x8_t*>(static_cast<bf16_t*>(e.post_out) + at) = c;
    }
    if (e.post_out8) {
      unsigned w[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        w[h] = code[4 * h] | code[4 * h + 1] << 8 | code[4 * h + 2] << 16 | code[4 * h + 3] << 24;
        // less the shift, byte by byte: bit 7 keeps a borrow inside (and is the shift itself with 8-bit codes)
        w[h] = e.post_shift == 128 ? w[h] ^ 0x80808080u : ((w[h] | 0x80808080u) - shift) ^ 0x80808080u;
      }
      *reinterpret_cast<uint2*>(e.post_out8 + at) = make_uint2(w[0], w[1]);
    }
  }
}
// What the backward pass needs of a stored value u in front of the GELU and its quantizer is a function of its 16 bits too: the
// derivative (outside the quantizer's range OUTSIDE, which gives zero whatever flows back, or NaN where that is no number), and the
// term of the step's gradient.  Values between 2^-11 and 8 are looked up
// (34 vector instructions when formed); 6 values in 10000 of N(0, 0.64) lie outside and are formed one by one.  A pass of its own
// read both tensors again and was bound by those instructions: 26 us for 4096 x 4096 values.  With it and the context's
// (POST_MASK, 8 us) in the products a step of six layers of 1024 over 4096 tokens takes 3975 us instead of 4112, over 16 x 384
// 5588 instead of 5802, three of 768 over 32 x 128 1541 instead of 1603.
struct GeluSlopes {
  static constexpr unsigned LOW = 116u << 7, N = 14u * 128u;  // bits of 2^-11; values of one sign
  static constexpr unsigned OUTSIDE = 0x80000000u;            // bits of -0, which no derivative inside has
  float2 of[2 * N];
  static __device__ __forceinline__ float2 form(unsigned bits, const QuantParam& q) {
    const float u = __uint_as_float(bits << 16), v = q_ratio_fma(gelu_t<bf16_t>(u), q);
    const bool in = q_inside(v, q);
    const float d = gelu_grad_t<bf16_t>(u);
    return make_float2(in ? d + 0.f : -fabsf(0.f * d), q_code(v, q) - (in ? v : 0.f));
  }
  __device__ __forceinline__ void fill(const QuantParam& q) {
    for (unsigned i = threadIdx.x; i < 2 * N; i += blockDim.x) of[i] = form((i < N ? LOW : 0x8000u + LOW - N) + i, q);
  }
};
template <int POST>
constexpr size_t post_table = POST == POST_DGELU ? sizeof(GeluSlopes) : POST == POST_GELU ? sizeof(GeluCodes) : 0;
template <int BM, int BN, int THREADS>
__device__ __forceinline__ void dgelu_tile(unsigned char* lds, const Epilogue& e, bf16_t* __restrict__ C, int ldc, int m0, int n0) {
  constexpr int CHUNKS = BN / 8, ROWS = THREADS / CHUNKS, R = 4;
  static_assert(BM % (ROWS * R) == 0 && ROWS * BN * 4 <= BM * post_stride<BN> * 2, "whole passes, column sums fit the tile");
  const bf16_t* tile = reinterpret_cast<const bf16_t*>(lds);
  GeluSlopes* table = reinterpret_cast<GeluSlopes*>(lds + BM * post_stride<BN> * sizeof(bf16_t));
  const QuantParam q = post_quantizer(e.post_q);
  const int row0 = threadIdx.x / CHUNKS, col = threadIdx.x % CHUNKS * 8;
  const size_t at0 = (size_t)(m0 + row0) * ldc + n0 + col;
  const bf16_t* const u = static_cast<const bf16_t*>(e.post_in) + at0;
  u32x4_t in[R];
  auto fetch = [&](int p) {
#pragma unroll
    for (int i = 0; i < R; ++i) in[i] = *reinterpret_cast<const u32x4_t*>(u + (size_t)(p + i * ROWS) * ldc);
  };
  fetch(0);
  table->fill(q);
  __syncthreads();
  float sum = 0.f, cols[8] = {};
  for (int p = 0; p < BM; p += ROWS * R) {
    if (p) fetch(p);
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const u32x4_t o = *reinterpret_cast<const u32x4_t*>(tile + (row0 + p + i * ROWS) * post_stride<BN> + col);
      float2 t[8];
      unsigned outside = 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const unsigned bits = (j & 1) ? in[i][j >> 1] >> 16 : in[i][j >> 1] & 0xffffu, k = (bits & 0x7fffu) - GeluSlopes::LOW;
        t[j] = table->of[min(k, GeluSlopes::N - 1) + (bits >> 15) * GeluSlopes::N];
        outside |= k < GeluSlopes::N ? 0u : 1u << j;
      }
      while (outside) {
        const int j = __ffs((int)outside) - 1;
        outside &= outside - 1;
        unsigned word = in[i][0];
#pragma unroll
        for (int k = 1; k < 4; ++k) word = j >> 1 == k ? in[i][k] : word;
        const float2 f = GeluSlopes::form((j & 1) ? word >> 16 : word & 0xffffu, q);
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (k == j) t[k] = f;
      }
      bf16x8_t d;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float g = __uint_as_float((j & 1) ? o[j >> 1] & 0xffff0000u : o[j >> 1] << 16);
        sum += g * t[j].y;
        d[j] = static_cast<bf16_t>(__float_as_uint(t[j].x) != GeluSlopes::OUTSIDE ? g * t[j].x : 0.f);
        cols[j] += static_cast<float>(d[j]);
      }
      *reinterpret_cast<bf16x8_t*>(C + at0 + (size_t)(p + i * ROWS) * ldc) = d;
    }
  }
  __syncthreads();  // nobody reads the tile any more
  float* const part = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int j = 0; j < 8; ++j) part[row0 * BN + col + j] = cols[j];
  __syncthreads();
  for (int n = threadIdx.x; n < BN; n += THREADS) {
    float c = 0.f;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) c += part[r * BN + n];
    e.post_col_parts[(size_t)(m0 / BM) * ldc + n0 + n] = c;
  }
  __syncthreads();
  sum = block_sum(sum, part);
  if (threadIdx.x == 0) e.post_parts[blockIdx.x] = sum;
}
template <int POST, int BM, int BN, int THREADS>
__device__ __forceinline__ void post_tile(unsigned char* lds, const Epilogue& e, bf16_t* __restrict__ C, int ldc, int m0, int n0) {
  constexpr int ROWS = THREADS / (BN / 8), R = 4;  // rows a pass, passes in flight
  static_assert(BM % (ROWS * R) == 0, "whole passes");
  if constexpr (POST == POST_GELU) return gelu_tile<BM, BN, THREADS>(lds, e, C, ldc, m0, n0);
  if constexpr (POST == POST_DGELU) return dgelu_tile<BM, BN, THREADS>(lds, e, C, ldc, m0, n0);
  const bf16_t* tile = reinterpret_cast<const bf16_t*>(lds);
  const int row0 = threadIdx.x / (BN / 8), col = threadIdx.x % (BN / 8) * 8;
  const size_t at0 = (size_t)(m0 + row0) * ldc + n0 + col;
  QuantParam q{};
  if constexpr (POST != POST_MSE) q = post_quantizer<POST>(e, n0 + col);
  auto get = [](const u32x4_t& w, int j) { return __uint_as_float((j & 1) ? w[j >> 1] & 0xffff0000u : w[j >> 1] << 16); };
  float sum = 0.f;
  for (int p = 0; p < BM; p += ROWS * R) {
    u32x4_t in[R];
#pragma unroll
    for (int i = 0; i < R && POST != POST_QKV; ++i) in[i] = *reinterpret_cast<const u32x4_t*>(static_cast<const bf16_t*>(e.post_in) + at0 + (size_t)(p + i * ROWS) * ldc);
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const size_t at = at0 + (size_t)(p + i * ROWS) * ldc;
      const u32x4_t o = *reinterpret_cast<const u32x4_t*>(tile + (row0 + p + i * ROWS) * post_stride<BN> + col);
      if constexpr (POST == POST_MSE) {
        bf16x8_t dy;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float d = get(o, j) - get(in[i], j);
          sum += d * d;
          dy[j] = static_cast<bf16_t>(2.0f * d * e.post_scale);
        }
        *reinterpret_cast<u32x4_t*>(C + at) = o;
        *reinterpret_cast<bf16x8_t*>(static_cast<bf16_t*>(e.post_out) + at) = dy;
      } else if constexpr (POST == POST_QKV) {
        bf16x8_t c;
#pragma unroll
        for (int j = 0; j < 8; ++j) c[j] = static_cast<bf16_t>(q_code(q_ratio_fma(get(o, j), q), q));
        *reinterpret_cast<u32x4_t*>(C + at) = o;
        *reinterpret_cast<bf16x8_t*>(static_cast<bf16_t*>(e.post_out) + at) = c;
      } else {
        bf16x8_t d;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float v = q_ratio_fma(get(in[i], j), q);
          const bool inside = q_inside(v, q);
          sum += get(o, j) * (q_code(v, q) - (inside ? v : 0.f));
          if constexpr (POST == POST_MASK) d[j] = static_cast<bf16_t>(inside ? get(o, j) : 0.f);
        }
        if constexpr (POST == POST_MASK) *reinterpret_cast<bf16x8_t*>(C + at) = d;
        else if (e.post_out) *reinterpret_cast<u32x4_t*>(C + at) = o;
      }
    }
  }
  if constexpr (POST != POST_QKV) {
    sum = block_sum(sum, reinterpret_cast<float*>(lds));
    if (threadIdx.x == 0) e.post_parts[blockIdx.x] = sum;
  }
}

// The ranges of a block's groups of columns (`groups` slots of lds, filled before; a slot holds them and its section) go out
// as one partial a section.
struct RangeSlot { MinMax r; int sec; };
__device__ __forceinline__ void store_ranges(const RangeSlot* lds, int groups, const Epilogue& e, int N) {
  __syncthreads();
  const int sections = e.range_cols ? N / e.range_cols : 1;
  for (int s = threadIdx.x; s < sections; s += blockDim.x) {
    MinMax r;
    for (int i = 0; i < groups; ++i)
      if (lds[i].sec == s) r.add(lds[i].r);
    r.store(e.range + ((size_t)s * gridDim.x + blockIdx.x) * 3);
  }
}
__device__ __forceinline__ void put_range(RangeSlot* lds, int slot, const MinMax& r, int n, const Epilogue& e, int lane) {
  const MinMax w = r.wave();
  if (lane == 0) {
    lds[slot].r = e.gelu ? w : w.rounded<bf16_t>();
    lds[slot].sec = e.range_cols ? n / e.range_cols : 0;
  }
}
template <class TO>
__device__ __forceinline__ void epilogue_store(TO* C, int ldc, int m, int n, float acc, const Epilogue& e, const EpiVals& ev) {
  float v = acc * (ev.alpha * (e.col_scale ? e.col_scale[n] : 1.f));
  if (e.beta) v += ev.beta * ((e.col_vec ? e.col_vec[n] : 0.f) + (e.row_vec ? e.row_vec[m] : 0.f));
  if (e.bias) v += e.bias[n];
  if (e.gelu) v = gelu_t<TO>(round_to<TO>(v));
  stf(C, (size_t)m * ldc + n, v);
}

// ------------------------------------------------------------------------------
// fp32 products (v_mfma_f32_32x32x2_f32: fp32 operands, products and sums), any M, N, K: the check mode.
// Its products are small (tens to hundreds of rows), so a launch is bound by latency, not by throughput: a block is one
// 32 x 32 output tile, its four wavefronts take every fourth group of 8 contraction values straight from memory (four
// groups' loads in flight), and their partial sums meet in LDS in wavefront order.  128 x 256 x 64 and the like: 64 x 64
// tiles of vector-ALU products, staged through LDS 16 values of k at a time without prefetch, took 18 us; a one-layer step
// of 128 tokens with 18 of them went from 370 to 283 us.  Wide modules, one layer: 768 over 512 tokens 2323 -> 922 us, 1024
// over 4096 tokens 10449 -> 9310 us (its forward passes alone 4477 and 4550).
// In a group, lane l holds row l % 32 and the k values 4 (l / 32) .. + 3 of both operands: MFMA j multiplies element j of
// both halves, so the four of them cover the group.
// ------------------------------------------------------------------------------
typedef float f32x16s_t __attribute__((ext_vector_type(16)));
// element (r, k) of an operand: k contiguous in whole 16-byte chunks (VEC), or any strides
template <bool VEC>
__device__ __forceinline__ float4 load_k4(const float* __restrict__ p, size_t sr, size_t sk, int r, int k, int K) {
  if constexpr (VEC) {
    if (k >= K) return make_float4(0.f, 0.f, 0.f, 0.f);
    return *reinterpret_cast<const float4*>(p + r * sr + k);
  } else {
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = k + j < K ? p[r * sr + (size_t)(k + j) * sk] : 0.f;
    return make_float4(v[0], v[1], v[2], v[3]);
  }
}
template <bool VA, bool VB>
__global__ __launch_bounds__(256) void gemm_f32_k(const float* __restrict__ A, size_t a_sr, size_t a_sk, const float* __restrict__ B, size_t b_sr,
                                                  size_t b_sk, float* __restrict__ C, int ldc, int M, int N, int K, Epilogue e) {
  __shared__ float part[4][16][64];
  constexpr int U = 4;  // groups in flight
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m0 = blockIdx.x * 32, n0 = blockIdx.y * 32;
  // rows beyond the matrix repeat the last one: what they give is not stored
  const int ra = min(m0 + (lane & 31), M - 1), rb = min(n0 + (lane & 31), N - 1);
  f32x16s_t acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  for (int k0 = 8 * wave; k0 < K; k0 += 32 * U) {
    float4 a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + 32 * u + 4 * (lane >> 5);
      a[u] = load_k4<VA>(A, a_sr, a_sk, ra, k, K);
      b[u] = load_k4<VB>(B, b_sr, b_sk, rb, k, K);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u].x, b[u].x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u].y, b[u].y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u].z, b[u].z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u].w, b[u].w, acc, 0, 0, 0);
    }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) part[wave][r][lane] = acc[r];
  __syncthreads();
  EpiVals ev;
  ev.alpha = e.alpha ? *e.alpha : 1.f;
  ev.beta = (e.beta ? *e.beta : 0.f) + e.beta_alpha * ev.alpha;
  // accumulator register r of a lane is row 8 (r / 4) + 4 (lane / 32) + r % 4, column lane % 32; wavefront w stores registers 4 w .. 4 w + 3
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 4 * wave + i;
    const int m = m0 + 8 * wave + 4 * (lane >> 5) + i, n = n0 + (lane & 31);
    const float v = ((part[0][r][lane] + part[1][r][lane]) + part[2][r][lane]) + part[3][r][lane];
    if (m < M && n < N) epilogue_store(C, ldc, m, n, v, e, ev);
  }
}
static void launch_f32(int a_t, int b_t, const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K, const Epilogue& e,
                       hipStream_t st) {
  const dim3 g((M + 31) / 32, (N + 31) / 32);
  const size_t asr = a_t ? 1 : lda, ask = a_t ? lda : 1, bsr = b_t ? 1 : ldb, bsk = b_t ? ldb : 1;
  auto vec = [&](int t, const void* p, int ld) { return !t && K % 4 == 0 && ld % 4 == 0 && (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  const bool va = vec(a_t, A, lda), vb = vec(b_t, B, ldb);
  auto go = [&](auto fa, auto fb) {
    hipLaunchKernelGGL((gemm_f32_k<decltype(fa)::value, decltype(fb)::value>), g, dim3(256), 0, st, (const float*)A, asr, ask, (const float*)B, bsr,
                       bsk, (float*)C, ldc, M, N, K, e);
  };
  if (va && vb) return go(std::true_type{}, std::true_type{});
  if (va) return go(std::true_type{}, std::false_type{});
  if (vb) return go(std::false_type{}, std::true_type{});
  go(std::false_type{}, std::false_type{});
}

// ------------------------------------------------------------------------------
// MFMA products (v_mfma_f32_32x32x16_bf16 with fp32 accumulation, v_mfma_i32_32x32x32_i8 with exact
// int32 accumulation): kernel gemm_dl_k in mrem_gemm_dl.h.  Integer codes (|q| <= 255) are exact in
// bf16 and their products and partial sums are exact in fp32 while they stay below 2^24 (always for
// 4-bit weights: K * 255 * 7 < 2^24 up to K = 9398; with 8-bit weights only up to K = 518, beyond
// that a product on bf16 codes rounds like any fp32 sum); the int8 mode is exact while sums stay in int32 (i8_sums_fit, which
// its callers ask).  Which sizes it takes: see gemm_launch (bf16) and gemm_i8_ok.
// ------------------------------------------------------------------------------
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef int i32x16_t __attribute__((ext_vector_type(16)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));

constexpr int kBK = 64;  // k-granularity of the MFMA kernels, in 2-byte elements

}  // namespace mrem
#include "mrem_gemm_dl.h"
#include "mrem_gemm_quad.h"
#include "mrem_gemm_chain.h"
namespace mrem {

// no tile of 128 x 128 and no stage of the contraction is partly filled
static bool whole_tiles(int M, int N, int K) { return M % 128 == 0 && N % 128 == 0 && K % kBK == 0; }

#if MREM_GEMM_REST
static void gemm_launch(int dt, int a_t, int b_t, const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K,
                        const Epilogue& e, hipStream_t st);

void gemm(int dt, int a_t, int b_t, const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K,
          const Epilogue& e, hipStream_t st, GemmProfile* prof) {
  if (!prof || !prof->on) {
    gemm_launch(dt, a_t, b_t, A, lda, B, ldb, C, ldc, M, N, K, e, st);
    return;
  }
  GemmRecord r;
  r.flops = 2.0 * (double)M * (double)N * (double)K;
  (void)hipEventCreate(&r.e0);
  (void)hipEventCreate(&r.e1);
  tl_launch_events.e0 = r.e0;
  tl_launch_events.e1 = r.e1;
  gemm_launch(dt, a_t, b_t, A, lda, B, ldb, C, ldc, M, N, K, e, st);
  tl_launch_events = LaunchEvents();
  prof->recs.push_back(r);
}

bool gemm_i8_ok(const void* A, int lda, const void* B, int ldb, int M, int N, int K) {
  return M % 128 == 0 && N % 128 == 0 && K % 128 == 0 && lda % 16 == 0 && ldb % 16 == 0 &&
         (reinterpret_cast<uintptr_t>(A) & 15) == 0 && (reinterpret_cast<uintptr_t>(B) & 15) == 0;
}
#endif
// int8 mode: two int8 codes travel as one 16-bit element, so leading dimensions and the contraction
// length are halved.
// Which tile serves a product, by how many compute units (256) the output's tiles can occupy.  Times of single
// products on rotating operands (bf16, us), each against the next candidate:
//   64 x 64, 8 wavefronts in two groups, up to 256 such tiles: a k-step is a chain of latencies, shorter the smaller
//     the tile (1000 x 768 x 3072: 15.6 against 18.5 for 128 x 64; weight gradient 768 x 768 x 4096: 20.2 against 24.2,
//     and 34.9 for 128 x 128);
//   128 x 64, 8 wavefronts in two groups, three stages, up to 256 such tiles (2304 x 768 x 3072: 20.0 against 22.6 for
//     64 x 64 and 26.0 for 128 x 128);
//   128 x 128 with 8 wavefronts (two groups of 4; each group multiplies every other 16-deep k-substep of a
//     stage and the groups' partial sums meet in LDS before the epilogue), four stages of 128-byte rows, one
//     block per compute unit, up to 256 such tiles -- one tile per compute unit, so the second wavefront on each
//     SIMD is what overlaps fragment reads, barriers and MFMA issue (4096 x 1024 x 4096: 41.4 against 52.9 for 128 x 64);
//   128 x 256 (mrem_gemm_quad.h) up to 256 such tiles: one round of blocks with 3/4 of the operand bytes per flop of two
//     128 x 128 tiles a compute unit (6144 x 1024 x 4096: 57.3 against 73.6, int8 30.1 and 37.6; 2310 x 3072 x 768: 17.1
//     and 21.2; 2000 x 4096 x 1024: 21.4 and 26.3; 1500 x 3072 x 768, 144 tiles: 14.8 and 16.6);
//   256 x 256 (mrem_gemm_quad.h) beyond that: half the operand bytes per flop of 128 x 128 (4096 x 4096 x 1024: 32.0; 3000 x
//     3072 x 768, 144 tiles: 24.4 against 28.2 for 288 tiles of 128 x 256).
// The two large tiles need an even number of whole stages (K a multiple of 128, 256 for int8).  Partly filled tiles sum the
// even and the odd k-substeps apart, as the tiles above do, so that a row's sums do not depend on how many rows there are,
// until 256 x 256 tiles take over: 128 x 256 does so in a second set of accumulators (2310 x 3072 x 768 inside a step: 20.7,
// 25.1 on 128 x 64), 256 x 256 has no registers for it, and the few sizes between the two (2800 x 3072 x 1024) stay on 128 x
// 64, where a second round of 128 x 256 would be nearly empty (41.7 and 47.2).  Other contractions take
//   256 x 256 (8 wavefronts of 64 x 128, two stages) from 144 such tiles on: half the
//     operand bytes per flop of the small tile, which is faster only while its tiles fit two a compute unit (against
//     128 x 128, bf16 and int8: 128 tiles, 4096 x 2048 x 1024: 29.0 and 24.0, int8 18.4 and 15.3; 144 tiles, 4608 x 2048 x
//     768: 23.4 and 26.6, int8 16.0 and 17.7; 160 tiles, 2560 x 4096 x 1024: 29.0 and 32.3, int8 19.1 and 20.4);
//   128 x 128 with 4 wavefronts of 64 x 64, four stages of 64-byte rows, two blocks per compute unit, otherwise:
//     the second block fills the barrier and epilogue gaps of the first (6144 x 768 x 3072: 51.6 against 57.3 for
//     128 x 64).  Sizes with partly filled tiles take 128 x 64 here (2310 x 3072 x 768: 22.2 against 23.1).
template <bool AT, bool BT, class TO, bool I8>
void launch_dl_tiles(const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K, const Epilogue& e,
                            hipStream_t st, int splits) {
  auto tiles = [&](int bm, int bn) { return (int64_t)((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  const bool whole = whole_tiles(M, N, K);
  // (each tile where it serves such a product without `post`, see post_ok and post_codes_ok)
  if constexpr (!AT) {
    if (e.post) {
      auto go = [&](auto post) {
        constexpr int POST = decltype(post)::value;
        if constexpr (POST == POST_GELU || POST == POST_QKV) {
          if (tiles(64, 64) <= 256) return launch_dl<64, 64, 2, 2, AT, BT, 4, 128, TO, I8, 2, 2, true, POST>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
          if (tiles(128, 64) <= 256) return launch_dl<128, 64, 2, 2, AT, BT, 3, 128, TO, I8, 2, 2, true, POST>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
        }
        if (tiles(128, 128) <= 256) return launch_dl<128, 128, 2, 2, AT, BT, 4, 128, TO, I8, 1, 2, false, POST>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
        if (tiles(128, 256) <= 256) return launch_quad<128, AT, BT, TO, I8, false, false, POST>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
        return launch_quad<256, AT, BT, TO, I8, false, false, POST>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
      };
      if constexpr (I8) {
        if (e.post == POST_GELU) return go(std::integral_constant<int, POST_GELU>{});
        if (e.post == POST_QKV) return go(std::integral_constant<int, POST_QKV>{});
      }
      if constexpr (BT) {
        if (e.post == POST_DGELU) return go(std::integral_constant<int, POST_DGELU>{});
        if (e.post == POST_MASK) return go(std::integral_constant<int, POST_MASK>{});
      }
      return go(std::integral_constant<int, BT ? POST_STEP : POST_MSE>{});
    }
  }
  if constexpr (AT && BT) {
    if (splits > 1) return launch_dl<128, 128, 2, 2, AT, BT, 4, 128, TO, I8, 1, 2>(A, lda, B, ldb, C, ldc, M, N, K, e, st, splits);
  }
  if (tiles(64, 64) <= 256)
    return launch_dl<64, 64, 2, 2, AT, BT, 4, 128, TO, I8, 2, 2, true>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
  if (tiles(128, 64) <= 256)
    return launch_dl<128, 64, 2, 2, AT, BT, 3, 128, TO, I8, 2, 2, true>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
  if (tiles(128, 128) <= 256) {
    if (!whole) return launch_dl<128, 128, 2, 2, AT, BT, 4, 128, TO, I8, 1, 2, true>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
    return launch_dl<128, 128, 2, 2, AT, BT, 4, 128, TO, I8, 1, 2>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
  }
  const bool pair = !I8 && !whole && tiles(256, 256) < 144;  // (sums of codes are exact in any order)
  if (quad_ok(K) && (tiles(128, 256) <= 256 || !pair)) {
    if (tiles(128, 256) <= 256) {
      if constexpr (!I8) {
        if (pair) return launch_quad<128, AT, BT, TO, I8, true, true>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
      }
      if (M % 128 == 0 && N % 256 == 0) return launch_quad<128, AT, BT, TO, I8, false>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
      return launch_quad<128, AT, BT, TO, I8, true>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
    }
    if (M % 256 == 0 && N % 256 == 0) return launch_quad<256, AT, BT, TO, I8, false>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
    return launch_quad<256, AT, BT, TO, I8, true>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
  }
  if (tiles(256, 256) >= 144) {
    if (whole && M % 256 == 0 && N % 256 == 0)
      return launch_dl<256, 256, 4, 2, AT, BT, 2, 128, TO, I8, 1>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
    return launch_dl<256, 256, 4, 2, AT, BT, 2, 128, TO, I8, 1, 1, true>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
  }
  if (!whole) return launch_dl<128, 64, 2, 2, AT, BT, 3, 128, TO, I8, 2, 2, true>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
  return launch_dl<128, 128, 2, 2, AT, BT, 4, 64, TO, I8, 2>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
}
#if defined(MREM_GEMM_PART)
#define MREM_TILES(AT, BT, TO, I8)                                                                                                              \
  template void launch_dl_tiles<AT, BT, TO, I8>(const void*, int, const void*, int, void*, int, int, int, int, const Epilogue&, hipStream_t, int)
#if MREM_GEMM_PART == 0
extern MREM_TILES(false, false, bf16_t, false);
extern MREM_TILES(false, false, bf16_t, true);
extern MREM_TILES(false, true, bf16_t, false);
extern MREM_TILES(true, true, float, false);
#elif MREM_GEMM_PART == 1
MREM_TILES(false, false, bf16_t, false);
#elif MREM_GEMM_PART == 2
MREM_TILES(false, false, bf16_t, true);
#elif MREM_GEMM_PART == 3
MREM_TILES(false, true, bf16_t, false);
#elif MREM_GEMM_PART == 4
MREM_TILES(true, true, float, false);
#endif
#endif

#if MREM_GEMM_REST
// Which sizes have kernels with Epilogue::post: whole tiles from 128 x 128 on.  (Backward passes in partly filled ones are neither
// built nor measured; in smaller tiles they would take the step gradients' sums in another order, which small steps pin.)
bool post_ok(int M, int N, int K) {
  auto tiles = [&](int bm, int bn) { return (int64_t)((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  if (!whole_tiles(M, N, K) || tiles(128, 64) <= 256) return false;
  if (tiles(128, 128) <= 256) return true;
  return quad_ok(K) && N % 256 == 0 && (tiles(128, 256) <= 256 || (tiles(256, 256) <= 2048 && M % 256 == 0));
}
// ... and for codes also smaller tiles, where a launch less counts most (ragged sizes on larger tiles lose up to 1.5% of a step
// beside the other stream's kernels: three layers of 768 over 30 x 77 tokens 1190 and 1196 us, four of 1024 over 8 x 141 1649
// and 1667).
bool post_codes_ok(int M, int N, int K) {
  return (int64_t)((M + 127) / 128) * ((N + 63) / 64) <= 256 || post_ok(M, N, K / 2);
}
static void gemm_i8_launch(const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K, const Epilogue& e,
                           hipStream_t st) {
  Epilogue ee = e;
  ee.apart = !whole_tiles(M, N, K / 2);
  launch_dl_tiles<false, false, bf16_t, true>(A, lda / 2, B, ldb / 2, C, ldc, M, N, K / 2, ee, st, 1);
}
void gemm_i8(const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K, const Epilogue& e, hipStream_t st,
             GemmProfile* prof) {
  if (!prof || !prof->on) {
    gemm_i8_launch(A, lda, B, ldb, C, ldc, M, N, K, e, st);
    return;
  }
  GemmRecord r;
  r.flops = 2.0 * (double)M * (double)N * (double)K;
  (void)hipEventCreate(&r.e0);
  (void)hipEventCreate(&r.e1);
  tl_launch_events.e0 = r.e0;
  tl_launch_events.e1 = r.e1;
  gemm_i8_launch(A, lda, B, ldb, C, ldc, M, N, K, e, st);
  tl_launch_events = LaunchEvents();
  r.cls = 1;
  prof->recs.push_back(r);
}

void gemm_nt(int dt, const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K, const Epilogue& e,
             hipStream_t st, GemmProfile* prof) {
  gemm(dt, 0, 0, A, lda, B, ldb, C, ldc, M, N, K, e, st, prof);
}

// Tiles for a quarter to half of the compute units and a long contraction (weight gradients of 1024 x 1024 and
// 2304 x 768): two k-slices; with fewer tiles the 64 x 64 ones take over (alone, over 4096 tokens, us: 512 x 512 18.5
// against 20.0, 768 x 768 18.4 and 21.3, 1536 x 512 19.2 and 23.0, 1024 x 1024 19.4 and 24.7; three layers' step of 768
// 1774 -> 1733).  64 x 64 tiles for 1024 x 1024 too cost the six-layer step 0.6%: twice the operand traffic beside the
// other stream's kernels.  (Larger weight gradients run beside the rest of the backward
// pass, where a second slice only adds atomic traffic.)  Two atomic adds onto a zeroed fp32 value
// commute exactly, so the result does not depend on which slice arrives first.
static int f32_k_slices(int M, int N, int K) {
  return (whole_tiles(M, N, K) && (M / 128) * (N / 128) <= 128 && (M / 64) * (N / 64) > 192 && K >= 2048 && (K / kBK) % 2 == 0) ? 2 : 1;
}
int gemm_f32_k_slices(int dt, int M, int N, int K) {
  return dt == DT_BF16 ? f32_k_slices(M, N, K) : 1;
}

// A layer's weight gradients in one launch: the smaller of the large tiles with which all of them fit into one round of blocks.
// More tiles than units (wider than about 1200) would leave a second round nearly empty.  A launch takes as long as one tile's
// contraction, so few tiles serve only short ones: steps, us, single products first, three layers of 256 (24 tiles) over 4096
// tokens 757 and 773, over 2560 681 and 635; of 320 (57 tiles) over 4096 923 and 886; of 512 (96 tiles) 1134 and 1099, over
// 2048 880 and 827; two of 1024 over 4096 1505 and 1463.  Token counts that are not whole stages: three of 768 over 2310 1323
// and 1271, six of 1024 over 3640 4299 and 4135, of 512 over 3589 2256 and 2091.  Fewer tokens: four of 768 over 1500 1527 and
// 1425, two of 1024 over 1111 939 and 912; below that the single products are short.
int wgrads_tile(int dt, const WgradJob* jobs, int njobs, int K) {
  if (dt != DT_BF16 || K < 1024) return 0;
  for (const int bm : {128, 256}) {
    int64_t tiles = 0;
    for (int i = 0; i < njobs; ++i) tiles += (int64_t)((jobs[i].M + bm - 1) / bm) * ((jobs[i].N + 255) / 256);
    if (128 * tiles < K) return 0;
    if (tiles <= 256) return bm;
  }
  return 0;
}
void gemm_wgrads(const WgradJob* jobs, int njobs, int K, int tile, hipStream_t st) {
  bool whole = quad_ok(K);
  for (int i = 0; i < njobs; ++i) whole = whole && jobs[i].M % tile == 0 && jobs[i].N % 256 == 0;
  if (tile == 128) return whole ? launch_quad_wgrads<128, false>(jobs, njobs, K, st) : launch_quad_wgrads<128, true>(jobs, njobs, K, st);
  whole ? launch_quad_wgrads<256, false>(jobs, njobs, K, st) : launch_quad_wgrads<256, true>(jobs, njobs, K, st);
}

// bf16 products fetch whole 16-byte chunks: the index that is contiguous in memory (the contraction index, or the row
// index of a transposed operand) and the leading dimensions are multiples of 8 and operands 16-byte aligned, which the
// entry points require of widths and pointers; everything else may be ragged.  The callers need three forms: codes or
// activations times weights, an input gradient (B transposed), and a weight gradient (both transposed, fp32 result).
static void gemm_launch(int dt, int a_t, int b_t, const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K,
                        const Epilogue& e, hipStream_t st) {
  if (dt == DT_F32) {
    const hipEvent_t t0 = tl_launch_events.e0, t1 = tl_launch_events.e1;  // these kernels are timed by recorded events
    if (t0) (void)hipEventRecord(t0, st);
    launch_f32(a_t, b_t, A, lda, B, ldb, C, ldc, M, N, K, e, st);
    if (t1) (void)hipEventRecord(t1, st);
  } else if (a_t) {
    const int splits = f32_k_slices(M, N, K);
    if (splits > 1 && !e.c_zeroed) fill_f32((float*)C, 0.f, (int64_t)M * ldc, st);
    launch_dl_tiles<true, true, float, false>(A, lda, B, ldb, C, ldc, M, N, K, e, st, splits);
  } else if (b_t) {
    launch_dl_tiles<false, true, bf16_t, false>(A, lda, B, ldb, C, ldc, M, N, K, e, st, 1);
  } else if (const bool whole = whole_tiles(M, N, K); e.chain && !whole) {
    launch_chain(A, lda, B, ldb, C, ldc, M, N, K, e, st);
  } else {
    Epilogue ee = e;
    ee.apart = !whole;
    launch_dl_tiles<false, false, bf16_t, false>(A, lda, B, ldb, C, ldc, M, N, K, ee, st, 1);
  }
}

#endif

}  // namespace mrem
