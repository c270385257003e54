// Products of real-valued bf16 operands whose result does not depend on the tile: C[m][n] = sum over k of A[m][k] B[n][k]
// as one fp32 fused multiply-add after the other, k ascending, for any M and N and K a multiple of 8.
//
// Why: the quantizers amplify rounding.  A sum taken in another order moves the clip ranges that a calibration finds and
// with them codes of every layer above; of a step of six layers of 1024 over 100 tokens that moved the second moments by
// up to 44 percent (a step size's gradient is a sum that cancels).  Whole tiles have one order each; for all other sizes
// this kernel keeps the sums the same whatever tile serves them, where the caller asks for it (Epilogue::chain).
//
// v_mfma_f32_16x16x4_f32 is such a chain: its result equals four fused multiply-adds with k ascending bit for bit, also
// where terms are subnormal.  It gives 64 flops a cycle and SIMD, a sixteenth of the bf16 product, which bounds the kernel
// (4000 x 4096 x 1024: 280 us, 214 at that rate and 2.4 GHz), and vector instructions do not run beside it: a form with
// direct loads that converts and rearranges operands per wavefront took 316 us.
//
// A block is BM x BN outputs, four wavefronts of (BM / 2) x (BN / 2).  LDS holds the stage's BK values of k as fp32, those
// with k % 4 = q together for the quarter q of a wavefront that multiplies them, so that a lane reads four products'
// operands (16 bytes) at once; with rows of one k each and 4-byte accesses that product took 305 us on 64 x 64 tiles
// (291 now) and 23 x 768 x 3072 30 us (28 now).  Groups of 16 bytes change places by row, so that 16 rows fall on
// different banks.  The next stage waits in registers while one is multiplied; two stages in LDS, one barrier each.
#pragma once

namespace mrem {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

template <int ROWS, int BK>
struct ChainOperand {
  static constexpr int CPR = BK / 8, PER = ROWS * CPR / 256, G = BK / 16, FLOATS = ROWS * BK;
  static_assert(PER >= 1 && ROWS * CPR % 256 == 0, "the chunks of a stage divide evenly over 256 threads");
  // [quarter][row][BK / 4] in groups of 4 values; group g of a row
  static __device__ __forceinline__ int at(int quarter, int row, int g) {
    return (quarter * ROWS + row) * (BK / 4) + 4 * (g ^ ((row / (16 / G)) & (G - 1)));
  }
  static __device__ __forceinline__ void load(u32x4_t (&v)[PER], const bf16_t* __restrict__ p, int ld, int row0, int rows, int k0, int K) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int id = threadIdx.x + 256 * i, r = min(row0 + id / CPR, rows - 1), k = k0 + id % CPR * 8;  // rows beyond the matrix repeat the last one
      v[i] = u32x4_t{0u, 0u, 0u, 0u};
      if (k < K) v[i] = *reinterpret_cast<const u32x4_t*>(p + (size_t)r * ld + k);
    }
  }
  // k = 8 c + 4 h + q of chunk c: value 2 c + h of quarter q
  static __device__ __forceinline__ void store(const u32x4_t (&v)[PER], float* dst) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int id = threadIdx.x + 256 * i, c = id % CPR;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const unsigned lo = v[i][q / 2], hi = v[i][2 + q / 2];
        const float2 f = q % 2 ? make_float2(__uint_as_float(lo & 0xffff0000u), __uint_as_float(hi & 0xffff0000u))
                               : make_float2(__uint_as_float(lo << 16), __uint_as_float(hi << 16));
        *reinterpret_cast<float2*>(dst + at(q, id / CPR, c / 2) + 2 * (c % 2)) = f;
      }
    }
  }
};

template <int BM, int BN, int BK>
__global__ __launch_bounds__(256) void gemm_chain_k(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ B, int ldb,
                                                    bf16_t* __restrict__ C, int ldc, int M, int N, int K, Epilogue e, int tiles_m, int tiles_n) {
  typedef ChainOperand<BM, BK> OpA;
  typedef ChainOperand<BN, BK> OpB;
  constexpr int MT = BM / 32, NT = BN / 32;
  __shared__ __attribute__((aligned(16))) float As[2][OpA::FLOATS];
  __shared__ __attribute__((aligned(16))) float Bs[2][OpB::FLOATS];
  int tm, tn;
  tile_of_block(tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, quarter = lane >> 4;
  const int wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * (BN / 2);
  u32x4_t va[OpA::PER], vb[OpB::PER];
  f32x4_t acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto load = [&](int k0) {
    OpA::load(va, A, lda, m0, M, k0, K);
    OpB::load(vb, B, ldb, n0, N, k0, K);
  };
  auto store = [&](int buf) {
    OpA::store(va, As[buf]);
    OpB::store(vb, Bs[buf]);
  };
  load(0);
  store(0);
  __syncthreads();
  for (int k0 = 0, buf = 0; k0 < K; k0 += BK, buf ^= 1) {
    const bool more = k0 + BK < K;
    if (more) load(k0 + BK);
    f32x4_t a[BK / 16][MT], b[BK / 16][NT];  // k = 16 g + 4 e + quarter: element e of group g
#pragma unroll
    for (int g = 0; g < BK / 16; ++g) {
#pragma unroll
      for (int i = 0; i < MT; ++i) a[g][i] = *reinterpret_cast<const f32x4_t*>(&As[buf][OpA::at(quarter, wm + 16 * i + l16, g)]);
#pragma unroll
      for (int j = 0; j < NT; ++j) b[g][j] = *reinterpret_cast<const f32x4_t*>(&Bs[buf][OpB::at(quarter, wn + 16 * j + l16, g)]);
    }
    // a single chain per wavefront: all fragments of the stage are read first
    if constexpr (MT * NT == 1) __builtin_amdgcn_sched_barrier(0);
    // rows of the accumulator tile are columns of C, so that a lane holds four neighbours of one row
#pragma unroll
    for (int s = 0; s < BK / 4; ++s)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[s / 4][j][s % 4], a[s / 4][i][s % 4], acc[i][j], 0, 0, 0);
    if (more) store(buf ^ 1);
    __syncthreads();
  }
  const float alpha = e.alpha ? *e.alpha : 1.f;
  const float beta = (e.beta ? *e.beta : 0.f) + e.beta_alpha * alpha;
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int n = n0 + wn + 16 * j + 4 * quarter;
    if (n >= N) continue;  // N is a multiple of 8
    float cs[4], cv[4], cb[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      cs[r] = alpha * (e.col_scale ? e.col_scale[n + r] : 1.f);
      cv[r] = e.beta && e.col_vec ? e.col_vec[n + r] : 0.f;
      cb[r] = e.bias ? e.bias[n + r] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int m = m0 + wm + 16 * i + l16;
      if (m >= M) continue;
      typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
      bf16x4_t out;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float t = e.beta && e.row_vec ? cv[r] + e.row_vec[m] : cv[r];
        float v = epilogue_apart(acc[i][j][r], cs[r], e.beta != nullptr, beta, t, e.bias != nullptr, cb[r]);
        if (e.gelu) v = gelu_t<bf16_t>(round_to<bf16_t>(v));
        out[r] = static_cast<bf16_t>(v);
      }
      *reinterpret_cast<bf16x4_t*>(C + (size_t)m * ldc + n) = out;
    }
  }
}

template <int BM, int BN, int BK>
static void launch_chain_tile(const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K, const Epilogue& e,
                              hipStream_t st) {
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  MREM_LAUNCH((gemm_chain_k<BM, BN, BK>), dim3(tiles_m * tiles_n), dim3(256), 0, st, (const bf16_t*)A, lda, (const bf16_t*)B, ldb, (bf16_t*)C, ldc, M,
              N, K, e, tiles_m, tiles_n);
}
// By how many tiles there are for the 256 compute units (us, against the next smaller tile): 128 x 128 from two a compute
// unit on (4000 x 4096 x 1024, 1024 tiles: 280 against 291; 2310 x 3072 x 768, 456: 110 against 100), 64 x 64 from one and
// a half on (924 x 3072 x 768, 720 tiles: 48 against 54; 924 x 768 x 3072, 180: 73 against 57).
static void launch_chain(const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K, const Epilogue& e, hipStream_t st) {
  auto tiles = [&](int b) { return (int64_t)((M + b - 1) / b) * ((N + b - 1) / b); };
  if (tiles(128) >= 512) return launch_chain_tile<128, 128, 16>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
  if (tiles(64) >= 384) return launch_chain_tile<64, 64, 32>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
  launch_chain_tile<32, 32, 64>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
}

}  // namespace mrem
