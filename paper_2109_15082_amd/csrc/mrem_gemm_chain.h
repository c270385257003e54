// Products of real-valued bf16 operands whose result does not depend on the tile: C[m][n] = sum over k of A[m][k] B[n][k]
// as one fp32 fused multiply-add after the other, k ascending, for any M and N and K a multiple of 8.
//
// Why: the quantizers amplify rounding.  A sum taken in another order moves the clip ranges that a calibration finds and
// with them codes of every layer above; of a step of six layers of 1024 over 100 tokens that moved the second moments by
// up to 44 percent (a step size's gradient is a sum that cancels).  Whole tiles have one order each; for all other sizes
// this kernel keeps the sums the same whatever tile serves them, where the caller asks for it (Epilogue::chain).
//
// v_mfma_f32_16x16x4_f32 is such a chain: its result equals four fused multiply-adds with k ascending bit for bit, also
// where terms are subnormal.  It gives 64 flops a cycle and SIMD, a sixteenth of the bf16 product, which bounds large
// products; small ones are bound by the chain itself, K / 4 instructions of 33.6 cycles each, whatever the tile.  One
// ordinary vector instruction between two of them costs 16 cycles, every further one 4 (they share the multipliers), an LDS
// read next to nothing up to two an instruction.  So the loop holds nothing else: operands go global -> LDS as they are
// (direct loads, three stages of 64 values of k ahead, swizzled as in mrem_gemm_dl.h), and a lane reads its value straight
// into the upper half of a register whose lower half is zero (ds_read_u16_d16_hi), which is the conversion.  Reads run AHEAD
// steps in front of the instruction that needs them and are waited for one step at a time; stage addresses advance in scalar
// registers.  23 x 768 x 3072: 17.1 us (43 cycles an instruction); with fp32 in LDS, converted by the threads that stored
// it, and a wait for all of a stage's reads 27.8 us.  500 x 1024 x 4096: 38 and 56 us.  4000 x 4096 x 1024: 268 and 283 us
// (214 at the instruction's rate and 2.4 GHz).
//
// A block is WM x WN wavefronts of MT x NT tiles of 16 x 16.
#pragma once

namespace mrem {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

template <int OFF>
__device__ __forceinline__ void lds_read_u16_hi(float& v, int addr) {
  asm volatile("ds_read_u16_d16_hi %0, %1 offset:%2" : "+v"(v) : "v"(addr), "n"(OFF));
}

// values of T tiles for one step (k = 4 STEP + quarter) of the stage OFF bytes on
template <int OFF, int STEP, int T>
__device__ __forceinline__ void chain_read(float (&f)[T], const int (&addr)[8]) {
  static_for<T>([&](auto i) { lds_read_u16_hi<OFF + 8 * (STEP & 1) + 2048 * i.value>(f[i.value], addr[STEP / 2]); });
}
template <int T>
__device__ __forceinline__ void chain_tie(float (&f)[T]) {
#pragma unroll
  for (int i = 0; i < T; ++i) asm volatile("" : "+v"(f[i]));
}
// at most N LDS reads may still be in flight (they return in order)
template <int N>
__device__ __forceinline__ void wait_lgkmcnt() {
  static_assert(N >= 0 && N < 16, "4-bit counter");
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory");
}

template <int MT, int NT, int WM, int WN, int AHEAD>
__global__ __launch_bounds__(64 * WM * WN) void gemm_chain_k(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ B, int ldb,
                                                             bf16_t* __restrict__ C, int ldc, int M, int N, int K, Epilogue e, int tiles_m, int tiles_n) {
  constexpr int BM = 16 * MT * WM, BN = 16 * NT * WN, BK = 64, RB = 2 * BK, NW = WM * WN, STAGES = 4, STEPS = BK / 4;
  constexpr int RING = AHEAD < 2 ? 2 : AHEAD < 3 ? 4 : 8;  // steps whose operands are in registers or on the way
  typedef DlOperand<false, BM, RB, 1> OpA;
  typedef DlOperand<false, BN, RB, 1> OpB;
  constexpr int STAGE_BYTES = OpA::BYTES + OpB::BYTES, LPW = (OpA::LOADS + OpB::LOADS) / NW;
  static_assert((OpA::LOADS + OpB::LOADS) % NW == 0, "the loads of a stage divide evenly over the wavefronts");
  static_assert((STAGES - 1) * STAGE_BYTES + 2048 * (MT > NT ? MT : NT) <= 65536, "an LDS read reaches every stage with its 16-bit offset");
  static_assert(AHEAD >= 1 && 2 * AHEAD <= RING && STEPS % RING == 0 && (2 * AHEAD - 1) * (MT + NT) < 16, "LDS reads in flight fit the 4-bit counter");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[STAGES * STAGE_BYTES];
  int tm, tn;
  tile_of_block(tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int lane = threadIdx.x & 63, l16 = lane & 15, quarter = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN * (16 * MT), wn = wave % WN * (16 * NT);
  const int KT = (K + BK - 1) / BK, tail = K % BK;

  // sources of this wavefront's loads: its operand's first row, and a lane's offset (rows beyond the matrix repeat the last one)
  const unsigned char* base[LPW];
  unsigned src[LPW];
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int gi = wave * LPW + i, p = gi * 1024 + lane * 16;
    base[i] = reinterpret_cast<const unsigned char*>(gi < OpA::LOADS ? A + (size_t)m0 * lda : B + (size_t)n0 * ldb);
    src[i] = (unsigned)(gi < OpA::LOADS ? OpA::src_offset_edge(p, lda, M - m0) : OpB::src_offset_edge(p - OpA::BYTES, ldb, N - n0));
  }
  // Fetch a stage into its slot.  Stages beyond the last are the last one again (nobody reads them): the loop has no case for
  // them.  Chunks beyond the contraction come from a block of zeros.
  auto issue = [&](int stage, int slot) {
    unsigned char* dst = smem + slot * STAGE_BYTES + wave * (LPW * 1024);
    const int kt = stage < KT ? stage : KT - 1;
    auto load = [&](int i, const unsigned char* s) {
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)s, (__attribute__((address_space(3))) void*)(dst + i * 1024), 16, 0, 0);
    };
    if (tail && kt == KT - 1) {
#pragma unroll
      for (int i = 0; i < LPW; ++i) {
        const int gi = wave * LPW + i, p = gi * 1024 + lane * 16;
        const int k = gi < OpA::LOADS ? OpA::k_of(p) : OpB::k_of(p - OpA::BYTES);
        load(i, k < tail ? base[i] + (size_t)kt * RB + src[i] : reinterpret_cast<const unsigned char*>(&kZeroChunk));
      }
    } else {
#pragma unroll
      for (int i = 0; i < LPW; ++i) load(i, base[i] + (size_t)kt * RB + src[i]);
    }
  };

  // LDS addresses of k values quarter and 4 + quarter (8 bytes on) of the eight chunks of a stage
  int a_addr[8], b_addr[8];
  const int lds0 = (int)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const int at = l16 * RB + ((c ^ OpA::swizzle_k(l16)) << 4) + 2 * quarter;  // 16 rows on: the swizzle is the same
    a_addr[c] = lds0 + wm * RB + at;
    b_addr[c] = lds0 + OpA::BYTES + wn * RB + at;
  }
  f32x4_t acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float fa[RING][MT], fb[RING][NT];  // the lower halves stay zero
#pragma unroll
  for (int s = 0; s < RING; ++s) {
#pragma unroll
    for (int i = 0; i < MT; ++i) fa[s][i] = 0.f;
#pragma unroll
    for (int j = 0; j < NT; ++j) fb[s][j] = 0.f;
  }
  auto read = [&](auto slot, auto step) {
    constexpr int off = decltype(slot)::value * STAGE_BYTES, s = decltype(step)::value;
    chain_read<off, s>(fa[s % RING], a_addr);
    chain_read<off, s>(fb[s % RING], b_addr);
  };
  // rows of the accumulator tile are columns of C, so that a lane holds four neighbours of one row; `later`: the steps that
  // have been read after this one
  auto multiply = [&](auto step, auto later) {
    constexpr int s = decltype(step)::value % RING;
    wait_lgkmcnt<decltype(later)::value * (MT + NT)>();
    chain_tie(fa[s]);
    chain_tie(fb[s]);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[s][j], fa[s][i], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  // The first steps of a stage have arrived.
  auto first_steps_arrived = [&]() {
    wait_lgkmcnt<0>();
    static_for<AHEAD>([&](auto s) {
      chain_tie(fa[s.value]);
      chain_tie(fb[s.value]);
    });
  };
  // Stage kt.  Its operands are read AHEAD steps before they are multiplied, those of the next stage's first steps behind
  // the barrier that hands it over, ahead of this stage's last steps.  A stage is straight code that begins and ends with
  // nothing in flight: a value that crosses a branch may be copied there, and a copy of what is still on its way into a
  // register is a copy of what was there before.  So the fetch, which has a branch, stands behind the last wait, which the
  // last steps' instructions cover (23 x 768 x 3072 in a calibration: 17.4 us with it and with values crossing the loop's
  // edge, 4000 x 4096 x 1024: 292 and 291).  The last stage reads on into the next slot, and what it reads is dropped.
  auto run_stage = [&](int kt, auto slot) {
    constexpr std::integral_constant<int, AHEAD> ahead{};
    static_for<STEPS - AHEAD>([&](auto s) {
      read(slot, std::integral_constant<int, s.value + AHEAD>{});
      multiply(s, ahead);
    });
    wait_vmcnt<LPW*(STAGES - 3)>();  // own loads of the next stage have landed
    __builtin_amdgcn_s_barrier();    // everybody's have, and everybody holds the operands of the stage before this one
    static_for<AHEAD>([&](auto s) { read(std::integral_constant<int, (slot.value + 1) % STAGES>{}, s); });
    static_for<AHEAD>([&](auto s) {
      multiply(std::integral_constant<int, STEPS - AHEAD + s.value>{}, std::integral_constant<int, 2 * AHEAD - 1 - s.value>{});
    });
    first_steps_arrived();
    issue(kt + STAGES - 1, (slot.value + STAGES - 1) % STAGES);
  };
  for (int s = 0; s < STAGES - 1; ++s) issue(s, s);
  wait_vmcnt<LPW*(STAGES - 2)>();
  __builtin_amdgcn_s_barrier();  // stage 0 has landed for everybody
  static_for<AHEAD>([&](auto s) { read(std::integral_constant<int, 0>{}, s); });
  first_steps_arrived();
  for (int kt = 0;;) {
    run_stage(kt, std::integral_constant<int, 0>{});
    if (++kt >= KT) break;
    run_stage(kt, std::integral_constant<int, 1>{});
    if (++kt >= KT) break;
    run_stage(kt, std::integral_constant<int, 2>{});
    if (++kt >= KT) break;
    run_stage(kt, std::integral_constant<int, 3>{});
    if (++kt >= KT) break;
  }
  // nothing is on its way into LDS when the block ends
  wait_vmcnt<0>();
  const float alpha = e.alpha ? *e.alpha : 1.f;
  const float beta = (e.beta ? *e.beta : 0.f) + e.beta_alpha * alpha;
  MinMax range[NT];
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
        if (e.range) range[j].add(v);
        out[r] = static_cast<bf16_t>(v);
      }
      *reinterpret_cast<bf16x4_t*>(C + (size_t)m * ldc + n) = out;
    }
  }
  if (e.range) {
    RangeSlot* const slots = reinterpret_cast<RangeSlot*>(smem);
    __syncthreads();  // nobody reads operands any more
#pragma unroll
    for (int j = 0; j < NT; ++j) put_range(slots, wave * NT + j, range[j], n0 + wn + 16 * j, e, lane);
    store_ranges(slots, NW * NT, e, N);
  }
}

template <int MT, int NT, int WM, int WN, int AHEAD>
static void launch_chain_tile(const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K, const Epilogue& e,
                              hipStream_t st) {
  constexpr int BM = 16 * MT * WM, BN = 16 * NT * WN;
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  if (e.blocks) *e.blocks = tiles_m * tiles_n;
  MREM_LAUNCH((gemm_chain_k<MT, NT, WM, WN, AHEAD>), dim3(tiles_m * tiles_n), dim3(64 * WM * WN), 0, st, (const bf16_t*)A, lda, (const bf16_t*)B,
              ldb, (bf16_t*)C, ldc, M, N, K, e, tiles_m, tiles_n);
}
// 64 x 64 from 480 such tiles on, almost two a compute unit (us, against 32 x 32: 500 x 4096 x 1024, 512 tiles: 38.9 and 41.5;
// 2048 x 960 x 320, 480: 15.5 and 16.7; 4000 x 1024 x 4096, 1008: 254 and 266; 2310 x 768 x 768, 444: 29.7 and 28.7).
// 128 x 128 tiles take as long as 64 x 64 ones (4000 x 4096 x 1024: 261 and 268; 4000 x 1024 x 4096: 255 and 254).
static void launch_chain(const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K, const Epilogue& e, hipStream_t st) {
  auto tiles = [&](int b) { return (int64_t)((M + b - 1) / b) * ((N + b - 1) / b); };
  if (tiles(64) >= 480) return launch_chain_tile<2, 2, 2, 2, 2>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
  launch_chain_tile<1, 1, 2, 2, 3>(A, lda, B, ldb, C, ldc, M, N, K, e, st);
}

}  // namespace mrem
