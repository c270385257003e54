// Large tiles of the matrix product: 256 x 256 and 128 x 256.  Same contract, operand modes and LDS layouts as gemm_dl_k
// (mrem_gemm_dl.h); what differs is how long a load may take to land, and what a wavefront issues when.  Sums are those of
// the gemm_dl_k tile that serves the same size where a contraction is no even number of stages: one chain over k, or (PAIR)
// two, of the even and of the odd k-substeps, which meet before the epilogue.
//
// Two stages of 64 KB are all that fit into LDS, and a stage that is refilled as a whole leaves its loads one k-step (about
// 1 us), while a quarter of them come from beyond the L2.  Here a stage is four halves, the first and second half of the
// rows of either operand, and a k-step is four phases, one quadrant of every wavefront's tile each, in an order in which
// every phase needs one half that the one before did not: A0 B0, A1 B0, A1 B1, A0 B1.  A half that has been read into
// registers is refilled in the next phase, so a load has seven phases (1.75 k-steps) to land and 12 to 14 KB a wavefront are
// on their way all the time.  A phase: wait for the oldest half on its way (the others stay), barrier, then the quadrant's
// matrix instructions on registers, with the refill of the half that the phase before read and the reads of the half that
// the next one needs between them -- not ahead of them, where eight wavefronts' reads queue up in front of an idle matrix
// pipe (8192^3: 905 us, 860 in this order).  Buffer loads take a uniform address and 32 bits a lane, so that addresses cost
// no vector registers.
//
// One block a compute unit.  us, against the tile of the same size that refills whole stages: 8192^3 860 and 980 (1.28
// PFLOP/s), 4096 x 4096 x 1024 32.0 and 38.1, its input gradient 32.8 and 39.4, on int8 codes 20.5 and 24.0.
#pragma once

namespace mrem {

// L direct loads of 1 KiB from p + o (a lane's bytes) on; bytes from `end` (if any) on are not read, LDS gets zeros for them
template <int L>
__device__ __forceinline__ void buffer_to_lds(const unsigned char* p, const unsigned char* end, const unsigned (&o)[L], unsigned char* dst) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass does not know the resource type
  int bytes = -1;
  if (end) bytes = p < end ? (int)(unsigned)min((size_t)(end - p), (size_t)0xffffffffu) : 0;
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(p), 0, bytes, 0x00027000);
#pragma unroll
  for (int i = 0; i < L; ++i)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)(dst + i * 1024), 16, o[i], 0, 0, 0);
#endif
}

// tile (tm, tn) of a product
template <int BM, bool AT, bool BT, class TO, bool I8, bool EDGE, bool PAIR, int POST = POST_NONE>
__device__ __forceinline__ void quad_tile(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ B, int ldb, TO* __restrict__ C, int ldc, int M,
                                          int N, int K, const Epilogue& e, int tm, int tn) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_quad[];
  constexpr int BN = 256, HA = BM / 2, HN = BN / 2, RB = 128, BK = RB / 2, KK = RB / 32;
  constexpr int WAVES_M = HA / 32, WAVES_N = 8 / WAVES_M, WN = HN / WAVES_N, NT = WN / 32;
  typedef DlOperand<AT, HA, RB, 1> OpA;
  typedef DlOperand<BT, HN, RB, NT> OpB;
  constexpr int SLOT_A = 2 * OpA::BYTES, SLOT_B = 2 * OpB::BYTES, B0 = 2 * SLOT_A;  // LDS: A's two slots, then B's
  constexpr int LA = OpA::LOADS / 8, LB = OpB::LOADS / 8;                            // direct loads of a half per wavefront
  static_assert(LA >= 1 && LB >= 1 && KK == 4, "whole loads of a half per wavefront; four k-substeps a stage");

  const int m0 = tm * BM, n0 = tn * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  // EDGE, both operands transposed: rows beyond the contraction are beyond the end of both operands and read as zeros, so any K
  // is an even number of stages
  const int KT = EDGE && AT && BT ? (K + 2 * BK - 1) / (2 * BK) * 2 : K / BK;

  // sources: the first element of a half's next stage (uniform) and this lane's offsets from it
  const size_t adv_a = AT ? (size_t)BK * lda * 2 : RB, adv_b = BT ? (size_t)BK * ldb * 2 : RB;
  const unsigned char *pa[2], *pb[2];
  unsigned oa[LA], ob[LB];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    pa[h] = reinterpret_cast<const unsigned char*>(AT ? A + m0 + h * HA : A + (size_t)(m0 + h * HA) * lda);
    pb[h] = reinterpret_cast<const unsigned char*>(BT ? B + n0 + h * HN : B + (size_t)(n0 + h * HN) * ldb);
  }
#pragma unroll
  for (int i = 0; i < LA; ++i) oa[i] = (unsigned)OpA::src_offset((wave * LA + i) * 1024 + lane * 16, lda);
#pragma unroll
  for (int i = 0; i < LB; ++i) ob[i] = (unsigned)OpB::src_offset((wave * LB + i) * 1024 + lane * 16, ldb);
  // EDGE: nothing is fetched from beyond the end of an operand (such bytes are zeros in LDS).  What a partly filled tile holds for rows that the matrix does
  // not have only enters results that are not stored.
  const unsigned char* const end_a = reinterpret_cast<const unsigned char*>(A + (size_t)((AT ? K : M) - 1) * lda + (AT ? M : K));
  const unsigned char* const end_b = reinterpret_cast<const unsigned char*>(B + (size_t)((BT ? K : N) - 1) * ldb + (BT ? N : K));
  auto fetch_a = [&](int h, int slot) {
    buffer_to_lds(pa[h], EDGE ? end_a : nullptr, oa, smem_quad + slot * SLOT_A + h * OpA::BYTES + wave * (LA * 1024));
    pa[h] += adv_a;
  };
  auto fetch_b = [&](int h, int slot) {
    buffer_to_lds(pb[h], EDGE ? end_b : nullptr, ob, smem_quad + B0 + slot * SLOT_B + h * OpB::BYTES + wave * (LB * 1024));
    pb[h] += adv_b;
  };

  int a_addr[OpA::NADDR], b_addr[OpB::NADDR];
  OpA::lane_addr(a_addr, wm * 32, lane, 0);
  OpB::lane_addr(b_addr, wn * WN, lane, 0);
  const int lds0 = (int)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem_quad;
#pragma unroll
  for (int i = 0; i < OpA::NADDR; ++i) a_addr[i] += lds0;
#pragma unroll
  for (int i = 0; i < OpB::NADDR; ++i) b_addr[i] += lds0 + B0;

  typedef typename std::conditional<I8, i32x16_t, f32x16_t>::type acc_t;
  constexpr int P = PAIR ? 2 : 1;
  acc_t acc[2][2][P][NT];  // quadrant (rows, columns), chain, tile
#pragma unroll
  for (int i = 0; i < 4 * P * NT; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i / (2 * P * NT)][i / (P * NT) % 2][i / NT % P][i % NT][r] = 0;
  typename OpA::frag_t fa[2][KK][1];
  typename OpB::frag_t fb[2][KK][NT];
  // k-substep `k` of a half that is read
  auto read_a = [&](typename OpA::frag_t (&f)[KK][1], auto at, auto k) {
    OpA::template read<decltype(k)::value, decltype(at)::value>(f[decltype(k)::value], a_addr, 0);
  };
  auto read_b = [&](typename OpB::frag_t (&f)[KK][NT], auto at, auto k) {
    OpB::template read<decltype(k)::value, decltype(at)::value>(f[decltype(k)::value], b_addr, 0);
  };
  // a quadrant's matrix instructions; `refill` sends out what the phase fetches, `read` (a k-substep) what it reads
  auto multiply = [&](acc_t (&acc_q)[P][NT], const typename OpA::frag_t (&a)[KK][1], const typename OpB::frag_t (&b)[KK][NT], auto refill, auto read) {
    auto substep = [&](auto kk) {
      constexpr int k = decltype(kk)::value;
      acc_t(&c)[NT] = acc_q[k % P];
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        if constexpr (I8) c[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(OpA::regs(a[k][0]), OpB::regs(b[k][j]), c[j], 0, 0, 0);
        else c[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, OpA::regs(a[k][0])), __builtin_bit_cast(bf16x8_t, OpB::regs(b[k][j])), c[j], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    constexpr std::integral_constant<int, 0> k0{};
    constexpr std::integral_constant<int, 1> k1{};
    constexpr std::integral_constant<int, 2> k2{};
    constexpr std::integral_constant<int, 3> k3{};
    __builtin_amdgcn_s_setprio(1);
    substep(k0);
    refill();
    read(k0);
    read(k1);
    __builtin_amdgcn_sched_barrier(0);
    substep(k1);
    read(k2);
    read(k3);
    __builtin_amdgcn_sched_barrier(0);
    substep(k2);
    substep(k3);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto arrived_a = [&](typename OpA::frag_t (&f)[KK][1]) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int k = 0; k < KK; ++k) OpA::tie(f[k]);
  };
  auto arrived_b = [&](typename OpB::frag_t (&f)[KK][NT]) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int k = 0; k < KK; ++k) OpB::tie(f[k]);
  };
  // The half that this phase reads has landed, for everybody, and everybody holds the one that the phase before read.  Loads
  // sent out after it, of NA halves of A and NB halves of B, may still be on their way.
  auto hand_over = [&](auto na, auto nb) {
    wait_vmcnt<decltype(na)::value * LA + decltype(nb)::value * LB>();
    __builtin_amdgcn_s_barrier();
  };
  constexpr std::integral_constant<int, 0> c0{};
  constexpr std::integral_constant<int, 1> c1{};
  constexpr std::integral_constant<int, 2> c2{};
  constexpr std::integral_constant<int, 3> c3{};
  constexpr std::integral_constant<int, 4> c4{};
  // A k-step in slot S.  LAST: 0 not one of the last two, 1 the last but one, 2 the last.  Halves go out in the order A0(kt + 2),
  // A1(kt + 2), B1(kt + 2), B0(kt + 3); `third` says whether there is a k-step kt + 3.
  auto k_step = [&](auto par, auto last_, bool third) {
    constexpr int S = decltype(par)::value, LAST = decltype(last_)::value, Q = S ^ 1;
    constexpr std::integral_constant<int, S * SLOT_A + OpA::BYTES> a1{};
    constexpr std::integral_constant<int, S * SLOT_B + OpB::BYTES> b1{};
    constexpr std::integral_constant<int, Q * SLOT_B> b0_next{};
    constexpr std::integral_constant<int, Q * SLOT_A> a0_next{};
    if constexpr (LAST == 0) hand_over(c2, c4);
    else if constexpr (LAST == 1) hand_over(c2, c3);
    else hand_over(c0, c1);
    multiply(acc[0][0], fa[S], fb[0], [&] { if constexpr (LAST == 0) fetch_a(0, S); }, [&](auto k) { read_a(fa[Q], a1, k); });
    arrived_a(fa[Q]);
    if constexpr (LAST == 0) hand_over(c3, c3);
    else if constexpr (LAST == 1) hand_over(c2, c2);
    else hand_over(c0, c0);
    multiply(acc[1][0], fa[Q], fb[0], [&] { if constexpr (LAST == 0) fetch_a(1, S); }, [&](auto k) { read_b(fb[1], b1, k); });
    arrived_b(fb[1]);
    if constexpr (LAST == 0) hand_over(c4, c2);
    else if constexpr (LAST == 1) hand_over(c2, c1);
    multiply(acc[1][1], fa[Q], fb[1], [&] { if constexpr (LAST == 0) fetch_b(1, S); }, [&](auto k) { if constexpr (LAST < 2) read_b(fb[0], b0_next, k); });
    if constexpr (LAST < 2) arrived_b(fb[0]);
    if constexpr (LAST == 0) hand_over(c3, c3);
    else if constexpr (LAST == 1) hand_over(c1, c1);
    multiply(acc[0][1], fa[S], fb[1], [&] { if (LAST == 0 && third) fetch_b(0, Q); }, [&](auto k) { if constexpr (LAST < 2) read_a(fa[Q], a0_next, k); });
    if constexpr (LAST < 2) arrived_a(fa[Q]);
  };

  fetch_b(0, 0); fetch_a(0, 0); fetch_a(1, 0); fetch_b(1, 0);
  fetch_b(0, 1); fetch_a(0, 1); fetch_a(1, 1); fetch_b(1, 1);
  hand_over(c3, c3);
  static_for<KK>([&](auto k) { read_b(fb[0], c0, k); });
  static_for<KK>([&](auto k) { read_a(fa[0], c0, k); });
  arrived_b(fb[0]);
  arrived_a(fa[0]);
  __builtin_amdgcn_s_barrier();
  if (KT > 2) fetch_b(0, 0);
  for (int kt = 0; kt + 2 < KT; kt += 2) {  // an even number of k-steps
    k_step(c0, c0, true);
    k_step(c1, c0, kt + 4 < KT);
  }
  k_step(c0, c1, false);
  k_step(c1, c2, false);
  if constexpr (PAIR) {
#pragma unroll
    for (int i = 0; i < 4 * NT; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i / (2 * NT)][i / NT % 2][0][i % NT][r] += acc[i / (2 * NT)][i / NT % 2][1][i % NT][r];
  }

  // epilogue: out = acc * (alpha * col_scale[n]) + beta * (col_vec[n] + row_vec[m]) + bias[n]
  const float alpha = e.alpha ? *e.alpha : 1.f;
  const float beta = (e.beta ? *e.beta : 0.f) + e.beta_alpha * alpha;
  auto write_out = [&](auto inside, auto with_row, auto with_gelu, auto apart, auto with_range) {
    auto write_group = [&](auto j_, int n, MinMax& range) {
      constexpr int j = decltype(j_)::value;
      const float cs = alpha * (e.col_scale ? e.col_scale[n] : 1.f);
      float cb = e.bias ? e.bias[n] : 0.f;
      const float cv = (e.beta && e.col_vec) ? e.col_vec[n] : 0.f;
      if (!decltype(apart)::value && e.beta && e.col_vec) cb += beta * cv;
      int shift = 0;
      if constexpr (I8 && decltype(apart)::value) shift = e.row_codes ? e.code_shift * e.row_codes[n] : 0;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int mb = m0 + i * HA + wm * 32 + 4 * (lane >> 5);
        TO* __restrict__ out = C + (size_t)mb * ldc + n;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int dm = 8 * (r >> 2) + (r & 3);
          if (!decltype(inside)::value && mb + dm >= M) continue;
          auto sum = acc[i][j / NT][0][j % NT][r];
          if constexpr (I8 && decltype(apart)::value) sum += shift;
          const float a = (float)sum;
          float v;
          if constexpr (decltype(apart)::value) {
            const float t = decltype(with_row)::value ? cv + e.row_vec[mb + dm] : cv;
            v = epilogue_apart(a, cs, e.beta != nullptr, beta, t, e.bias != nullptr, cb);
          } else {
            v = a * cs + cb;
            if constexpr (decltype(with_row)::value) v += beta * e.row_vec[mb + dm];
          }
          if constexpr (decltype(with_gelu)::value) v = gelu_t<TO>(round_to<TO>(v));
          if constexpr (decltype(with_range)::value) range.add(v);
          if constexpr (POST != POST_NONE) stf(reinterpret_cast<bf16_t*>(smem_quad), (mb - m0 + dm) * post_stride<BN> + n - n0, v);
          else stf(out, (size_t)dm * ldc, v);
        }
      }
    };
    if constexpr (decltype(with_range)::value) __syncthreads();  // nobody reads operands any more
    static_for<2 * NT>([&](auto j) {
      const int n = n0 + j.value / NT * HN + wn * WN + j.value % NT * 32;
      MinMax range;
      if (decltype(inside)::value || n + (lane & 31) < N) write_group(j, n + (lane & 31), range);
      if constexpr (decltype(with_range)::value) {
        // each group's range leaves the registers before the next group (93 registers spilled without the barrier)
        put_range(reinterpret_cast<RangeSlot*>(smem_quad), wave * 2 * NT + j.value, range, n, e, lane);
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    if constexpr (decltype(with_range)::value) store_ranges(reinterpret_cast<RangeSlot*>(smem_quad), 16 * NT, e, N);
  };
  const bool row_term = e.beta && e.row_vec;
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  if constexpr (POST != POST_NONE) {
    static_assert(!EDGE && !PAIR && !AT, "whole tiles");
    __syncthreads();  // nobody reads operands any more
    write_out(yes, no, no, no, no);
    __syncthreads();
    post_tile<POST, BM, BN, 512>(smem_quad, e, C, ldc, m0, n0);
    return;
  }
  auto choose = [&](auto inside) {
    if constexpr (EDGE && I8) {
      if (e.apart) return write_out(inside, no, no, yes, no);
    }
    if constexpr (EDGE && !AT && !BT && !I8) {
      if (e.apart && e.gelu) return row_term ? write_out(inside, yes, yes, yes, no) : write_out(inside, no, yes, yes, no);
      if (e.apart) return row_term ? write_out(inside, yes, no, yes, no) : write_out(inside, no, no, yes, no);
    }
    if constexpr (!AT && !BT && !I8 && !PAIR) {
      if (e.range) return e.gelu ? write_out(inside, no, yes, no, yes) : write_out(inside, no, no, no, yes);
    }
    if (e.gelu) return row_term ? write_out(inside, yes, yes, no, no) : write_out(inside, no, yes, no, no);
    return row_term ? write_out(inside, yes, no, no, no) : write_out(inside, no, no, no, no);
  };
  // (a test per stored value costs a tenth of 4096 x 4096 x 1024)
  if (!EDGE || (m0 + BM <= M && n0 + BN <= N)) choose(yes);
  else choose(no);
}

template <int BM, bool AT, bool BT, class TO, bool I8, bool EDGE, bool PAIR, int POST>
__global__ __launch_bounds__(512, 1) void gemm_quad_k(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ B, int ldb,
                                                      TO* __restrict__ C, int ldc, int M, int N, int K, Epilogue e, int tiles_m, int tiles_n) {
  int tm, tn;
  tile_of_block(tiles_m, tiles_n, tm, tn);
  quad_tile<BM, AT, BT, TO, I8, EDGE, PAIR, POST>(A, lda, B, ldb, C, ldc, M, N, K, e, tm, tn);
}

// The weight gradients of a layer in one launch, at most one tile a compute unit.  Products of
// their own took 64 x 64 or 128 x 128 tiles or slices of the contraction to fill the chip, with up to four times the operand
// bytes per flop; the step has another stream's kernels for the units that one round of large tiles leaves over.
// Steps, us: six layers of 1024 over 32 x 128 tokens
// 4480 -> 4261, 16 x 384 6490 -> 6133, three of 768 over 32 x 128 1720 -> 1652, six of 320 over 4096 1774 -> 1636.
struct QuadJob {
  WgradJob j;
  int tiles_m, tiles_n, first;  // its tiles, and how many the jobs before it have
};
struct QuadJobs { QuadJob job[kMaxWgradJobs]; };
template <int BM, bool EDGE>
__global__ __launch_bounds__(512, 1) void gemm_quad_wgrads_k(QuadJobs jobs, int njobs, int K) {
  // each XCD takes a contiguous range of all tiles (see tile_of_block); what eight do not divide goes in order
  int pid = blockIdx.x;
  const int each = (int)gridDim.x >> 3;
  if (pid < 8 * each) pid = (pid & 7) * each + (pid >> 3);
  int i = 0;
  while (i + 1 < njobs && pid >= jobs.job[i + 1].first) ++i;
  const QuadJob& q = jobs.job[i];
  int tm, tn;
  tile_of_index(pid - q.first, q.tiles_m, q.tiles_n, tm, tn);
  Epilogue e;
  e.alpha = q.j.alpha;
  quad_tile<BM, true, true, float, false, EDGE, false>((const bf16_t*)q.j.dy, q.j.M, (const bf16_t*)q.j.x, q.j.N, q.j.dw, q.j.N, q.j.M, q.j.N, K, e, tm, tn);
}

// whole stages, an even number of them
static bool quad_ok(int K) { return K % (2 * kBK) == 0; }

// LDS of a kernel of BM x 256 tiles, beyond what is allowed without asking
template <int BM, int POST = POST_NONE>
static size_t quad_lds(const void* kernel, std::atomic<int>& configured_dev) {
  constexpr size_t stages = 2 * (BM + 256) * 128, lds = POST != POST_NONE ? std::max(stages, BM * post_stride<256> * sizeof(bf16_t) + post_table<POST>) : stages;
  static_assert(lds <= 160 * 1024, "LDS of a compute unit");
  int dev = -1;
  (void)hipGetDevice(&dev);
  if (dev != configured_dev.load()) {
    (void)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    configured_dev.store(dev);
  }
  return lds;
}

template <int BM, bool AT, bool BT, class TO, bool I8, bool EDGE, bool PAIR = false, int POST = POST_NONE>
static void launch_quad(const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K, const Epilogue& e, hipStream_t st) {
  constexpr int BN = 256;
  static std::atomic<int> configured_dev{-1};
  const size_t lds = quad_lds<BM, POST>(reinterpret_cast<const void*>(&gemm_quad_k<BM, AT, BT, TO, I8, EDGE, PAIR, POST>), configured_dev);
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  if (e.blocks) *e.blocks = tiles_m * tiles_n;
  if (e.row_tiles) *e.row_tiles = tiles_m;
  MREM_LAUNCH((gemm_quad_k<BM, AT, BT, TO, I8, EDGE, PAIR, POST>), dim3(tiles_m * tiles_n), dim3(512), lds, st, (const bf16_t*)A, lda, (const bf16_t*)B, ldb, (TO*)C,
              ldc, M, N, K, e, tiles_m, tiles_n);
}

template <int BM, bool EDGE>
static void launch_quad_wgrads(const WgradJob* jobs, int njobs, int K, hipStream_t st) {
  static std::atomic<int> configured_dev{-1};
  const size_t lds = quad_lds<BM>(reinterpret_cast<const void*>(&gemm_quad_wgrads_k<BM, EDGE>), configured_dev);
  QuadJobs q{};
  int tiles = 0;
  for (int i = 0; i < njobs; ++i) {
    q.job[i] = QuadJob{jobs[i], (jobs[i].M + BM - 1) / BM, (jobs[i].N + 255) / 256, tiles};
    tiles += q.job[i].tiles_m * q.job[i].tiles_n;
  }
  hipLaunchKernelGGL((gemm_quad_wgrads_k<BM, EDGE>), dim3(tiles), dim3(512), lds, st, q, njobs, K);
}

}  // namespace mrem
