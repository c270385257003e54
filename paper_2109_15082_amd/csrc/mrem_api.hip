// C ABI of the MREM module step (Algorithm 2) and the host-side orchestration of
// its kernels.  Host code only enqueues kernels on the caller's stream; all
// arithmetic of the method runs on the device.
#include "../../include/mrem.h"
#include "mrem_kernels.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

using namespace mrem;

static thread_local std::string g_err;

struct mrem_ctx {
  mrem_config cfg;
  int dt, L, H, F, nh, d;
  int64_t foff[MREM_F_COUNT], fsize[MREM_F_COUNT];
  int64_t layer_stride;
  int64_t tc_off[4], tc_layer_stride;  // teacher cache, in elements
  int wN[4], wK[4];                    // the four linear layers [N,K]
  std::string err;
  // side stream for the teacher's forward pass of a step (created on the first step, on the
  // device that is current then; default priority) and the two events of its fork and join
  hipStream_t side = nullptr;
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;
  hipEvent_t ev_codes = nullptr;     // the side stream has prepared the weights of the layers above the first
  std::vector<hipEvent_t> ev_layer;  // "the backward pass of layer l is enqueued", one per layer
  std::vector<hipEvent_t> ev_ready;  // [4 * l + i]: the output gradient of linear layer i of layer l is written
  std::vector<hipEvent_t> ev_done;   // [4 * l + i]: its weight-gradient product has read it
  int side_device = -1;
  GemmProfile prof;                // per-launch timing of the matrix products (measurement aid)
  int32_t* nonfinite_flag = nullptr;  // device, caller-owned, optional
};

static mrem_status fail(const mrem_ctx* ctx, mrem_status st, const std::string& msg) {
  g_err = msg;
  if (ctx) const_cast<mrem_ctx*>(ctx)->err = msg;
  return st;
}

static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

extern "C" const char* mrem_last_error(const mrem_ctx* ctx) { return ctx ? ctx->err.c_str() : g_err.c_str(); }

static void count_contexts(int more);

extern "C" mrem_status mrem_create(const mrem_config* cfg, mrem_ctx** out) {
  if (!cfg || !out) return fail(nullptr, MREM_EINVAL, "mrem_create: null argument");
  const mrem_config& c = *cfg;
  if (c.n_layers < 1 || c.n_layers > 32) return fail(nullptr, MREM_ESHAPE, "n_layers must be in 1..32");
  if (c.hidden < 8 || c.hidden % 8 || c.hidden > 2048) return fail(nullptr, MREM_ESHAPE, "hidden must be a multiple of 8, <= 2048");
  if (c.ffn < 8 || c.ffn % 8) return fail(nullptr, MREM_ESHAPE, "ffn must be a multiple of 8");
  if (c.n_heads < 1 || c.hidden % c.n_heads) return fail(nullptr, MREM_ESHAPE, "hidden must be divisible by n_heads");
  const int d = c.hidden / c.n_heads;
  if (d % 8 || d > 128) return fail(nullptr, MREM_ESHAPE, "head dimension must be a multiple of 8, <= 128");
  if (c.max_seq < 1 || c.max_seq > 512) return fail(nullptr, MREM_ESHAPE, "max_seq must be in 1..512");
  if (c.max_batch < 1) return fail(nullptr, MREM_ESHAPE, "max_batch must be >= 1");
  if (!(c.w_bits == 0 || (c.w_bits >= 2 && c.w_bits <= 8))) return fail(nullptr, MREM_EINVAL, "w_bits must be 0 or 2..8");
  if (!(c.a_bits == 0 || (c.a_bits >= 2 && c.a_bits <= 8))) return fail(nullptr, MREM_EINVAL, "a_bits must be 0 or 2..8");
  if (c.act_dtype != MREM_BF16 && c.act_dtype != MREM_FP32) return fail(nullptr, MREM_EINVAL, "act_dtype must be MREM_BF16 or MREM_FP32");
  if (c.per_channel != 0 && c.per_channel != 1) return fail(nullptr, MREM_EINVAL, "per_channel must be 0 or 1");
  mrem_ctx* x = new mrem_ctx();
  x->cfg = c;
  x->dt = c.act_dtype == MREM_BF16 ? DT_BF16 : DT_F32;
  x->L = c.n_layers; x->H = c.hidden; x->F = c.ffn; x->nh = c.n_heads; x->d = d;
  const int64_t H = x->H, F = x->F;
  const int64_t sizes[MREM_F_COUNT] = {3 * H * H, H * H, F * H, H * F, 3 * H, H, H, H, F, H, H, H, 3 * H, H, F, H, 8, 8};
  int64_t off = 0;
  for (int f = 0; f < MREM_F_COUNT; ++f) { x->foff[f] = off; x->fsize[f] = sizes[f]; off += sizes[f]; }
  x->layer_stride = off;
  x->wN[0] = 3 * H; x->wK[0] = H; x->wN[1] = H; x->wK[1] = H; x->wN[2] = F; x->wK[2] = H; x->wN[3] = H; x->wK[3] = F;
  int64_t t = 0;
  for (int i = 0; i < 4; ++i) { x->tc_off[i] = t; t += (int64_t)x->wN[i] * x->wK[i]; }
  x->tc_layer_stride = t;
  count_contexts(1);
  *out = x;
  return MREM_OK;
}

// Releases the side stream and its events (null handles are skipped, so it also cleans up after
// a creation that failed half way).
static void release_side(mrem_ctx* ctx) {
  if (ctx->side) (void)hipStreamSynchronize(ctx->side);
  for (hipEvent_t* e : {&ctx->ev_fork, &ctx->ev_join, &ctx->ev_codes}) {
    if (*e) (void)hipEventDestroy(*e);
    *e = nullptr;
  }
  for (std::vector<hipEvent_t>* evs : {&ctx->ev_layer, &ctx->ev_ready, &ctx->ev_done}) {
    for (hipEvent_t e : *evs)
      if (e) (void)hipEventDestroy(e);
    evs->clear();
  }
  if (ctx->side) (void)hipStreamDestroy(ctx->side);
  ctx->side = nullptr;
  ctx->side_device = -1;
}
// All or nothing: on failure nothing is left behind and the next call tries again.
static bool create_side(mrem_ctx* ctx, int dev) {
  bool ok = hipStreamCreateWithFlags(&ctx->side, hipStreamNonBlocking) == hipSuccess &&
            hipEventCreateWithFlags(&ctx->ev_fork, hipEventDisableTiming) == hipSuccess &&
            hipEventCreateWithFlags(&ctx->ev_join, hipEventDisableTiming) == hipSuccess &&
            hipEventCreateWithFlags(&ctx->ev_codes, hipEventDisableTiming) == hipSuccess;
  ctx->ev_layer.assign((size_t)ctx->L, nullptr);
  ctx->ev_ready.assign((size_t)ctx->L * 4, nullptr);
  ctx->ev_done.assign((size_t)ctx->L * 4, nullptr);
  for (std::vector<hipEvent_t>* evs : {&ctx->ev_layer, &ctx->ev_ready, &ctx->ev_done})
    for (hipEvent_t& e : *evs) ok = ok && hipEventCreateWithFlags(&e, hipEventDisableTiming) == hipSuccess;
  if (!ok) {
    release_side(ctx);
    (void)hipGetLastError();  // the failure is reported by the caller's return value
    return false;
  }
  ctx->side_device = dev;
  return true;
}

// Streams for the full-precision pass of mrem_module_forward: one for each stream that such calls come from, whichever their
// contexts.  What one caller's stream holds is in order anyway, so nobody waits for another caller's work, and a new context
// finds the stream of its caller's earlier ones (creating a stream takes 0.1 to 3.5 ms, a call over a sentence 0.25).  There
// are up to kPassStreams; a further caller takes over one that has nothing left to do, or gets none.  With the last context
// they are given back but for the one used last, which the next context's first call finds.  (Not a step's side stream, which
// may be part of a capture.)
struct PassStream {
  hipStream_t caller, st;
  std::thread::id thread;  // of the caller where its handle means another stream in each thread
  int dev;
  hipEvent_t fork, join;
  std::mutex lock;  // held from the recording of an event to the wait for it: several threads may call on one stream
  int calls = 0;    // that are using it now
  uint64_t used = 0;
};
constexpr int kPassStreams = 16;
struct PassPool {
  std::mutex lock;
  std::vector<PassStream*> all;
  int contexts = 0;
  uint64_t used = 0;
};
static PassPool& pass_pool() {
  static PassPool* const pool = new PassPool;  // never destroyed: the runtime may be gone before this library's statics
  return *pool;
}

static bool pass_idle(const PassStream* p) {
  if (p->calls) return false;
  const bool idle = hipStreamQuery(p->st) == hipSuccess;
  (void)hipGetLastError();
  return idle;
}
static PassStream* new_pass_stream(int dev) {
  hipStream_t st = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
  if (hipStreamCreateWithFlags(&st, hipStreamNonBlocking) != hipSuccess || hipEventCreateWithFlags(&fork, hipEventDisableTiming) != hipSuccess ||
      hipEventCreateWithFlags(&join, hipEventDisableTiming) != hipSuccess) {
    if (fork) (void)hipEventDestroy(fork);
    if (st) (void)hipStreamDestroy(st);
    (void)hipGetLastError();
    return nullptr;
  }
  PassStream* p = new PassStream;
  p->st = st; p->dev = dev; p->fork = fork; p->join = join;
  return p;
}
// null: the passes run one after the other
static PassStream* take_pass_stream(hipStream_t caller) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return nullptr;
  const std::thread::id thread = caller == hipStreamPerThread ? std::this_thread::get_id() : std::thread::id();
  PassPool& pool = pass_pool();
  const std::lock_guard<std::mutex> hold(pool.lock);
  PassStream* found = nullptr;
  for (PassStream* p : pool.all)
    if (p->caller == caller && p->dev == dev && p->thread == thread) found = p;
  if (!found) {
    if (pool.all.size() < kPassStreams) {
      if ((found = new_pass_stream(dev))) pool.all.push_back(found);
    } else {
      for (PassStream* p : pool.all)
        if (p->dev == dev && (!found || p->used < found->used) && pass_idle(p)) found = p;
    }
    if (!found) return nullptr;
    found->caller = caller;
    found->thread = thread;
  }
  ++found->calls;
  found->used = ++pool.used;
  return found;
}
static void leave_pass_stream(PassStream* p) {
  const std::lock_guard<std::mutex> hold(pass_pool().lock);
  --p->calls;
}
static void count_contexts(int more) {
  PassPool& pool = pass_pool();
  const std::lock_guard<std::mutex> hold(pool.lock);
  if ((pool.contexts += more) > 0) return;
  std::vector<PassStream*> kept;
  for (PassStream* p : pool.all) {
    if (p->used == pool.used || !pass_idle(p)) {
      kept.push_back(p);
      continue;
    }
    (void)hipEventDestroy(p->fork);
    (void)hipEventDestroy(p->join);
    (void)hipStreamDestroy(p->st);
    delete p;
  }
  pool.all.swap(kept);
}

extern "C" void mrem_destroy(mrem_ctx* ctx) {
  if (!ctx) return;
  release_side(ctx);
  delete ctx;
  count_contexts(-1);
}
extern "C" int64_t mrem_param_count(const mrem_ctx* ctx) { return ctx ? ctx->layer_stride * ctx->L : -1; }
extern "C" int64_t mrem_teacher_count(const mrem_ctx* ctx) { return mrem_param_count(ctx); }
extern "C" int64_t mrem_param_offset(const mrem_ctx* ctx, int32_t layer, int32_t field) {
  if (!ctx || layer < 0 || layer >= ctx->L || field < 0 || field >= MREM_F_COUNT) return -1;
  return ctx->layer_stride * layer + ctx->foff[field];
}
extern "C" int64_t mrem_param_size(const mrem_ctx* ctx, int32_t field) {
  if (!ctx || field < 0 || field >= MREM_F_COUNT) return -1;
  return ctx->fsize[field];
}
extern "C" size_t mrem_teacher_cache_bytes(const mrem_ctx* ctx) {
  return ctx ? (size_t)(ctx->tc_layer_stride * ctx->L) * dt_size(ctx->dt) : 0;
}

// ------------------------------------------------------------------------------
// workspace plan
// ------------------------------------------------------------------------------
namespace {

struct Bump {
  size_t off = 0;
  size_t take(size_t bytes) {
    const size_t o = off;
    off += (bytes + 255) & ~size_t(255);
    return o;
  }
};

struct LayerWs {
  size_t wcodes[4], what[4], zcorr[4];
  size_t wcodes8[4], xcodes8, ctxcodes8, x1codes8, gcodes8;  // int8 copies of the codes the forward products read
  size_t xcodes, qkv, qkvcodes, ctx, ctxcodes, o, x1, x1codes, u, gcodes, y, mu1, rstd1, mu2, rstd2, stat_m, stat_l;
};

struct Plan {
  LayerWs lw[32];
  // teacher scratch
  size_t t_qkv, t_ctx, t_o, t_x1, t_g, t_y, t_mu, t_rstd;
  // backward scratch
  size_t dr2, dr1, dxh, dx1h, dch, dc, dgh, du, dqkvh, dqkv, s_da, s_ph, partials, partials_per_layer, grads, pmax, xmix;
  size_t total;
};

// The forward products of the quantized module run on int8 codes (exact int32 accumulation) when
// the storage type is bf16 and both bit widths are between 1 and 8, for any number of tokens.  Where these are no whole tiles
// it takes half the k-steps of bf16 codes: steps of three layers of 768 over 30 x 77 tokens 1254 -> 1215 us, both passes of one over 23
// tokens 231 -> 222.
bool i8_config(const mrem_ctx* c) {
  return c->dt == DT_BF16 && c->cfg.a_bits >= 1 && c->cfg.a_bits <= 8 && c->cfg.w_bits >= 1 && c->cfg.w_bits <= 8 && c->H % 128 == 0 &&
         c->F % 128 == 0;
}
// ... and no sum can leave int32: the largest codes are the GELU's, recentred in whole tiles (8 bits: ffn <= 132104), added up
// before that in others (ffn <= 66311), where the sums of the weight codes' rows, formed in fp32, have to be exact too.
bool i8_products(const mrem_ctx* c, int64_t T) {
  if (!i8_config(c)) return false;
  const int a = 1 << (c->cfg.a_bits - 1), w = (1 << (c->cfg.w_bits - 1)) - 1;
  return T % 128 == 0 ? i8_sums_fit(c->F, a, w) : i8_sums_fit(c->F, 2 * a - 1, w) && (int64_t)c->F * w <= 1 << 24;
}

Plan make_plan(const mrem_ctx* c, int B, int S) {
  Plan p;
  Bump b;
  const size_t T = (size_t)B * S, H = c->H, F = c->F, es = dt_size(c->dt);
  for (int l = 0; l < c->L; ++l) {
    LayerWs& w = p.lw[l];
    for (int i = 0; i < 4; ++i) {
      const size_t n = (size_t)c->wN[i] * c->wK[i];
      w.wcodes[i] = b.take(n * es);
      w.what[i] = b.take(n * es);
      w.zcorr[i] = b.take((size_t)c->wN[i] * 4);
      w.wcodes8[i] = b.take(i8_config(c) ? n : 0);
    }
    w.xcodes8 = b.take(i8_config(c) ? T * H : 0); w.ctxcodes8 = b.take(i8_config(c) ? T * H : 0);
    w.x1codes8 = b.take(i8_config(c) ? T * H : 0); w.gcodes8 = b.take(i8_config(c) ? T * F : 0);
    w.xcodes = b.take(T * H * es); w.qkv = b.take(T * 3 * H * es); w.qkvcodes = b.take(T * 3 * H * es);
    w.ctx = b.take(T * H * es); w.ctxcodes = b.take(T * H * es); w.o = b.take(T * H * es);
    w.x1 = b.take(T * H * es); w.x1codes = b.take(T * H * es); w.u = b.take(T * F * es); w.gcodes = b.take(T * F * es);
    w.y = b.take(T * H * es);
    w.mu1 = b.take(T * 4); w.rstd1 = b.take(T * 4); w.mu2 = b.take(T * 4); w.rstd2 = b.take(T * 4);
    w.stat_m = b.take((size_t)B * c->nh * S * 4); w.stat_l = b.take((size_t)B * c->nh * S * 4);
  }
  p.t_qkv = b.take(T * 3 * H * es); p.t_ctx = b.take(T * H * es); p.t_o = b.take(T * H * es); p.t_x1 = b.take(T * H * es);
  p.t_g = b.take(T * F * es); p.t_y = b.take(T * H * es); p.t_mu = b.take(T * 4); p.t_rstd = b.take(T * 4);
  p.dr2 = b.take(T * H * es); p.dr1 = b.take(T * H * es); p.dxh = b.take(T * H * es);
  p.dx1h = b.take(T * H * es); p.dch = b.take(T * H * es); p.dc = b.take(T * H * es);
  p.dgh = b.take(T * F * es); p.du = b.take(T * F * es); p.dqkvh = b.take(T * 3 * H * es); p.dqkv = b.take(T * 3 * H * es);
  const size_t s_pad = ((size_t)S + 31) / 32 * 32;
  const size_t pp = (size_t)B * c->nh * s_pad * s_pad;
  // scalar attention keeps two fp32 matrices a head; the matrix-core kernels use less of it (see attn_bwd_mfma)
  p.s_da = b.take(pp * 4); p.s_ph = b.take(pp * 4);
  p.pmax = b.take((size_t)B * c->nh * S * 4);
  // first-stage partial sums of one layer's backward pass (all of them stay until the single
  // second-stage launch at the end of the backward pass): two LayerNorms, two bias column sums,
  // the elementwise kernels (at most 2048 blocks, up to 3 values each) and the attention rows
  // (in the forward pass, the sums of the weight codes' rows)
  size_t np = 2 * (size_t)ln_bwd_parts((int)T) * (3 * H + 2) + (size_t)kColMaxParts * (F + 3 * H) + 8 * 2048 + (size_t)B * c->nh * S;
  static_assert(8 * 3 * kCalibParts <= 8 * 2048, "the partial ranges of a layer's eight quantizers fit too");
  np = (np + 63) & ~size_t(63);
  p.partials_per_layer = np;
  p.partials = b.take(np * 4 * c->L);
  p.grads = b.take((size_t)mrem_param_count(c) * 4);
  p.xmix = b.take(T * H * es);  // Eq. 4: the mixed module input, when a step is given a lambda > 0
  p.total = b.off;
  return p;
}

struct Run {
  const mrem_ctx* c;
  Plan p;
  char* ws;
  hipStream_t st;
  int B, S, T;
  const int32_t* seqlens;
  GemmProfile* prof = nullptr;
  template <class X = void> X* at(size_t off) const { return reinterpret_cast<X*>(ws + off); }
  bool i8() const { return i8_products(c, T); }
  int8_t* at8(size_t off) const { return i8() ? reinterpret_cast<int8_t*>(ws + off) : nullptr; }
};

// One launch of a bandwidth-bound kernel; while a context's timing is on, the launch carries an event pair and
// is recorded with its algorithmic bytes (what the kernel must read and write at least) under `label`.
template <class F>
void timed(const Run& r, const char* label, double bytes, F&& launch) {
  if (!r.prof || !r.prof->on) { launch(); return; }
  GemmRecord rec;
  rec.flops = bytes; rec.cls = 2; rec.label = label;
  (void)hipEventCreate(&rec.e0);
  (void)hipEventCreate(&rec.e1);
  tl_launch_events.e0 = rec.e0;
  tl_launch_events.e1 = rec.e1;
  launch();
  tl_launch_events = LaunchEvents();
  r.prof->recs.push_back(rec);
}

// Second-stage reductions of a backward pass, collected while the first-stage kernels are enqueued.
struct Reductions {
  std::vector<ReduceJob> jobs;
  float* next = nullptr;  // bump pointer into the partials area
  float* take(size_t n) { float* p = next; next += (n + 63) & ~size_t(63); return p; }
  void add(const float* partials, int nparts, int width, int begin, int len, float* out, float scale = 1.f) {
    ReduceJob j;
    j.partials = partials; j.nparts = nparts; j.width = width; j.begin = begin; j.len = len; j.out = out; j.scale = scale;
    jobs.push_back(j);
  }
};

QArg make_q(const mrem_ctx* c, const float* params, int layer, int idx) {
  QArg q;
  q.on = c->cfg.a_bits > 0;
  if (!q.on) return q;
  const float* base = params + c->layer_stride * layer;
  q.s = base + c->foff[MREM_F_S_A] + idx;
  const bool uns = (idx == 3 || idx == 7);
  q.z = (idx == 7) ? base + c->foff[MREM_F_Z_A] + idx : nullptr;
  if (uns) { q.qn = 0.f; q.qp = (float)((1 << c->cfg.a_bits) - 1); }
  else { q.qp = (float)((1 << (c->cfg.a_bits - 1)) - 1); q.qn = -q.qp; }
  return q;
}

AttnQ make_attn_q(const mrem_ctx* c, const float* params, int layer, bool quant) {
  AttnQ a;
  if (!quant) return a;
  a.q = make_q(c, params, layer, 1); a.k = make_q(c, params, layer, 2); a.p = make_q(c, params, layer, 3);
  a.v = make_q(c, params, layer, 4); a.c = make_q(c, params, layer, 5);
  return a;
}

const int kWField[4] = {MREM_F_W_QKV, MREM_F_W_O, MREM_F_W_1, MREM_F_W_2};
const int kBField[4] = {MREM_F_B_QKV, MREM_F_B_O, MREM_F_B_1, MREM_F_B_2};
const int kSField[4] = {MREM_F_SW_QKV, MREM_F_SW_O, MREM_F_SW_1, MREM_F_SW_2};
const int kInQuant[4] = {0, 5, 6, 7};  // activation quantizer feeding each linear layer

// sums of the weight codes of linear layer i's rows; they wait in the layer's partial sums, which only the backward pass forms
int* row_codes(const Run& r, int l, int i) {
  int* at = r.at<int>(r.p.partials) + r.p.partials_per_layer * l;
  for (int k = 0; k < i; ++k) at += r.c->wN[k];
  return at;
}
// quantized linear layer i of layer l: out = codes_in * wcodes^T with the steps in the epilogue; `post`: what else its kernel does
void student_linear(const Run& r, const float* params, int l, int i, const void* in_codes, const int8_t* in_codes8, void* out,
                    const Epilogue& post = Epilogue()) {
  const mrem_ctx* c = r.c;
  const float* base = params + c->layer_stride * l;
  Epilogue e = post;
  const QArg q = make_q(c, params, l, kInQuant[i]);
  if (q.on) e.alpha = q.s;
  if (c->cfg.w_bits > 0) e.col_scale = base + c->foff[kSField[i]];
  if (q.on && q.z) { e.beta = q.z; e.col_vec = r.at<float>(r.p.lw[l].zcorr[i]); }
  e.bias = base + c->foff[kBField[i]];
  e.chain = !(q.on && c->cfg.w_bits > 0);  // sums of integer codes are exact in any order
  if (r.i8() && in_codes8) {
    // unsigned codes (GELU output) are stored recentred by half their range; the epilogue adds that back, in whole tiles to the
    // result, in others to the sum of codes, which then is that of a product of bf16 codes
    if (q.z && r.T % 128 == 0) e.beta_alpha = 0.5f * (q.qp + 1.f);
    else if (q.z) { e.row_codes = row_codes(r, l, i); e.code_shift = (int)(0.5f * (q.qp + 1.f)); }
    gemm_i8(in_codes8, c->wK[i], r.at8(r.p.lw[l].wcodes8[i]), c->wK[i], out, c->wN[i], r.T, c->wN[i], c->wK[i], e, r.st, r.prof);
    return;
  }
  gemm_nt(c->dt, in_codes, c->wK[i], r.at(r.p.lw[l].wcodes[i]), c->wK[i], out, c->wN[i], r.T, c->wN[i], c->wK[i], e, r.st, r.prof);
}

// (layers [l0, l1); l1 < 0: to the last layer; backward: also the dequantized copy that the input gradients read)
void prepare_weights(const Run& r, const float* params, bool backward, int l0 = 0, int l1 = -1) {
  const mrem_ctx* c = r.c;
  if (l1 < 0) l1 = c->L;
  if (l0 >= l1) return;
  std::vector<WeightJob> jobs;
  jobs.reserve((size_t)(l1 - l0) * 4);
  for (int l = l0; l < l1; ++l) {
    const float* base = params + c->layer_stride * l;
    for (int i = 0; i < 4; ++i) {
      WeightJob j;
      j.w = base + c->foff[kWField[i]]; j.sw = base + c->foff[kSField[i]];
      j.codes8 = r.at8(r.p.lw[l].wcodes8[i]);
      // (the forward reads one or the other; beside int8 ones of a call that has no whole tiles they are left for inspection)
      j.codes = j.codes8 && r.T % 128 == 0 ? nullptr : r.at(r.p.lw[l].wcodes[i]);
      j.row_codes = j.codes8 ? row_codes(r, l, i) : nullptr;
      j.what = backward ? r.at(r.p.lw[l].what[i]) : nullptr; j.zcorr = r.at<float>(r.p.lw[l].zcorr[i]);
      j.N = c->wN[i]; j.K = c->wK[i];
      jobs.push_back(j);
    }
  }
  double nw = 0;
  for (const WeightJob& j : jobs) nw += (double)j.N * j.K;
  // fp32 master in; codes (int8, or the storage type) and the dequantized copy out
  timed(r, "weight_codes_k", nw * (4 + (r.i8() ? 1 : 0) + (r.i8() && r.T % 128 == 0 ? 0 : dt_size(c->dt)) + (backward ? dt_size(c->dt) : 0)),
        [&] { weight_prepare(c->dt, jobs.data(), (int)jobs.size(), c->cfg.w_bits, r.st); });
}

// Layers [l0, l1) of the quantized module (l1 < 0: to the last layer).  backward: with what only a backward pass reads, the codes
// in the storage type (where the products read int8 ones) and the first feed-forward projection's output (where its kernel forms
// the codes of its GELU).  Without it both passes of six layers of 1024 over 4096 tokens take 1575 us, 1740 with it.
// mix_fp != null (with 0 < lambda <= 1): the module input is lambda * mix_fp + (1 - lambda) * x_in (Eq. 4), formed and
// stored in x_q (a workspace buffer) by the kernel that quantizes the first layer's input.
void student_forward(const Run& r, const float* params, const void* x_q, void* per_layer_q, bool backward, int l0 = 0, int l1 = -1,
                     const void* mix_fp = nullptr, const void* mix_in = nullptr, float lambda = 0.f) {
  const mrem_ctx* c = r.c;
  const size_t es = dt_size(c->dt);
  const int H = c->H, F = c->F, T = r.T;
  const size_t slice = (size_t)T * H * es;
  if (l1 < 0) l1 = c->L;
  const bool only8 = !backward && r.i8();
  auto codes = [&](size_t off) { return only8 ? nullptr : r.at(off); };
  const double es_codes = only8 ? 1 : es + (r.i8() ? 1 : 0);
  for (int l = l0; l < l1; ++l) {
    const LayerWs& w = r.p.lw[l];
    const float* base = params + c->layer_stride * l;
    const void* x = l == 0 ? x_q : (const char*)per_layer_q + slice * (l - 1);
    void* f = (char*)per_layer_q + slice * l;
    // every code tensor that feeds a linear layer is also written as int8 when the int8 products are in use
    // (the input codes of layers 1.. come from the second LayerNorm of the layer before)
    if (l == 0 && mix_fp)
      mix_quantize(c->dt, mix_fp, mix_in, lambda, 1.f - lambda, const_cast<void*>(x), r.at(w.xcodes), (int64_t)T * H, make_q(c, params, l, 0), r.st,
                   r.at8(w.xcodes8));
    else if (l == 0)
      timed(r, "act_quantize_k", (double)T * H * (es + es_codes),
            [&] { act_quantize(c->dt, x, codes(w.xcodes), (int64_t)T * H, make_q(c, params, l, 0), r.st, r.at8(w.xcodes8)); });
    const AttnQ aq = make_attn_q(c, params, l, true);
    if (r.i8() && post_codes_ok(T, 3 * H, H)) {
      Epilogue post;
      post.post = POST_QKV; post.post_q = aq.q; post.post_q1 = aq.k; post.post_q2 = aq.v; post.post_cols = H; post.post_out = r.at(w.qkvcodes);
      student_linear(r, params, l, 0, r.at(w.xcodes), r.at8(w.xcodes8), r.at(w.qkv), post);
    } else {
      student_linear(r, params, l, 0, r.at(w.xcodes), r.at8(w.xcodes8), r.at(w.qkv));
      timed(r, "qkv_quantize_k", (double)T * 3 * H * 2 * es, [&] { qkv_quantize(c->dt, r.at(w.qkv), r.at(w.qkvcodes), T, H, aq.q, aq.k, aq.v, r.st); });
    }
    if (attn_mfma_ok(c->dt, c->d)) {
      attn_fwd_mfma(r.at(w.qkvcodes), r.at(w.ctx), codes(w.ctxcodes), aq, r.seqlens, r.B, r.S, c->nh, c->d, nullptr, r.at<float>(w.stat_m),
                    r.at<float>(w.stat_l), r.st, true, r.at8(w.ctxcodes8));
    } else {
      attn_fwd(c->dt, r.at(w.qkvcodes), r.at(w.ctx), r.at(w.ctxcodes), aq, r.seqlens, r.B, r.S, c->nh, c->d, nullptr, r.st);
      if (r.i8()) codes_to_i8(c->dt, r.at(w.ctxcodes), r.at8(w.ctxcodes8), (int64_t)T * H, 0.f, r.st);
    }
    student_linear(r, params, l, 1, r.at(w.ctxcodes), r.at8(w.ctxcodes8), r.at(w.o));
    const double ln_q_bytes = (double)T * H * (3 * es + es_codes);  // x, r in; y and its codes out
    timed(r, "ln_fwd_k", ln_q_bytes, [&] {
      ln_fwd(c->dt, x, r.at(w.o), base + c->foff[MREM_F_LN1_G], base + c->foff[MREM_F_LN1_B], r.at(w.x1), codes(w.x1codes),
             make_q(c, params, l, 6), r.at<float>(w.mu1), r.at<float>(w.rstd1), T, H, c->cfg.ln_eps, r.st, r.at8(w.x1codes8));
    });
    const QArg qg = make_q(c, params, l, 7);
    if (r.i8() && post_codes_ok(T, F, H)) {
      Epilogue post;
      post.post = POST_GELU; post.post_q = qg; post.post_out = codes(w.gcodes); post.post_out8 = r.at8(w.gcodes8); post.post_shift = (int)(0.5f * (qg.qp + 1.f));
      student_linear(r, params, l, 2, r.at(w.x1codes), r.at8(w.x1codes8), backward ? r.at(w.u) : nullptr, post);
    } else {
      student_linear(r, params, l, 2, r.at(w.x1codes), r.at8(w.x1codes8), r.at(w.u));
      timed(r, "gelu_quantize_k", (double)T * F * (es + es_codes),
            [&] { gelu_quantize(c->dt, r.at(w.u), codes(w.gcodes), (int64_t)T * F, qg, r.st, r.at8(w.gcodes8), 0.5f * (qg.qp + 1.f)); });
    }
    student_linear(r, params, l, 3, r.at(w.gcodes), r.at8(w.gcodes8), r.at(w.y));
    if (l + 1 < c->L) {
      // the layer output and, in the same pass, its codes under the next layer's input quantizer
      const LayerWs& wn = r.p.lw[l + 1];
      timed(r, "ln_fwd_k", ln_q_bytes, [&] {
        ln_fwd(c->dt, r.at(w.x1), r.at(w.y), base + c->foff[MREM_F_LN2_G], base + c->foff[MREM_F_LN2_B], f, codes(wn.xcodes),
               make_q(c, params, l + 1, 0), r.at<float>(w.mu2), r.at<float>(w.rstd2), T, H, c->cfg.ln_eps, r.st, r.at8(wn.xcodes8));
      });
    } else {
      timed(r, "ln_fwd_k", (double)T * H * 3 * es, [&] {
        ln_fwd(c->dt, r.at(w.x1), r.at(w.y), base + c->foff[MREM_F_LN2_G], base + c->foff[MREM_F_LN2_B], f, nullptr, QArg(),
               r.at<float>(w.mu2), r.at<float>(w.rstd2), T, H, c->cfg.ln_eps, r.st);
      });
    }
  }
}

// Where the full-precision module's products keep one order of sums (Epilogue::chain).  Its calibration always does: the
// steps it finds decide every code of the quantized module.  In a step or a forward pass only the targets f_l depend on
// it, and what rounding moves there averages out over the tokens: with bf16 matrix products instead, the second moments
// of 1 to 6 layers moved by up to 2.3 percent under 128 tokens and by up to 0.7 percent from 300 on (100 shapes), and the
// ordered products take 3 to 5 times as long (both passes of six layers of 1024 over 4000 tokens: 7264 against 2611 us).
constexpr int kChainTokens = 512;

// Where a calibration's partial ranges go and what turns them into steps and offsets; `first`, `last`: of the module's layers.
struct Calibration {
  float* params;  // of the layer that the pass runs
  float* parts;
  std::vector<CalibJob>* jobs;
  bool first, last;
};

// Full-precision module, layers [l0, l1) (l1 < 0: to the last layer).  With `cal` (one layer) the ranges of the inputs of the
// activation quantizers are taken on the way, by the kernels that write them where these can: a pass of its own for each
// (5 to 7 us, 18 with the GELU) was a fifth of a calibration of six layers of 1024 over 4096 tokens (1198 -> 990 us).
void teacher_forward(const Run& r, const float* teacher, const void* cache, const void* x_fp, void* per_layer_fp, int l0 = 0, int l1 = -1,
                     Calibration* cal = nullptr) {
  const mrem_ctx* c = r.c;
  const size_t es = dt_size(c->dt);
  const int H = c->H, F = c->F, T = r.T;
  const size_t slice = (size_t)T * H * es;
  const float qp_s = (float)((1 << (c->cfg.a_bits > 0 ? c->cfg.a_bits - 1 : 1)) - 1);
  const float qp_u = (float)((1 << (c->cfg.a_bits > 0 ? c->cfg.a_bits : 1)) - 1);
  // quantizer idx of the layer, or of the one above it
  auto job = [&](int idx, int nparts, int mode, bool above = false) {
    float* base = cal->params + (above ? c->layer_stride : 0);
    cal->jobs->push_back(CalibJob{cal->parts, base + c->foff[MREM_F_S_A] + idx, base + c->foff[MREM_F_Z_A] + idx, nparts, mode, mode == 0 ? qp_s : qp_u});
    cal->parts += 3 * nparts;
  };
  auto calib = [&](int idx, const void* a, int dt, int rows, int cols, int mode) { job(idx, absminmax(dt, a, rows, cols, 1, cols, cal->parts, r.st), mode); };
  // ranges from the products' epilogues: the partials of the smallest tiles (32 x 32) fit the area, with those of the other kernels
  auto tiles = [&](int n) { return (size_t)((T + 31) / 32) * ((n + 31) / 32); };
  const bool attn_mfma = attn_mfma_ok(c->dt, c->d);
  const bool ranges = cal && c->dt == DT_BF16 && H % 32 == 0 &&
                      3 * (3 * tiles(3 * H) + tiles(F) + 2 * (size_t)T + 2 * (size_t)attn_fwd_mfma_parts(r.B, r.S, c->nh, c->d) + 2 * kCalibParts) <= r.p.partials_per_layer;
  const bool chain = cal || T < kChainTokens;
  if (l1 < 0) l1 = c->L;
  for (int l = l0; l < l1; ++l) {
    const float* base = teacher + c->layer_stride * l;
    const char* wc = (const char*)cache + (size_t)c->tc_layer_stride * l * es;
    auto W = [&](int i) { return (const void*)(wc + (size_t)c->tc_off[i] * es); };
    const void* x = l == 0 ? x_fp : (const char*)per_layer_fp + slice * (l - 1);
    void* f = (char*)per_layer_fp + slice * l;
    Epilogue e;
    e.chain = chain;
    int nparts = 0;
    auto with_range = [&](const Epilogue& plain, int cols) {
      Epilogue er = plain;
      if (ranges) { er.range = cal->parts; er.range_cols = cols; er.blocks = &nparts; }
      return er;
    };
    if (cal && (cal->first || !ranges)) calib(0, x, c->dt, T, H, 0);
    e.bias = base + c->foff[MREM_F_B_QKV];
    gemm_nt(c->dt, x, H, W(0), H, r.at(r.p.t_qkv), 3 * H, T, 3 * H, H, with_range(e, H), r.st, r.prof);
    if (cal) {
      if (!ranges) nparts = absminmax(c->dt, r.at(r.p.t_qkv), T, H, 3, 3 * H, cal->parts, r.st);
      job(1, nparts, 0);
      job(2, nparts, 0);
      job(4, nparts, 0);
    }
    const bool attn_ranges = cal && attn_mfma;  // (24 floats a head and query in the area, against 12.4 that these take at most)
    if (attn_mfma)
      nparts = attn_fwd_mfma(r.at(r.p.t_qkv), r.at(r.p.t_ctx), nullptr, AttnQ(), r.seqlens, r.B, r.S, c->nh, c->d, attn_ranges ? cal->parts : nullptr, nullptr,
                             nullptr, r.st, chain);
    else
      attn_fwd(c->dt, r.at(r.p.t_qkv), r.at(r.p.t_ctx), nullptr, AttnQ(), r.seqlens, r.B, r.S, c->nh, c->d,
               cal ? r.at<float>(r.p.pmax) : nullptr, r.st);
    if (attn_ranges) {
      job(3, nparts, 1);
      job(5, nparts, 0);
    } else if (cal) {
      calib(3, r.at(r.p.pmax), DT_F32, 1, r.B * c->nh * r.S, 1);
      calib(5, r.at(r.p.t_ctx), c->dt, T, H, 0);
    }
    e.bias = base + c->foff[MREM_F_B_O];
    gemm_nt(c->dt, r.at(r.p.t_ctx), H, W(1), H, r.at(r.p.t_o), H, T, H, H, e, r.st, r.prof);
    timed(r, "ln_fwd_k", (double)T * H * 3 * es, [&] {
      ln_fwd(c->dt, x, r.at(r.p.t_o), base + c->foff[MREM_F_LN1_G], base + c->foff[MREM_F_LN1_B], r.at(r.p.t_x1), nullptr, QArg(),
             r.at<float>(r.p.t_mu), r.at<float>(r.p.t_rstd), T, H, c->cfg.ln_eps, r.st, nullptr, ranges ? cal->parts : nullptr);
    });
    if (ranges) job(6, T, 0);
    else if (cal) calib(6, r.at(r.p.t_x1), c->dt, T, H, 0);
    e.bias = base + c->foff[MREM_F_B_1];
    e.gelu = !cal || ranges;
    gemm_nt(c->dt, r.at(r.p.t_x1), H, W(2), H, r.at(r.p.t_g), F, T, F, H, with_range(e, 0), r.st, r.prof);
    e.gelu = 0;
    // (the range of gelu(u) is that of its unrounded values)
    if (ranges) job(7, nparts, 2);
    else if (cal) job(7, gelu_minmax(c->dt, r.at(r.p.t_g), (int64_t)T * F, cal->parts, r.st), 2);
    e.bias = base + c->foff[MREM_F_B_2];
    gemm_nt(c->dt, r.at(r.p.t_g), F, W(3), F, r.at(r.p.t_y), H, T, H, F, e, r.st, r.prof);
    // the layer's output is the next one's input
    const bool above = ranges && !cal->last;
    timed(r, "ln_fwd_k", (double)T * H * 3 * es, [&] {
      ln_fwd(c->dt, r.at(r.p.t_x1), r.at(r.p.t_y), base + c->foff[MREM_F_LN2_G], base + c->foff[MREM_F_LN2_B], f, nullptr, QArg(),
             r.at<float>(r.p.t_mu), r.at<float>(r.p.t_rstd), T, H, c->cfg.ln_eps, r.st, nullptr, above ? cal->parts : nullptr);
    });
    if (above) job(0, T, 0, true);
  }
}

// weight-gradient product of linear layer i: grads[w] = (dY^T * codes_in) * s_a (+ z * db);
// dy is [T, N_out], codes_in is [T, K_in]: the token index is the contraction index of both
void wgrad(const Run& r, const float* params, float* grads, int l, int i, const void* dy, const void* codes_in) {
  const mrem_ctx* c = r.c;
  float* g = grads + c->layer_stride * l;
  Epilogue e;
  const QArg q = make_q(c, params, l, kInQuant[i]);
  if (q.on) e.alpha = q.s;  // the offset term z * db[n] of an asymmetric input quantizer is added by the update kernel
  e.out_f32 = 1;
  e.c_zeroed = 1;  // the step starts by zeroing the gradients that are formed in k-slices
  gemm(c->dt, 1, 1, dy, c->wN[i], codes_in, c->wK[i], g + c->foff[kWField[i]], c->wK[i], c->wN[i], c->wK[i], r.T, e, r.st, r.prof);
}
// ... and all four of layer l as one list; dy and codes_in by linear layer
std::vector<WgradJob> wgrad_jobs(const Run& r, const float* params, float* grads, int l, const size_t (&dy)[4]) {
  const mrem_ctx* c = r.c;
  const LayerWs& w = r.p.lw[l];
  const size_t codes[4] = {w.xcodes, w.ctxcodes, w.x1codes, w.gcodes};
  std::vector<WgradJob> jobs;
  for (int i = 3; i >= 0; --i) {
    const QArg q = make_q(c, params, l, kInQuant[i]);
    jobs.push_back(WgradJob{r.at(dy[i]), r.at(codes[i]), grads + c->layer_stride * l + c->foff[kWField[i]], q.on ? q.s : nullptr, c->wN[i], c->wK[i]});
  }
  return jobs;
}
// input-gradient product: d(in^) = dY * W^ with the dequantized weights [N_out, K_in]
void dgrad(const Run& r, int l, int i, const void* dy, void* out, const Epilogue& e = Epilogue()) {
  const mrem_ctx* c = r.c;
  gemm(c->dt, 0, 1, dy, c->wN[i], r.at(r.p.lw[l].what[i]), c->wK[i], out, c->wK[i], r.T, c->wK[i], c->wN[i], e, r.st, r.prof);
}

// Zeroes what the backward pass adds into (weight gradients formed in two k-slices) or never
// writes (the slots of the fixed quantizer offsets; the vectors of a layer are one region).
// `together`: those of the layers above the lowest are written by one launch a layer, whole.
void zero_gradient_slots(const Run& r, float* grads, bool together) {
  const mrem_ctx* c = r.c;
  std::vector<FillRegion> regions;
  for (int l = 0; l < c->L; ++l) {
    float* g = grads + c->layer_stride * l;
    regions.push_back(FillRegion{g + c->foff[MREM_F_B_QKV], c->layer_stride - c->foff[MREM_F_B_QKV]});
    for (int i = 0; i < 4 && !(together && l > 0); ++i)
      if (gemm_f32_k_slices(c->dt, c->wN[i], c->wK[i], r.T) > 1)
        regions.push_back(FillRegion{g + c->foff[kWField[i]], (int64_t)c->wN[i] * c->wK[i]});
  }
  zero_regions(regions.data(), (int)regions.size(), r.st);
}

// What the backward pass needs to update the weight matrices of a layer as soon as that layer's
// gradients are complete (Algorithm 2, last line), on `side` if there is one.
struct Update {
  float* params;
  float* m;
  float* v;
  AdamArg a;
  int write_grads;
  hipStream_t side;            // nullptr: everything on the caller's stream
  const hipEvent_t* ev_layer;  // one per layer when side != nullptr
  const hipEvent_t* ev_ready;  // four per layer
  const hipEvent_t* ev_done;   // four per layer
  hipEvent_t ev_join;
  bool by_layer;               // one handover to `side` a layer instead of one a product
  int wgrad_tile;              // then, above the lowest layer: the tile that serves a layer's weight gradients in one launch (0: none)
};
void update_matrices(const Run& r, const Update& u, float* grads, int l, hipStream_t st);

void student_backward(const Run& r, const float* params, const void* x_q, const void* per_layer_fp, const void* per_layer_q,
                      float* grads, float* loss_out, const Update& up) {
  const mrem_ctx* c = r.c;
  const size_t es = dt_size(c->dt);
  const int H = c->H, F = c->F, T = r.T, L = c->L;
  const size_t slice = (size_t)T * H * es;
  const int64_t numel = (int64_t)T * H;
  Reductions red;
  for (int l = L - 1; l >= 0; --l) {
    const size_t first_job = red.jobs.size();
    const LayerWs& w = r.p.lw[l];
    const float* base = params + c->layer_stride * l;
    float* g = grads + c->layer_stride * l;
    const void* x = l == 0 ? x_q : (const char*)per_layer_q + slice * (l - 1);
    const void* fq = (const char*)per_layer_q + slice * l;
    const void* ffp = (const char*)per_layer_fp + slice * l;
    const bool in_loss = (c->cfg.loss_layer_mask >> l) & 1u;
    red.next = r.at<float>(r.p.partials) + r.p.partials_per_layer * l;
    // The weight-gradient products feed nothing but the update, so with a side stream they run
    // there, beside the input-gradient products and the bandwidth-bound kernels of this stream.
    // Handed over one by one, each output gradient has one buffer, which this stream overwrites in the layer below only
    // when the product has read it.  Handed over by the layer, two layers alternate between two sets of buffers (the
    // second is the full-precision pass's scratch, which nobody needs any more).
    // The lowest layer's products, with nothing to run beside them afterwards, are not held back for one launch.
    const bool sets = up.side && up.by_layer, second = sets && (l & 1), by_layer = sets && (l > 0 || !up.wgrad_tile);
    const size_t dr2 = second ? r.p.t_y : r.p.dr2, dr1 = second ? r.p.t_o : r.p.dr1, du = second ? r.p.t_g : r.p.du, dqkv = second ? r.p.t_qkv : r.p.dqkv;
    const size_t dr1_above = sets && !second ? r.p.t_o : r.p.dr1;
    if (sets && l + 2 < L) (void)hipStreamWaitEvent(r.st, up.ev_done[4 * (l + 2)], 0);
    Run rs = r;
    if (up.side) rs.st = up.side;
    auto issue_wgrad = [&](int i, const void* dy, const void* codes) {
      if (by_layer) return;
      if (up.side) {
        (void)hipEventRecord(up.ev_ready[4 * l + i], r.st);
        (void)hipStreamWaitEvent(up.side, up.ev_ready[4 * l + i], 0);
      }
      wgrad(rs, params, grads, l, i, dy, codes);
      if (up.side) (void)hipEventRecord(up.ev_done[4 * l + i], up.side);
    };
    auto before_overwrite = [&](int i) {
      if (up.side && !sets && l < L - 1) (void)hipStreamWaitEvent(r.st, up.ev_done[4 * (l + 1) + i], 0);
    };
    // all that the side stream does for this layer, once everything it reads is enqueued on this one
    auto hand_over = [&]() {
      (void)hipEventRecord(up.ev_layer[l], r.st);
      (void)hipStreamWaitEvent(up.side, up.ev_layer[l], 0);
      if (!by_layer) return;
      if (up.wgrad_tile) {
        const std::vector<WgradJob> jobs = wgrad_jobs(r, params, grads, l, {dqkv, dr1, du, dr2});
        gemm_wgrads(jobs.data(), (int)jobs.size(), r.T, up.wgrad_tile, rs.st);
        if (l >= 2) (void)hipEventRecord(up.ev_done[4 * l], up.side);
        return;
      }
      wgrad(rs, params, grads, l, 3, r.at(dr2), r.at(w.gcodes));
      wgrad(rs, params, grads, l, 2, r.at(du), r.at(w.x1codes));
      wgrad(rs, params, grads, l, 1, r.at(dr1), r.at(w.ctxcodes));
      wgrad(rs, params, grads, l, 0, r.at(dqkv), r.at(w.xcodes));
      if (l >= 2) (void)hipEventRecord(up.ev_done[4 * l], up.side);
    };
    // second LayerNorm: dy = [dr1 + dxh*mask of the layer above] + gradient of this layer's Eq. 3 term,
    // which the same kernel forms from the two layer outputs (it also returns the squared-error sum)
    {
      const bool top = (l == L - 1);
      const QArg q_above = top ? QArg() : make_q(c, params, l + 1, 0);
      const float scale = c->cfg.loss_mean ? 1.0f / (float)numel : 1.0f;
      const int wd = 3 * H + 2;
      float* parts = red.take((size_t)ln_bwd_parts(T) * wd);
      before_overwrite(3);
      int n = 0;
      // in: layer output, the two LayerNorm inputs, the full-precision output (loss), above the top layer also the two
      // gradients from above; out: the gradient of the LayerNorm input
      timed(r, "ln_bwd_k", (double)T * H * es * ((top ? 4 : 6) + (in_loss ? 1 : 0)), [&] {
        n = ln_bwd(c->dt, top ? nullptr : r.at(dr1_above), top ? nullptr : r.at(r.p.dxh), fq, q_above, r.at(w.x1), r.at(w.y),
                   r.at<float>(w.mu2), r.at<float>(w.rstd2), base + c->foff[MREM_F_LN2_G], r.at(dr2), parts, T, H, r.st,
                   in_loss ? ffp : nullptr, scale);
      });
      red.add(parts, n, wd, 0, H, g + c->foff[MREM_F_LN2_G]);
      red.add(parts, n, wd, H, H, g + c->foff[MREM_F_LN2_B]);
      red.add(parts, n, wd, 2 * H, H, g + c->foff[MREM_F_B_2]);
      if (!top) red.add(parts, n, wd, 3 * H, 1, grads + c->layer_stride * (l + 1) + c->foff[MREM_F_S_A] + 0);
      // a layer outside the loss mask contributes an exact zero (its partial sums are zero)
      red.add(parts, n, wd, 3 * H + 1, 1, loss_out + 1 + l, in_loss ? scale : 0.f);
    }
    // second feed-forward projection
    issue_wgrad(3, r.at(dr2), r.at(w.gcodes));
    // GELU and its output quantizer
    {
      // the kernel also leaves the column sums of du per row slab: the bias gradient of the first projection
      float* parts = red.take(2048);
      float* cols = red.take((size_t)kColMaxParts * F);
      const QArg qg = make_q(c, params, l, 7);
      before_overwrite(2);
      int n = 0, slabs = 0;
      if (c->dt == DT_BF16 && qg.on && post_ok(T, F, H) && T / 128 <= kColMaxParts) {
        Epilogue post;
        post.post = POST_DGELU; post.post_in = r.at(w.u); post.post_q = qg; post.post_parts = parts; post.post_col_parts = cols; post.blocks = &n; post.row_tiles = &slabs;
        dgrad(r, l, 3, r.at(dr2), r.at(du), post);
      } else {
        dgrad(r, l, 3, r.at(dr2), r.at(r.p.dgh));
        timed(r, "gelu_quant_bwd_k", (double)T * F * 3 * es, [&] {
          const ColGrid cg = gelu_quant_bwd(c->dt, r.at(r.p.dgh), r.at(w.u), r.at(du), T, F, qg, parts, cols, r.st);
          n = cg.gx * cg.gy;
          slabs = cg.gy;
        });
      }
      red.add(parts, n, 1, 0, 1, g + c->foff[MREM_F_S_A] + 7);
      red.add(cols, slabs, F, 0, F, g + c->foff[MREM_F_B_1]);
    }
    // first feed-forward projection
    issue_wgrad(2, r.at(du), r.at(w.x1codes));
    dgrad(r, l, 2, r.at(du), r.at(r.p.dx1h));
    // first LayerNorm: dy = dr2 (residual) + dx1h through the FFN-input quantizer
    {
      float* parts = red.take((size_t)ln_bwd_parts(T) * (3 * H + 2));
      before_overwrite(1);
      int n = 0;
      timed(r, "ln_bwd_k", (double)T * H * es * 6, [&] {
        n = ln_bwd(c->dt, r.at(dr2), r.at(r.p.dx1h), r.at(w.x1), make_q(c, params, l, 6), x, r.at(w.o),
                   r.at<float>(w.mu1), r.at<float>(w.rstd1), base + c->foff[MREM_F_LN1_G], r.at(dr1), parts, T, H, r.st);
      });
      const int wd = 3 * H + 2;
      red.add(parts, n, wd, 0, H, g + c->foff[MREM_F_LN1_G]);
      red.add(parts, n, wd, H, H, g + c->foff[MREM_F_LN1_B]);
      red.add(parts, n, wd, 2 * H, H, g + c->foff[MREM_F_B_O]);
      red.add(parts, n, wd, 3 * H, 1, g + c->foff[MREM_F_S_A] + 6);
    }
    // attention output projection
    issue_wgrad(1, r.at(dr1), r.at(w.ctxcodes));
    {
      float* parts = red.take(2048);
      const QArg qc = make_q(c, params, l, 5);
      int n = 0;
      if (c->dt == DT_BF16 && qc.on && post_ok(T, H, H)) {
        Epilogue post;
        post.post = POST_MASK; post.post_in = r.at(w.ctx); post.post_q = qc; post.post_parts = parts; post.blocks = &n;
        dgrad(r, l, 1, r.at(dr1), r.at(r.p.dc), post);
      } else {
        dgrad(r, l, 1, r.at(dr1), r.at(r.p.dch));
        timed(r, "quant_bwd_k", (double)numel * 3 * es, [&] { n = quant_bwd(c->dt, r.at(r.p.dch), r.at(w.ctx), r.at(r.p.dc), numel, qc, parts, r.st); });
      }
      red.add(parts, n, 1, 0, 1, g + c->foff[MREM_F_S_A] + 5);
    }
    // attention
    const AttnQ aq = make_attn_q(c, params, l, true);
    {
      int n = r.B * c->nh * r.S;
      float* parts = red.take((size_t)n);
      if (attn_mfma_ok(c->dt, c->d))
        n = attn_bwd_mfma(r.at(w.qkvcodes), r.at(r.p.dc), r.at(r.p.dqkvh), aq, r.seqlens, r.B, r.S, c->nh, c->d,
                          r.at<float>(w.stat_m), r.at<float>(w.stat_l), r.at(r.p.s_ph), r.at(r.p.s_da), parts, r.st);
      else
        attn_bwd(c->dt, r.at(w.qkvcodes), r.at(r.p.dc), r.at(r.p.dqkvh), aq, r.seqlens, r.B, r.S, c->nh, c->d, r.at<float>(r.p.s_da),
                 r.at<float>(r.p.s_ph), parts, r.st);
      red.add(parts, n, 1, 0, 1, g + c->foff[MREM_F_S_A] + 3);
    }
    {
      // the kernel also leaves the column sums of dqkv per row slab: the bias gradient of the projection
      float* parts = red.take(2048 * 3);
      float* cols = red.take((size_t)kColMaxParts * 3 * H);
      before_overwrite(0);
      ColGrid cg{};
      timed(r, "qkv_quant_bwd_k", (double)T * 3 * H * 3 * es,
            [&] { cg = qkv_quant_bwd(c->dt, r.at(r.p.dqkvh), r.at(w.qkv), r.at(dqkv), T, H, aq.q, aq.k, aq.v, parts, cols, r.st); });
      const int n = cg.gx * cg.gy;
      red.add(parts, n, 3, 0, 1, g + c->foff[MREM_F_S_A] + 1);
      red.add(parts, n, 3, 1, 1, g + c->foff[MREM_F_S_A] + 2);
      red.add(parts, n, 3, 2, 1, g + c->foff[MREM_F_S_A] + 4);
      red.add(cols, cg.gy, 3 * H, 0, 3 * H, g + c->foff[MREM_F_B_QKV]);
    }
    // query/key/value projection
    issue_wgrad(0, r.at(dqkv), r.at(w.xcodes));
    if (by_layer && l > 0) hand_over();
    dgrad(r, l, 0, r.at(dqkv), r.at(r.p.dxh));
    if (l == 0) {
      // nothing flows out of the module (Section 4.2); only the input quantizer's step needs dxh
      float* parts = red.take(2048);
      const int n = quant_bwd_reduce(c->dt, r.at(r.p.dxh), x, numel, make_q(c, params, 0, 0), parts, r.st);
      red.add(parts, n, 1, 0, 1, g + c->foff[MREM_F_S_A] + 0);
    }
    // This layer's gradients are complete and nothing below reads its matrices or their steps
    // again (the input gradients used the dequantized copies): its second-stage reductions and
    // the update of its four matrices, which is bound by memory traffic, run beside the
    // matrix products of the layers below.
    if (up.side && (!by_layer || l == 0)) hand_over();
    reduce_jobs(red.jobs.data() + first_job, (int)(red.jobs.size() - first_job), rs.st);
    update_matrices(r, up, grads, l, rs.st);
  }
  if (up.side) {
    (void)hipEventRecord(up.ev_join, up.side);
    (void)hipStreamWaitEvent(r.st, up.ev_join, 0);
  }
  loss_total(loss_out, L, c->nonfinite_flag, r.st);
}

AdamArg adam_arg(const mrem_ctx* c, int64_t step, float lr) {
  AdamArg a;
  a.lr = lr; a.beta1 = c->cfg.beta1; a.beta2 = c->cfg.beta2; a.eps = c->cfg.adam_eps; a.wd = c->cfg.weight_decay;
  a.bc1 = (float)(1.0 - std::pow((double)c->cfg.beta1, (double)step));
  a.bc2 = (float)(1.0 - std::pow((double)c->cfg.beta2, (double)step));
  a.floor = c->cfg.step_floor;
  return a;
}
// AdamW on the four weight matrices of layer l and their steps (they read the bias gradient and the
// activation offset of their layer, so the layer's reductions come first on the same stream)
void update_matrices(const Run& r, const Update& u, float* grads, int l, hipStream_t st) {
  const mrem_ctx* c = r.c;
  AdamJob jobs[4];
  const int64_t o = c->layer_stride * l;
  for (int i = 0; i < 4; ++i) {
    const int64_t ow = o + c->foff[kWField[i]], os = o + c->foff[kSField[i]];
    // the second feed-forward projection reads the GELU output through an asymmetric quantizer with offset z
    const bool zterm = (i == 3 && c->cfg.a_bits > 0);
    AdamJob& j = jobs[i];
    j.w = u.params + ow; j.sw = u.params + os; j.g_w = grads + ow; j.g_sw = grads + os;
    j.m_w = u.m + ow; j.v_w = u.v + ow; j.m_sw = u.m + os; j.v_sw = u.v + os;
    j.z_in = zterm ? u.params + o + c->foff[MREM_F_Z_A] + 7 : nullptr;
    j.db = zterm ? grads + o + c->foff[MREM_F_B_2] : nullptr;
    j.N = c->wN[i]; j.K = c->wK[i];
  }
  double nw = 0;
  for (int i = 0; i < 4; ++i) nw += (double)c->wN[i] * c->wK[i];
  Run rs = r;
  rs.st = st;
  // parameter, gradient and both moments in; parameter and both moments out (the masked gradient too when it is exported)
  timed(rs, "adam_matrix_k", nw * (28 + (u.write_grads ? 4 : 0)),
        [&] { adam_matrix(jobs, 4, c->cfg.w_bits, u.a, u.write_grads, c->cfg.per_channel ? 0 : 1, st); });
}
// AdamW (no decay) on everything that is not a matrix: biases, LayerNorm parameters, activation steps
void update_vectors(const Run& r, const Update& u, float* grads) {
  const mrem_ctx* c = r.c;
  AdamArg nodecay = u.a;
  nodecay.wd = 0.f;
  std::vector<VecJob> vjobs;
  for (int l = 0; l < c->L; ++l) {
    const int64_t o = c->layer_stride * l;
    vjobs.push_back(VecJob{o + c->foff[MREM_F_B_QKV], c->foff[MREM_F_SW_QKV] - c->foff[MREM_F_B_QKV], 0});
    if (c->cfg.a_bits > 0) vjobs.push_back(VecJob{o + c->foff[MREM_F_S_A], 8, 1});
  }
  adam_vector(u.params, grads, u.m, u.v, vjobs.data(), (int)vjobs.size(), nodecay, r.st);
}

mrem_status check_common(const mrem_ctx* ctx, int32_t batch, int32_t seq, const void* workspace, size_t workspace_bytes, const char* who,
                         Plan* plan) {
  if (!ctx) return fail(nullptr, MREM_EINVAL, std::string(who) + ": null context");
  if (batch < 1 || batch > ctx->cfg.max_batch) return fail(ctx, MREM_ESHAPE, std::string(who) + ": batch outside 1..max_batch");
  if (seq < 1 || seq > ctx->cfg.max_seq) return fail(ctx, MREM_ESHAPE, std::string(who) + ": seq outside 1..max_seq");
  if (!workspace || !aligned16(workspace)) return fail(ctx, MREM_EINVAL, std::string(who) + ": workspace null or misaligned");
  *plan = make_plan(ctx, batch, seq);
  if (workspace_bytes < plan->total) return fail(ctx, MREM_EWORKSPACE, std::string(who) + ": workspace too small");
  return MREM_OK;
}

mrem_status finish(const mrem_ctx* ctx, const char* who) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(ctx, MREM_EHIP, std::string(who) + ": " + hipGetErrorString(e));
  return MREM_OK;
}

#define REQUIRE_PTR(p, who)                                                                  \
  do {                                                                                       \
    if (!(p) || !aligned16(p)) return fail(ctx, MREM_EINVAL, std::string(who) + ": " #p " is null or not 16-byte aligned"); \
  } while (0)

}  // namespace

extern "C" size_t mrem_workspace_bytes(const mrem_ctx* ctx, int32_t batch, int32_t seq) {
  if (!ctx || batch < 1 || seq < 1) return 0;
  return make_plan(ctx, batch, seq).total;
}

extern "C" int64_t mrem_workspace_offset(const mrem_ctx* ctx, int32_t batch, int32_t seq, int32_t layer, int32_t item) {
  if (!ctx || batch < 1 || seq < 1 || layer < 0 || layer >= ctx->L) return -1;
  const Plan p = make_plan(ctx, batch, seq);
  const LayerWs& w = p.lw[layer];
  const int64_t T = (int64_t)batch * seq;
  const bool i8 = T % 128 == 0 && i8_products(ctx, T);
  if (item >= MREM_WS_WCODES8 && item < MREM_WS_WCODES8 + 4) return i8 ? (int64_t)w.wcodes8[item - MREM_WS_WCODES8] : -1;
  if (item >= MREM_WS_WCODES && item < MREM_WS_WCODES + 4) return i8 ? -1 : (int64_t)w.wcodes[item - MREM_WS_WCODES];
  if (item == MREM_WS_QKV) return (int64_t)w.qkv;
  if (item == MREM_WS_XCODES8) return i8 ? (int64_t)w.xcodes8 : -1;
  return -1;
}

extern "C" mrem_status mrem_quantize(const float* w, int64_t N, int64_t K, int32_t bits, int32_t per_channel, int32_t init_scale,
                                     float* scale, int8_t* codes, void* hip_stream) {
  const mrem_ctx* ctx = nullptr;
  REQUIRE_PTR(w, "mrem_quantize");
  REQUIRE_PTR(scale, "mrem_quantize");
  REQUIRE_PTR(codes, "mrem_quantize");
  if (bits < 2 || bits > 8) return fail(nullptr, MREM_EINVAL, "mrem_quantize: bits must be in 2..8");
  if (N < 1 || K < 1 || N > 0x7fffffff) return fail(nullptr, MREM_ESHAPE, "mrem_quantize: N and K must be >= 1 (N < 2^31)");
  if (per_channel != 0 && per_channel != 1) return fail(nullptr, MREM_EINVAL, "mrem_quantize: per_channel must be 0 or 1");
  weight_quantize_i8(w, scale, codes, N, K, bits, per_channel, init_scale, (hipStream_t)hip_stream);
  return finish(nullptr, "mrem_quantize");
}

extern "C" mrem_status mrem_module_init_steps(mrem_ctx* ctx, float* params, void* hip_stream) {
  if (!ctx) return fail(nullptr, MREM_EINVAL, "mrem_module_init_steps: null context");
  REQUIRE_PTR(params, "mrem_module_init_steps");
  if (ctx->cfg.w_bits == 0) return fail(ctx, MREM_EINVAL, "mrem_module_init_steps: weight quantizers are off (w_bits = 0)");
  for (int l = 0; l < ctx->L; ++l)
    for (int i = 0; i < 4; ++i) {
      float* sw = params + ctx->layer_stride * l + ctx->foff[kSField[i]];
      weight_step_init(params + ctx->layer_stride * l + ctx->foff[kWField[i]], sw, ctx->wN[i], ctx->wK[i], ctx->cfg.w_bits,
                       (hipStream_t)hip_stream);
      // one step per matrix: max|W| / Qp is the largest of the rows' quotients (the division is monotone)
      if (!ctx->cfg.per_channel) tie_steps_max(sw, ctx->wN[i], (hipStream_t)hip_stream);
    }
  return finish(ctx, "mrem_module_init_steps");
}

extern "C" mrem_status mrem_teacher_prepare(mrem_ctx* ctx, const float* teacher, void* cache, void* hip_stream) {
  if (!ctx) return fail(nullptr, MREM_EINVAL, "mrem_teacher_prepare: null context");
  REQUIRE_PTR(teacher, "mrem_teacher_prepare");
  REQUIRE_PTR(cache, "mrem_teacher_prepare");
  const size_t es = dt_size(ctx->dt);
  for (int l = 0; l < ctx->L; ++l)
    for (int i = 0; i < 4; ++i)
      convert_f32(ctx->dt, teacher + ctx->layer_stride * l + ctx->foff[kWField[i]],
                  (char*)cache + ((size_t)ctx->tc_layer_stride * l + ctx->tc_off[i]) * es, (int64_t)ctx->wN[i] * ctx->wK[i],
                  (hipStream_t)hip_stream);
  return finish(ctx, "mrem_teacher_prepare");
}

extern "C" mrem_status mrem_module_calibrate(mrem_ctx* ctx, float* params, const float* teacher, const void* teacher_cache, const void* x_fp,
                                             const int32_t* seqlens, int32_t batch, int32_t seq, void* workspace, size_t workspace_bytes,
                                             void* hip_stream) {
  Plan plan;
  mrem_status s = check_common(ctx, batch, seq, workspace, workspace_bytes, "mrem_module_calibrate", &plan);
  if (s != MREM_OK) return s;
  REQUIRE_PTR(params, "mrem_module_calibrate");
  REQUIRE_PTR(teacher, "mrem_module_calibrate");
  REQUIRE_PTR(teacher_cache, "mrem_module_calibrate");
  REQUIRE_PTR(x_fp, "mrem_module_calibrate");
  if (ctx->cfg.a_bits == 0) return fail(ctx, MREM_EINVAL, "mrem_module_calibrate: activation quantizers are off (a_bits = 0)");
  Run r{ctx, plan, (char*)workspace, (hipStream_t)hip_stream, batch, seq, batch * seq, seqlens, &ctx->prof};
  // Layer by layer with two alternating output buffers: only the ranges are wanted, not the per-layer outputs.  Nothing
  // of the pass depends on the steps, so all of them are formed at the end.
  {
    std::vector<CalibJob> jobs;
    jobs.reserve((size_t)ctx->L * 8);
    mrem_ctx one = *ctx;
    one.L = 1;
    const size_t es = dt_size(ctx->dt);
    void* bufs[2] = {r.at(r.p.dr1), r.at(r.p.dr2)};
    const void* x = x_fp;
    for (int l = 0; l < ctx->L; ++l) {
      Run rl = r;
      rl.c = &one;
      Calibration cal{params + ctx->layer_stride * l, r.at<float>(r.p.partials) + r.p.partials_per_layer * l, &jobs, l == 0, l + 1 == ctx->L};
      teacher_forward(rl, teacher + ctx->layer_stride * l, (const char*)teacher_cache + (size_t)ctx->tc_layer_stride * l * es, x, bufs[l & 1], 0, -1, &cal);
      x = bufs[l & 1];
    }
    calib_finalize(jobs.data(), (int)jobs.size(), r.st);
  }
  return finish(ctx, "mrem_module_calibrate");
}

namespace {
struct Bytes { const void* p; size_t n; };
bool overlap(const Bytes& a, const Bytes& b) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a.p), y = reinterpret_cast<uintptr_t>(b.p);
  return a.p && b.p && x < y + b.n && y < x + a.n;
}
// Whether either forward pass writes what the other one reads or writes: a quantized pass over the full-precision pass's
// outputs, or one that leaves its outputs in place of the input that both read.
bool passes_depend(const mrem_ctx* c, int batch, int seq, const float* params, const float* teacher, const void* teacher_cache, const void* x_fp,
                   const void* x_q, const int32_t* seqlens, const void* per_layer_fp, const void* per_layer_q) {
  const size_t io = (size_t)batch * seq * c->H * dt_size(c->dt), vec = (size_t)mrem_param_count(c) * sizeof(float);
  const Bytes out_fp{per_layer_fp, io * c->L}, out_q{per_layer_q, io * c->L}, lens{seqlens, (size_t)batch * sizeof(int32_t)};
  for (const Bytes& b : {out_q, Bytes{x_q, io}, Bytes{params, vec}, lens})
    if (overlap(out_fp, b)) return true;
  for (const Bytes& b : {Bytes{x_fp, io}, Bytes{teacher, vec}, Bytes{teacher_cache, mrem_teacher_cache_bytes(c)}, lens})
    if (overlap(out_q, b)) return true;
  return false;
}

// Whether two streams are worth the 30 us that forking and joining cost the host.  Small calls are bound by the host and the
// device has little to do beside them.  Measured over widths 64 to 1024, 1 to 12 layers and 8 to 4096 tokens, both passes
// (change in percent with two streams, a call by itself / calls behind each other):
//   from 640 columns in all layers together: 2 of 320 over 8 tokens 0/-3, over 128 -8/-7; 6 of 128 -9/-4 and -15/-16; 3 of 256
//     -9/-11 and -13/-15; 1 of 768 -1/-11 and 3/-6; 3 of 768 -26/-34 and -29/-33; 6 of 1024 over 4096 -7/-9;
//   512 to 640: 2 of 256 over 23 -1/-4, over 64 -3/-4, over 1024 -6/-10; 4 of 128 over 23 1/2, over 128 -3/-3;
//   384 to 512: 3 of 128 over 128 2/3, over 400 -2/-1, over 2048 -7/-6; 6 of 64 over 64 0/5, over 400 -9/-3;
//   fewer: 4 of 64 over 256 0/3, over 1024 -10/0; 3 of 64 over 1024 4/6, over 2048 -15/-12; 2 of 128 over 1024 7/13, over 2048
//     6/5, over 4096 -2/-5; 2 of 64 over 4096 6/12;
//   single layers: 512 over 1024 2/-2, over 2048 -2/-15; 320 over 4096 5/-12; 256 over 128 26/24.
bool worth_forking(int L, int H, int T) {
  const int64_t width = (int64_t)L * H;
  if (width >= 640) return true;
  if (L == 1) return H >= 512 && T >= 2048;
  if (width >= 512) return (int64_t)T * H >= 1 << 14;
  if (L == 2) return width * T >= 1 << 20;
  return width >= 384 ? T >= 384 : width * T >= 1 << 18;
}

mrem_status forward_impl(mrem_ctx* ctx, const float* params, const float* teacher, const void* teacher_cache, const void* x_fp,
                         const void* x_q, const int32_t* seqlens, int32_t batch, int32_t seq, void* per_layer_fp, void* per_layer_q,
                         void* workspace, size_t workspace_bytes, void* hip_stream, bool two_streams, const char* who) {
  Plan plan;
  mrem_status s = check_common(ctx, batch, seq, workspace, workspace_bytes, who, &plan);
  if (s != MREM_OK) return s;
  if (!per_layer_fp && !per_layer_q) return fail(ctx, MREM_EINVAL, std::string(who) + ": both outputs are null");
  Run r{ctx, plan, (char*)workspace, (hipStream_t)hip_stream, batch, seq, batch * seq, seqlens, &ctx->prof};
  if (per_layer_fp) {
    REQUIRE_PTR(teacher, who);
    REQUIRE_PTR(teacher_cache, who);
    REQUIRE_PTR(x_fp, who);
    if (!aligned16(per_layer_fp)) return fail(ctx, MREM_EINVAL, std::string(who) + ": per_layer_fp misaligned");
  }
  if (per_layer_q) {
    REQUIRE_PTR(params, who);
    REQUIRE_PTR(x_q, who);
    if (!aligned16(per_layer_q)) return fail(ctx, MREM_EINVAL, std::string(who) + ": per_layer_q misaligned");
  }
  // Where the passes share nothing but their inputs the full-precision one runs on a side stream, forked from the caller's and
  // joined to it (both passes of a 23-token sentence through three layers of 768: 373 us one after the other, 264 now; six
  // layers of 1024 over 4096 tokens: 1840 and 1660).  Not while the caller's stream is being captured: another thread that
  // calls on that stream would find the side stream in the capture.  Nor where worth_forking says so.
  hipStreamCaptureStatus capture = hipStreamCaptureStatusActive;
  bool fork = two_streams && per_layer_fp && per_layer_q && !ctx->prof.on &&
              worth_forking(ctx->L, ctx->H, r.T) && !passes_depend(ctx, batch, seq, params, teacher, teacher_cache, x_fp, x_q, seqlens, per_layer_fp, per_layer_q);
  if (fork && (hipStreamIsCapturing(r.st, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone)) {
    (void)hipGetLastError();
    fork = false;
  }
  PassStream* const side = fork ? take_pass_stream(r.st) : nullptr;
  if (side) {
    Run rt = r;
    rt.st = side->st;
    {
      const std::lock_guard<std::mutex> lock(side->lock);
      (void)hipEventRecord(side->fork, r.st);
      (void)hipStreamWaitEvent(side->st, side->fork, 0);
    }
    prepare_weights(r, params, false);
    // layer by layer in turn, so that both streams have work from the start
    for (int l = 0; l < ctx->L; ++l) {
      teacher_forward(rt, teacher, teacher_cache, x_fp, per_layer_fp, l, l + 1);
      student_forward(r, params, x_q, per_layer_q, false, l, l + 1);
    }
    {
      const std::lock_guard<std::mutex> lock(side->lock);
      (void)hipEventRecord(side->join, side->st);
      (void)hipStreamWaitEvent(r.st, side->join, 0);
    }
    leave_pass_stream(side);
    return finish(ctx, who);
  }
  if (per_layer_fp) teacher_forward(r, teacher, teacher_cache, x_fp, per_layer_fp);
  if (per_layer_q) {
    prepare_weights(r, params, false);
    student_forward(r, params, x_q, per_layer_q, false);
  }
  return finish(ctx, who);
}
}  // namespace

extern "C" mrem_status mrem_module_forward(mrem_ctx* ctx, const float* params, const float* teacher, const void* teacher_cache,
                                           const void* x_fp, const void* x_q, const int32_t* seqlens, int32_t batch, int32_t seq,
                                           void* per_layer_fp, void* per_layer_q, void* workspace, size_t workspace_bytes, void* hip_stream) {
  return forward_impl(ctx, params, teacher, teacher_cache, x_fp, x_q, seqlens, batch, seq, per_layer_fp, per_layer_q, workspace,
                      workspace_bytes, hip_stream, true, "mrem_module_forward");
}

// ------------------------------------------------------------------------------
// The forward passes for callers that cannot allocate: the workspace is a static device array.
// ------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[MREM_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
// Device address of `scratch` on each device (every device holds its own copy of the array at its
// own address; the array's name itself is only a host-side handle).  Looked up once per device,
// with that device current.
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

extern "C" size_t mrem_static_scratch_bytes(void) { return MREM_STATIC_SCRATCH_BYTES; }

extern "C" mrem_status mrem_module_forward_static(mrem_ctx* ctx, const float* params, const float* teacher, const void* teacher_cache,
                                                  const void* x_fp, const void* x_q, const int32_t* seqlens, int32_t batch,
                                                  int32_t seq, void* per_layer_fp, void* per_layer_q, void* hip_stream) {
  const char* who = "mrem_module_forward_static";
  if (!ctx) return fail(nullptr, MREM_EINVAL, std::string(who) + ": null context");
  if (batch < 1 || seq < 1) return fail(ctx, MREM_ESHAPE, std::string(who) + ": batch and seq must be >= 1");
  const size_t need = make_plan(ctx, batch, seq).total;
  if (need > (size_t)MREM_STATIC_SCRATCH_BYTES)
    return fail(ctx, MREM_EWORKSPACE, std::string(who) + ": this module at this batch and seq needs " + std::to_string(need) +
                                          " bytes of scratch, the static array holds " + std::to_string((size_t)MREM_STATIC_SCRATCH_BYTES) +
                                          "; use mrem_module_forward with a caller-owned workspace");
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return fail(ctx, MREM_EHIP, std::string(who) + ": no current device");
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return fail(ctx, MREM_EHIP, std::string(who) + ": hipGetSymbolAddress: " + hipGetErrorString(e));
    g_scratch_ptr[dev] = p;
  }
  // Nothing in the forward passes reads scratch memory that the same call has not written, so the
  // contents a previous call left behind need no clearing.
  return forward_impl(ctx, params, teacher, teacher_cache, x_fp, x_q, seqlens, batch, seq, per_layer_fp, per_layer_q,
                      g_scratch_ptr[dev], MREM_STATIC_SCRATCH_BYTES, hip_stream, false, who);
}

extern "C" mrem_status mrem_module_step(mrem_ctx* ctx, float* params, float* adam_m, float* adam_v, int64_t step_index, float lr,
                                        float lambda, const float* teacher, const void* teacher_cache, const void* x_fp, const void* x_q,
                                        const int32_t* seqlens, int32_t batch, int32_t seq, float* loss_out, void* per_layer_fp,
                                        void* per_layer_q, float* grads_out, void* workspace, size_t workspace_bytes, void* hip_stream) {
  Plan plan;
  mrem_status s = check_common(ctx, batch, seq, workspace, workspace_bytes, "mrem_module_step", &plan);
  if (s != MREM_OK) return s;
  REQUIRE_PTR(params, "mrem_module_step");
  REQUIRE_PTR(adam_m, "mrem_module_step");
  REQUIRE_PTR(adam_v, "mrem_module_step");
  REQUIRE_PTR(teacher, "mrem_module_step");
  REQUIRE_PTR(teacher_cache, "mrem_module_step");
  REQUIRE_PTR(x_fp, "mrem_module_step");
  REQUIRE_PTR(x_q, "mrem_module_step");
  REQUIRE_PTR(loss_out, "mrem_module_step");
  REQUIRE_PTR(per_layer_fp, "mrem_module_step");
  REQUIRE_PTR(per_layer_q, "mrem_module_step");
  if (grads_out && !aligned16(grads_out)) return fail(ctx, MREM_EINVAL, "mrem_module_step: grads_out misaligned");
  if (step_index < 1) return fail(ctx, MREM_EINVAL, "mrem_module_step: step_index is 1-based");
  if (!(lambda >= 0.f && lambda <= 1.f)) return fail(ctx, MREM_EINVAL, "mrem_module_step: lambda must be in [0,1]");
  Run r{ctx, plan, (char*)workspace, (hipStream_t)hip_stream, batch, seq, batch * seq, seqlens, &ctx->prof};
  float* grads = grads_out ? grads_out : r.at<float>(r.p.grads);
  // The teacher's forward pass shares nothing with the quantized forward pass (its own scratch, its
  // own outputs), so it runs on a side stream, forked from the caller's stream and joined before
  // the loss: kernels of the two passes fill each other's tails.
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return fail(ctx, MREM_EHIP, "mrem_module_step: no current device");
  if (!ctx->side && !create_side(ctx, dev))
    return fail(ctx, MREM_EHIP, "mrem_module_step: cannot create the side stream and its events");
  if (dev != ctx->side_device) return fail(ctx, MREM_EINVAL, "mrem_module_step: the context was first used on another device");
  // What the second stream is worth depends on the size.  A wait for an event takes the host 11 us, five launches' time, and
  // with a handover for every product a layer needs nine of them, so a step of few tokens is bound by the host: 3 layers of
  // 256 over 66 tokens 718 us, 532 with one handover a layer, 551 on one stream; 3 of 512 over 427: 735, 664, 786; 6 of 1024
  // over 495: 2512, 2396, 2949.  From about 2^19 activations a layer on the device is the limit, and products that start
  // later cost up to 1.5% (2 of 768 over 992 tokens: 670, 681, 762; 6 of 1024 over 4096: 4305, 4350) unless the weight
  // gradients of a layer are one launch (wgrads_tile: 4261).  With one layer there is nothing to overlap the update with (1
  // of 1024 over 400: 435, 450, 469), and the shortest steps are quickest on one stream (1 of 64 over 128, fp32: 290, 235,
  // 198; 1 of 512 over 200: 282, 262, 255; 2 of 128 over 80: 494, 405, 332).
  const int64_t acts = (int64_t)r.T * ctx->H;
  const bool fork = !ctx->prof.on &&  // per-launch timing wants every product alone on the device
                    acts * ctx->L * ctx->L > (1 << 17);
  const bool few = ctx->L > 1 && acts <= (1 << 19);
  int wgrad_tile = 0;
  if (fork && ctx->L > 1 && !few) {
    const std::vector<WgradJob> jobs = wgrad_jobs(r, params, grads, 0, {r.p.dqkv, r.p.dr1, r.p.du, r.p.dr2});
    wgrad_tile = wgrads_tile(ctx->dt, jobs.data(), (int)jobs.size(), r.T);
  }
  // Eq. 4: with lambda > 0 the quantized module reads lambda * x_fp + (1 - lambda) * x_q, formed by its first kernel
  const bool mix = lambda > 0.f && x_fp != x_q;
  const void* x_in = mix ? r.at(r.p.xmix) : x_q;
  const void* mix_fp = mix ? x_fp : nullptr;
  // Before the passes: the gradient slots that are added into or never written are zeroed.
  if (fork) {
    Run rt = r;
    rt.st = ctx->side;
    (void)hipEventRecord(ctx->ev_fork, r.st);
    (void)hipStreamWaitEvent(ctx->side, ctx->ev_fork, 0);
    zero_gradient_slots(r, grads, wgrad_tile > 0);
    // Only the first layer's weights are prepared on this stream; those of the layers above are prepared on the side
    // stream ahead of the teacher's pass (which has slack before the loss needs it), so the quantized pass starts after
    // one layer's worth of that work instead of the whole module's.
    prepare_weights(r, params, true, 0, few ? -1 : 1);
    if (ctx->L > 1 && !few) {
      prepare_weights(rt, params, true, 1, ctx->L);
      (void)hipEventRecord(ctx->ev_codes, ctx->side);
    }
    // the two passes are enqueued layer by layer in turn, so that both streams have work from the
    // start also when the caller's queue was empty
    for (int l = 0; l < ctx->L; ++l) {
      teacher_forward(rt, teacher, teacher_cache, x_fp, per_layer_fp, l, l + 1);
      if (l == 1 && !few) (void)hipStreamWaitEvent(r.st, ctx->ev_codes, 0);
      student_forward(r, params, x_in, per_layer_q, true, l, l + 1, mix_fp, x_q, lambda);
    }
    (void)hipEventRecord(ctx->ev_join, ctx->side);
  } else {
    teacher_forward(r, teacher, teacher_cache, x_fp, per_layer_fp);
    zero_gradient_slots(r, grads, false);
    prepare_weights(r, params, true);
    student_forward(r, params, x_in, per_layer_q, true, 0, -1, mix_fp, x_q, lambda);
  }
  if (fork) (void)hipStreamWaitEvent(r.st, ctx->ev_join, 0);
  const Update up{params, adam_m, adam_v, adam_arg(ctx, step_index, lr), grads_out != nullptr, fork ? ctx->side : nullptr,
                  ctx->ev_layer.data(), ctx->ev_ready.data(), ctx->ev_done.data(), ctx->ev_join, few || wgrad_tile > 0, wgrad_tile};
  student_backward(r, params, x_in, per_layer_fp, per_layer_q, grads, loss_out, up);
  update_vectors(r, up, grads);
  return finish(ctx, "mrem_module_step");
}

// ------------------------------------------------------------------------------
// REM: the reconstruction step of ONE matrix product (Section 3.2, Eq. 2)
// ------------------------------------------------------------------------------
namespace {
struct RemPlan {
  size_t wt, wcodes, what, zcorr, xcodes, dy, dxh, partials, grads, total;
  int64_t n_vec;  // length of the flat vector [w | s_w | s_a, padded]
};
RemPlan rem_plan(int dt, int64_t T, int64_t N, int64_t K) {
  RemPlan p;
  Bump b;
  const size_t es = dt_size(dt);
  p.n_vec = ((N * K + N + 1 + 3) / 4) * 4;
  p.wt = b.take((size_t)N * K * es); p.wcodes = b.take((size_t)N * K * es); p.what = b.take((size_t)N * K * es);
  p.zcorr = b.take((size_t)N * 4);  // (nothing is kept here: the size of the workspace stays what callers have stored)
  p.xcodes = b.take((size_t)T * K * es); p.dy = b.take((size_t)T * N * es); p.dxh = b.take((size_t)T * K * es);
  p.partials = b.take(2 * 2048 * 4);
  p.grads = b.take((size_t)p.n_vec * 4);
  p.total = b.off;
  return p;
}
}  // namespace

extern "C" int64_t mrem_rem_vector_count(int64_t N, int64_t K) { return (N < 1 || K < 1) ? -1 : ((N * K + N + 1 + 3) / 4) * 4; }
extern "C" size_t mrem_rem_workspace_bytes(const mrem_ctx* ctx, int64_t T, int64_t N, int64_t K) {
  if (!ctx || T < 1 || N < 1 || K < 1) return 0;
  return rem_plan(ctx->dt, T, N, K).total;
}

extern "C" mrem_status mrem_rem_step(mrem_ctx* ctx, int64_t T, int64_t N, int64_t K, float* vec, float* adam_m, float* adam_v,
                                     int64_t step_index, float lr, const float* w_fp, const void* a_fp, const void* a_q, float* loss_out,
                                     void* y_fp, void* y_q, float* grads_out, void* workspace, size_t workspace_bytes, void* hip_stream) {
  const char* who = "mrem_rem_step";
  if (!ctx) return fail(nullptr, MREM_EINVAL, std::string(who) + ": null context");
  if (T < 1 || N < 1 || K < 1 || T % 8 || N % 8 || K % 8 || T * std::max(N, K) > 0x7fffffff || N * K > 0x7fffffff)
    return fail(ctx, MREM_ESHAPE, std::string(who) + ": T, N, K must be positive multiples of 8 (products below 2^31)");
  if (ctx->cfg.w_bits == 0 || ctx->cfg.a_bits == 0) return fail(ctx, MREM_EINVAL, std::string(who) + ": both quantizer families must be on");
  if (step_index < 1) return fail(ctx, MREM_EINVAL, std::string(who) + ": step_index is 1-based");
  REQUIRE_PTR(vec, who); REQUIRE_PTR(adam_m, who); REQUIRE_PTR(adam_v, who); REQUIRE_PTR(w_fp, who); REQUIRE_PTR(a_fp, who);
  REQUIRE_PTR(a_q, who); REQUIRE_PTR(loss_out, who); REQUIRE_PTR(y_fp, who); REQUIRE_PTR(y_q, who); REQUIRE_PTR(workspace, who);
  if (grads_out && !aligned16(grads_out)) return fail(ctx, MREM_EINVAL, std::string(who) + ": grads_out misaligned");
  const RemPlan p = rem_plan(ctx->dt, T, N, K);
  if (workspace_bytes < p.total) return fail(ctx, MREM_EWORKSPACE, std::string(who) + ": workspace too small");
  const int dt = ctx->dt;
  hipStream_t st = (hipStream_t)hip_stream;
  char* ws = (char*)workspace;
  float* w = vec;
  float* sw = vec + N * K;
  float* sa = vec + N * K + N;
  float* grads = grads_out ? grads_out : reinterpret_cast<float*>(ws + p.grads);
  float* parts = reinterpret_cast<float*>(ws + p.partials);
  GemmProfile* prof = &ctx->prof;
  // one launch for both weight sets: the frozen ones rounded to the storage type; codes and the dequantized copy of the trained ones
  WeightJob wj[2];
  // Whole tiles multiply int8 codes (4096 x 4096 x 1024: 20 us, 31 on bf16 ones); those of the weights take the place of their
  // bf16 codes, those of the input that of its gradient, which is written behind the product.  Not where a sum could leave int32.
  int8_t* const wcodes8 = reinterpret_cast<int8_t*>(ws + p.wcodes);
  int8_t* const xcodes8 = reinterpret_cast<int8_t*>(ws + p.dxh);
  const bool i8 = dt == DT_BF16 && gemm_i8_ok(xcodes8, (int)K, wcodes8, (int)K, (int)T, (int)N, (int)K) &&
                  i8_sums_fit(K, (1 << (ctx->cfg.a_bits - 1)) - 1, (1 << (ctx->cfg.w_bits - 1)) - 1);
  wj[0].w = w; wj[0].sw = sw; wj[0].codes = i8 ? nullptr : ws + p.wcodes; wj[0].what = ws + p.what; wj[0].zcorr = nullptr;
  wj[0].codes8 = i8 ? wcodes8 : nullptr;
  wj[0].N = (int)N; wj[0].K = (int)K;
  wj[1] = wj[0];
  wj[1].w = w_fp; wj[1].sw = nullptr; wj[1].codes = ws + p.wt; wj[1].codes8 = nullptr; wj[1].what = nullptr;
  weight_prepare(dt, wj, 2, ctx->cfg.w_bits, st);
  // full-precision product  y = a W^T  on the original weights
  gemm_nt(dt, a_fp, (int)K, ws + p.wt, (int)K, y_fp, (int)N, (int)T, (int)N, (int)K, Epilogue(), st, prof);
  // quantized product  y^ = Q(a) Q(w)^T: codes of both operands, the two steps in the epilogue
  QArg qa;
  qa.on = 1; qa.s = sa; qa.qp = (float)((1 << (ctx->cfg.a_bits - 1)) - 1); qa.qn = -qa.qp;
  act_quantize(dt, a_q, ws + p.xcodes, T * K, qa, st, i8 ? xcodes8 : nullptr);
  // Eq. 2 and its gradient with respect to y^, by the product's kernel where it can (4096 x 4096 x 1024: 33 us for what took 31 on bf16 codes and 16 in a pass over three tensors)
  const float scale = ctx->cfg.loss_mean ? 1.0f / (float)((double)T * (double)N) : 1.0f;
  int nl = 0, ns = 0;
  Epilogue e;
  e.alpha = sa; e.col_scale = sw;
  const bool fused_loss = dt == DT_BF16 && post_ok((int)T, (int)N, (int)(i8 ? K / 2 : K));
  if (fused_loss) {
    e.post = POST_MSE; e.post_in = y_fp; e.post_out = ws + p.dy; e.post_parts = parts; e.post_scale = scale; e.blocks = &nl;
  }
  if (i8) gemm_i8(xcodes8, (int)K, wcodes8, (int)K, y_q, (int)N, (int)T, (int)N, (int)K, e, st, prof);
  else gemm_nt(dt, ws + p.xcodes, (int)K, ws + p.wcodes, (int)K, y_q, (int)N, (int)T, (int)N, (int)K, e, st, prof);
  if (!fused_loss) nl = mse_grad(dt, y_q, y_fp, ws + p.dy, T * N, scale, parts, st);
  // straight-through backward: d w^ = dy^T a^ (the update kernel applies the mask and forms ds_w), d a^ = dy W^ for ds_a
  Epilogue ew;
  ew.alpha = sa; ew.out_f32 = 1;
  gemm(dt, 1, 1, ws + p.dy, (int)N, ws + p.xcodes, (int)K, grads, (int)K, (int)N, (int)K, (int)T, ew, st, prof);
  Epilogue ex;
  const bool fused_step = dt == DT_BF16 && post_ok((int)T, (int)K, (int)N);
  if (fused_step) {
    // (only its sum is needed; it is left in the workspace where gradients are asked for)
    ex.post = POST_STEP; ex.post_in = a_q; ex.post_out = grads_out ? ws + p.dxh : nullptr; ex.post_parts = parts + 2048; ex.post_q = qa; ex.blocks = &ns;
  }
  gemm(dt, 0, 1, ws + p.dy, (int)N, ws + p.what, (int)K, ws + p.dxh, (int)K, (int)T, (int)K, (int)N, ex, st, prof);
  if (!fused_step) ns = quant_bwd_reduce(dt, ws + p.dxh, a_q, T * K, qa, parts + 2048, st);
  ReduceJob jobs[2];
  jobs[0].partials = parts; jobs[0].nparts = nl; jobs[0].width = 1; jobs[0].begin = 0; jobs[0].len = 1; jobs[0].out = loss_out; jobs[0].scale = scale;
  jobs[1].partials = parts + 2048; jobs[1].nparts = ns; jobs[1].width = 1; jobs[1].begin = 0; jobs[1].len = 1; jobs[1].out = grads + N * K + N;
  // AdamW on w (decay) and s_w, and on s_a (no decay, floor) behind its gradient
  const AdamArg a = adam_arg(ctx, step_index, lr);
  AdamJob aj;
  aj.w = w; aj.sw = sw; aj.g_w = grads; aj.g_sw = grads + N * K; aj.m_w = adam_m; aj.v_w = adam_v; aj.m_sw = adam_m + N * K; aj.v_sw = adam_v + N * K;
  aj.z_in = nullptr; aj.db = nullptr; aj.N = (int)N; aj.K = (int)K;
  adam_matrix(&aj, 1, ctx->cfg.w_bits, a, grads_out != nullptr, ctx->cfg.per_channel ? 0 : 1, st);
  AdamArg nodecay = a;
  nodecay.wd = 0.f;
  reduce_and_step(jobs[0], jobs[1], sa, adam_m + N * K + N, adam_v + N * K + N, nodecay, st);
  return finish(ctx, who);
}

extern "C" mrem_status mrem_mix_inputs(mrem_ctx* ctx, const void* x_fp, const void* x_q, float lambda, void* out, int64_t n,
                                       void* hip_stream) {
  if (!ctx) return fail(nullptr, MREM_EINVAL, "mrem_mix_inputs: null context");
  REQUIRE_PTR(x_fp, "mrem_mix_inputs");
  REQUIRE_PTR(x_q, "mrem_mix_inputs");
  REQUIRE_PTR(out, "mrem_mix_inputs");
  if (n < 1) return fail(ctx, MREM_ESHAPE, "mrem_mix_inputs: n must be >= 1");
  if (!(lambda >= 0.f && lambda <= 1.f)) return fail(ctx, MREM_EINVAL, "mrem_mix_inputs: lambda must be in [0,1]");
  axpby(ctx->dt, x_fp, x_q, lambda, 1.f - lambda, out, n, (hipStream_t)hip_stream);
  return finish(ctx, "mrem_mix_inputs");
}

extern "C" mrem_status mrem_profile_gemm_begin(mrem_ctx* ctx) {
  if (!ctx) return fail(nullptr, MREM_EINVAL, "mrem_profile_gemm_begin: null context");
  gemm_profile_begin(&ctx->prof);
  return MREM_OK;
}
extern "C" mrem_status mrem_profile_gemm_end(mrem_ctx* ctx, double* ms, double* flops, int64_t* launches) {
  if (!ctx || !ms || !flops || !launches) return fail(ctx, MREM_EINVAL, "mrem_profile_gemm_end: null argument");
  return gemm_profile_end(&ctx->prof, ms, flops, launches) == 0 ? MREM_OK : fail(ctx, MREM_EHIP, "mrem_profile_gemm_end: event query failed");
}

extern "C" int32_t mrem_profile_kernel_count(const mrem_ctx* ctx) { return ctx ? (int32_t)ctx->prof.stats.size() : -1; }
extern "C" mrem_status mrem_profile_kernel_get(const mrem_ctx* ctx, int32_t i, char* name, int32_t name_bytes, double* ms, double* bytes,
                                               int64_t* launches) {
  if (!ctx || !name || name_bytes < 1 || !ms || !bytes || !launches) return fail(ctx, MREM_EINVAL, "mrem_profile_kernel_get: null argument");
  if (i < 0 || i >= (int32_t)ctx->prof.stats.size()) return fail(ctx, MREM_EINVAL, "mrem_profile_kernel_get: no such entry");
  const KernelStat& k = ctx->prof.stats[(size_t)i];
  snprintf(name, (size_t)name_bytes, "%s", k.label);
  *ms = k.ms; *bytes = k.bytes; *launches = k.launches;
  return MREM_OK;
}

extern "C" mrem_status mrem_set_nonfinite_flag(mrem_ctx* ctx, int32_t* device_flag) {
  if (!ctx) return fail(nullptr, MREM_EINVAL, "mrem_set_nonfinite_flag: null context");
  if (device_flag && (reinterpret_cast<uintptr_t>(device_flag) & 3u)) return fail(ctx, MREM_EINVAL, "mrem_set_nonfinite_flag: misaligned flag");
  ctx->nonfinite_flag = device_flag;
  return MREM_OK;
}
extern "C" mrem_status mrem_check_nonfinite(mrem_ctx* ctx, void* hip_stream) {
  if (!ctx) return fail(nullptr, MREM_EINVAL, "mrem_check_nonfinite: null context");
  if (!ctx->nonfinite_flag) return fail(ctx, MREM_EINVAL, "mrem_check_nonfinite: no flag has been set");
  int32_t host = 0;
  if (hipStreamSynchronize((hipStream_t)hip_stream) != hipSuccess ||
      hipMemcpy(&host, ctx->nonfinite_flag, sizeof(host), hipMemcpyDeviceToHost) != hipSuccess)
    return fail(ctx, MREM_EHIP, "mrem_check_nonfinite: cannot read the flag");
  if (host) return fail(ctx, MREM_ENONFINITE, "a step since the flag was last cleared produced a non-finite loss");
  return MREM_OK;
}

// ------------------------------------------------------------------------------
// schedules (host arithmetic) and the input queue of Algorithm 1
// ------------------------------------------------------------------------------
extern "C" double mrem_schedule_lr(double lr0, int64_t t, int64_t total) {
  if (total < 1 || t < 0) return 0.0;
  return lr0 * (1.0 - (double)t / (double)total);
}
extern "C" double mrem_schedule_lambda(int64_t t, int64_t tf_steps) {
  if (tf_steps < 1 || t < 0) return 0.0;
  const double l = 1.0 - (double)t / (double)tf_steps;
  return l > 0.0 ? l : 0.0;
}

struct mrem_queue {
  int depth;            // readable entries
  size_t half_bytes, len_bytes;
  char* mem;            // device, caller-owned: (depth + 1) slots of [fp half | q half | lengths]
  int64_t published;    // entries handed over so far
  size_t slot_bytes() const { return 2 * half_bytes + len_bytes; }
};
static size_t round256(size_t b) { return (b + 255) & ~size_t(255); }
extern "C" size_t mrem_queue_bytes(int32_t depth, size_t half_bytes, size_t lengths_bytes) {
  if (depth < 1) return 0;
  return (size_t)(depth + 1) * (2 * round256(half_bytes) + round256(lengths_bytes));
}
extern "C" mrem_status mrem_queue_create(int32_t depth, size_t half_bytes, size_t lengths_bytes, void* device_mem, mrem_queue** out) {
  if (!out || !device_mem || !aligned16(device_mem)) return fail(nullptr, MREM_EINVAL, "mrem_queue_create: null or misaligned argument");
  if (depth < 1 || half_bytes < 1) return fail(nullptr, MREM_ESHAPE, "mrem_queue_create: depth and half_bytes must be >= 1");
  mrem_queue* q = new mrem_queue();
  q->depth = depth; q->half_bytes = round256(half_bytes); q->len_bytes = round256(lengths_bytes); q->mem = (char*)device_mem; q->published = 0;
  *out = q;
  return MREM_OK;
}
extern "C" void mrem_queue_destroy(mrem_queue* q) { delete q; }
extern "C" int32_t mrem_queue_size(const mrem_queue* q) { return q ? (int32_t)(q->published < q->depth ? q->published : q->depth) : -1; }
extern "C" mrem_status mrem_queue_write_slot(mrem_queue* q, void** fp, void** qd, void** lengths) {
  if (!q || !fp || !qd) return fail(nullptr, MREM_EINVAL, "mrem_queue_write_slot: null argument");
  char* slot = q->mem + (size_t)(q->published % (q->depth + 1)) * q->slot_bytes();
  *fp = slot; *qd = slot + q->half_bytes;
  if (lengths) *lengths = q->len_bytes ? slot + 2 * q->half_bytes : nullptr;
  return MREM_OK;
}
extern "C" mrem_status mrem_queue_push(mrem_queue* q, const void* fp, const void* qd, const void* lengths, size_t half_bytes,
                                       size_t lengths_bytes, void* hip_stream) {
  if (!q || !fp || !qd) return fail(nullptr, MREM_EINVAL, "mrem_queue_push: null argument");
  if (half_bytes > q->half_bytes || lengths_bytes > q->len_bytes) return fail(nullptr, MREM_ESHAPE, "mrem_queue_push: entry larger than a slot");
  void *dfp, *dq, *dl;
  (void)mrem_queue_write_slot(q, &dfp, &dq, &dl);
  hipStream_t st = (hipStream_t)hip_stream;
  bool ok = hipMemcpyAsync(dfp, fp, half_bytes, hipMemcpyDeviceToDevice, st) == hipSuccess &&
            hipMemcpyAsync(dq, qd, half_bytes, hipMemcpyDeviceToDevice, st) == hipSuccess;
  if (lengths && lengths_bytes) ok = ok && hipMemcpyAsync(dl, lengths, lengths_bytes, hipMemcpyDeviceToDevice, st) == hipSuccess;
  return ok ? MREM_OK : fail(nullptr, MREM_EHIP, "mrem_queue_push: copy failed");
}
extern "C" mrem_status mrem_queue_publish(mrem_queue* q) {
  if (!q) return fail(nullptr, MREM_EINVAL, "mrem_queue_publish: null queue");
  q->published += 1;
  return MREM_OK;
}
extern "C" mrem_status mrem_queue_entry(const mrem_queue* q, int32_t age, void** fp, void** qd, void** lengths) {
  if (!q || !fp || !qd) return fail(nullptr, MREM_EINVAL, "mrem_queue_entry: null argument");
  if (age < 0 || age >= mrem_queue_size(q)) return fail(nullptr, MREM_EINVAL, "mrem_queue_entry: no entry of that age");
  char* slot = q->mem + (size_t)((q->published - 1 - age) % (q->depth + 1)) * q->slot_bytes();
  *fp = slot; *qd = slot + q->half_bytes;
  if (lengths) *lengths = q->len_bytes ? slot + 2 * q->half_bytes : nullptr;
  return MREM_OK;
}
