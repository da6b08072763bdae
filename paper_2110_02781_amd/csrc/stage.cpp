// Model description, stage object and the C ABI entry points for
// forward / loss / backward / update / weight stashing / profiling.
//
// A stage executes its units as a fixed sequence of kernel launches on the
// caller's stream.  Every convolution writes its raw output z once; the
// following BatchNorm is reduced to a per-channel scale/shift that the NEXT
// kernel applies on load together with the activation ("view"), so activated
// tensors are never written except at block outputs (where the residual is
// added) and at the stage boundary.  Backward mirrors this: per convolution a
// reduction for d(gamma), d(beta), one elementwise pass that forms dz, then
// weight- and data-gradient kernels.
#include <hip/hip_runtime.h>
#include <sys/mman.h>
#include <unistd.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/ftp.h"
#include "kernels.h"

using namespace ftp;

// ------------------------------------------------------------------ errors
static thread_local char g_err[512] = "";
void ftp_set_error(const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
}
extern "C" const char* ftp_last_error(void) { return g_err; }

#define HIP_TRY(expr)                                                              \
  do {                                                                             \
    hipError_t e_ = (expr);                                                        \
    if (e_ != hipSuccess) {                                                        \
      ftp_set_error("%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), __FILE__, __LINE__); \
      return FTP_ERR_HIP;                                                          \
    }                                                                              \
  } while (0)

static const float kBnEps = 1e-5f, kBnMomentum = 0.1f;
// What the stores of a stage that defers its weight gradients may take whatever its layers' sizes: bytes, floats.  (Emptying them
// earlier costs launches that no longer fill the GPU: with 64 MB of partials and no more than two activations of dz a step at 224x224
// was 1.5 - 2.5 % longer, fp32 batch 32 and 64, bfloat16 batch 32 and 128.)
static const size_t kDzStore = (size_t)128 << 20, kPartStore = (size_t)32 << 20, kDzRing = (size_t)64 << 20;

static inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
static inline int conv_out(int n, int k, int s, int p) { return (n + 2 * p - k) / s + 1; }

// ------------------------------------------------------------------- model
enum SubType { SUB_DIRECT = 0, SUB_PW = 1, SUB_DW = 2 };

struct Sub {           // convolution + BatchNorm + activation
  int type;
  ConvGeom g;          // N filled in per stage
  int act;
  size_t w_off, w_n;   // offsets relative to the unit's parameter vector
  size_t gamma_off, beta_off;
  size_t bn_off;       // channel offset relative to the unit's BatchNorm channels
};

struct UnitInfo {
  ftp_unit_desc d;
  int inH, inW, inC, outH, outW, outC;
  std::vector<Sub> subs;
  bool residual;
  size_t n_param, n_bn;
};

struct ftp_model {
  std::vector<UnitInfo> units;
  int dtype;
  int inH, inW, inC;
};

static int build_unit(const ftp_unit_desc& d, int H, int W, int C, int idx, UnitInfo* u) {
  u->d = d;
  u->inH = H; u->inW = W; u->inC = C;
  u->residual = false;
  u->n_param = 0; u->n_bn = 0;
  auto add_sub = [&](int type, int Hin, int Win, int Cin, int Cout, int kh, int kw, int s, int ph, int pw, int act) {
    Sub sb;
    sb.type = type;
    sb.g = ConvGeom{0, Hin, Win, Cin, conv_out(Hin, kh, s, ph), conv_out(Win, kw, s, pw), Cout, kh, kw, s, ph, pw};
    sb.act = act;
    sb.w_off = u->n_param;
    sb.w_n = (size_t)Cout * kh * kw * (type == SUB_DW ? 1 : Cin);
    sb.gamma_off = sb.w_off + sb.w_n;
    sb.beta_off = sb.gamma_off + Cout;
    sb.bn_off = u->n_bn;
    u->n_param = sb.beta_off + Cout;
    u->n_bn += Cout;
    u->subs.push_back(sb);
    return sb;
  };
  switch (d.kind) {
    case FTP_UNIT_CONV: {
      if (d.cin != C || d.cout < 8 || d.cout % 8 || d.kh < 1 || d.kw < 1 || d.stride < 1 || d.pad_h < 0 || d.pad_w < 0 ||
          d.act < 0 || d.act > 2) {
        ftp_set_error("unit %d (CONV): cin=%d must equal incoming channels %d, cout=%d a multiple of 8", idx, d.cin, C, d.cout);
        return FTP_ERR_SHAPE;
      }
      if (H + 2 * d.pad_h < d.kh || W + 2 * d.pad_w < d.kw) { ftp_set_error("unit %d: kernel larger than padded input", idx); return FTP_ERR_SHAPE; }
      bool pw = d.kh == 1 && d.kw == 1 && d.stride == 1 && d.pad_h == 0 && d.pad_w == 0 && C % 8 == 0;
      Sub sb = add_sub(pw ? SUB_PW : SUB_DIRECT, H, W, C, d.cout, d.kh, d.kw, d.stride, d.pad_h, d.pad_w, d.act);
      if (!pw && !conv_direct_supported(sb.g)) {
        ftp_set_error("unit %d: dense %dx%d conv with cin*cout=%d > 8192 is not supported", idx, d.kh, d.kw, C * d.cout);
        return FTP_ERR_UNSUPPORTED;
      }
      u->outH = sb.g.Hout; u->outW = sb.g.Wout; u->outC = d.cout;
      break;
    }
    case FTP_UNIT_INVRES: {
      if (d.cin != C || C % 8 || d.cout < 8 || d.cout % 8 || d.expand < 1 || (d.stride != 1 && d.stride != 2)) {
        ftp_set_error("unit %d (INVRES): cin=%d must equal incoming channels %d; channels multiples of 8; stride 1 or 2", idx, d.cin, C);
        return FTP_ERR_SHAPE;
      }
      int ce = C * d.expand;
      // the depthwise kernels address inside one image with 32-bit offsets formed from 24-bit factors
      if ((size_t)H * W >= ((size_t)1 << 24) || (size_t)H * W * ce >= ((size_t)1 << 31) || ce >= (1 << 24)) {
        ftp_set_error("unit %d (INVRES): a %dx%dx%d expanded feature map is beyond the depthwise kernels' in-image offsets "
                      "(H*W < 2^24 and H*W*C < 2^31)", idx, H, W, ce);
        return FTP_ERR_UNSUPPORTED;
      }
      if (d.expand != 1) add_sub(SUB_PW, H, W, C, ce, 1, 1, 1, 0, 0, FTP_ACT_RELU6);
      Sub dw = add_sub(SUB_DW, H, W, ce, ce, 3, 3, d.stride, 1, 1, FTP_ACT_RELU6);
      add_sub(SUB_PW, dw.g.Hout, dw.g.Wout, ce, d.cout, 1, 1, 1, 0, 0, FTP_ACT_NONE);
      u->outH = dw.g.Hout; u->outW = dw.g.Wout; u->outC = d.cout;
      u->residual = d.stride == 1 && d.cin == d.cout;
      break;
    }
    case FTP_UNIT_GAP:
      if (C % 8) { ftp_set_error("unit %d (GAP): channels must be a multiple of 8", idx); return FTP_ERR_SHAPE; }
      u->outH = 1; u->outW = 1; u->outC = C;
      break;
    case FTP_UNIT_FC:
      if (H != 1 || W != 1 || d.cin != C || d.cout < 1 || C % 8) {
        ftp_set_error("unit %d (FC): needs a [batch,1,1,%d] input with cin %% 8 == 0 (got %dx%dx%d)", idx, d.cin, H, W, C);
        return FTP_ERR_SHAPE;
      }
      u->n_param = (size_t)d.cout * C + d.cout;
      u->outH = 1; u->outW = 1; u->outC = d.cout;
      break;
    case FTP_UNIT_LOSS:
      if (H != 1 || W != 1 || d.cin != C) { ftp_set_error("unit %d (LOSS): needs [batch,1,1,classes] logits", idx); return FTP_ERR_SHAPE; }
      u->outH = 1; u->outW = 1; u->outC = C;
      break;
    default:
      ftp_set_error("unit %d: unknown kind %d", idx, d.kind);
      return FTP_ERR_ARG;
  }
  if (u->outH < 1 || u->outW < 1) { ftp_set_error("unit %d: empty output", idx); return FTP_ERR_SHAPE; }
  return FTP_OK;
}

extern "C" int ftp_model_create(const ftp_unit_desc* units, int L, int in_h, int in_w, int in_c, ftp_dtype act_dtype,
                                ftp_model** out) {
  if (!units || !out || L < 1 || in_h < 1 || in_w < 1 || in_c < 1 || (act_dtype != FTP_F32 && act_dtype != FTP_BF16)) {
    ftp_set_error("model_create: bad argument");
    return FTP_ERR_ARG;
  }
  ftp_model* m = new (std::nothrow) ftp_model();
  if (!m) { ftp_set_error("model_create: out of host memory"); return FTP_ERR_NOMEM; }
  m->dtype = (int)act_dtype;
  m->inH = in_h; m->inW = in_w; m->inC = in_c;
  int H = in_h, W = in_w, C = in_c;
  for (int i = 0; i < L; ++i) {
    UnitInfo u;
    int rc = build_unit(units[i], H, W, C, i, &u);
    if (rc != FTP_OK) { delete m; return rc; }
    if (units[i].kind == FTP_UNIT_LOSS && i + 1 != L) { ftp_set_error("unit %d: LOSS must be the last unit", i); delete m; return FTP_ERR_SHAPE; }
    if (units[i].kind == FTP_UNIT_LOSS && i > 0 && units[i - 1].kind == FTP_UNIT_CONV) {
      ftp_set_error("unit %d: LOSS may not directly follow a CONV unit", i); delete m; return FTP_ERR_SHAPE;
    }
    H = u.outH; W = u.outW; C = u.outC;
    m->units.push_back(u);
  }
  *out = m;
  return FTP_OK;
}

extern "C" void ftp_model_destroy(ftp_model* m) { delete m; }
extern "C" int ftp_model_num_units(const ftp_model* m) { return m ? (int)m->units.size() : FTP_ERR_ARG; }

extern "C" int ftp_model_unit_in_shape(const ftp_model* m, int u, int* h, int* w, int* c) {
  if (!m || u < 0 || u > (int)m->units.size() || !h || !w || !c) { ftp_set_error("unit_in_shape: bad argument"); return FTP_ERR_ARG; }
  if (u == (int)m->units.size()) { const UnitInfo& x = m->units.back(); *h = x.outH; *w = x.outW; *c = x.outC; }
  else { const UnitInfo& x = m->units[u]; *h = x.inH; *w = x.inW; *c = x.inC; }
  return FTP_OK;
}
extern "C" int ftp_model_unit_param_count(const ftp_model* m, int u, size_t* n) {
  if (!m || u < 0 || u >= (int)m->units.size() || !n) { ftp_set_error("unit_param_count: bad argument"); return FTP_ERR_ARG; }
  *n = m->units[u].n_param;
  return FTP_OK;
}
extern "C" int ftp_model_unit_bn_channels(const ftp_model* m, int u, size_t* n) {
  if (!m || u < 0 || u >= (int)m->units.size() || !n) { ftp_set_error("unit_bn_channels: bad argument"); return FTP_ERR_ARG; }
  *n = m->units[u].n_bn;
  return FTP_OK;
}

// -------------------------------------------------------------------- stage
struct UnitPlan {
  const UnitInfo* info;
  size_t p_off;                    // float offset of the unit's parameters in the flat buffers
  size_t bn_off;                   // channel offset in the running-stat arrays
  std::vector<size_t> z_off;       // per sub: byte offset of z in the slot stash
  std::vector<size_t> st_off;      // per sub: float offset of mean|invstd|scale|shift in the slot stats
  std::vector<size_t> part;        // per sub: floats of its partial weight gradients (stages that defer them)
  size_t late_part, late_floats;   // floats in front of its depthwise layer's place in ws_late, and those of the place
  std::vector<char> at_once;       // per sub: a pointwise layer of such a stage whose weight gradient runs next to its data gradient all the same
  std::vector<char> axis;          // per sub: a convolution along one axis that the kernels for those run
  size_t out_off;                  // byte offset of the materialised unit output (if any)
  bool out_virtual;                // CONV unit whose output stays a view
  size_t in_mat_off;               // residual block fed by a view: materialised copy of its input
  bool need_in_mat;
  size_t open_off;                 // an average behind a convolution: byte offset of what its forward leaves of the activation (gap_fwd's open)
};

struct Slot {
  char* stash = nullptr;     // intermediates; with recomputation all slots point at the stage's one shared stash
  char* xin_keep = nullptr;  // recomputation: the slot's own copy of its stage input
  float* stats = nullptr;
  float* snap_w = nullptr;   // fp32 parameter snapshot
  int timer_idx = -1;        // ring entry of the batch in this slot when execution timing is on
  void* snap_lp = nullptr;   // bfloat16 working-copy snapshot
  void* dlogits = nullptr;
  bool busy = false, has_snap = false, has_loss = false;
};

struct ProfEvents {          // optional per-unit timing (profile_layers)
  std::vector<hipEvent_t> f0, f1, b0, b1;
};

// Optional per-batch execution time of the stage (the online profiling that feeds the capacity estimate):
// a ring of event quadruples, one per forwarded batch, harvested by ftp_stage_timing_read.
struct ExecTimer {
  enum { kRing = 256 };
  hipEvent_t ev[kRing][4];       // forward begin/end, backward begin/end
  bool bwd_done[kRing];
  int used = 0;                  // entries handed out since the last read
  bool created = false;
};

struct ftp_stage {
  const ftp_model* model;
  int a, b, batch, dt, device;
  size_t es;
  std::vector<UnitPlan> plan;
  size_t n_param = 0, n_bn = 0;
  float *params = nullptr, *grads = nullptr, *mom = nullptr, *run_mean = nullptr, *run_var = nullptr;
  void* w_lp = nullptr;
  size_t stash_bytes = 0, stats_floats = 0, xin_bytes = 0, max_act_bytes = 0;
  std::vector<Slot> slots;
  char *gbuf[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};   // boundary A/B, dz (even), dA, dz (odd); no dz ones in a stage that defers
  // Weight gradients depend on nothing downstream, so in backward they run on a second stream next to the
  // data-gradient chain: fork after dz is formed, join before that dz buffer is overwritten / at the end.
  hipStream_t side = nullptr;
  // fork / join of the side stream: one pair per dz buffer, and a third for the partial sums of the one-pass expand backward
  hipEvent_t ev_fork[3] = {nullptr, nullptr, nullptr}, ev_join[3] = {nullptr, nullptr, nullptr};
  bool join_pending[3] = {false, false, false};
  // Weight gradients of an inverted-residual unit whose tensors are small (kernels of 10 - 40 us): an event record
  // between two kernels of a stream costs about 3 us and a wait for a recent event of the other stream about 2 (both
  // measured), per layer as much as a finalize kernel.  Such a unit forks ONCE, behind its last layer: its layers write
  // their dz into a set of three buffers of their own (two sets, alternating from unit to unit), the weight gradients
  // are noted and all enqueued on the side stream at the end of the unit.
  struct PendingWgrad { const void* dz; HView in; ConvGeom g; size_t M; float* gw; };
  PendingWgrad pend[3];
  int n_pend = 0;
  char* dzring[6] = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
  size_t dzring_bytes = 0;
  hipEvent_t ev_bfork[2] = {nullptr, nullptr}, ev_bjoin[2] = {nullptr, nullptr};
  bool bjoin_pending[2] = {false, false};
  int bset = 0;
  bool bset_open = false;      // a layer of the current unit has written into the set
  // A stage that does not run weight gradients on a second stream (ftp_stage_create_ex says when) notes them instead: the
  // layers' dz and partial sums lie one behind the other in two stores, and the pointwise weight gradients of all layers run together at the
  // end of the backward call, a few launches for all of them, or earlier where the next layer does not fit a store any more.
  bool defers = false;
  char* dz_store = nullptr;
  float* parts = nullptr;
  size_t dz_cap = 0, dz_used = 0, part_cap = 0, part_used = 0;      // bytes, floats
  PwShare share{0, 0};         // pointwise layers that share the launches of weight gradients
  std::vector<PwWgradJob> q_pw;
  std::vector<ReduceJob> q_red;
  // Partial weight gradients that a stage on two streams leaves on the caller's until the end of the call: those of depthwise layers
  // (a place for each in ws_late) and of its first unit's expand layer, behind which nothing is left to run beside.
  std::vector<ReduceJob> q_late;
  float* ws_late = nullptr;
  size_t ws_late_floats = 0;
  unsigned n_sub_bwd = 0;
  float *bn_part = nullptr, *coef = nullptr, *ws = nullptr, *row_loss = nullptr;
  unsigned* arrived = nullptr;
  // A second partial-sum workspace for the weight gradient of the stage's very first layer when the stage forks
  // its weight gradients: that layer has no data gradient, so nothing follows it on the caller's stream and it
  // runs there, next to whatever the side stream still has queued, instead of behind it.
  float* ws_tail = nullptr;
  size_t ws_tail_floats = 0;
  // partial sums of the one-pass backward of the expand layers: it runs on the caller's stream while the side stream
  // may be using ws, so it has a workspace of its own
  float* ws_fused = nullptr;
  size_t ws_fused_floats = 0;
  int n_direct = 0;           // sublayers that use the patch-matrix buffer
  void* im2col = nullptr;     // patch matrix for the weight gradient of small dense convolutions
  // The conv output whose input patches the buffer holds right now (nullptr: none).  A forward that goes through the
  // patch matrix leaves it behind; if nothing has used the buffer since, the weight gradient of the same layer and
  // slot takes it as it is instead of writing the same matrix again.
  const void* im2col_of = nullptr;
  // BatchNorm-backward partial sums that the data gradient of a layer has left while it wrote the gradient tensor `of` (nullptr: none), for the
  // layer that reads that tensor next: where in bn_part they are, and how many.  Whoever leaves them sets all three (leave_sums), whoever needs
  // sums asks for them by its gradient tensor (take_sums).
  struct LeftSums { const void* of = nullptr; float* partial = nullptr; int P = 0; } left;
  size_t im2col_elems = 0;
  size_t ws_floats = 0;
  int max_c = 0;
  bool has_loss = false;
  int classes = 0;
  ProfEvents* prof = nullptr;
  ExecTimer* timer = nullptr;   // non-null while execution timing is enabled
  // Recomputation: slots keep only their stage input; the intermediates of the batch whose forward ran last
  // live in one shared stash, and a backward of any other slot first runs the forward again.
  bool recompute = false;
  char* shared_stash = nullptr;
  int stash_owner = -1;         // slot whose intermediates the shared stash holds
  float bn_mom = kBnMomentum;   // 0 while a forward is being recomputed: running statistics stay put
  size_t dev_bytes = 0;         // device memory the stage allocated
};

static inline void dfree(void* p) { if (p) (void)hipFree(p); }

static void stage_free(ftp_stage* s) {
  if (!s) return;
  dfree(s->params); dfree(s->grads); dfree(s->mom); dfree(s->run_mean); dfree(s->run_var); dfree(s->w_lp);
  for (auto& sl : s->slots) { if (!s->recompute) dfree(sl.stash); dfree(sl.xin_keep); dfree(sl.stats); dfree(sl.snap_w); dfree(sl.snap_lp); dfree(sl.dlogits); }
  dfree(s->shared_stash);
  for (int i = 0; i < 5; ++i) dfree(s->gbuf[i]);
  if (s->side) (void)hipStreamDestroy(s->side);
  for (int i = 0; i < 3; ++i) {
    if (s->ev_fork[i]) (void)hipEventDestroy(s->ev_fork[i]);
    if (s->ev_join[i]) (void)hipEventDestroy(s->ev_join[i]);
  }
  for (int i = 0; i < 2; ++i) {
    if (s->ev_bfork[i]) (void)hipEventDestroy(s->ev_bfork[i]);
    if (s->ev_bjoin[i]) (void)hipEventDestroy(s->ev_bjoin[i]);
  }
  for (int i = 0; i < 6; ++i) dfree(s->dzring[i]);
  dfree(s->bn_part); dfree(s->coef); dfree(s->ws); dfree(s->ws_tail); dfree(s->ws_fused); dfree(s->ws_late); dfree(s->row_loss); dfree(s->arrived); dfree(s->im2col);
  dfree(s->dz_store); dfree(s->parts);
  if (s->timer) {
    if (s->timer->created)
      for (auto& q : s->timer->ev)
        for (auto& e : q) (void)hipEventDestroy(e);
    delete s->timer;
  }
  delete s;
}

extern "C" void ftp_stage_destroy(ftp_stage* s) { stage_free(s); }

static thread_local size_t g_alloc_total = 0;

template <typename P>
static int dev_alloc(P** p, size_t bytes) {
  void* q = nullptr;
  hipError_t e = hipMalloc(&q, align_up(bytes ? bytes : 1, 256));
  if (e != hipSuccess) { ftp_set_error("hipMalloc(%zu bytes) failed: %s", bytes, hipGetErrorString(e)); return FTP_ERR_NOMEM; }
  *p = (P*)q;
  g_alloc_total += align_up(bytes ? bytes : 1, 256);
  return FTP_OK;
}

extern "C" int ftp_stage_create_ex(const ftp_model* m, int a, int b, int batch, int n_slots, unsigned flags, ftp_stage** out) {
  if (!m || !out) { ftp_set_error("stage_create: NULL argument"); return FTP_ERR_ARG; }
  if (flags & ~(unsigned)FTP_STAGE_RECOMPUTE) { ftp_set_error("stage_create: unknown flags 0x%x", flags); return FTP_ERR_ARG; }
  int L = (int)m->units.size();
  if (a < 0 || a >= b || b > L) { ftp_set_error("stage_create: bad unit range [%d,%d) for %d units", a, b, L); return FTP_ERR_ARG; }
  if (batch < 1 || n_slots < 1 || n_slots > 64) { ftp_set_error("stage_create: batch >= 1 and 1 <= n_slots <= 64 required"); return FTP_ERR_ARG; }
  ftp_stage* s = new (std::nothrow) ftp_stage();
  if (!s) { ftp_set_error("stage_create: out of host memory"); return FTP_ERR_NOMEM; }
  s->model = m; s->a = a; s->b = b; s->batch = batch; s->dt = m->dtype;
  s->recompute = (flags & FTP_STAGE_RECOMPUTE) != 0;
  g_alloc_total = 0;
  s->es = m->dtype == FTP_F32 ? 4 : 2;
  if (hipGetDevice(&s->device) != hipSuccess) { ftp_set_error("stage_create: no HIP device"); delete s; return FTP_ERR_HIP; }

  size_t stash = 0, stats = 0, max_act = 0, ws_floats = 1024, layer_ws = 0, n_convs = 0, z_values = 0;
  size_t dz_bytes = 0, dz_max = 0, part_floats = 0, part_max = 0;
  size_t n_long = 0, n_narrow = 0, short_rows = 0, short_products = 0;      // pointwise layers outside the transposing kernel
  int max_c = 8;
  auto act_bytes = [&](int H, int W, int C) { return align_up((size_t)batch * H * W * C * s->es, 256); };
  const UnitInfo& first = m->units[a];
  s->xin_bytes = act_bytes(first.inH, first.inW, first.inC);
  stash += s->xin_bytes;
  max_act = s->xin_bytes;
  for (int i = a; i < b; ++i)
    for (const Sub& sb : m->units[i].subs) {
      const size_t M = (size_t)batch * sb.g.Hout * sb.g.Wout;
      z_values += M * sb.g.Cout;
      ++n_convs;
      if (sb.type != SUB_PW || (m->dtype == FTP_BF16 && pw_bwd_fused_ws(M, sb.g.Cin, sb.g.Cout) > 0)) continue;
      if (pw_wgrad_tr_ok(m->dtype, M, sb.g.Cin, sb.g.Cout)) { ++s->share.tr; continue; }
      ++s->share.other;
      if (M > 2048) { ++n_long; n_narrow += sb.g.Cout <= 32 && M >= 16384; continue; }
      short_rows += M;
      short_products += M * sb.g.Cin * sb.g.Cout;
    }
  // Two ways to keep weight gradients off the data-gradient chain: all of them at the end of the call, or each on a second
  // stream as soon as its dz is there.  The second costs event calls and a division of the memory bandwidth, and pays only where
  // single layers fill the GPU for long: from about 20 M values per convolution output on average.  A step at 224x224, ms,
  // second stream / end of the call: whole network batch 32 fp32 4.9 / 4.0, 128 fp32 11.6 / 11.3, 32 bfloat16 (width 1.4) 4.0 / 3.2,
  // 128 bfloat16 5.8 / 5.6 (16.5 M values); block 2 alone bfloat16 batch 16 0.25 / 0.20, 32 (16.8 M) 0.295 / 0.289, 64 (34 M)
  // 0.490 / 0.509; units 1-4 bfloat16 batch 32 1.03 / 0.88, 64 (22 M) 1.42 / 1.45; width 1.4 batch 128 bfloat16 (26 M) 7.4 / 7.5.
  s->defers = n_convs == 0 || z_values / n_convs < ((size_t)20 << 20);
  // A launch for the weight gradients of a few short layers, and one for their partial sums, cost more than it costs to run each next to
  // its data gradient, in that one's launch.  A step (forward and backward), us, at once / together: 64 <-> 384 channels, fp32, 512 rows one layer
  // 18.2 / 26.1, two 35.8 / 41.2, three 52.2 / 56.6, four (2048 rows in all) 70.1 / 72.0, six 104 / 106; 2048 rows one 33.1 / 37.8, two 65.0 / 66.7, three
  // 94 / 92; 128 rows twelve 190 / 184; bfloat16 512 rows one 18.0 / 24.3, three 52.1 / 52.4, four 69.1 / 67.5; 2048 rows one 30.8 / 33.8, two 64.3 / 60.5; one
  // block of 64 channels, 512 rows fp32 42.7 / 48.0, bfloat16 42.3 / 45.1.  Blocks with their depthwise layer: one of 64 -> 384 -> 96, fp32, 900 rows
  // 55.7 / 62.2, 1600 rows 76.6 / 82.3, of 88 channels 900 rows 65.8 / 67.9, 1600 rows (149 M products) 88.0 / 86.7, two of 64 channels 820 rows 101 / 102,
  // 1040 rows 118 / 114; bfloat16 one of 64 channels 900 rows 51.2 / 54.3, 1040 rows 59.3 / 58.7, 1600 rows 72.7 / 69.1, of 48 channels 1040 rows
  // 55.8 / 51.8, two of 64 channels 700 rows 96.4 / 93.4, 1040 rows 118 / 107: in bfloat16 the two are even near 1000 rows of one block, and the line
  // below lies some hundred rows beyond that.  From about 300 M products on the together form is the faster one; without a data gradient from somewhat less
  // (512 rows, 320 -> 1280, 210 M, fp32 41.0 / 44.4, 1024 rows 56.5 / 52.1; 512 -> 512 1024 rows, 268 M, 39.0 / 40.6, 2048 rows 61.8 / 53.7).  With a longer layer
  // in the stage the launch is there anyway.
  // A single bfloat16 layer of 16384 rows and more with at most 32 outputs has a kernel that multiplies in bfloat16 and reads 128 rows at
  // once: 96 -> 24 channels 32768 rows 34.8 / 40.0; 32 -> 16 131072 rows 43.5 / 51.4; a block of one depthwise and one such layer
  // 131072 rows 98.3 / 103.4.
  const size_t n_short = s->share.other - n_long;
  const bool narrow_at_once = m->dtype == FTP_BF16 && s->share.other == 1 && n_narrow == 1;
  const size_t rows_at_once = n_short > 4 || short_products > 150000000 ? 1600 : m->dtype == FTP_F32 ? 3200 : n_short == 2 ? 2080 : 1600;
  const bool short_at_once = n_long == 0 && (n_short == 1 || short_rows <= rows_at_once) && short_products <= 300000000;
  for (int i = a; i < b; ++i) {
    const UnitInfo& u = m->units[i];
    UnitPlan p;
    p.info = &u;
    p.late_part = p.late_floats = 0;
    p.p_off = s->n_param; s->n_param += align_up(u.n_param, 8);
    p.bn_off = s->n_bn; s->n_bn += u.n_bn;
    for (const Sub& sb : u.subs) {
      size_t zb = act_bytes(sb.g.Hout, sb.g.Wout, sb.g.Cout);
      p.z_off.push_back(stash); stash += zb;
      p.st_off.push_back(stats); stats += (size_t)4 * sb.g.Cout;
      if (zb > max_act) max_act = zb;
      size_t ib = act_bytes(sb.g.Hin, sb.g.Win, sb.g.Cin);
      if (ib > max_act) max_act = ib;
      if (sb.g.Cout > max_c) max_c = sb.g.Cout;
      ConvGeom g = sb.g; g.N = batch;
      size_t M = (size_t)batch * g.Hout * g.Wout;
      const bool c1 = sb.type == SUB_DIRECT && conv1d_ok(g) && conv1d_pays(m->dtype, g, i == 0, n_convs == 1, !s->defers);
      const bool patches = sb.type == SUB_DIRECT && !c1;
      p.axis.push_back(c1);
      size_t need = c1 ? conv1d_wgrad_ws(g) : patches ? conv_direct_wgrad_ws(g) : sb.type == SUB_DW ? dw_bwd_ws(m->dtype, g) : pw_wgrad_ws(M, g.Cin, g.Cout);
      if (patches && need > ws_floats) ws_floats = need;
      if (sb.type != SUB_DW && need > layer_ws) layer_ws = need;
      if (i == a && &sb == &u.subs[0] && sb.type != SUB_DW) s->ws_tail_floats = need;
      size_t part = patches ? 0 : need;
      bool at_once = false;
      bool dz_stored = true;             // a layer whose dz is not always stored still counts in dz_max
      if (sb.type == SUB_PW) {
        const bool narrow = M >= 16384 && g.Cout <= 32 && narrow_at_once;
        at_once = s->defers && (narrow || (M <= 2048 && short_at_once));
        part = narrow ? pw_wgrad_ws(M, g.Cin, g.Cout) : at_once ? 0 : pw_wgrad_group_ws(m->dtype, M, g.Cin, g.Cout, s->share);
        const size_t fused = m->dtype == FTP_BF16 ? pw_bwd_fused_ws(M, g.Cin, g.Cout) : 0;
        if (fused > 0 && &sb == &u.subs[0]) dz_stored = false;
        if (fused > part) part = fused;
      } else if (sb.type == SUB_DW) {
        // the short kernel, which leaves no partials, is for stages that defer: on two streams every layer has a place of its own until the call's end
        const bool in_one = s->defers && u.subs.size() == 3 && dw_bwd_small_ok(g);
        if (!s->defers) { p.late_part = s->ws_late_floats; p.late_floats = need; s->ws_late_floats += align_up(need, 64); }
        if (in_one) part = 0;
        dz_stored = !in_one && bn_bwd_small_ok(M, g.Cout);
      }
      if (zb > dz_max) dz_max = zb;
      dz_bytes += dz_stored ? zb : 0;
      part = align_up(part, 64);
      p.part.push_back(part);
      p.at_once.push_back(at_once);
      if (part > part_max) part_max = part;
      part_floats += part;
      if (sb.type == SUB_PW && m->dtype == FTP_BF16 && pw_bwd_fused_ws(M, g.Cin, g.Cout) > s->ws_fused_floats)
        s->ws_fused_floats = pw_bwd_fused_ws(M, g.Cin, g.Cout);
      if (patches) ++s->n_direct;
      if (patches && conv_direct_gemm_ok(g) && conv_direct_gemm_wpad_elems(g) > ws_floats)
        ws_floats = conv_direct_gemm_wpad_elems(g);      // padded weight copy of the GEMM forward (at most 4 bytes each)
      if (patches && conv_direct_im2col_elems(g) > s->im2col_elems) s->im2col_elems = conv_direct_im2col_elems(g);
      if (patches && conv_direct_dgrad_gemm_ok(g)) {
        if (conv_direct_dgrad_gemm_im2col_elems(g) > s->im2col_elems) s->im2col_elems = conv_direct_dgrad_gemm_im2col_elems(g);
        if (conv_direct_dgrad_gemm_w_elems(g) > ws_floats) ws_floats = conv_direct_dgrad_gemm_w_elems(g);
      }
    }
    p.out_virtual = (u.d.kind == FTP_UNIT_CONV);
    p.out_off = 0;
    if (!p.out_virtual && u.d.kind != FTP_UNIT_LOSS) {
      size_t ob = act_bytes(u.outH, u.outW, u.outC);
      p.out_off = stash; stash += ob;
      if (ob > max_act) max_act = ob;
    }
    p.need_in_mat = u.residual && i > a && m->units[i - 1].d.kind == FTP_UNIT_CONV;
    p.in_mat_off = 0;
    if (p.need_in_mat) { p.in_mat_off = stash; stash += act_bytes(u.inH, u.inW, u.inC); }
    p.open_off = stash;
    if (u.d.kind == FTP_UNIT_GAP && i > a && m->units[i - 1].d.kind == FTP_UNIT_CONV) stash += align_up((size_t)batch * 2 * u.inC * 4, 256);
    if (u.d.kind == FTP_UNIT_FC) {
      size_t need = pw_wgrad_ws((size_t)batch, u.inC, u.outC);
      if (need > ws_floats) ws_floats = need;
    }
    if (u.d.kind == FTP_UNIT_LOSS) { s->has_loss = true; s->classes = u.inC; }
    s->plan.push_back(p);
  }
  if (s->defers) {
    // The stores take every layer of the stage where that is little, and otherwise no more dz than a stage on two streams has
    // buffers for.  MobileNetV2 at 224x224, bfloat16 batch 128: 4.16 GB (two streams 4.05, with places for all layers 4.97); fp32
    // batch 32: 2.37 GB (2.25, 2.56); units 15 - 18, bfloat16 batch 64: 197 MB (147, 215).
    const size_t two = 2 * max_act + 6 * (max_act < kDzRing ? max_act : kDzRing);
    const size_t dz_lim = two > kDzStore ? two : kDzStore, part_lim = part_max > kPartStore ? part_max : kPartStore;
    s->dz_cap = dz_bytes < dz_max ? dz_max : dz_bytes < dz_lim ? dz_bytes : dz_lim;
    s->part_cap = part_floats < part_lim ? part_floats : part_lim;
  } else if (layer_ws > ws_floats) ws_floats = layer_ws;
  s->stash_bytes = stash; s->stats_floats = stats; s->max_act_bytes = max_act; s->ws_floats = ws_floats; s->max_c = max_c;

  s->q_pw.reserve(n_convs); s->q_red.reserve(n_convs); s->q_late.reserve(n_convs);      // a layer leaves at most one of each
  int rc = FTP_OK;
  size_t np = s->n_param ? s->n_param : 8;
  size_t nb = s->n_bn ? s->n_bn : 8;
  if ((rc = dev_alloc(&s->params, np * 4)) || (rc = dev_alloc(&s->grads, np * 4)) || (rc = dev_alloc(&s->mom, np * 4)) ||
      (rc = dev_alloc(&s->run_mean, nb * 4)) || (rc = dev_alloc(&s->run_var, nb * 4))) { stage_free(s); return rc; }
  if (s->dt == FTP_BF16 && (rc = dev_alloc(&s->w_lp, np * 2))) { stage_free(s); return rc; }
  s->slots.resize(n_slots);
  if (s->recompute && (rc = dev_alloc(&s->shared_stash, stash))) { stage_free(s); return rc; }
  for (auto& sl : s->slots) {
    if (s->recompute) {
      sl.stash = s->shared_stash;
      if ((rc = dev_alloc(&sl.xin_keep, s->xin_bytes))) { stage_free(s); return rc; }
    } else if ((rc = dev_alloc(&sl.stash, stash))) { stage_free(s); return rc; }
    if ((rc = dev_alloc(&sl.stats, (stats ? stats : 8) * 4)) ||
        (rc = dev_alloc(&sl.snap_w, np * 4))) { stage_free(s); return rc; }
    if (s->dt == FTP_BF16 && (rc = dev_alloc(&sl.snap_lp, np * 2))) { stage_free(s); return rc; }
    if (s->has_loss && (rc = dev_alloc(&sl.dlogits, (size_t)batch * s->classes * s->es))) { stage_free(s); return rc; }
  }
  for (int i = 0; i < 5; ++i)
    if (!(s->defers && (i == 2 || i == 4)) && (rc = dev_alloc(&s->gbuf[i], max_act))) { stage_free(s); return rc; }
  {
    hipError_t e = hipStreamCreateWithFlags(&s->side, hipStreamNonBlocking);     // default priority
    for (int i = 0; i < 3 && e == hipSuccess; ++i) {
      e = hipEventCreateWithFlags(&s->ev_fork[i], hipEventDisableTiming);
      if (e == hipSuccess) e = hipEventCreateWithFlags(&s->ev_join[i], hipEventDisableTiming);
    }
    for (int i = 0; i < 2 && e == hipSuccess; ++i) {
      e = hipEventCreateWithFlags(&s->ev_bfork[i], hipEventDisableTiming);
      if (e == hipSuccess) e = hipEventCreateWithFlags(&s->ev_bjoin[i], hipEventDisableTiming);
    }
    if (e != hipSuccess) { ftp_set_error("stage_create: stream/event creation failed: %s", hipGetErrorString(e)); stage_free(s); return FTP_ERR_HIP; }
  }
  if (!s->defers) {
    s->dzring_bytes = max_act < kDzRing ? max_act : kDzRing;
    for (int i = 0; i < 6; ++i)
      if ((rc = dev_alloc(&s->dzring[i], s->dzring_bytes))) { stage_free(s); return rc; }
  }
  if ((rc = dev_alloc(&s->bn_part, (size_t)kBnPartials * 2 * max_c * 4)) || (rc = dev_alloc(&s->coef, (size_t)3 * max_c * 4)) ||
      (rc = dev_alloc(&s->ws, ws_floats * 4)) || (rc = dev_alloc(&s->row_loss, align_up((size_t)batch, 8) * 4)) || (s->has_loss && (rc = dev_alloc(&s->arrived, kCeCounters * 4)))) { stage_free(s); return rc; }
  if (s->im2col_elems && (rc = dev_alloc(&s->im2col, s->im2col_elems * s->es))) { stage_free(s); return rc; }
  if (s->defers && ((rc = dev_alloc(&s->dz_store, s->dz_cap)) || (rc = dev_alloc(&s->parts, s->part_cap * 4)))) { stage_free(s); return rc; }
  if (!s->defers && s->ws_fused_floats && (rc = dev_alloc(&s->ws_fused, s->ws_fused_floats * 4))) { stage_free(s); return rc; }
  if (!s->defers && s->ws_late_floats && (rc = dev_alloc(&s->ws_late, s->ws_late_floats * 4))) { stage_free(s); return rc; }
  if (!s->defers && s->ws_tail_floats && s->n_direct <= 1 &&
      (rc = dev_alloc(&s->ws_tail, s->ws_tail_floats * 4))) { stage_free(s); return rc; }

  // initial state: zero weights / momentum / gradients, running mean 0, running variance 1
  std::vector<float> ones(nb, 1.0f);
  hipError_t e = hipMemset(s->params, 0, np * 4);
  if (e == hipSuccess) e = hipMemset(s->grads, 0, np * 4);
  if (e == hipSuccess) e = hipMemset(s->mom, 0, np * 4);
  if (e == hipSuccess) e = hipMemset(s->run_mean, 0, nb * 4);
  if (e == hipSuccess) e = hipMemcpy(s->run_var, ones.data(), nb * 4, hipMemcpyHostToDevice);
  if (e == hipSuccess && s->arrived) e = hipMemset(s->arrived, 0, kCeCounters * 4);
  if (e == hipSuccess && s->w_lp) e = hipMemset(s->w_lp, 0, np * 2);
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) { ftp_set_error("stage_create: initialisation failed: %s", hipGetErrorString(e)); stage_free(s); return FTP_ERR_HIP; }
  s->dev_bytes = g_alloc_total;
  *out = s;
  return FTP_OK;
}

extern "C" int ftp_stage_create(const ftp_model* m, int a, int b, int batch, int n_slots, ftp_stage** out) {
  return ftp_stage_create_ex(m, a, b, batch, n_slots, 0u, out);
}

extern "C" int ftp_stage_device_bytes(const ftp_stage* s, size_t* bytes) {
  if (!s || !bytes) { ftp_set_error("stage_device_bytes: NULL argument"); return FTP_ERR_ARG; }
  *bytes = s->dev_bytes;
  return FTP_OK;
}

// ---- parameter import / export ------------------------------------------------
static int unit_check(const ftp_stage* s, int unit, size_t n, size_t expect, const void* p, const char* who) {
  if (!s || !p) { ftp_set_error("%s: NULL argument", who); return FTP_ERR_ARG; }
  if (unit < s->a || unit >= s->b) { ftp_set_error("%s: unit %d outside the stage [%d,%d)", who, unit, s->a, s->b); return FTP_ERR_ARG; }
  if (n != expect) { ftp_set_error("%s: unit %d has %zu values, caller passed %zu", who, unit, expect, n); return FTP_ERR_SHAPE; }
  return FTP_OK;
}

extern "C" int ftp_stage_import_weights(ftp_stage* s, int unit, const float* host_w, size_t n) {
  int rc = unit_check(s, unit, n, s ? (unit >= s->a && unit < s->b ? s->plan[unit - s->a].info->n_param : 0) : 0, host_w, "import_weights");
  if (rc) return rc;
  if (n == 0) return FTP_OK;
  const UnitPlan& p = s->plan[unit - s->a];
  HIP_TRY(hipMemcpy(s->params + p.p_off, host_w, n * 4, hipMemcpyHostToDevice));
  if (s->w_lp) {
    f32_to_storage(FTP_BF16, nullptr, s->params + p.p_off, (char*)s->w_lp + p.p_off * 2, n);
    HIP_TRY(hipGetLastError());
  if (const char* why = launch_plan_failure_take()) { ftp_set_error("%s", why); return FTP_ERR_UNSUPPORTED; }
    HIP_TRY(hipDeviceSynchronize());
  }
  return FTP_OK;
}

// A caller's new array has no pages yet, and the copy would take a fault for each.  They are asked for together instead, while the GPU may still
// be busy; contents stay as they are, and where the kernel does not know the request the copy takes its faults as before.  Only where the last
// page is missing: going through pages that are there costs 0.25 ms for 14 MB.  The weights of MobileNetV2 (20 units, 14 MB) into new arrays
// 2.65 -> 1.88 ms, into ones used before 1.05.
static void populate(void* p, size_t bytes) {
#ifndef MADV_POPULATE_WRITE
#define MADV_POPULATE_WRITE 23
#endif
  if (bytes < ((size_t)256 << 10)) return;
  const uintptr_t page = (uintptr_t)sysconf(_SC_PAGESIZE), lo = ((uintptr_t)p + page - 1) / page * page, hi = ((uintptr_t)p + bytes) / page * page;
  unsigned char here = 1;
  if (mincore((void*)(hi - page), page, &here) == 0 && (here & 1)) return;      // written before: nothing to ask for
  (void)madvise((void*)lo, hi - lo, MADV_POPULATE_WRITE);
}

static int export_from(const ftp_stage* s, const float* base, int unit, float* host, size_t n, const char* who) {
  int rc = unit_check(s, unit, n, s ? (unit >= s->a && unit < s->b ? s->plan[unit - s->a].info->n_param : 0) : 0, host, who);
  if (rc) return rc;
  if (n == 0) return FTP_OK;
  populate(host, n * 4);
  HIP_TRY(hipDeviceSynchronize());
  HIP_TRY(hipMemcpy(host, base + s->plan[unit - s->a].p_off, n * 4, hipMemcpyDeviceToHost));
  return FTP_OK;
}
extern "C" int ftp_stage_export_weights(const ftp_stage* s, int unit, float* h, size_t n) { return export_from(s, s ? s->params : nullptr, unit, h, n, "export_weights"); }
extern "C" int ftp_stage_export_grads(const ftp_stage* s, int unit, float* h, size_t n) { return export_from(s, s ? s->grads : nullptr, unit, h, n, "export_grads"); }
extern "C" int ftp_stage_export_momentum(const ftp_stage* s, int unit, float* h, size_t n) { return export_from(s, s ? s->mom : nullptr, unit, h, n, "export_momentum"); }

extern "C" int ftp_stage_export_bn_stats(const ftp_stage* s, int unit, float* host, size_t n) {
  int rc = unit_check(s, unit, n, s ? (unit >= s->a && unit < s->b ? 2 * s->plan[unit - s->a].info->n_bn : 0) : 0, host, "export_bn_stats");
  if (rc) return rc;
  if (n == 0) return FTP_OK;
  const UnitPlan& p = s->plan[unit - s->a];
  HIP_TRY(hipDeviceSynchronize());
  // per BatchNorm: running_mean then running_var
  size_t o = 0;
  for (const Sub& sb : p.info->subs) {
    size_t C = sb.g.Cout;
    HIP_TRY(hipMemcpy(host + o, s->run_mean + p.bn_off + sb.bn_off, C * 4, hipMemcpyDeviceToHost));
    HIP_TRY(hipMemcpy(host + o + C, s->run_var + p.bn_off + sb.bn_off, C * 4, hipMemcpyDeviceToHost));
    o += 2 * C;
  }
  return FTP_OK;
}

static int inspect_check_owner(const ftp_stage* s, int slot, const char* who) {
  if (s->recompute && s->stash_owner != slot) {
    ftp_set_error("%s: with recomputation only the slot forwarded (or recomputed) last has intermediates, not slot %d", who, slot);
    return FTP_ERR_SLOT;
  }
  return FTP_OK;
}
static int inspect_check(const ftp_stage* s, int slot, int unit, int conv, const void* host, const char* who) {
  if (!s || !host) { ftp_set_error("%s: NULL argument", who); return FTP_ERR_ARG; }
  if (slot < 0 || slot >= (int)s->slots.size()) { ftp_set_error("%s: slot %d out of range", who, slot); return FTP_ERR_ARG; }
  if (unit < s->a || unit >= s->b) { ftp_set_error("%s: unit %d outside the stage [%d,%d)", who, unit, s->a, s->b); return FTP_ERR_ARG; }
  if (conv < 0 || conv >= (int)s->plan[unit - s->a].info->subs.size()) { ftp_set_error("%s: unit %d has no convolution %d", who, unit, conv); return FTP_ERR_ARG; }
  if (!s->slots[slot].busy) { ftp_set_error("%s: slot %d holds no forwarded batch", who, slot); return FTP_ERR_SLOT; }
  return FTP_OK;
}

extern "C" int ftp_stage_export_conv_output(const ftp_stage* s, int slot, int unit, int conv, float* host_z, size_t n) {
  int rc = inspect_check(s, slot, unit, conv, host_z, "export_conv_output");
  if (!rc) rc = inspect_check_owner(s, slot, "export_conv_output");
  if (rc) return rc;
  const UnitPlan& p = s->plan[unit - s->a];
  const Sub& sb = p.info->subs[conv];
  size_t expect = (size_t)s->batch * sb.g.Hout * sb.g.Wout * sb.g.Cout;
  if (n != expect) { ftp_set_error("export_conv_output: tensor has %zu values, caller passed %zu", expect, n); return FTP_ERR_SHAPE; }
  HIP_TRY(hipDeviceSynchronize());
  const char* src = s->slots[slot].stash + p.z_off[conv];
  if (s->dt == FTP_F32) {
    HIP_TRY(hipMemcpy(host_z, src, n * 4, hipMemcpyDeviceToHost));
  } else {
    std::vector<uint16_t> tmp(n);
    HIP_TRY(hipMemcpy(tmp.data(), src, n * 2, hipMemcpyDeviceToHost));
    for (size_t i = 0; i < n; ++i) { uint32_t u = (uint32_t)tmp[i] << 16; memcpy(&host_z[i], &u, 4); }
  }
  return FTP_OK;
}

extern "C" int ftp_stage_export_bn_batch_stats(const ftp_stage* s, int slot, int unit, int conv, float* host_s, size_t n) {
  int rc = inspect_check(s, slot, unit, conv, host_s, "export_bn_batch_stats");
  if (rc) return rc;
  const UnitPlan& p = s->plan[unit - s->a];
  size_t expect = (size_t)4 * p.info->subs[conv].g.Cout;
  if (n != expect) { ftp_set_error("export_bn_batch_stats: %zu values, caller passed %zu", expect, n); return FTP_ERR_SHAPE; }
  HIP_TRY(hipDeviceSynchronize());
  HIP_TRY(hipMemcpy(host_s, s->slots[slot].stats + p.st_off[conv], n * 4, hipMemcpyDeviceToHost));
  return FTP_OK;
}

// ---- helpers for the compute calls ------------------------------------------------
struct WeightSet { const float* w32; const char* lp; };

static inline const void* conv_w(const ftp_stage* s, const WeightSet& ws, size_t off) {
  return s->dt == FTP_F32 ? (const void*)(ws.w32 + off) : (const void*)(ws.lp + off * 2);
}

static int check_call(ftp_stage* s, int slot, const char* who) {
  if (!s) { ftp_set_error("%s: NULL stage", who); return FTP_ERR_ARG; }
  if (slot < 0 || slot >= (int)s->slots.size()) { ftp_set_error("%s: slot %d out of range (n_slots=%zu)", who, slot, s->slots.size()); return FTP_ERR_ARG; }
  return FTP_OK;
}

static HView plain(const void* p) { return HView{p, nullptr, nullptr, 0}; }

// Input view of every unit and of every convolution inside it, from the slot's buffers.
struct Views {
  std::vector<HView> unit_in;                 // per unit
  std::vector<std::vector<HView>> sub_out;    // per unit, per sub
};

static void build_views(const ftp_stage* s, const Slot& sl, Views* v) {
  HView cur = plain(sl.stash);                // stashed stage input at offset 0
  size_t n = s->plan.size();
  v->unit_in.resize(n);
  v->sub_out.resize(n);
  for (size_t i = 0; i < n; ++i) {
    const UnitPlan& p = s->plan[i];
    if (p.need_in_mat) cur = plain(sl.stash + p.in_mat_off);
    v->unit_in[i] = cur;
    for (size_t k = 0; k < p.info->subs.size(); ++k) {
      const Sub& sb = p.info->subs[k];
      float* st = sl.stats + p.st_off[k];
      v->sub_out[i].push_back(HView{sl.stash + p.z_off[k], st + 2 * sb.g.Cout, st + 3 * sb.g.Cout, sb.act});
    }
    if (p.out_virtual) cur = v->sub_out[i].back();
    else if (p.info->d.kind != FTP_UNIT_LOSS) cur = plain(sl.stash + p.out_off);
  }
}

// A block output that nobody has written yet: the raw output of its project layer, the statistics as partial sums, the residual
// (nullptr: none) and where it goes.  The pointwise layer behind it forms it on the way in (pw_fwd_pro).
struct OutPending { BnPending pend{}; HView z{}; const void* res = nullptr; void* out = nullptr; };

// the second half of the partial sums' buffer, for a layer that reads the first half while it leaves its own
static float* other_partials(const ftp_stage* s) { return s->bn_part + (size_t)kBnPartials / 2 * 2 * s->max_c; }

static void finish_now(const ftp_stage* s, hipStream_t st, const BnPending& b, int C) {
  bn_finalize(st, b.partial, b.P, b.M, C, b.gamma, b.beta, b.mean, b.invstd, b.scale, b.shift, b.run_mean, b.run_var, kBnEps, s->bn_mom);
}

// pend (in/out): on entry the unfinished BatchNorm of `in` (partial == nullptr: none); on exit, when
// defer is set and the statistics of this layer were left as partial sums, their description
static void sub_forward(ftp_stage* s, Slot& sl, const UnitPlan& p, size_t k, HView in, const WeightSet& W, hipStream_t st,
                        BnPending* pend = nullptr, bool defer = false, OutPending* block = nullptr) {
  const Sub& sb = p.info->subs[k];
  ConvGeom g = sb.g; g.N = s->batch;
  void* z = sl.stash + p.z_off[k];
  const void* w = conv_w(s, W, p.p_off + sb.w_off);
  size_t M = (size_t)s->batch * g.Hout * g.Wout;
  int P = 0;
  float* stt = sl.stats + p.st_off[k];
  int C = g.Cout;
  if (s->im2col_of == z) s->im2col_of = nullptr;     // this layer's input is a new one: patches kept from before are stale
  const float* gamma = W.w32 + p.p_off + sb.gamma_off;
  const float* beta = W.w32 + p.p_off + sb.beta_off;
  float* rm = s->run_mean + p.bn_off + sb.bn_off;
  float* rv = s->run_var + p.bn_off + sb.bn_off;
  if (sb.type == SUB_DW && dw_fwd_bn_small_ok(g)) {
    BnPending none{};
    dw_fwd_bn_small(s->dt, st, in, pend ? *pend : none, w, g, gamma, beta, stt, stt + C, stt + 2 * C, stt + 3 * C, rm, rv, kBnEps,
                    s->bn_mom, z);
    if (pend) pend->partial = nullptr;
    return;
  }
  if (sb.type == SUB_PW) {
    float* part = s->bn_part;
    if (block && block->pend.partial) {
      part = other_partials(s);
      pw_fwd_pro(s->dt, st, block->pend, block->z, block->res, block->out, kBnEps, s->bn_mom, w, M, g.Cin, g.Cout, z, part, &P);
      block->pend.partial = nullptr;
    } else {
      pw_fwd(s->dt, st, in, w, nullptr, M, g.Cin, g.Cout, z, part, &P);       // statistics in the epilogue
    }
    if (defer && pend) {
      *pend = BnPending{part, P, M, gamma, beta, stt, stt + C, stt + 2 * C, stt + 3 * C, rm, rv};
      return;
    }
    bn_finalize(st, part, P, M, C, gamma, beta, stt, stt + C, stt + 2 * C, stt + 3 * C, rm, rv, kBnEps, s->bn_mom);
    return;
  } else if (p.axis[k]) {
    // the partials of the input's BatchNorm, if it is pending, are read by every block: this layer's go to the other half
    float* part = s->bn_part;
    if (pend && pend->partial && !conv1d_small_ok(g) && !conv1d_finish_ok(g, pend->P)) {
      finish_now(s, st, *pend, g.Cin);
      pend->partial = nullptr;
    }
    if (pend && pend->partial == part) part = other_partials(s);
    const BnPending none{};
    conv1d_fwd(s->dt, st, in, pend ? *pend : none, kBnEps, s->bn_mom, w, g, z, part, &P);
    if (pend) pend->partial = nullptr;
    if (defer && pend) {
      *pend = BnPending{part, P, M, gamma, beta, stt, stt + C, stt + 2 * C, stt + 3 * C, rm, rv};
      return;
    }
    bn_finalize(st, part, P, M, C, gamma, beta, stt, stt + C, stt + 2 * C, stt + 3 * C, rm, rv, kBnEps, s->bn_mom);
    return;
  } else if (sb.type == SUB_DIRECT && conv_direct_gemm_ok(g) && s->im2col &&
             conv_direct_gemm_wpad_elems(g) * s->es <= s->ws_floats * sizeof(float)) {
    // the float workspace is free during a forward: the padded weight copy lives there
    conv_direct_fwd_gemm(s->dt, st, in, w, g, s->im2col, s->ws, z, s->bn_part, &P);
    s->im2col_of = z;
  } else {
    if (sb.type == SUB_DW && dw_fwd_stats_ok(s->dt, g)) {
      dw_fwd(s->dt, st, in, w, g, z, s->bn_part, &P);           // few tiles: their sums are the partials
    } else {
      if (sb.type == SUB_DW) dw_fwd(s->dt, st, in, w, g, z);
      else conv_direct_fwd(s->dt, st, in, w, g, z);
      bn_stats(s->dt, st, z, M, g.Cout, s->bn_part, &P);
    }
  }
  bn_finalize(st, s->bn_part, P, M, C, gamma, beta, stt, stt + C, stt + 2 * C, stt + 3 * C, rm, rv, kBnEps, s->bn_mom);
}

// the unit behind unit i of the stage starts with a pointwise layer that can form unit i's output
static bool next_forms_block(const ftp_stage* s, size_t i) {
  if (i + 1 >= s->plan.size() || s->plan[i + 1].info->subs.empty()) return false;
  const Sub& n = s->plan[i + 1].info->subs[0];
  return n.type == SUB_PW && pw_pro_ok(s->dt, (size_t)s->batch * n.g.Hout * n.g.Wout, n.g.Cin, n.g.Cout);
}

// A short 1-D convolution that does its own BatchNorm backward from sums the layer behind has left, and whether unit i's convolution
// can leave them for the one in front.
static bool conv1d_takes_sums(const ftp_stage* s, const UnitPlan& p) {
  if (p.info->d.kind != FTP_UNIT_CONV || !p.axis[0] || !s->defers) return false;
  ConvGeom g = p.info->subs[0].g; g.N = s->batch;
  return conv1d_bwd_sums_ok(s->dt, g) && bn_bwd_small_ok((size_t)g.N * g.Wout, g.Cout);
}
static bool conv1d_leaves_sums(const ftp_stage* s, size_t i) { return i > 0 && conv1d_takes_sums(s, s->plan[i - 1]); }

// what the forward of unit i, an average, leaves of the activation in front for that BatchNorm's backward sums (nullptr: nothing, its backward
// does not take sums)
static float* open_sums(const ftp_stage* s, const Slot& sl, size_t i) {
  if (i == 0 || s->plan[i - 1].info->d.kind != FTP_UNIT_CONV) return nullptr;
  const UnitPlan& q = s->plan[i - 1];
  const ConvGeom& g = q.info->subs[0].g;
  if (!conv1d_takes_sums(s, q) && bn_bwd_small_ok((size_t)s->batch * g.Hout * g.Wout, g.Cout)) return nullptr;
  return (float*)(sl.stash + s->plan[i].open_off);
}

// every unit of the stage over the input at offset 0 of the slot's stash, with the weights W
// y: where the caller wants the stage's output (nullptr: nowhere); *y_written: it is there
static int forward_units(ftp_stage* s, Slot& sl, const Views& v, const WeightSet& W, hipStream_t st, void* y = nullptr, bool* y_written = nullptr) {
  OutPending block{};      // the output of a short block, left to the pointwise layer behind it
  BnPending carry{};       // a short 1-D convolution leaves its statistics to the short 1-D convolution or the average behind it
  for (size_t i = 0; i < s->plan.size(); ++i) {
    const UnitPlan& p = s->plan[i];
    const UnitInfo& u = *p.info;
    if (s->prof) HIP_TRY(hipEventRecord(s->prof->f0[i], st));
    if (p.need_in_mat) {
      // the previous CONV unit's output, materialised so the residual can read it
      HView prev = v.sub_out[i - 1].back();
      bn_apply(s->dt, st, prev, (size_t)s->batch * u.inH * u.inW, u.inC, nullptr, sl.stash + p.in_mat_off);
    }
    HView in = v.unit_in[i];
    switch (u.d.kind) {
      case FTP_UNIT_CONV:
      {
        // the statistics of a convolution on the 1-D kernels are left to the one behind, and those of a short one to an average too
        auto on_axis = [&](size_t j) { return s->plan[j].info->d.kind == FTP_UNIT_CONV && s->plan[j].axis[0]; };
        ConvGeom g = u.subs[0].g; g.N = s->batch;
        const bool defer = on_axis(i) && i + 1 < s->plan.size() &&
                           (on_axis(i + 1) || (s->plan[i + 1].info->d.kind == FTP_UNIT_GAP && conv1d_small_ok(g)));
        sub_forward(s, sl, p, 0, in, W, st, &carry, defer, &block);
        break;
      }
      case FTP_UNIT_INVRES: {
        HView h = in;
        BnPending pend{};
        for (size_t k = 0; k < u.subs.size(); ++k) {
          // an expand layer in front of a short depthwise layer leaves its statistics to that layer's kernel
          bool defer = false;
          if (k + 1 < u.subs.size() && u.subs[k].type == SUB_PW && u.subs[k + 1].type == SUB_DW) {
            ConvGeom gn = u.subs[k + 1].g; gn.N = s->batch;
            defer = dw_fwd_bn_small_ok(gn) && (size_t)s->batch * u.subs[k].g.Hout * u.subs[k].g.Wout <= 16 * 128;
          }
          // ... and the project layer leaves them to whatever writes the block output
          if (k + 1 == u.subs.size() && u.subs[k].type == SUB_PW) defer = true;
          sub_forward(s, sl, p, k, h, W, st, &pend, defer, k == 0 ? &block : nullptr);
          h = v.sub_out[i][k];
        }
        const size_t Mo = (size_t)s->batch * u.outH * u.outW;
        const void* res = u.residual ? in.z : nullptr;
        // the stage's output goes to the caller at once where its vectors allow it: nothing here reads it again (block 2 at 112x112, batch 64, bfloat16: a step
        // 0.427 -> 0.423 ms without the copy)
        const bool direct = y && i + 1 == s->plan.size() && ((uintptr_t)y & 15) == 0;
        char* out = direct ? (char*)y : sl.stash + p.out_off;
        if (direct) *y_written = true;
        if (bn_finalize_apply_small_ok(Mo, u.outC)) {
          if (next_forms_block(s, i)) block = OutPending{pend, h, res, out};
          else bn_finalize_apply_small(s->dt, st, pend, h.z, Mo, u.outC, h.act, kBnEps, s->bn_mom, res, out);
        } else if (bn_finish_ok(Mo, u.outC, pend.P)) {
          bn_finish_apply(s->dt, st, pend, h.z, Mo, u.outC, h.act, kBnEps, s->bn_mom, res, out);
        } else {
          finish_now(s, st, pend, u.outC);
          bn_apply(s->dt, st, h, Mo, u.outC, res, out);
        }
        break;
      }
      case FTP_UNIT_GAP:
        gap_fwd(s->dt, st, in, carry, kBnEps, s->bn_mom, s->batch, u.inH * u.inW, u.inC, sl.stash + p.out_off, open_sums(s, sl, i));
        carry.partial = nullptr;
        break;
      case FTP_UNIT_FC:
        pw_fwd(s->dt, st, in, conv_w(s, W, p.p_off), W.w32 + p.p_off + (size_t)u.outC * u.inC, (size_t)s->batch, u.inC,
               u.outC, sl.stash + p.out_off, nullptr, nullptr);
        break;
      default:
        break;  // LOSS: evaluated by ftp_stage_loss
    }
    if (s->prof) HIP_TRY(hipEventRecord(s->prof->f1[i], st));
  }
  return FTP_OK;
}

extern "C" int ftp_stage_forward(ftp_stage* s, int slot, const void* x_dev, void* y_dev, void* stream) {
  int rc = check_call(s, slot, "stage_forward");
  if (rc) return rc;
  if (!x_dev) { ftp_set_error("stage_forward: x_dev is NULL"); return FTP_ERR_ARG; }
  Slot& sl = s->slots[slot];
  if (sl.busy) { ftp_set_error("stage_forward: slot %d is busy (its backward has not run)", slot); return FTP_ERR_SLOT; }
  hipStream_t st = (hipStream_t)stream;
  const UnitInfo& first = *s->plan[0].info;
  size_t xin = (size_t)s->batch * first.inH * first.inW * first.inC * s->es;
  sl.timer_idx = -1;
  if (s->timer && s->timer->used < ExecTimer::kRing) {
    sl.timer_idx = s->timer->used++;
    s->timer->bwd_done[sl.timer_idx] = false;
    HIP_TRY(hipEventRecord(s->timer->ev[sl.timer_idx][0], st));
  }
  HIP_TRY(hipMemcpyAsync(sl.stash, x_dev, xin, hipMemcpyDeviceToDevice, st));
  if (s->recompute) {
    HIP_TRY(hipMemcpyAsync(sl.xin_keep, x_dev, xin, hipMemcpyDeviceToDevice, st));
    s->stash_owner = slot;
  }
  Views v;
  build_views(s, sl, &v);
  WeightSet W{s->params, (const char*)s->w_lp};
  bool y_written = false;
  if ((rc = forward_units(s, sl, v, W, st, y_dev, &y_written))) return rc;
  if (y_dev && !y_written) {
    size_t li = s->plan.size() - 1;
    const UnitPlan& p = s->plan[li];
    const UnitInfo& u = *p.info;
    size_t M = (size_t)s->batch * u.outH * u.outW;
    if (p.out_virtual) {
      bn_apply(s->dt, st, v.sub_out[li].back(), M, u.outC, nullptr, y_dev);
    } else {
      const void* src = u.d.kind == FTP_UNIT_LOSS ? v.unit_in[li].z : (const void*)(sl.stash + p.out_off);
      HIP_TRY(hipMemcpyAsync(y_dev, src, M * u.outC * s->es, hipMemcpyDeviceToDevice, st));
    }
  }
  if (s->timer && sl.timer_idx >= 0) HIP_TRY(hipEventRecord(s->timer->ev[sl.timer_idx][1], st));
  HIP_TRY(hipGetLastError());
  if (const char* why = launch_plan_failure_take()) { ftp_set_error("%s", why); return FTP_ERR_UNSUPPORTED; }
  sl.busy = true; sl.has_snap = false; sl.has_loss = false;
  return FTP_OK;
}

extern "C" int ftp_stage_loss(ftp_stage* s, int slot, const int32_t* labels_dev, float* loss_dev, void* stream) {
  int rc = check_call(s, slot, "stage_loss");
  if (rc) return rc;
  if (!s->has_loss) { ftp_set_error("stage_loss: the stage does not end with the LOSS unit"); return FTP_ERR_ARG; }
  if (!labels_dev || !loss_dev) { ftp_set_error("stage_loss: NULL argument"); return FTP_ERR_ARG; }
  Slot& sl = s->slots[slot];
  if (!sl.busy) { ftp_set_error("stage_loss: slot %d holds no forwarded batch", slot); return FTP_ERR_SLOT; }
  if (s->recompute && s->stash_owner != slot) {
    ftp_set_error("stage_loss: with recomputation the loss of slot %d has to follow its forward directly (the logits are gone)", slot);
    return FTP_ERR_SLOT;
  }
  hipStream_t st = (hipStream_t)stream;
  Views v;
  build_views(s, sl, &v);
  size_t li = s->plan.size() - 1;
  if (s->prof) HIP_TRY(hipEventRecord(s->prof->f0[li], st));
  softmax_ce(s->dt, st, v.unit_in[li].z, labels_dev, s->batch, s->classes, s->row_loss, sl.dlogits, loss_dev, s->arrived);
  if (s->prof) HIP_TRY(hipEventRecord(s->prof->f1[li], st));
  HIP_TRY(hipGetLastError());
  if (const char* why = launch_plan_failure_take()) { ftp_set_error("%s", why); return FTP_ERR_UNSUPPORTED; }
  sl.has_loss = true;
  return FTP_OK;
}

extern "C" int ftp_stage_snapshot_weights(ftp_stage* s, int slot, void* stream) {
  int rc = check_call(s, slot, "stage_snapshot_weights");
  if (rc) return rc;
  Slot& sl = s->slots[slot];
  if (!sl.busy) { ftp_set_error("stage_snapshot_weights: slot %d holds no forwarded batch", slot); return FTP_ERR_SLOT; }
  hipStream_t st = (hipStream_t)stream;
  if (s->n_param) {
    HIP_TRY(hipMemcpyAsync(sl.snap_w, s->params, s->n_param * 4, hipMemcpyDeviceToDevice, st));
    if (s->w_lp) HIP_TRY(hipMemcpyAsync(sl.snap_lp, s->w_lp, s->n_param * 2, hipMemcpyDeviceToDevice, st));
  }
  sl.has_snap = true;
  return FTP_OK;
}

extern "C" int ftp_stage_copy_units(ftp_stage* dst, const ftp_stage* src, int unit_lo, int unit_hi, void* stream) {
  if (!dst || !src) { ftp_set_error("stage_copy_units: NULL stage"); return FTP_ERR_ARG; }
  if (dst->model != src->model || dst->dt != src->dt) {
    ftp_set_error("stage_copy_units: the two stages must come from the same model and storage type");
    return FTP_ERR_ARG;
  }
  if (unit_lo < 0 || unit_hi < unit_lo || unit_lo < dst->a || unit_hi > dst->b || unit_lo < src->a || unit_hi > src->b) {
    ftp_set_error("stage_copy_units: units [%d,%d) must lie inside both stages (dst [%d,%d), src [%d,%d))", unit_lo, unit_hi,
                  dst->a, dst->b, src->a, src->b);
    return FTP_ERR_ARG;
  }
  hipStream_t st = (hipStream_t)stream;
  for (int u = unit_lo; u < unit_hi; ++u) {
    const UnitPlan& pd = dst->plan[u - dst->a];
    const UnitPlan& ps = src->plan[u - src->a];
    const size_t n = pd.info->n_param, nb = pd.info->n_bn;
    if (n) {
      HIP_TRY(hipMemcpyAsync(dst->params + pd.p_off, src->params + ps.p_off, n * 4, hipMemcpyDeviceToDevice, st));
      HIP_TRY(hipMemcpyAsync(dst->mom + pd.p_off, src->mom + ps.p_off, n * 4, hipMemcpyDeviceToDevice, st));
      if (dst->w_lp) f32_to_storage(FTP_BF16, st, dst->params + pd.p_off, (char*)dst->w_lp + pd.p_off * 2, n);
    }
    if (nb) {
      HIP_TRY(hipMemcpyAsync(dst->run_mean + pd.bn_off, src->run_mean + ps.bn_off, nb * 4, hipMemcpyDeviceToDevice, st));
      HIP_TRY(hipMemcpyAsync(dst->run_var + pd.bn_off, src->run_var + ps.bn_off, nb * 4, hipMemcpyDeviceToDevice, st));
    }
  }
  HIP_TRY(hipGetLastError());
  if (const char* why = launch_plan_failure_take()) { ftp_set_error("%s", why); return FTP_ERR_UNSUPPORTED; }
  return FTP_OK;
}

extern "C" int ftp_stage_aggregate_weights(ftp_stage* s, const int* slots, int n, void* stream) {
  if (!s || !slots) { ftp_set_error("stage_aggregate_weights: NULL argument"); return FTP_ERR_ARG; }
  if (n < 1 || n > 8) { ftp_set_error("stage_aggregate_weights: 1 <= n <= 8 required, got %d", n); return FTP_ERR_ARG; }
  AggSources src{};
  for (int j = 0; j < n; ++j) {
    const int slot = slots[j];
    if (slot < 0 || slot >= (int)s->slots.size()) {
      ftp_set_error("stage_aggregate_weights: slot %d out of range (n_slots=%zu)", slot, s->slots.size());
      return FTP_ERR_ARG;
    }
    for (int q = 0; q < j; ++q)
      if (slots[q] == slot) { ftp_set_error("stage_aggregate_weights: slot %d listed twice", slot); return FTP_ERR_ARG; }
    if (!s->slots[slot].has_snap) {
      ftp_set_error("stage_aggregate_weights: slot %d holds no weight snapshot", slot);
      return FTP_ERR_SLOT;
    }
    src.p[j] = s->slots[slot].snap_w;
  }
  if (s->n_param) aggregate_weights((hipStream_t)stream, s->params, s->w_lp, src, n, s->n_param);
  HIP_TRY(hipGetLastError());
  if (const char* why = launch_plan_failure_take()) { ftp_set_error("%s", why); return FTP_ERR_UNSUPPORTED; }
  return FTP_OK;
}

// Backward of one convolution+BN+act: dA is the gradient of the activated output.
// Forms dz in one of two alternating buffers; accumulates weight / gamma / beta gradients; when dIn is
// non-NULL writes the gradient of the (activated) input there (+ res for pointwise).  The weight
// gradient runs on the stage's side stream unless per-unit profiling is on.
// mode: the whole layer, or from a dz that the caller formed (passed as dA)
enum { BWD_FULL = 0, BWD_FROM_DZ = 1 };
// stage_forks: the stage runs weight gradients on its second stream (decides which kernels a
// layer uses); stage_overlaps: it does so now (not while per-unit profiling needs everything on one stream)
static bool stage_forks(const ftp_stage* s) { return !s->defers; }
static bool stage_overlaps(const ftp_stage* s) { return s->prof == nullptr && stage_forks(s); }

static int join_side(ftp_stage* s, hipStream_t st);
static int flush_unit_fork(ftp_stage* s, hipStream_t st);
static void run_noted(ftp_stage* s, hipStream_t st);

// Places for one layer's dz (bytes; 0: none) and partial weight gradients in the stores of a stage that defers.  Both at once: where
// one does not fit, what is noted so far runs and the stores start again, and nothing not yet noted may lie in them then.
struct Places { void* dz; float* part; };
static Places take_places(ftp_stage* s, size_t dz_bytes, size_t part_floats, hipStream_t st) {
  if (s->dz_used + dz_bytes > s->dz_cap || s->part_used + part_floats > s->part_cap) run_noted(s, st);
  const Places at{s->dz_store + s->dz_used, s->parts + s->part_used};
  s->dz_used += dz_bytes;
  s->part_used += part_floats;
  return at;
}
static size_t dz_size(const ftp_stage* s, const Sub& sb) {
  return align_up((size_t)s->batch * sb.g.Hout * sb.g.Wout * sb.g.Cout * s->es, 256);
}

static void leave_sums(ftp_stage* s, const void* of, float* partial, int P) { s->left = ftp_stage::LeftSums{of, partial, P}; }
// the sums left for the gradient dA, if there are any (P > 0): they can be taken once
static ftp_stage::LeftSums take_sums(ftp_stage* s, const void* dA) {
  const ftp_stage::LeftSums l = s->left.of == dA ? s->left : ftp_stage::LeftSums{};
  s->left.of = nullptr;
  return l;
}

// A short project layer (no activation, k the last of its block) whose BatchNorm backward is done on the way into its data gradient,
// from sums that the layer behind has left: dIn is wanted, the weight gradient waits for the end of the call.
static bool takes_sums(const ftp_stage* s, const UnitPlan& p, size_t k) {
  const UnitInfo& u = *p.info;
  const Sub& sb = u.subs[k];
  const size_t M = (size_t)s->batch * sb.g.Hout * sb.g.Wout;
  return s->defers && u.d.kind == FTP_UNIT_INVRES && k + 1 == u.subs.size() && sb.type == SUB_PW && !p.at_once[k] &&
         bn_bwd_small_ok(M, sb.g.Cout) && pw_pro_ok(s->dt, M, sb.g.Cout, sb.g.Cin);
}
// the raw output of the project layer in front of unit i, whose BatchNorm takes backward sums that unit i's first layer may leave; else nullptr
static const void* leaves_sums(const ftp_stage* s, const Views& v, size_t i) {
  if (i == 0) return nullptr;
  const UnitPlan& p = s->plan[i];
  const UnitPlan& q = s->plan[i - 1];
  if (p.info->subs.empty() || p.info->subs[0].type != SUB_PW || p.at_once[0] || q.info->subs.empty()) return nullptr;
  const ConvGeom& g = p.info->subs[0].g;
  const size_t M = (size_t)s->batch * g.Hout * g.Wout;
  const HView of{v.sub_out[i - 1].back().z, nullptr, nullptr, FTP_ACT_NONE};
  if (q.info->d.kind != FTP_UNIT_INVRES) return nullptr;
  return !bn_bwd_small_ok(M, g.Cin) || (takes_sums(s, q, q.info->subs.size() - 1) && pw_dgrad_sums_ok(s->dt, M, g.Cin, g.Cout, of)) ? of.z : nullptr;
}

// part: BWD_FROM_DZ in a stage that defers, where the caller has taken the layer's places
// z_sum: dIn is the gradient of a BatchNorm without activation over this tensor, whose backward can use the sums (leaves_sums)
static int sub_backward(ftp_stage* s, Slot& sl, const UnitPlan& p, size_t k, const void* dA, HView in, HView out,
                        void* dIn, const void* res, const WeightSet& W, hipStream_t st, int mode = BWD_FULL,
                        bool unit_fork = false, float* part = nullptr, const void* z_sum = nullptr) {
  const Sub& sb = p.info->subs[k];
  ConvGeom g = sb.g; g.N = s->batch;
  int C = g.Cout;
  size_t M = (size_t)s->batch * g.Hout * g.Wout;
  float* stt = sl.stats + p.st_off[k];
  // the fork and join cost four event calls per layer and a cross-stream dependency: long kernels only
  const bool overlap = mode == BWD_FULL && stage_overlaps(s) && M * (size_t)C >= ((size_t)1 << 20);
  int b = 0, rc_join = 0;
  void* dz = const_cast<void*>(dA);
  // one fork for the whole unit (see PendingWgrad): this layer's dz goes into the unit's buffer set
  const bool batched = unit_fork && overlap && k < 3 && sb.type == SUB_PW && dIn != nullptr && s->dzring[0] != nullptr &&
                       M * (size_t)C * s->es <= s->dzring_bytes;
  // An expand layer in bfloat16: behind the BatchNorm reductions the rest of its backward (dz, data gradient,
  // weight gradient) is one pass on this stream; dz never reaches memory.
  if (mode == BWD_FULL && sb.type == SUB_PW && dIn && !bn_bwd_small_ok(M, C) && pw_bwd_fused_ok(s->dt, M, g.Cin, g.Cout, in) &&
      (s->defers || (s->ws_fused && pw_bwd_fused_ws(M, g.Cin, g.Cout) <= s->ws_fused_floats))) {
    ftp_stage::LeftSums sums = take_sums(s, dA);
    if (!sums.of) bn_bwd_reduce(s->dt, st, dA, out.z, M, C, out.scale, out.shift, sb.act, sums.partial = s->bn_part, &sums.P);
    bn_bwd_finalize(st, sums.partial, sums.P, M, C, W.w32 + p.p_off + sb.gamma_off, stt, stt + C, s->grads + p.p_off + sb.gamma_off,
                    s->grads + p.p_off + sb.beta_off, s->coef);
    // the sum of the kernel's partial weight gradients is off the data-gradient chain: it goes to the side stream,
    // and the next user of the partial buffer waits for it
    const bool last = !s->defers && &p == &s->plan[0], aside = stage_overlaps(s) && !last;
    const int sums_in = z_sum ? pw_bwd_fused_sums(M, g.Cin, g.Cout) : 0;
    if (s->join_pending[2]) {
      HIP_TRY(hipStreamWaitEvent(st, s->ev_join[2], 0));
      s->join_pending[2] = false;
    }
    pw_bwd_fused(st, dA, out, s->coef, conv_w(s, W, p.p_off + sb.w_off), in.z, res, M, g.Cin, g.Cout,
                 s->defers ? take_places(s, 0, p.part[k], st).part : s->ws_fused, s->grads + p.p_off + sb.w_off, dIn, aside ? s->side : st,
                 aside ? s->ev_fork[2] : nullptr, s->defers ? &s->q_red : last ? &s->q_late : nullptr, sums_in > 0 ? z_sum : nullptr, s->bn_part);
    if (sums_in > 0) leave_sums(s, dIn, s->bn_part, sums_in);
    if (aside) {
      HIP_TRY(hipEventRecord(s->ev_join[2], s->side));
      s->join_pending[2] = true;
    }
    return FTP_OK;
  }
  // A depthwise layer: behind the sums of its BatchNorm one pass does the rest, and leaves the sums of the BatchNorm in front
  // and the weight gradient's partials.  dIn is not dA.
  if (sb.type == SUB_DW) {
    const bool small = bn_bwd_small_ok(M, C) != 0;
    if (dw_bwd_ws(s->dt, g) > (s->defers ? p.part[k] : p.late_floats)) {
      ftp_set_error("stage_backward: no place for a depthwise layer's partial weight gradients"); return FTP_ERR_UNSUPPORTED;
    }
    Places at{nullptr, s->ws_late + p.late_part};
    if (s->defers) {
      at = take_places(s, small ? dz_size(s, sb) : 0, p.part[k], st);
    } else if (small) {
      b = (int)(s->n_sub_bwd++ & 1u);
      at.dz = s->gbuf[b ? 4 : 2];
      if (s->join_pending[b]) {            // the weight gradient that last read this dz buffer must be done
        HIP_TRY(hipStreamWaitEvent(st, s->ev_join[b], 0));
        s->join_pending[b] = false;
      }
    }
    const float* gamma = W.w32 + p.p_off + sb.gamma_off;
    float *gg = s->grads + p.p_off + sb.gamma_off, *gb = s->grads + p.p_off + sb.beta_off;
    const int P = dw_bwd_partials(s->dt, g);
    ftp_stage::LeftSums sums = take_sums(s, dA);
    BnPending left{};
    float* fill = s->bn_part;
    if (small) {
      bn_bwd_small(s->dt, st, dA, out.z, M, C, out.scale, out.shift, sb.act, gamma, stt, stt + C, gg, gb, at.dz);
    } else {
      if (!sums.of) bn_bwd_reduce(s->dt, st, dA, out.z, M, C, out.scale, out.shift, sb.act, sums.partial = s->bn_part, &sums.P);
      if (bn_finish_ok(M, C, sums.P) && P <= kBnPartials / 2) {
        left = BnPending{sums.partial, sums.P, M, gamma, nullptr, stt, stt + C, nullptr, nullptr, nullptr, nullptr};
        if (sums.partial == fill) fill = other_partials(s);
      } else {
        bn_bwd_finalize(st, sums.partial, sums.P, M, C, gamma, stt, stt + C, gg, gb, s->coef);
      }
    }
    // behind another layer's BatchNorm: dIn is the gradient of its activated output
    if (!dIn || in.scale == nullptr || bn_bwd_small_ok((size_t)s->batch * g.Hin * g.Win, g.Cin)) fill = nullptr;
    dw_bwd(s->dt, st, small ? at.dz : dA, small ? nullptr : &out, left.partial ? &left : nullptr, s->coef, gg, gb, conv_w(s, W, p.p_off + sb.w_off), g, dIn, in,
           fill, at.part);
    if (fill) leave_sums(s, dIn, fill, P);
    (s->defers ? s->q_red : s->q_late).push_back(ReduceJob{at.part, s->grads + p.p_off + sb.w_off, P, 9 * C, C, 1, 9, C});
    return FTP_OK;
  }
  // A pointwise layer's data gradient, with the backward sums of the BatchNorm in front where its kernel can leave them and that layer takes them: the one
  // in front within the block, or that of the block in front (z_sum).  Convolutions as units of their own keep the pass, and with it the gradients of a stage of
  // one layer bit for bit.
  auto run_pw_dgrad = [&]() {
    const HView of = z_sum ? HView{z_sum, nullptr, nullptr, FTP_ACT_NONE} : k > 0 && in.scale && !bn_bwd_small_ok(M, g.Cin) ? in : HView{};
    float* const sums = of.z && pw_dgrad_sums_ok(s->dt, M, g.Cin, g.Cout, of) ? s->bn_part : nullptr;
    int P = 0;
    pw_dgrad(s->dt, st, dz, conv_w(s, W, p.p_off + sb.w_off), res, M, g.Cin, g.Cout, dIn, of, sums, &P);
    if (sums) leave_sums(s, dIn, sums, P);
  };
  // noted for the end of the backward call: dz stays where it is written until then
  const bool noted = s->defers && (sb.type != SUB_DIRECT || p.axis[k]);
  if (mode != BWD_FROM_DZ) {
    ftp_stage::LeftSums sums = take_sums(s, dA);
    const BnPending left{sums.partial, sums.P, M, W.w32 + p.p_off + sb.gamma_off, nullptr, stt, stt + C, nullptr, nullptr, nullptr, nullptr};
    const BnBwdIn own{dA, out, nullptr, nullptr, nullptr, s->grads + p.p_off + sb.gamma_off, s->grads + p.p_off + sb.beta_off};
    if (noted && sums.of && conv1d_takes_sums(s, p)) {         // no dz, and no partial weight gradients: it needs no places
      float* const fill = !dIn || !conv1d_leaves_sums(s, &p - s->plan.data()) ? nullptr : sums.partial == s->bn_part ? other_partials(s) : s->bn_part;
      int P = 0;
      conv1d_bwd_small(s->dt, st, nullptr, conv_w(s, W, p.p_off + sb.w_off), in, g, s->grads + p.p_off + sb.w_off, dIn, &left, &own, fill, &P);
      if (fill) leave_sums(s, dIn, fill, P);
      return FTP_OK;
    }
    if (batched) dz = s->dzring[s->bset * 3 + (int)k];
    else if (s->defers) {
      const Places at = take_places(s, dz_size(s, sb), p.part[k], st);
      dz = at.dz;
      part = at.part;
    } else {
      b = (int)(s->n_sub_bwd++ & 1u);
      dz = s->gbuf[b ? 4 : 2];
    }
    const bool small = bn_bwd_small_ok(M, C) != 0;
    bool finishes = false;
    if (noted && sums.of && takes_sums(s, p, k)) {
      s->q_pw.push_back(PwWgradJob{dz, in, M, g.Cin, g.Cout, part, s->grads + p.p_off + sb.w_off});
      pw_dgrad_pro(s->dt, st, left, own, dz, conv_w(s, W, p.p_off + sb.w_off), M, g.Cin, g.Cout, dIn);
      return FTP_OK;
    }
    if (!small) {
      if (!sums.of) bn_bwd_reduce(s->dt, st, dA, out.z, M, C, out.scale, out.shift, sb.act, sums.partial = s->bn_part, &sums.P);
      finishes = bn_finish_ok(M, C, sums.P) != 0;
      if (!finishes)
        bn_bwd_finalize(st, sums.partial, sums.P, M, C, W.w32 + p.p_off + sb.gamma_off, stt, stt + C, s->grads + p.p_off + sb.gamma_off,
                        s->grads + p.p_off + sb.beta_off, s->coef);
    }
    if (batched) {
      if (!s->bset_open) {                // the unit's first write into this set: the weight gradients that last read it must be done
        if (s->bjoin_pending[s->bset]) {
          HIP_TRY(hipStreamWaitEvent(st, s->ev_bjoin[s->bset], 0));
          s->bjoin_pending[s->bset] = false;
        }
        s->bset_open = true;
      }
    } else if (s->join_pending[b]) {      // the weight gradient that last read this dz buffer must be done
      HIP_TRY(hipStreamWaitEvent(st, s->ev_join[b], 0));
      s->join_pending[b] = false;
    }
    if (small)
      bn_bwd_small(s->dt, st, dA, out.z, M, C, out.scale, out.shift, sb.act, W.w32 + p.p_off + sb.gamma_off, stt, stt + C,
                   s->grads + p.p_off + sb.gamma_off, s->grads + p.p_off + sb.beta_off, dz);
    else if (finishes)
      bn_bwd_finish_apply(s->dt, st, dA, out.z, M, C, out.scale, out.shift, sb.act,
                          BnPending{sums.partial, sums.P, M, W.w32 + p.p_off + sb.gamma_off, nullptr, stt, stt + C, nullptr, nullptr, nullptr, nullptr},
                          s->grads + p.p_off + sb.gamma_off, s->grads + p.p_off + sb.beta_off, dz);
    else
      bn_bwd_apply(s->dt, st, dA, out.z, M, C, out.scale, out.shift, sb.act, s->coef, dz);
  }
  hipStream_t ws = st;
  s->left.of = nullptr;                // where the caller formed dz
  auto run_conv1d_dgrad = [&]() {
    // behind another convolution of the stage: this is the dA of that one's BatchNorm + activation
    const bool sums = in.scale != nullptr && !bn_bwd_small_ok((size_t)s->batch * g.Hin * g.Win, g.Cin);
    int P = 0;
    conv1d_dgrad(s->dt, st, dz, conv_w(s, W, p.p_off + sb.w_off), g, dIn, in, sums ? s->bn_part : nullptr, &P);
    if (sums) leave_sums(s, dIn, s->bn_part, P);
  };
  if (batched && mode == BWD_FULL) {
    // noted for the unit's fork; the data gradient goes on as it would behind a forked weight gradient
    if (s->n_pend >= 3) { ftp_set_error("stage_backward: more weight gradients noted for a unit than it has layers"); return FTP_ERR_UNSUPPORTED; }
    s->pend[s->n_pend++] = ftp_stage::PendingWgrad{dz, in, g, M, s->grads + p.p_off + sb.w_off};
    run_pw_dgrad();
    return FTP_OK;
  }
  if (noted) {
    float* gw = s->grads + p.p_off + sb.w_off;
    const void* w = conv_w(s, W, p.p_off + sb.w_off);
    if (p.at_once[k]) {
      if (dIn) pw_bwd(s->dt, st, dz, w, res, in, M, g.Cin, g.Cout, part, gw, dIn);
      else pw_wgrad(s->dt, st, dz, in, M, g.Cin, g.Cout, part, gw);
    } else if (sb.type == SUB_PW) {
      s->q_pw.push_back(PwWgradJob{dz, in, M, g.Cin, g.Cout, part, gw});
      if (dIn) run_pw_dgrad();
    } else if (dIn && conv1d_small_ok(g)) {
      float* const fill = conv1d_leaves_sums(s, &p - s->plan.data()) ? s->bn_part : nullptr;
      int P = 0;
      conv1d_bwd_small(s->dt, st, dz, w, in, g, gw, dIn, nullptr, nullptr, fill, &P);
      if (fill) leave_sums(s, dIn, fill, P);
    } else {
      conv1d_wgrad(s->dt, st, dz, in, g, part, gw, &s->q_red);
      if (dIn) run_conv1d_dgrad();
    }
    return FTP_OK;
  }
  // the first layer of the stage, last in this pass and without a data gradient: its weight gradient is all that is
  // left for this stream, so it runs here with a workspace of its own while the side stream works off its queue
  const bool tail_here = overlap && dIn == nullptr && s->ws_tail != nullptr && &p == &s->plan[0] && k == 0;
  float* wsp = tail_here ? s->ws_tail : s->ws;
  if (overlap && !tail_here) {
    HIP_TRY(hipEventRecord(s->ev_fork[b], st));
    HIP_TRY(hipStreamWaitEvent(s->side, s->ev_fork[b], 0));
    ws = s->side;
  }
  const void* w = conv_w(s, W, p.p_off + sb.w_off);
  float* gw = s->grads + p.p_off + sb.w_off;
  // a layer too short to fork still takes the partial-sum workspace: in a stage that forks its longer layers the
  // side stream may be in the middle of using it, so that work is waited for first
  if (!overlap && stage_overlaps(s) && (rc_join = join_side(s, st))) return rc_join;
  if (sb.type == SUB_PW && !overlap && dIn) {
    pw_bwd(s->dt, st, dz, w, res, in, M, g.Cin, g.Cout, s->ws, gw, dIn);
    return FTP_OK;
  }
  if (p.axis[k]) {
    if (!overlap && dIn && conv1d_small_ok(g)) { conv1d_bwd_small(s->dt, st, dz, w, in, g, gw, dIn); return FTP_OK; }
    conv1d_wgrad(s->dt, ws, dz, in, g, wsp, gw, &s->q_red);
    reduce_group(ws, s->q_red.data(), (int)s->q_red.size());
    s->q_red.clear();
  }
  else if (sb.type == SUB_DIRECT) {
    conv_direct_wgrad(s->dt, ws, dz, in, g, s->im2col, wsp, gw, s->im2col_of == out.z);
    s->im2col_of = nullptr;      // one weight gradient per forward: nobody else can want these patches
  }
  else pw_wgrad(s->dt, ws, dz, in, M, g.Cin, g.Cout, wsp, gw);
  if (overlap && !tail_here) {
    HIP_TRY(hipEventRecord(s->ev_join[b], s->side));
    s->join_pending[b] = true;
  }
  if (dIn) {
    if (p.axis[k]) run_conv1d_dgrad();
    else if (sb.type == SUB_DIRECT) {
      // the scratch buffers are shared with the weight gradients: fine on one stream, but a stage that runs them on
      // the side stream keeps the direct kernel
      if (conv_direct_dgrad_gemm_ok(g) && !stage_forks(s) && s->im2col) {
        conv_direct_dgrad_gemm(s->dt, st, dz, w, g, s->im2col, s->ws, dIn);
        s->im2col_of = nullptr;
      }
      else conv_direct_dgrad(s->dt, st, dz, w, g, dIn);
    }
    else run_pw_dgrad();
  }
  return FTP_OK;
}

// every weight gradient noted so far, and the sums of what the kernels left
static void run_noted(ftp_stage* s, hipStream_t st) {
  pw_wgrad_group(s->dt, st, s->q_pw.data(), (int)s->q_pw.size(), s->share, &s->q_red);
  reduce_group(st, s->q_red.data(), (int)s->q_red.size());
  reduce_group(st, s->q_late.data(), (int)s->q_late.size());
  s->q_pw.clear(); s->q_red.clear(); s->q_late.clear();
  s->dz_used = s->part_used = 0;         // what reads the stores is ahead of what this stream writes there next
}

// the weight gradients a unit has noted: one fork behind everything the unit has enqueued, all of them on the side
// stream, one join event for the unit's buffer set
static int flush_unit_fork(ftp_stage* s, hipStream_t st) {
  if (s->n_pend == 0) { s->bset_open = false; return FTP_OK; }
  HIP_TRY(hipEventRecord(s->ev_bfork[s->bset], st));
  HIP_TRY(hipStreamWaitEvent(s->side, s->ev_bfork[s->bset], 0));
  for (int i = 0; i < s->n_pend; ++i) {
    const ftp_stage::PendingWgrad& w = s->pend[i];
    pw_wgrad(s->dt, s->side, w.dz, w.in, w.M, w.g.Cin, w.g.Cout, s->ws, w.gw);
  }
  HIP_TRY(hipEventRecord(s->ev_bjoin[s->bset], s->side));
  s->bjoin_pending[s->bset] = true;
  s->n_pend = 0;
  s->bset ^= 1;
  s->bset_open = false;
  return FTP_OK;
}

// all side-stream work of this backward is ordered before whatever the caller enqueues next
static int join_side(ftp_stage* s, hipStream_t st) {
  for (int b = 0; b < 3; ++b)
    if (s->join_pending[b]) {
      HIP_TRY(hipStreamWaitEvent(st, s->ev_join[b], 0));
      s->join_pending[b] = false;
    }
  for (int b = 0; b < 2; ++b)
    if (s->bjoin_pending[b]) {
      HIP_TRY(hipStreamWaitEvent(st, s->ev_bjoin[b], 0));
      s->bjoin_pending[b] = false;
    }
  return FTP_OK;
}

extern "C" int ftp_stage_backward(ftp_stage* s, int slot, const void* dy_dev, void* dx_dev, void* stream) {
  int rc = check_call(s, slot, "stage_backward");
  if (rc) return rc;
  Slot& sl = s->slots[slot];
  if (!sl.busy) { ftp_set_error("stage_backward: slot %d holds no forwarded batch", slot); return FTP_ERR_SLOT; }
  if (!dy_dev && !(s->has_loss && sl.has_loss)) {
    ftp_set_error("stage_backward: dy_dev is NULL and ftp_stage_loss has not seeded slot %d", slot);
    return FTP_ERR_ARG;
  }
  hipStream_t st = (hipStream_t)stream;
  if (s->timer && sl.timer_idx >= 0) HIP_TRY(hipEventRecord(s->timer->ev[sl.timer_idx][2], st));
  Views v;
  build_views(s, sl, &v);
  WeightSet W{sl.has_snap ? sl.snap_w : s->params, (const char*)(sl.has_snap ? sl.snap_lp : s->w_lp)};
  if (s->recompute && s->stash_owner != slot) {
    // the intermediates of this batch are gone: forward again from the kept input with the weights of its
    // forward; not a training forward, so the running statistics stay as they are
    const UnitInfo& first = *s->plan[0].info;
    HIP_TRY(hipMemcpyAsync(sl.stash, sl.xin_keep, (size_t)s->batch * first.inH * first.inW * first.inC * s->es,
                           hipMemcpyDeviceToDevice, st));
    s->bn_mom = 0.f;
    rc = forward_units(s, sl, v, W, st);
    s->bn_mom = kBnMomentum;
    if (rc) return rc;
    s->stash_owner = slot;
  }
  s->q_pw.clear(); s->q_red.clear(); s->q_late.clear();
  s->dz_used = s->part_used = 0;
  s->left.of = nullptr;
  s->n_pend = 0; s->bset_open = false;              // nothing is left noted by a call that ended in an error
  const void* d = dy_dev ? dy_dev : sl.dlogits;     // gradient of the current unit's output (read only)
  int flip = 0;
  bool gap_done = false;
  for (int i = (int)s->plan.size() - 1; i >= 0; --i) {
    const UnitPlan& p = s->plan[i];
    const UnitInfo& u = *p.info;
    if (s->prof) HIP_TRY(hipEventRecord(s->prof->b0[i], st));
    // where the gradient of this unit's input goes: the boundary buffer that does not hold d
    void* next = i > 0 ? (void*)s->gbuf[flip] : dx_dev;
    bool produced = true;
    HView in = v.unit_in[i];
    switch (u.d.kind) {
      case FTP_UNIT_LOSS:
        produced = false;   // the logits gradient passes through unchanged
        if (i == 0 && dx_dev) HIP_TRY(hipMemcpyAsync(dx_dev, d, (size_t)s->batch * u.inC * s->es, hipMemcpyDeviceToDevice, st));
        break;
      case FTP_UNIT_FC: {
        size_t woff = p.p_off;
        if (fc_bwd_ok(s->batch, u.outC, u.inC)) {
          // behind an average (not the stage's first unit): its backward is part of the data gradient's last step
          const UnitInfo* pu = i > 1 ? s->plan[i - 1].info : nullptr;
          const int HW = pu && pu->d.kind == FTP_UNIT_GAP && s->prof == nullptr && fc_bwd_gap_ok(s->batch, pu->inH * pu->inW, u.inC)
                             ? pu->inH * pu->inW : 0;
          const float* open = HW > 0 ? open_sums(s, sl, i - 1) : nullptr;
          int P = 0;
          fc_bwd(s->dt, st, d, in, conv_w(s, W, woff), s->batch, u.outC, u.inC, s->grads + woff, s->grads + woff + (size_t)u.outC * u.inC, next, HW,
                 open, open ? s->bn_part : nullptr, &P);
          if (open) leave_sums(s, next, s->bn_part, P);
          gap_done = HW > 0;
          break;
        }
        pw_wgrad(s->dt, st, d, in, (size_t)s->batch, u.inC, u.outC, s->ws, s->grads + woff);
        bias_grad(s->dt, st, d, s->batch, u.outC, s->grads + woff + (size_t)u.outC * u.inC);
        if (next) pw_dgrad(s->dt, st, d, conv_w(s, W, woff), nullptr, (size_t)s->batch, u.inC, u.outC, next);
        break;
      }
      case FTP_UNIT_GAP:
        if (gap_done) { produced = false; gap_done = false; }         // d is its input's gradient already
        else if (next) {
          const float* open = open_sums(s, sl, i);
          int P = 0;
          gap_bwd(s->dt, st, d, s->batch, u.inH * u.inW, u.inC, next, open, open ? s->bn_part : nullptr, &P);
          if (open) leave_sums(s, next, s->bn_part, P);
        }
        break;
      case FTP_UNIT_CONV:
        if ((rc = sub_backward(s, sl, p, 0, d, in, v.sub_out[i][0], next, nullptr, W, st, BWD_FULL, false, nullptr, leaves_sums(s, v, i)))) return rc;
        break;
      case FTP_UNIT_INVRES: {
        size_t ns = u.subs.size();
        // the gradients of the depthwise layer's output and input lie in different buffers; the boundary buffer that the unit's input gradient will take is
        // free until then
        void *tmp = s->gbuf[3], *mid = ns == 3 || u.residual ? (void*)s->gbuf[flip] : tmp;
        // project: gradient of the activated depthwise output
        // one fork for the unit when every layer's dz fits the small buffer sets
        bool uf = ns == 3 && s->dzring[0] != nullptr;
        for (const Sub& sb : u.subs)
          if ((size_t)s->batch * sb.g.Hout * sb.g.Wout * sb.g.Cout * s->es > s->dzring_bytes) uf = false;
        if ((rc = sub_backward(s, sl, p, ns - 1, d, v.sub_out[i][ns - 2], v.sub_out[i][ns - 1], mid, nullptr, W, st, BWD_FULL, uf))) return rc;
        ConvGeom gd = ns == 3 ? u.subs[1].g : ConvGeom{};
        gd.N = s->batch;
        if (ns == 3 && s->defers && dw_bwd_small_ok(gd)) {
          // short tensors: depthwise dgrad + wgrad and the expand layer's BatchNorm backward in one launch
          const Sub& s0 = u.subs[0];
          const Sub& s1 = u.subs[1];
          // the depthwise layer's own BatchNorm backward happens inside too: its dz never reaches memory
          const Places at = take_places(s, dz_size(s, s0), p.part[0], st);
          void* dz1 = at.dz;
          float* st0 = sl.stats + p.st_off[0];
          float* st1 = sl.stats + p.st_off[1];
          BnBwdIn bo{mid, v.sub_out[i][1], W.w32 + p.p_off + s1.gamma_off, st1, st1 + s1.g.Cout,
                     s->grads + p.p_off + s1.gamma_off, s->grads + p.p_off + s1.beta_off};
          dw_bwd_small(s->dt, st, bo, conv_w(s, W, p.p_off + s1.w_off), v.sub_out[i][0], gd, W.w32 + p.p_off + s0.gamma_off, st0,
                       st0 + s0.g.Cout, s->grads + p.p_off + s1.w_off, s->grads + p.p_off + s0.gamma_off,
                       s->grads + p.p_off + s0.beta_off, dz1);
          if ((rc = sub_backward(s, sl, p, 0, dz1, in, v.sub_out[i][0], next, u.residual ? d : nullptr, W, st, BWD_FROM_DZ, false, at.part,
                                 leaves_sums(s, v, i)))) return rc;
        } else if (ns == 3) {
          if ((rc = sub_backward(s, sl, p, 1, mid, v.sub_out[i][0], v.sub_out[i][1], tmp, nullptr, W, st, BWD_FULL, uf))) return rc;
          if ((rc = sub_backward(s, sl, p, 0, tmp, in, v.sub_out[i][0], next, u.residual ? d : nullptr, W, st, BWD_FULL, uf, nullptr,
                                 leaves_sums(s, v, i)))) return rc;
          if ((rc = flush_unit_fork(s, st))) return rc;
        } else {
          if (next && u.residual) {
            if ((rc = sub_backward(s, sl, p, 0, mid, in, v.sub_out[i][0], tmp, nullptr, W, st))) return rc;
            bn_apply(s->dt, st, plain(tmp), (size_t)s->batch * u.inH * u.inW, u.inC, d, next);
          } else {
            if ((rc = sub_backward(s, sl, p, 0, mid, in, v.sub_out[i][0], next, nullptr, W, st))) return rc;
          }
        }
        break;
      }
      default:
        break;
    }
    if (s->prof) {                                    // a unit's time includes its weight gradients
      run_noted(s, st);
      HIP_TRY(hipEventRecord(s->prof->b1[i], st));
    }
    if (produced && next) { d = next; if (i > 0) flip ^= 1; }
  }
  run_noted(s, st);
  if ((rc = join_side(s, st))) return rc;
  if (s->timer && sl.timer_idx >= 0) {
    HIP_TRY(hipEventRecord(s->timer->ev[sl.timer_idx][3], st));
    s->timer->bwd_done[sl.timer_idx] = true;
    sl.timer_idx = -1;
  }
  HIP_TRY(hipGetLastError());
  if (const char* why = launch_plan_failure_take()) { ftp_set_error("%s", why); return FTP_ERR_UNSUPPORTED; }
  sl.busy = false; sl.has_snap = false; sl.has_loss = false;
  return FTP_OK;
}

extern "C" int ftp_stage_timing(ftp_stage* s, int enable) {
  if (!s) { ftp_set_error("stage_timing: NULL stage"); return FTP_ERR_ARG; }
  for (auto& sl : s->slots)
    if (sl.busy) { ftp_set_error("stage_timing: switch it while no batch is in flight"); return FTP_ERR_SLOT; }
  if (!enable) {
    if (s->timer) {
      if (s->timer->created)
        for (auto& q : s->timer->ev)
          for (auto& e : q) (void)hipEventDestroy(e);
      delete s->timer;
      s->timer = nullptr;
    }
    return FTP_OK;
  }
  if (!s->timer) {
    s->timer = new ExecTimer();
    for (auto& q : s->timer->ev)
      for (auto& e : q) HIP_TRY(hipEventCreate(&e));
    s->timer->created = true;
  }
  s->timer->used = 0;
  return FTP_OK;
}

extern "C" int ftp_stage_timing_read(ftp_stage* s, double* mean_ns, int* n_batches) {
  if (!s || !mean_ns || !n_batches) { ftp_set_error("stage_timing_read: NULL argument"); return FTP_ERR_ARG; }
  if (!s->timer) { ftp_set_error("stage_timing_read: execution timing is not enabled"); return FTP_ERR_ARG; }
  double sum = 0.0;
  int n = 0;
  for (int i = 0; i < s->timer->used; ++i) {
    if (!s->timer->bwd_done[i]) continue;              // forwarded, not yet backwarded: not a whole batch
    float f = 0.f, b = 0.f;
    HIP_TRY(hipEventSynchronize(s->timer->ev[i][3]));
    HIP_TRY(hipEventElapsedTime(&f, s->timer->ev[i][0], s->timer->ev[i][1]));
    HIP_TRY(hipEventElapsedTime(&b, s->timer->ev[i][2], s->timer->ev[i][3]));
    sum += ((double)f + (double)b) * 1e6;
    ++n;
  }
  for (auto& sl : s->slots) sl.timer_idx = -1;         // batches in flight are dropped from the measurement
  s->timer->used = 0;
  *n_batches = n;
  *mean_ns = n ? sum / n : 0.0;
  return FTP_OK;
}

extern "C" int ftp_stage_update(ftp_stage* s, const ftp_sgd* opt, void* stream) {
  if (!s || !opt) { ftp_set_error("stage_update: NULL argument"); return FTP_ERR_ARG; }
  if (!(std::isfinite(opt->lr) && std::isfinite(opt->momentum) && std::isfinite(opt->weight_decay))) {
    ftp_set_error("stage_update: non-finite hyper-parameter");
    return FTP_ERR_VALUE;
  }
  if (s->n_param) sgd_update((hipStream_t)stream, s->params, s->grads, s->mom, s->w_lp, s->n_param, opt->lr, opt->momentum, opt->weight_decay);
  HIP_TRY(hipGetLastError());
  if (const char* why = launch_plan_failure_take()) { ftp_set_error("%s", why); return FTP_ERR_UNSUPPORTED; }
  return FTP_OK;
}

// ------------------------------------------------------------ loss without a stage, without allocation
// Row losses of ftp_softmax_ce_static, or sums of eight: partial results inside the call.  One copy per GPU, held until the
// process ends; in host code the name is only a handle for hipGetSymbolAddress, the kernels get the address.
enum { kStaticLossMaxBatch = FTP_STATIC_LOSS_MAX_BATCH, kStaticMaxDevices = 64, kStaticStreams = 64 };
static __device__ __align__(256) float scratch[kStaticLossMaxBatch + kStaticStreams * kCeCounters];
static float* g_scratch_ptr[kStaticMaxDevices];     // per device: the address of that GPU's copy
static std::mutex g_scratch_mu;
// Behind the losses: counters for the one-launch form, those of each stream its own (calls of one stream follow one another).  The first
// kStaticStreams streams of a GPU have some; a stream that comes later, the handle that stands for a stream of each thread, and a call that is being
// captured (its graph may run on any stream) take two launches.
static hipStream_t g_scratch_stream[kStaticMaxDevices][kStaticStreams];
static int g_scratch_streams[kStaticMaxDevices];

static int static_scratch(hipStream_t st, bool counters, float** out, unsigned** arrived) {
  int dev = -1;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kStaticMaxDevices) { ftp_set_error("softmax_ce_static: device ordinal %d not supported", dev); return FTP_ERR_UNSUPPORTED; }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    float* p = nullptr;
    HIP_TRY(hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch)));    // with `dev` current: this GPU's copy
    if (!p) { ftp_set_error("softmax_ce_static: no device address for the scratch array"); return FTP_ERR_HIP; }
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  *arrived = nullptr;
  if (!counters) return FTP_OK;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cap) != hipSuccess) { (void)hipGetLastError(); return FTP_OK; }
  if (st == hipStreamPerThread || cap != hipStreamCaptureStatusNone) return FTP_OK;
  int i = 0;
  for (; i < g_scratch_streams[dev] && g_scratch_stream[dev][i] != st; ++i) {}
  if (i == kStaticStreams) return FTP_OK;
  if (i == g_scratch_streams[dev]) g_scratch_stream[dev][g_scratch_streams[dev]++] = st;
  *arrived = (unsigned*)*out + kStaticLossMaxBatch + i * kCeCounters;
  return FTP_OK;
}

extern "C" int ftp_softmax_ce_static(const void* logits_dev, const int32_t* labels_dev, int batch, int classes, ftp_dtype dtype,
                                     void* dlogits_dev, float* loss_dev, void* stream) {
  if (!logits_dev || !labels_dev || !dlogits_dev || !loss_dev) { ftp_set_error("softmax_ce_static: NULL argument"); return FTP_ERR_ARG; }
  if (dtype != FTP_F32 && dtype != FTP_BF16) { ftp_set_error("softmax_ce_static: unknown dtype %d", (int)dtype); return FTP_ERR_ARG; }
  if (batch < 1 || classes < 1) { ftp_set_error("softmax_ce_static: batch and classes must be positive"); return FTP_ERR_ARG; }
  if (batch > kStaticLossMaxBatch) {
    ftp_set_error("softmax_ce_static: batch %d is beyond the %d rows the static scratch array holds", batch, (int)kStaticLossMaxBatch);
    return FTP_ERR_ARG;
  }
  float* rows = nullptr;
  unsigned* arrived = nullptr;
  int rc = static_scratch((hipStream_t)stream, softmax_ce_arrives(batch, classes) != 0, &rows, &arrived);
  if (rc) return rc;
  // every row < batch is written before it is read and nothing beyond is read: nothing has to start at zero
  softmax_ce((int)dtype, (hipStream_t)stream, logits_dev, labels_dev, batch, classes, rows, dlogits_dev, loss_dev, arrived);
  HIP_TRY(hipGetLastError());
  if (const char* why = launch_plan_failure_take()) { ftp_set_error("%s", why); return FTP_ERR_UNSUPPORTED; }
  return FTP_OK;
}

// ------------------------------------------------------------ profile_layers
__global__ void synth_fill_k(float* p, size_t n, uint32_t salt, float amp) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    uint32_t h = (uint32_t)i * 2654435761u + salt;
    h ^= h >> 15; h *= 2246822519u; h ^= h >> 13; h *= 3266489917u; h ^= h >> 16;
    p[i] = ((float)(h >> 8) * (1.0f / 8388608.0f) - 1.0f) * amp;
  }
}

extern "C" int ftp_profile_layers(const ftp_model* m, int batch, int reps, double* t_ns, int64_t* out_bytes, void* stream) {
  if (!m || !t_ns || !out_bytes || batch < 1 || reps < 1) { ftp_set_error("profile_layers: bad argument"); return FTP_ERR_ARG; }
  int L = (int)m->units.size();
  ftp_stage* s = nullptr;
  int rc = ftp_stage_create(m, 0, L, batch, 1, &s);
  if (rc) return rc;
  hipStream_t st = (hipStream_t)stream;
  ProfEvents ev;
  float *x32 = nullptr, *loss = nullptr;
  void *x = nullptr, *dy = nullptr;
  int32_t* labels = nullptr;
  const UnitInfo& last = m->units[L - 1];
  size_t n_in = (size_t)batch * m->inH * m->inW * m->inC;
  size_t n_out = (size_t)batch * last.outH * last.outW * last.outC;
  size_t es = s->es;
  auto cleanup = [&]() {
    for (auto* vec : {&ev.f0, &ev.f1, &ev.b0, &ev.b1})
      for (hipEvent_t e : *vec) (void)hipEventDestroy(e);
    dfree(x32); dfree(x); dfree(dy); dfree(labels); dfree(loss);
    s->prof = nullptr;
    stage_free(s);
  };
#define PROF_TRY(expr)                                                                   \
  do {                                                                                   \
    hipError_t e_ = (expr);                                                              \
    if (e_ != hipSuccess) {                                                              \
      ftp_set_error("profile_layers: %s failed: %s", #expr, hipGetErrorString(e_));     \
      cleanup();                                                                         \
      return FTP_ERR_HIP;                                                                \
    }                                                                                    \
  } while (0)
  size_t nmax = n_in > n_out ? n_in : n_out;
  PROF_TRY(hipMalloc((void**)&x32, align_up(nmax * 4, 256)));
  PROF_TRY(hipMalloc(&x, align_up(n_in * es, 256)));
  PROF_TRY(hipMalloc(&dy, align_up(n_out * es, 256)));
  PROF_TRY(hipMalloc((void**)&labels, align_up((size_t)batch * 4, 256)));
  PROF_TRY(hipMalloc((void**)&loss, 256));
  // synthetic weights (uniform, variance 2/fan_in-like scale is irrelevant for timing), input and output gradient
  hipLaunchKernelGGL(synth_fill_k, dim3(1024), dim3(256), 0, st, s->params, s->n_param, 17u, 0.1f);
  if (s->w_lp) f32_to_storage(FTP_BF16, st, s->params, s->w_lp, s->n_param);
  hipLaunchKernelGGL(synth_fill_k, dim3(1024), dim3(256), 0, st, x32, n_in, 29u, 1.7f);
  f32_to_storage(s->dt, st, x32, x, n_in);
  hipLaunchKernelGGL(synth_fill_k, dim3(1024), dim3(256), 0, st, x32, n_out, 31u, 0.01f);
  f32_to_storage(s->dt, st, x32, dy, n_out);
  fill_zero(st, labels, align_up((size_t)batch * 4, 256));
  // gamma = 1 so that activations keep a sane scale
  for (const UnitPlan& p : s->plan)
    for (const Sub& sb : p.info->subs) {
      std::vector<float> ones(sb.g.Cout, 1.0f);
      PROF_TRY(hipMemcpyAsync(s->params + p.p_off + sb.gamma_off, ones.data(), ones.size() * 4, hipMemcpyHostToDevice, st));
      PROF_TRY(hipStreamSynchronize(st));
    }
  for (auto* vec : {&ev.f0, &ev.f1, &ev.b0, &ev.b1}) {
    vec->resize(L);
    for (int i = 0; i < L; ++i) PROF_TRY(hipEventCreate(&(*vec)[i]));
  }
  std::vector<double> acc(L, 0.0);
  bool has_loss = s->has_loss;
  for (int r = 0; r < reps + 2; ++r) {
    s->prof = &ev;
    rc = ftp_stage_forward(s, 0, x, nullptr, st);
    if (!rc && has_loss) rc = ftp_stage_loss(s, 0, labels, loss, st);
    if (!rc) rc = ftp_stage_backward(s, 0, has_loss ? nullptr : dy, nullptr, st);
    s->prof = nullptr;
    if (rc) { cleanup(); return rc; }
    PROF_TRY(hipStreamSynchronize(st));
    if (r < 2) continue;   // discarded warm-up runs
    for (int i = 0; i < L; ++i) {
      float f = 0.f, b = 0.f;
      PROF_TRY(hipEventElapsedTime(&f, ev.f0[i], ev.f1[i]));
      PROF_TRY(hipEventElapsedTime(&b, ev.b0[i], ev.b1[i]));
      acc[i] += ((double)f + (double)b) * 1e6;
    }
  }
  // The per-unit events need every unit to begin and end on the caller's stream, so a stage that normally runs its
  // weight gradients on a second stream was just timed without that overlap.  The per-unit times keep their
  // proportions and are scaled so that they add up to what a batch costs under the plan training really runs
  // (forward + loss + backward, timed like ftp_stage_timing does): the capacity equation divides a worker's
  // measured batch time by this sum, and the same device then comes out at capacity 1.
  double sum_units = 0.0, whole = 0.0;
  for (int i = 0; i < L; ++i) sum_units += acc[i] / reps;
  for (int r = 0; r < reps + 1; ++r) {
    PROF_TRY(hipEventRecord(ev.f0[0], st));
    rc = ftp_stage_forward(s, 0, x, nullptr, st);
    if (!rc && has_loss) rc = ftp_stage_loss(s, 0, labels, loss, st);
    if (!rc) rc = ftp_stage_backward(s, 0, has_loss ? nullptr : dy, nullptr, st);
    if (rc) { cleanup(); return rc; }
    PROF_TRY(hipEventRecord(ev.f1[0], st));
    PROF_TRY(hipStreamSynchronize(st));
    float ms = 0.f;
    PROF_TRY(hipEventElapsedTime(&ms, ev.f0[0], ev.f1[0]));
    if (r > 0) whole += (double)ms * 1e6;   // first run discarded: the other plan's kernels load their code
  }
  whole /= reps;
  const double k_plan = sum_units > 0.0 && whole > 0.0 ? whole / sum_units : 1.0;
  for (int i = 0; i < L; ++i) {
    double t = std::floor(acc[i] / reps * k_plan + 0.5);
    t_ns[i] = t < 1.0 ? 1.0 : t;
    const UnitInfo& u = m->units[i];
    out_bytes[i] = (int64_t)((size_t)batch * u.outH * u.outW * u.outC * es);
  }
  cleanup();
#undef PROF_TRY
  return FTP_OK;
}
