// C ABI of libstill: argument validation, workspace layout and the launch sequence of the prefill path.
// See include/still.h for the contract of every entry point.
#include "../../include/still.h"

#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <mutex>

#include "still_kernels.h"

namespace {

thread_local char g_err[512] = "";

still_status_t fail(still_status_t code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

// per-thread kernel timing (host-side event objects only): one (begin, end) pair per kernel, recorded on the
// stream that kernel runs on, in a ring of kProfRing sets so that a run of calls can be timed without a
// synchronisation in between
constexpr int kProfRing = 64;
struct Profile {
  bool on = false, created = false;
  bool last_only = false;   // record the last kernel's pair only (fewer markers in the stream)
  int calls = 0;   // prefill calls recorded since profiling was enabled
  hipEvent_t beg[kProfRing][STILL_PROFILE_SLOTS], end[kProfRing][STILL_PROFILE_SLOTS];
};
thread_local Profile g_prof;
const char* const kSlotNames[STILL_PROFILE_SLOTS] = {"transpose_v", "transpose_w", "score_select", "gather",
                                                     "keep_mask",   "la_states",   "la_prefix",    "sparse_attn_merge"};

void prof_begin(int slot, hipStream_t stream) {
  if (!g_prof.on || (g_prof.last_only && slot != STILL_PROFILE_SLOTS - 1)) return;
  if (!g_prof.created) {
    for (int r = 0; r < kProfRing; ++r)
      for (int i = 0; i < STILL_PROFILE_SLOTS; ++i)
        if (hipEventCreate(&g_prof.beg[r][i]) != hipSuccess || hipEventCreate(&g_prof.end[r][i]) != hipSuccess) {
          g_prof.on = false;
          return;
        }
    g_prof.created = true;
  }
  (void)hipEventRecord(g_prof.beg[g_prof.calls % kProfRing][slot], stream);
}

void prof_end(int slot, hipStream_t stream) {
  if (!g_prof.on || !g_prof.created || (g_prof.last_only && slot != STILL_PROFILE_SLOTS - 1)) return;
  (void)hipEventRecord(g_prof.end[g_prof.calls % kProfRing][slot], stream);
  if (slot == STILL_PROFILE_SLOTS - 1) ++g_prof.calls;
}

// The layout kernels (transposes of v and of the projection weights) do not depend on the scores and are bound by
// memory, the score kernel by the vector ALU: they run side by side, the layout kernels on a second stream of
// default priority that forks from the caller's stream at the start of the call and joins it again before the
// first kernel that reads their output.  The backward pass runs its softmax branch there.  One side stream and its events
// per host thread and device.
struct SideStream {
  bool ok = false;
  int dev = -1;
  hipStream_t s = nullptr;
  hipEvent_t fork = nullptr, join = nullptr, mid = nullptr;
};
thread_local SideStream g_side;

// Between a captured call and the end of its capture the helper stream belongs to that capture: a call on a stream outside it
// (eager, or in a capture of its own) that waited for the helper would be drawn into it, and the capture end unjoined.  Such
// a call takes its own stream alone.
bool in_another_capture(hipStream_t helper, hipStream_t stream) {
  hipStreamCaptureStatus own = hipStreamCaptureStatusNone, his = hipStreamCaptureStatusNone;
  unsigned long long own_id = 0, his_id = 0;
  if (hipStreamGetCaptureInfo(helper, &own, &own_id) != hipSuccess) return true;
  if (own == hipStreamCaptureStatusNone) return false;
  return hipStreamGetCaptureInfo(stream, &his, &his_id) != hipSuccess || his != own || his_id != own_id;
}

// the helper stream for a call on `stream`, or nullptr
SideStream* side_stream(hipStream_t stream) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return nullptr;
  if (g_side.ok && g_side.dev == dev) return in_another_capture(g_side.s, stream) ? nullptr : &g_side;
  if (g_side.ok) {   // the thread moved to another device: drop the old objects
    (void)hipEventDestroy(g_side.fork);
    (void)hipEventDestroy(g_side.join);
    (void)hipEventDestroy(g_side.mid);
    (void)hipStreamDestroy(g_side.s);
    g_side.ok = false;
  }
  if (hipStreamCreateWithFlags(&g_side.s, hipStreamNonBlocking) != hipSuccess) return nullptr;
  if (hipEventCreateWithFlags(&g_side.fork, hipEventDisableTiming) != hipSuccess) {
    (void)hipStreamDestroy(g_side.s);
    return nullptr;
  }
  if (hipEventCreateWithFlags(&g_side.join, hipEventDisableTiming) != hipSuccess) {
    (void)hipEventDestroy(g_side.fork);
    (void)hipStreamDestroy(g_side.s);
    return nullptr;
  }
  if (hipEventCreateWithFlags(&g_side.mid, hipEventDisableTiming) != hipSuccess) {
    (void)hipEventDestroy(g_side.fork);
    (void)hipEventDestroy(g_side.join);
    (void)hipStreamDestroy(g_side.s);
    return nullptr;
  }
  g_side.dev = dev;
  g_side.ok = true;
  return &g_side;
}

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline size_t esize(int dtype) { return dtype == STILL_BF16 ? 2 : 4; }
// A range of memory (empty for a null pointer), and whether two of them meet.
struct Span {
  uintptr_t lo, hi;
};
inline Span flat_span(const void* x, size_t bytes) {
  const uintptr_t lo = reinterpret_cast<uintptr_t>(x);
  return {lo, x != nullptr ? lo + bytes : lo};
}
inline bool meet(const Span& a, const Span& b) { return a.lo < b.hi && b.lo < a.hi; }
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }
inline int retained_budget(const still_params_t* p) { return p->max_retained > 0 ? p->max_retained : still::kNoBudget; }

still_status_t validate_params(const still_params_t* p, bool need_n) {
  if (p == nullptr) return fail(STILL_ERR_INVALID_ARG, "params is NULL");
  if (p->dtype != STILL_F32 && p->dtype != STILL_BF16) return fail(STILL_ERR_INVALID_ARG, "dtype %d unknown", p->dtype);
  if (p->B < 1 || p->Hq < 1 || p->Hkv < 1) return fail(STILL_ERR_INVALID_ARG, "B, Hq, Hkv must be >= 1");
  if (need_n && p->N < 1) return fail(STILL_ERR_INVALID_ARG, "N must be >= 1 (got %d)", p->N);
  if (p->lambda < 0 || p->lambda > p->C) return fail(STILL_ERR_INVALID_ARG, "lambda %d outside [0, C=%d]", p->lambda, p->C);
  if (p->W < 1) return fail(STILL_ERR_INVALID_ARG, "W must be >= 1");
  if (p->gate_activation != 0 && p->gate_activation != 1)
    return fail(STILL_ERR_INVALID_ARG, "gate_activation %d unknown (0: none, 1: sigmoid)", p->gate_activation);
  if (p->budget_policy != 0 && p->budget_policy != 1)
    return fail(STILL_ERR_INVALID_ARG, "budget_policy %d unknown (0: stop adding, 1: evict the lowest score)",
                p->budget_policy);
  if (p->budget_policy == 1) {
    if (p->max_retained < 1) return fail(STILL_ERR_INVALID_ARG, "budget_policy 1 needs max_retained >= 1");
    if (p->shared_selection) return fail(STILL_ERR_UNSUPPORTED, "budget_policy 1 is defined per query head");
    if (p->max_retained > still::kMaxEvictBudget)
      return fail(STILL_ERR_UNSUPPORTED, "budget_policy 1: max_retained %d > %d", p->max_retained,
                  still::kMaxEvictBudget);
  }
  if (!(p->eps > 0.f)) return fail(STILL_ERR_INVALID_ARG, "eps must be > 0");
  if (!(p->scale > 0.f)) return fail(STILL_ERR_INVALID_ARG, "scale must be > 0");
  if (p->Hq > still::kMaxHq) return fail(STILL_ERR_UNSUPPORTED, "Hq %d > %d", p->Hq, still::kMaxHq);
  if (p->kv_head_of_q == nullptr) {
    if (p->Hq % p->Hkv != 0) return fail(STILL_ERR_INVALID_ARG, "Hq %% Hkv != 0 and no kv_head_of_q map given");
  } else {
    for (int h = 0; h < p->Hq; ++h)
      if (p->kv_head_of_q[h] < 0 || p->kv_head_of_q[h] >= p->Hkv)
        return fail(STILL_ERR_INVALID_ARG, "kv_head_of_q[%d] = %d outside [0, Hkv)", h, p->kv_head_of_q[h]);
  }
  if (p->d != 64 && p->d != 128) return fail(STILL_ERR_UNSUPPORTED, "d = %d (supported: 64, 128)", p->d);
  if (p->d_f != p->d) return fail(STILL_ERR_UNSUPPORTED, "d_f = %d (supported: d_f == d)", p->d_f);
  if (p->C != 64 && p->C != 128) return fail(STILL_ERR_UNSUPPORTED, "C = %d (supported: 64, 128)", p->C);
  if (p->W > 256 || p->W > 4 * p->C)   // nine band tiles at most; a decode state keeps the last 4 C tokens
    return fail(STILL_ERR_UNSUPPORTED, "W = %d (supported: 1..min(256, 4 C))", p->W);
  if (need_n && (int64_t)p->N > (int64_t)1 << 24) return fail(STILL_ERR_UNSUPPORTED, "N = %d too large", p->N);
  return STILL_OK;
}

// What the two side entry points (global score, selection overlap) need from the problem description: they do not
// touch the linear branch, so its restrictions (d_f, W, the fp32 LDS budget) do not apply to them.
still_status_t validate_score_params(const still_params_t* p, bool with_qk) {
  if (p == nullptr) return fail(STILL_ERR_INVALID_ARG, "params is NULL");
  if (p->B < 1 || p->Hq < 1 || p->N < 1) return fail(STILL_ERR_INVALID_ARG, "B, Hq, N must be >= 1");
  if ((int64_t)p->N > (int64_t)1 << 24) return fail(STILL_ERR_UNSUPPORTED, "N = %d too large", p->N);
  if (p->Hq > still::kMaxHq) return fail(STILL_ERR_UNSUPPORTED, "Hq %d > %d", p->Hq, still::kMaxHq);
  if (with_qk) {
    if (p->dtype != STILL_F32 && p->dtype != STILL_BF16) return fail(STILL_ERR_INVALID_ARG, "dtype %d unknown", p->dtype);
    if (p->Hkv < 1) return fail(STILL_ERR_INVALID_ARG, "Hkv must be >= 1");
    if (!(p->eps > 0.f)) return fail(STILL_ERR_INVALID_ARG, "eps must be > 0");
    if (!(p->scale > 0.f)) return fail(STILL_ERR_INVALID_ARG, "scale must be > 0");
    if (p->d != 64 && p->d != 128) return fail(STILL_ERR_UNSUPPORTED, "d = %d (supported: 64, 128)", p->d);
    if (p->kv_head_of_q == nullptr) {
      if (p->Hq % p->Hkv != 0) return fail(STILL_ERR_INVALID_ARG, "Hq %% Hkv != 0 and no kv_head_of_q map given");
    } else {
      for (int h = 0; h < p->Hq; ++h)
        if (p->kv_head_of_q[h] < 0 || p->kv_head_of_q[h] >= p->Hkv)
          return fail(STILL_ERR_INVALID_ARG, "kv_head_of_q[%d] = %d outside [0, Hkv)", h, p->kv_head_of_q[h]);
    }
  } else {
    if (p->C < 1 || p->C > 128) return fail(STILL_ERR_UNSUPPORTED, "C = %d (supported by the overlap count: 1..128)", p->C);
    if (p->lambda < 0 || p->lambda > p->C) return fail(STILL_ERR_INVALID_ARG, "lambda %d outside [0, C=%d]", p->lambda, p->C);
  }
  return STILL_OK;
}

still_status_t validate_strides(const still_params_t* p, bool with_g) {
  const int64_t unit = 16 / (int64_t)esize(p->dtype);
  const int64_t s[] = {p->q_sb, p->q_st, p->q_sh, p->k_sb, p->k_st, p->k_sh, p->v_sb, p->v_st, p->v_sh,
                       p->o_sb, p->o_st, p->o_sh};
  for (int64_t x : s)
    if (x < 0 || x % unit != 0) return fail(STILL_ERR_INVALID_ARG, "stride %lld is negative or not a multiple of 16 bytes", (long long)x);
  if (p->q_st < p->d || p->k_st < p->d || p->v_st < p->d || p->o_st < p->d)
    return fail(STILL_ERR_INVALID_ARG, "token stride smaller than d");
  if (with_g) {
    const int64_t gs[] = {p->g_sb, p->g_st, p->g_sh};
    for (int64_t x : gs)
      if (x < 0 || x % unit != 0) return fail(STILL_ERR_INVALID_ARG, "gate stride %lld invalid", (long long)x);
  }
  return STILL_OK;
}

void fill_map(const still_params_t* p, still::HeadMap* m) {
  for (int h = 0; h < still::kMaxHq; ++h) m->kv[h] = 0;
  for (int h = 0; h < p->Hq; ++h) m->kv[h] = p->kv_head_of_q ? p->kv_head_of_q[h] : h / (p->Hq / p->Hkv);
}

void layout_with_segments(const still_params_t* p, int64_t G, still_ws_layout_t* L) {
  const size_t es = esize(p->dtype);
  const int64_t B = p->B, N = p->N, Hq = p->Hq, Hkv = p->Hkv, d = p->d, df = p->d_f;
  const int64_t nc = (N + p->C - 1) / p->C, ncf = N / p->C;
  const int64_t npad = (N + 127) / 128 * 128;
  const bool evict = p->budget_policy == 1;   // then the retained rows of the workspace are ALL offers, under masks
  const int64_t cap = ((int64_t)still::retained_rows((int)ncf, p->lambda, evict ? still::kNoBudget : retained_budget(p)) + 63) / 64 * 64;
  const int64_t nseg = (nc + G - 1) / G;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + (bytes ? bytes : 16), 256);
    return o;
  };
  L->score = take((size_t)B * Hq * N * 4);
  L->sel = take((size_t)B * Hq * ncf * p->lambda * 4);
  L->vt = take((size_t)B * Hkv * d * npad * es);
  L->kret = take((size_t)B * Hq * cap * d * es);
  L->vrett = take((size_t)B * Hq * cap * d * es);
  L->wqt = take((size_t)Hq * df * d * es);
  L->wkf = take((size_t)Hq * df * d * es);
  L->seg = take((size_t)B * Hq * nseg * (2 * df * (d + 1)) * 4);
  L->snap = take((size_t)B * Hq * nc * d * (2 * df) * es);
  L->zsnap = take((size_t)B * Hq * nc * (2 * df) * 4);
  L->pimg = take((size_t)B * Hq * nseg * d * (2 * df) * es);
  L->zpre = take((size_t)B * Hq * nseg * (2 * df) * 4);
  L->kmask = take((size_t)B * Hq * ncf * (p->C / 32) * 4);
  L->n_la = take(p->emit_terms ? (size_t)B * Hq * N * d * 4 : 0);
  L->d_la = take(p->emit_terms ? (size_t)B * Hq * N * 4 : 0);
  L->vfr = take((size_t)B * Hkv * d * npad * es);
  const size_t M = evict ? (size_t)p->max_retained : 0;
  L->ev_src = take(evict ? (size_t)B * Hq * N * 4 : 0);
  L->ev_alive = take(evict ? (size_t)B * Hq * nc * (cap / 64) * 8 : 0);
  L->ev_fin = take(evict ? (size_t)B * Hq * (2 * M + 1) * 4 : 0);
  L->ev_vfr = take(evict ? (size_t)B * Hq * d * npad * es : 0);
  L->lse = take((size_t)B * Hq * N * 4);
  L->total = off;
  L->n_pad = (int32_t)npad;
  L->cap = (int32_t)cap;
  L->nseg = (int32_t)nseg;
  L->seg_chunks = (int32_t)G;
}

// Chunks per segment of the scan.  The scan walks in rounds of RT tokens, a segment is a whole number of rounds, and the
// device holds one of its workgroups per CU at a time.  A workgroup costs its rounds and about one more (its weights, its
// total); the cheapest number of passes over the CUs wins, the smaller number of segments among equals.  (Cutting for one
// workgroup per CU, whatever that leaves, put 5 sequences of 3001 tokens, 32 heads, into 320 workgroups, i.e. two
// passes of twelve chunks: call 505 us; three segments, two passes of eight: 446 us.  Counting two workgroups per CU at
// d = 64, where two fit, was 2 % slower at 4 x 4096 tokens.)
void compute_layout(const still_params_t* p, still_ws_layout_t* L) {
  constexpr int64_t kCus = 256;
  const int64_t nc = ((int64_t)p->N + p->C - 1) / p->C, units = (int64_t)p->B * p->Hq;
  const int64_t rt = still::la_round_tokens((int)esize(p->dtype), p->d), per_round = rt > p->C ? rt / p->C : 1;
  auto whole_rounds = [&](int64_t g) { return (g + per_round - 1) / per_round * per_round; };
  int64_t G = 0, best = 0;
  for (int64_t ns = 1; ns <= nc && (ns == 1 || units * ns <= 4 * kCus); ++ns) {
    int64_t g = (nc + ns - 1) / ns;
    g = whole_rounds(g < 2 ? 2 : g);
    const int64_t groups = units * ((nc + g - 1) / g);
    const int64_t cost = (groups + kCus - 1) / kCus * ((g * p->C + rt - 1) / rt + 1);
    if (G == 0 || cost < best) G = g, best = cost;
  }
  layout_with_segments(p, G, L);
  // More segments take more workspace: a problem that only fits the built-in scratch array with fewer keeps fewer (d = 64,
  // C = 128, bf16, 512 to 1024 tokens and 129 or more heads over the batch, for instance 5 x 768 tokens with 26 heads).  The
  // rule does not ask which entry point called: both give the same bits, so both cut alike.
  const int64_t g_few = whole_rounds(std::min(nc, std::max<int64_t>(2, (nc * units + kCus - 1) / kCus)));
  if (g_few > G && L->total > (size_t)STILL_STATIC_WORKSPACE_BYTES) {
    still_ws_layout_t F;
    layout_with_segments(p, g_few, &F);
    if (F.total <= (size_t)STILL_STATIC_WORKSPACE_BYTES) *L = F;
  }
}

still_status_t validate_state_params(const still_params_t* p) {
  still_status_t st = validate_params(p, false);
  if (st != STILL_OK) return st;
  if (p->max_tokens < 1) return fail(STILL_ERR_INVALID_ARG, "max_tokens must be >= 1 for a decode state");
  if ((int64_t)p->max_tokens > (int64_t)1 << 24) return fail(STILL_ERR_UNSUPPORTED, "max_tokens too large");
  return STILL_OK;
}

void compute_state_layout(const still_params_t* p, still_state_layout_t* L) {
  const size_t es = esize(p->dtype);
  const int64_t B = p->B, Hq = p->Hq, Hkv = p->Hkv, d = p->d, df = p->d_f;
  const int64_t nch = ((int64_t)p->max_tokens + p->C - 1) / p->C;
  const int64_t cap = ((int64_t)still::retained_rows((int)nch, p->lambda, retained_budget(p)) + 63) / 64 * 64 + 64;
  const int64_t R = 4 * (int64_t)p->C;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + (bytes ? bytes : 16), 256);
    return o;
  };
  const int64_t slices = p->shared_selection ? Hkv : Hq;   // group-shared selection: retained rows once per kv head
  L->S = take((size_t)B * Hq * (2 * df * (d + 1)) * 4);
  L->kret = take((size_t)B * slices * cap * d * es);
  L->vret = take((size_t)B * slices * cap * d * es);
  L->sel = take((size_t)B * Hq * nch * p->lambda * 4);
  L->kring = take((size_t)B * Hkv * R * d * es);
  L->vring = take((size_t)B * Hkv * R * d * es);
  L->score = take((size_t)B * Hq * R * 4);
  L->part = take((size_t)B * Hq * 32 * (d + 2) * 4);
  L->ret_score = take(p->budget_policy == 1 ? (size_t)B * Hq * cap * 4 : 0);
  L->ret_tok = take(p->budget_policy == 1 ? (size_t)B * Hq * cap * 4 : 0);
  L->total = off;
  L->cap = (int32_t)cap;
  L->R = (int32_t)R;
  L->n_chunks = (int32_t)nch;
}

}  // namespace

extern "C" {

// 0.3.0: budget_policy in the params, more regions in both layouts
// 0.4.0: backward pass, attention map, rotary pre-pass
// 0.5.0: state images in blocks, other regions in the backward workspace
// 0.5.1: values in tiles of 64 tokens, the blocks of the images in operand order, counters in the decode scratch
int32_t still_version(void) { return 501; }

const char* still_last_error(void) { return g_err; }

still_status_t still_fwd_workspace_layout(const still_params_t* p, still_ws_layout_t* layout) {
  if (layout == nullptr) return fail(STILL_ERR_INVALID_ARG, "layout is NULL");
  still_status_t st = validate_params(p, true);
  if (st != STILL_OK) return st;
  compute_layout(p, layout);
  return STILL_OK;
}

size_t still_fwd_workspace_bytes(const still_params_t* p) {
  still_ws_layout_t L;
  if (still_fwd_workspace_layout(p, &L) != STILL_OK) return 0;
  return L.total;
}

}  // extern "C"

namespace {

// Scratch of the allocation-free entry point: one fixed array in device memory per GPU, part of the library's code
// object (it exists from the moment the library is loaded on a device until the process ends).  In host code the
// array's name is only a handle for hipGetSymbolAddress; the address each device holds it at is looked up once per
// device and kept here.
constexpr size_t kStaticWorkspaceBytes = (size_t)STILL_STATIC_WORKSPACE_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticWorkspaceBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

still_status_t static_workspace(void** ptr) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(STILL_ERR_HIP, "hipGetDevice: %s", hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices) return fail(STILL_ERR_UNSUPPORTED, "device index %d outside [0, %d)", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* sym = nullptr;
    e = hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch));
    if (e != hipSuccess || sym == nullptr)
      return fail(STILL_ERR_HIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
    g_scratch_ptr[dev] = sym;
  }
  *ptr = g_scratch_ptr[dev];
  return STILL_OK;
}

// The prefill behind both entry points.  two_streams: run the layout kernels on the library's helper stream (created
// on first use) and record timing events if profiling is on; without it everything is enqueued on `stream` and no
// host or device object is created.
still_status_t fwd_impl(const still_params_t* p, const void* q, const void* k, const void* v,
                        const void* g, const void* Wq, const void* bq, const void* Wk,
                        const void* bk, void* out, float* score_out, int32_t* sel_idx,
                        int32_t sel_idx_is_input, void* state_out, void* workspace,
                        size_t workspace_bytes, void* stream_v, bool two_streams, bool static_ws) {
  still_status_t st = validate_params(p, true);
  if (st != STILL_OK) return st;
  st = validate_strides(p, g != nullptr);
  if (st != STILL_OK) return st;
  if (p->budget_policy != 0) {
    if (sel_idx_is_input || static_ws)
      return fail(STILL_ERR_UNSUPPORTED, "budget_policy 1 with injected indices or the built-in scratch array");
    const int64_t offers = (int64_t)(p->N / p->C) * p->lambda;
    if (offers > still::kMaxEvictOffers)
      return fail(STILL_ERR_UNSUPPORTED, "budget_policy 1: %lld offers per head > %d", (long long)offers,
                  still::kMaxEvictOffers);
  }
  if (!q || !k || !v || !Wq || !Wk || !out || (!workspace && !static_ws))
    return fail(STILL_ERR_INVALID_ARG, "a required pointer (q, k, v, Wq, Wk, out, workspace) is NULL");
  const void* ptrs[] = {q, k, v, g, Wq, bq, Wk, bk, out, score_out, sel_idx, workspace};
  for (const void* x : ptrs)
    if (x != nullptr && !aligned16(x)) return fail(STILL_ERR_INVALID_ARG, "pointer %p is not 16-byte aligned", x);
  if (p->seq_len != nullptr && (reinterpret_cast<uintptr_t>(p->seq_len) & 3) != 0)
    return fail(STILL_ERR_INVALID_ARG, "seq_len is not 4-byte aligned");
  if (sel_idx_is_input && sel_idx == nullptr && p->lambda > 0 && p->N >= p->C)
    return fail(STILL_ERR_INVALID_ARG, "sel_idx_is_input set but sel_idx is NULL");
  if (state_out != nullptr) {
    if (!aligned16(state_out)) return fail(STILL_ERR_INVALID_ARG, "state_out is not 16-byte aligned");
    if (p->max_tokens < p->N) return fail(STILL_ERR_INVALID_ARG, "state_out needs max_tokens >= N");
    if ((int64_t)p->max_tokens > (int64_t)1 << 24) return fail(STILL_ERR_UNSUPPORTED, "max_tokens too large");
    // the state carries the scores of the local span; with injected indices they are only computed on request
    if (sel_idx_is_input && score_out == nullptr)
      return fail(STILL_ERR_INVALID_ARG,
                  "state_out needs the scores: do not combine it with sel_idx_is_input unless score_out is given");
  }
  still_ws_layout_t L;
  compute_layout(p, &L);
  if (static_ws) {
    if (L.total > kStaticWorkspaceBytes)
      return fail(STILL_ERR_WORKSPACE_TOO_SMALL,
                  "this problem needs %zu bytes of workspace, the built-in scratch array holds %zu: use "
                  "still_hybrid_attn_fwd with a caller-owned workspace", L.total, kStaticWorkspaceBytes);
    st = static_workspace(&workspace);
    if (st != STILL_OK) return st;
  } else if (workspace_bytes < L.total) {
    return fail(STILL_ERR_WORKSPACE_TOO_SMALL, "workspace has %zu bytes, %zu needed", workspace_bytes, L.total);
  }
  // timing events are host objects created on demand: the allocation-free entry point records none
  struct ProfPause {
    bool was;
    explicit ProfPause(bool pause) : was(g_prof.on) { if (pause) g_prof.on = false; }
    ~ProfPause() { g_prof.on = was; }
  } prof_pause(!two_streams);

  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  const int B = p->B, N = p->N, d = p->d, C = p->C;
  const int nc = (N + C - 1) / C, ncf = N / C;
  still::HeadMap map;
  fill_map(p, &map);
  float* score = reinterpret_cast<float*>(ws + L.score);
  int32_t* sel = (sel_idx != nullptr) ? sel_idx : reinterpret_cast<int32_t*>(ws + L.sel);
  const bool have_sel = p->lambda > 0 && ncf > 0;
  hipError_t e;

  // layout preparation, on the side stream (the caller's stream if it could not be created)
  SideStream* side = two_streams ? side_stream(stream) : nullptr;
  hipStream_t s2 = stream;
  if (side != nullptr) {
    if (hipEventRecord(side->fork, stream) == hipSuccess && hipStreamWaitEvent(side->s, side->fork, 0) == hipSuccess)
      s2 = side->s;
    else
      side = nullptr;
  }
  // From here on the helper stream may hold work that depends on the caller's stream.  A launch failure must not
  // leave it dangling (under stream capture an unjoined fork invalidates the capture): every error return below
  // goes through hip_fail, which joins the helper stream back into `stream` first.
  bool joined = false;
  auto join_side = [&]() -> hipError_t {
    if (side == nullptr || joined) return hipSuccess;
    joined = true;
    hipError_t je = hipEventRecord(side->join, s2);
    if (je == hipSuccess) je = hipStreamWaitEvent(stream, side->join, 0);
    return je;
  };
  auto hip_fail = [&](const char* what, hipError_t err) -> still_status_t {
    (void)join_side();
    return fail(STILL_ERR_HIP, "%s: %s", what, hipGetErrorString(err));
  };
  prof_begin(0, s2);
  const bool evict = p->budget_policy == 1;
  const int budget = evict ? still::kNoBudget : retained_budget(p);   // under eviction every chunk offers its lam best
  still::TransposeVArgs tv{v, p->v_sb, p->v_st, p->v_sh, ws + L.vt, evict ? nullptr : ws + L.vfr, N, L.n_pad, p->Hkv, d,
                           C, p->seq_len};
  if ((e = still::launch_transpose_v(tv, p->dtype, B, s2)) != hipSuccess)
    return hip_fail("transpose_v", e);
  prof_end(0, s2);
  prof_begin(1, s2);
  still::TransposeWArgs twq{Wq, ws + L.wqt, p->Hq, d, p->d_f, 0};   // rows of W_q^T: tiles of the query feature map
  still::TransposeWArgs twk{Wk, ws + L.wkf, p->Hq, d, p->d_f, 1};   // W_k^T in operand order: the key projection
  if ((e = still::launch_transpose_w(twq, p->dtype, s2)) != hipSuccess ||
      (e = still::launch_transpose_w(twk, p->dtype, s2)) != hipSuccess)
    return hip_fail("transpose_w", e);
  prof_end(1, s2);

  prof_begin(2, stream);
  // Self-Saliency Score + Top-lambda
  still::ScoreArgs sa{};
  sa.q = q; sa.k = k;
  sa.q_sb = p->q_sb; sa.q_st = p->q_st; sa.q_sh = p->q_sh;
  sa.k_sb = p->k_sb; sa.k_st = p->k_st; sa.k_sh = p->k_sh;
  sa.map = map;
  sa.N = N; sa.C = C; sa.W = p->W; sa.lam = p->lambda; sa.Hq = p->Hq; sa.ncf = ncf; sa.rcap = budget;
  sa.scale = p->scale; sa.eps = p->eps;
  sa.score = score;
  const bool group_sel = p->shared_selection != 0;
  sa.sel = (have_sel && !sel_idx_is_input && !group_sel) ? sel : nullptr;
  sa.seq_len = p->seq_len;
  const bool mask_done = sa.sel != nullptr && !evict;
  if (mask_done) sa.kmask = reinterpret_cast<uint32_t*>(ws + L.kmask);
  const bool need_scores = !sel_idx_is_input || score_out != nullptr;
  if (need_scores) {
    if ((e = still::launch_score(sa, p->dtype, d, B, nc, stream)) != hipSuccess)
      return hip_fail("score_select", e);
    if (have_sel && !sel_idx_is_input && group_sel) {
      sa.sel = sel;
      if ((e = still::launch_group_select(sa, B, p->Hkv, stream)) != hipSuccess)
        return hip_fail("group_select", e);
    }
    if (score_out != nullptr) {
      e = hipMemcpyAsync(score_out, score, (size_t)B * p->Hq * N * sizeof(float), hipMemcpyDeviceToDevice, stream);
      if (e != hipSuccess) return hip_fail("score copy", e);
    }
  }
  prof_end(2, stream);

  prof_begin(3, stream);
  // retained K/V of every full chunk
  still::GatherArgs ga{};
  ga.k = k; ga.v = v;
  ga.k_sb = p->k_sb; ga.k_st = p->k_st; ga.k_sh = p->k_sh;
  ga.v_sb = p->v_sb; ga.v_st = p->v_st; ga.v_sh = p->v_sh;
  ga.map = map;
  ga.sel = sel;
  ga.nsel = have_sel ? still::retained_rows(ncf, p->lambda, budget) : 0;
  ga.sel_stride = ncf * p->lambda;
  ga.C = C; ga.lam = p->lambda; ga.rcap = budget; ga.seq_len = p->seq_len;
  ga.cap = L.cap; ga.Hq = p->Hq; ga.d = d; ga.N = N;
  ga.kret = ws + L.kret; ga.vrett = ws + L.vrett;
  if ((e = still::launch_gather(ga, p->dtype, B, stream)) != hipSuccess)
    return hip_fail("gather", e);
  prof_end(3, stream);
  // everything below reads the transposed copies
  if ((e = join_side()) != hipSuccess) return hip_fail("side stream", e);

  // NP-Map of the keys + scan of the linear-attention state: per-chunk sums inside every segment, prefix over segments
  still::LaArgs la{};
  la.k = k;
  la.k_sb = p->k_sb; la.k_st = p->k_st; la.k_sh = p->k_sh;
  la.vfr = ws + L.vfr; la.wkf = ws + L.wkf; la.bk = bk;
  la.kmask = reinterpret_cast<const uint32_t*>(ws + L.kmask);
  la.map = map;
  la.N = N; la.Np = L.n_pad; la.C = C; la.Hq = p->Hq; la.Hkv = p->Hkv;
  la.nc = nc; la.ncf = ncf; la.seq_len = p->seq_len;
  la.seg_chunks = L.seg_chunks; la.nseg = L.nseg;
  la.seg = reinterpret_cast<float*>(ws + L.seg);
  la.snap = ws + L.snap;
  la.zsnap = reinterpret_cast<float*>(ws + L.zsnap);
  la.pimg = ws + L.pimg;
  la.zpre = reinterpret_cast<float*>(ws + L.zpre);
  still_state_layout_t SL{};
  unsigned char* stp = static_cast<unsigned char*>(state_out);
  if (state_out != nullptr) compute_state_layout(p, &SL);
  la.s_final = state_out != nullptr ? reinterpret_cast<float*>(stp + SL.S) : nullptr;
  prof_begin(4, stream);
  const bool plan = evict && have_sel;
  int32_t* fin_tok = reinterpret_cast<int32_t*>(ws + L.ev_fin);
  float* fin_score = reinterpret_cast<float*>(ws + L.ev_fin) + (size_t)B * p->Hq * (plan ? p->max_retained : 0);
  int32_t* fin_n = fin_tok + (size_t)2 * B * p->Hq * (plan ? p->max_retained : 0);
  if (plan) {
    // which offers are retained for which rows, and which token every position carries into the state scan
    still::EvictPlanArgs ep{};
    ep.score = score; ep.sel = sel;
    ep.src = reinterpret_cast<int32_t*>(ws + L.ev_src); ep.alive = ws + L.ev_alive;
    ep.fin_tok = fin_tok; ep.fin_score = fin_score; ep.fin_n = fin_n;
    ep.seq_len = p->seq_len;
    ep.N = N; ep.C = C; ep.lam = p->lambda; ep.M = p->max_retained; ep.Hq = p->Hq; ep.ncf_all = ncf; ep.nc_all = nc;
    ep.AW = L.cap / 64;
    if ((e = still::launch_evict_plan(ep, B, stream)) != hipSuccess) return hip_fail("evict_plan", e);
    still::VfrGatherArgs vg{};
    vg.v = v; vg.v_sb = p->v_sb; vg.v_st = p->v_st; vg.v_sh = p->v_sh;
    vg.src = ep.src; vg.vfr = ws + L.ev_vfr; vg.map = map; vg.seq_len = p->seq_len;
    vg.N = N; vg.Np = L.n_pad; vg.Hq = p->Hq; vg.d = d; vg.C = C;
    if ((e = still::launch_vfr_gather(vg, p->dtype, B, stream)) != hipSuccess) return hip_fail("vfr_gather", e);
    la.src = ep.src;
    la.vfr = ws + L.ev_vfr;
  } else if (!mask_done) {   // lists that do not come from the score kernel (also budget_policy 1 without any offers)
    still::KeepMaskArgs km{sel, reinterpret_cast<uint32_t*>(ws + L.kmask), p->Hq, ncf, C, have_sel ? p->lambda : 0,
                           retained_budget(p)};
    if ((e = still::launch_keep_mask(km, B, stream)) != hipSuccess)
      return hip_fail("keep_mask", e);
  }
  prof_end(4, stream);
  prof_begin(5, stream);
  if ((e = still::launch_la_states(la, p->dtype, d, B, stream)) != hipSuccess)
    return hip_fail("la_states", e);
  prof_end(5, stream);
  prof_begin(6, stream);
  if ((e = still::launch_la_prefix(la, p->dtype, d, B, stream)) != hipSuccess)
    return hip_fail("la_prefix", e);
  prof_end(6, stream);

  prof_begin(7, stream);
  // sparse softmax branch, the rows' linear terms, merge
  still::SaArgs sx{};
  sx.q = q; sx.k = k;
  sx.q_sb = p->q_sb; sx.q_st = p->q_st; sx.q_sh = p->q_sh;
  sx.k_sb = p->k_sb; sx.k_st = p->k_st; sx.k_sh = p->k_sh;
  sx.vt = ws + L.vt; sx.kret = ws + L.kret; sx.vrett = ws + L.vrett;
  sx.wqt = ws + L.wqt; sx.bq = bq;
  sx.g = g; sx.g_sb = p->g_sb; sx.g_st = p->g_st; sx.g_sh = p->g_sh; sx.gate_act = p->gate_activation != 0;
  sx.snap = la.snap; sx.zsnap = la.zsnap; sx.nc = nc;
  sx.pimg = la.pimg; sx.zpre = la.zpre; sx.seg_chunks = L.seg_chunks; sx.nseg = L.nseg;
  sx.n_la_out = p->emit_terms ? reinterpret_cast<float*>(ws + L.n_la) : nullptr;
  sx.d_la_out = p->emit_terms ? reinterpret_cast<float*>(ws + L.d_la) : nullptr;
  sx.lse = reinterpret_cast<float*>(ws + L.lse);
  sx.out = out; sx.o_sb = p->o_sb; sx.o_st = p->o_st; sx.o_sh = p->o_sh;
  sx.map = map;
  sx.N = N; sx.Np = L.n_pad; sx.C = C; sx.lam = have_sel ? p->lambda : 0; sx.Hq = p->Hq; sx.Hkv = p->Hkv;
  sx.rcap = budget; sx.seq_len = p->seq_len;
  if (plan) {
    sx.alive = ws + L.ev_alive;
    sx.AW = L.cap / 64;
  }
  sx.cap = L.cap; sx.ntiles = (N + still::kSaRows - 1) / still::kSaRows; sx.B_ = B;
  sx.scale = p->scale;
  if ((e = still::launch_sa(sx, p->dtype, d, B, stream)) != hipSuccess)
    return hip_fail("sparse_attention", e);
  prof_end(7, stream);

  // decode state standing after token N-1: (S, z) through chunk c_last-2 came from the linear pass above
  if (state_out != nullptr) {
    still::StateFillArgs sf{};
    sf.k = k; sf.v = v;
    sf.k_sb = p->k_sb; sf.k_st = p->k_st; sf.k_sh = p->k_sh;
    sf.v_sb = p->v_sb; sf.v_st = p->v_st; sf.v_sh = p->v_sh;
    sf.score = score; sf.sel = sel; sf.map = map;
    sf.kret = stp + SL.kret; sf.vret = stp + SL.vret;
    sf.sel_state = reinterpret_cast<int32_t*>(stp + SL.sel);
    sf.kring = stp + SL.kring; sf.vring = stp + SL.vring;
    sf.score_ring = reinterpret_cast<float*>(stp + SL.score);
    sf.N = N; sf.R = SL.R; sf.Hq = p->Hq; sf.Hkv = p->Hkv; sf.d = d; sf.lam = have_sel ? p->lambda : 0;
    sf.cap = SL.cap; sf.ncf = ncf; sf.nchunks = SL.n_chunks; sf.rcap = budget;
    sf.shared = p->shared_selection != 0; sf.C = C; sf.seq_len = p->seq_len;
    sf.lists_only = plan;      // under eviction the lists are the offers and the rows come from the plan's last set
    const int n_routed = nc >= 2 ? nc - 2 : 0;
    if ((e = still::launch_state_fill(sf, p->dtype, B, n_routed, stream)) != hipSuccess)
      return hip_fail("state_fill", e);
    if (plan) {
      still::StateFillEvictArgs fe{};
      fe.k = k; fe.v = v;
      fe.k_sb = p->k_sb; fe.k_st = p->k_st; fe.k_sh = p->k_sh;
      fe.v_sb = p->v_sb; fe.v_st = p->v_st; fe.v_sh = p->v_sh;
      fe.fin_tok = fin_tok; fe.fin_score = fin_score; fe.fin_n = fin_n;
      fe.kret = stp + SL.kret; fe.vret = stp + SL.vret;
      fe.ret_score = reinterpret_cast<float*>(stp + SL.ret_score);
      fe.ret_tok = reinterpret_cast<int32_t*>(stp + SL.ret_tok);
      fe.map = map; fe.M = p->max_retained; fe.cap = SL.cap; fe.Hq = p->Hq; fe.d = d;
      if ((e = still::launch_state_fill_evict(fe, p->dtype, B, stream)) != hipSuccess)
        return hip_fail("state_fill_evict", e);
    }
  }
  g_err[0] = 0;
  return STILL_OK;
}

}  // namespace

extern "C" {

still_status_t still_hybrid_attn_fwd(const still_params_t* p, const void* q, const void* k, const void* v,
                                     const void* g, const void* Wq, const void* bq, const void* Wk,
                                     const void* bk, void* out, float* score_out, int32_t* sel_idx,
                                     int32_t sel_idx_is_input, void* state_out, void* workspace,
                                     size_t workspace_bytes, void* stream_v) {
  return fwd_impl(p, q, k, v, g, Wq, bq, Wk, bk, out, score_out, sel_idx, sel_idx_is_input, state_out, workspace,
                  workspace_bytes, stream_v, /*two_streams=*/true, /*static_ws=*/false);
}

still_status_t still_hybrid_attn_fwd_static(const still_params_t* p, const void* q, const void* k, const void* v,
                                            const void* g, const void* Wq, const void* bq, const void* Wk,
                                            const void* bk, void* out, float* score_out, int32_t* sel_idx,
                                            int32_t sel_idx_is_input, void* state_out, void* stream_v) {
  return fwd_impl(p, q, k, v, g, Wq, bq, Wk, bk, out, score_out, sel_idx, sel_idx_is_input, state_out, nullptr, 0,
                  stream_v, /*two_streams=*/false, /*static_ws=*/true);
}

void still_profile_enable(int32_t on) {
  g_prof.on = on != 0;
  g_prof.last_only = on == 2;
  g_prof.calls = 0;
}

still_status_t still_profile_read(float* ms, int32_t n) {
  if (ms == nullptr || n < 0) return fail(STILL_ERR_INVALID_ARG, "ms is NULL or n < 0");
  if (!g_prof.created || g_prof.calls == 0) return fail(STILL_ERR_STATE, "no profiled call recorded on this thread");
  const int last = (g_prof.calls - 1) % kProfRing;
  const int kept = g_prof.calls < kProfRing ? g_prof.calls : kProfRing;
  if (hipEventSynchronize(g_prof.end[last][STILL_PROFILE_SLOTS - 1]) != hipSuccess)
    return fail(STILL_ERR_HIP, "event synchronize failed");
  for (int i = 0; i < n && i < STILL_PROFILE_SLOTS; ++i) {
    double sum = 0.0;
    if (g_prof.last_only && i != STILL_PROFILE_SLOTS - 1) {
      ms[i] = 0.f;
      continue;
    }
    for (int c = 0; c < kept; ++c) {
      const int r = (g_prof.calls - 1 - c) % kProfRing;
      float t = 0.f;
      if (hipEventElapsedTime(&t, g_prof.beg[r][i], g_prof.end[r][i]) != hipSuccess)
        return fail(STILL_ERR_HIP, "event elapsed failed for slot %d", i);
      sum += t;
    }
    ms[i] = (float)(sum / kept);
  }
  return STILL_OK;
}

const char* still_profile_kernel_name(int32_t i) {
  return (i >= 0 && i < STILL_PROFILE_SLOTS) ? kSlotNames[i] : nullptr;
}

size_t still_state_bytes(const still_params_t* p) {
  still_state_layout_t L;
  if (still_state_layout(p, &L) != STILL_OK) return 0;
  return L.total;
}

still_status_t still_state_layout(const still_params_t* p, still_state_layout_t* layout) {
  if (layout == nullptr) return fail(STILL_ERR_INVALID_ARG, "layout is NULL");
  still_status_t st = validate_state_params(p);
  if (st != STILL_OK) return st;
  compute_state_layout(p, layout);
  return STILL_OK;
}

still_status_t still_state_init(const still_params_t* p, void* state, void* stream) {
  still_status_t st = validate_state_params(p);
  if (st != STILL_OK) return st;
  if (state == nullptr || !aligned16(state)) return fail(STILL_ERR_INVALID_ARG, "state is NULL or misaligned");
  still_state_layout_t L;
  compute_state_layout(p, &L);
  hipError_t e = still::launch_fill_zero(state, L.total, static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return fail(STILL_ERR_HIP, "state_init: %s", hipGetErrorString(e));
  g_err[0] = 0;
  return STILL_OK;
}

}  // extern "C"

namespace {

// One decode step.  t_dev == nullptr: every sequence is at token t.  Otherwise t_dev holds each sequence's own
// token index on the device and t is an upper bound of them, used only to size the launch.
still_status_t decode_step(const still_params_t* p, void* state, int32_t t, const int32_t* t_dev, const void* q_t,
                           const void* k_t, const void* v_t, const void* g_t, const void* Wq, const void* bq,
                           const void* Wk, const void* bk, void* out_t, void* stream_v) {
  still_status_t st = validate_state_params(p);
  if (st != STILL_OK) return st;
  if (!state || !q_t || !k_t || !v_t || !Wq || !Wk || !out_t)
    return fail(STILL_ERR_INVALID_ARG, "a required pointer (state, q_t, k_t, v_t, Wq, Wk, out_t) is NULL");
  const void* ptrs[] = {state, q_t, k_t, v_t, g_t, Wq, bq, Wk, bk, out_t};
  for (const void* x : ptrs)
    if (x != nullptr && !aligned16(x)) return fail(STILL_ERR_INVALID_ARG, "pointer %p is not 16-byte aligned", x);
  if (t < 0 || t >= p->max_tokens)
    return fail(STILL_ERR_STATE, "token index %d outside the state capacity [0, %d)", t, p->max_tokens);
  still_state_layout_t L;
  compute_state_layout(p, &L);
  unsigned char* sp = static_cast<unsigned char*>(state);
  still::DecArgs a{};
  a.S = reinterpret_cast<float*>(sp + L.S);
  a.kret = sp + L.kret; a.vret = sp + L.vret;
  a.sel = reinterpret_cast<int32_t*>(sp + L.sel);
  a.kring = sp + L.kring; a.vring = sp + L.vring;
  a.score = reinterpret_cast<float*>(sp + L.score);
  a.part = reinterpret_cast<float*>(sp + L.part);
  a.q = q_t; a.k = k_t; a.v = v_t; a.g = g_t; a.wq = Wq; a.wk = Wk; a.bq = bq; a.bk = bk; a.out = out_t;
  fill_map(p, &a.map);
  a.B = p->B; a.Hq = p->Hq; a.Hkv = p->Hkv; a.C = p->C; a.W = p->W; a.lam = p->lambda;
  a.cap = L.cap; a.R = L.R; a.nchunks = L.n_chunks; a.t = t; a.rcap = retained_budget(p);
  a.scale = p->scale; a.eps = p->eps;
  a.tpos = t_dev; a.max_tokens = p->max_tokens; a.shared = p->shared_selection != 0;
  a.gate_act = p->gate_activation != 0;
  a.evict = p->budget_policy == 1;
  a.ret_score = reinterpret_cast<float*>(sp + L.ret_score);
  a.ret_tok = reinterpret_cast<int32_t*>(sp + L.ret_tok);
  const int c = t / p->C;
  const int rows = still::retained_rows(c >= 1 ? c - 1 : 0, p->lambda, a.rcap) + (t - (c >= 1 ? c - 1 : 0) * p->C + 1);
  const int units = p->B * (p->shared_selection ? p->Hkv : p->Hq);   // workgroups per split
  int nsplit = (1024 + units - 1) / units;
  if (nsplit > still::kMaxSplits) nsplit = still::kMaxSplits;
  if (nsplit > (rows + 63) / 64) nsplit = (rows + 63) / 64;
  if (nsplit < 1) nsplit = 1;
  a.nsplit = nsplit;
  // The step merges a head as soon as its parts are there, while other workgroups still read the token's rows (the score, the
  // ring copy, other heads).  Where out_t lies over what they read, the merge is a launch behind them.  (Not g_t: only the
  // merge reads it, each element by the thread that writes the output's.)
  const size_t es = esize(p->dtype), rows_q = (size_t)p->B * p->Hq * p->d * es, rows_kv = (size_t)p->B * p->Hkv * p->d * es;
  const Span read[] = {flat_span(q_t, rows_q), flat_span(k_t, rows_kv), flat_span(v_t, rows_kv),
                       flat_span(Wq, (size_t)p->Hq * p->d * p->d_f * es), flat_span(bq, (size_t)p->Hq * p->d_f * es),
                       flat_span(t_dev, (size_t)p->B * sizeof(int32_t))};
  for (const Span& x : read) a.merge_apart = a.merge_apart || meet(flat_span(out_t, rows_q), x);
  a.merge_apart = a.merge_apart || a.shared;
  // with per-sequence positions any sequence at a chunk start >= 2C routes; the others leave the kernel at once
  const bool route = t_dev != nullptr ? c >= 2 : ((t % p->C == 0) && c >= 2);
  hipError_t e = still::launch_decode_step(a, p->dtype, p->d, route, static_cast<hipStream_t>(stream_v));
  if (e != hipSuccess) return fail(STILL_ERR_HIP, "decode_step: %s", hipGetErrorString(e));
  g_err[0] = 0;
  return STILL_OK;
}

}  // namespace

extern "C" {

still_status_t still_hybrid_attn_decode_step(const still_params_t* p, void* state, int32_t t, const void* q_t,
                                             const void* k_t, const void* v_t, const void* g_t, const void* Wq,
                                             const void* bq, const void* Wk, const void* bk, void* out_t,
                                             void* stream_v) {
  return decode_step(p, state, t, nullptr, q_t, k_t, v_t, g_t, Wq, bq, Wk, bk, out_t, stream_v);
}

still_status_t still_hybrid_attn_decode_step_at(const still_params_t* p, void* state, const int32_t* t_dev,
                                                int32_t t_max, const void* q_t, const void* k_t, const void* v_t,
                                                const void* g_t, const void* Wq, const void* bq, const void* Wk,
                                                const void* bk, void* out_t, void* stream_v) {
  if (t_dev == nullptr) return fail(STILL_ERR_INVALID_ARG, "t_dev is NULL");
  if ((reinterpret_cast<uintptr_t>(t_dev) & 3) != 0) return fail(STILL_ERR_INVALID_ARG, "t_dev is not 4-byte aligned");
  return decode_step(p, state, t_max, t_dev, q_t, k_t, v_t, g_t, Wq, bq, Wk, bk, out_t, stream_v);
}

still_status_t still_global_score(const still_params_t* p, const void* q, const void* k, float* score_out,
                                  void* stream_v) {
  still_status_t st = validate_score_params(p, true);
  if (st != STILL_OK) return st;
  {
    const int64_t unit = 16 / (int64_t)esize(p->dtype);
    const int64_t s[] = {p->q_sb, p->q_st, p->q_sh, p->k_sb, p->k_st, p->k_sh};
    for (int64_t x : s)
      if (x < 0 || x % unit != 0) return fail(STILL_ERR_INVALID_ARG, "stride %lld is negative or not a multiple of 16 bytes", (long long)x);
    if (p->q_st < p->d || p->k_st < p->d) return fail(STILL_ERR_INVALID_ARG, "token stride smaller than d");
  }
  if (!q || !k || !score_out) return fail(STILL_ERR_INVALID_ARG, "a required pointer (q, k, score_out) is NULL");
  if (!aligned16(q) || !aligned16(k) || !aligned16(score_out))
    return fail(STILL_ERR_INVALID_ARG, "q, k and score_out must be 16-byte aligned");
  still::GScoreArgs ga{};
  ga.q = q; ga.k = k;
  ga.q_sb = p->q_sb; ga.q_st = p->q_st; ga.q_sh = p->q_sh;
  ga.k_sb = p->k_sb; ga.k_st = p->k_st; ga.k_sh = p->k_sh;
  fill_map(p, &ga.map);
  ga.N = p->N; ga.Hq = p->Hq; ga.scale = p->scale; ga.eps = p->eps; ga.score = score_out;
  hipError_t e = still::launch_global_score(ga, p->dtype, p->d, p->B, static_cast<hipStream_t>(stream_v));
  if (e != hipSuccess) return fail(STILL_ERR_HIP, "global_score: %s", hipGetErrorString(e));
  g_err[0] = 0;
  return STILL_OK;
}

still_status_t still_selection_overlap(const still_params_t* p, const float* score_a, const float* score_b,
                                       int32_t* overlap, void* stream_v) {
  still_status_t st = validate_score_params(p, false);
  if (st != STILL_OK) return st;
  if (!score_a || !score_b || !overlap) return fail(STILL_ERR_INVALID_ARG, "a required pointer (score_a, score_b, overlap) is NULL");
  if ((reinterpret_cast<uintptr_t>(score_a) & 3) || (reinterpret_cast<uintptr_t>(score_b) & 3) ||
      (reinterpret_cast<uintptr_t>(overlap) & 3))
    return fail(STILL_ERR_INVALID_ARG, "score_a, score_b and overlap must be 4-byte aligned");
  hipError_t e = still::launch_topk_overlap(score_a, score_b, overlap, p->N, p->C, p->lambda, p->Hq, p->B,
                                            static_cast<hipStream_t>(stream_v));
  if (e != hipSuccess) return fail(STILL_ERR_HIP, "selection_overlap: %s", hipGetErrorString(e));
  g_err[0] = 0;
  return STILL_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------------------------------------
// Backward pass of the prefill (the routing held fixed)
// ---------------------------------------------------------------------------------------------------------
namespace {

still_status_t validate_bwd_params(const still_params_t* p) {
  still_status_t st = validate_params(p, true);
  if (st != STILL_OK) return st;
  if (p->budget_policy != 0) return fail(STILL_ERR_UNSUPPORTED, "the backward pass does not cover budget_policy 1");
  if (p->seq_len != nullptr) return fail(STILL_ERR_UNSUPPORTED, "the backward pass does not cover right-padded batches");
  if (p->dtype == STILL_F32 && p->d != 64)
    return fail(STILL_ERR_UNSUPPORTED, "the backward pass in fp32 is built for d = 64 only");
  return STILL_OK;
}

void compute_bwd_layout(const still_params_t* p, still_bwd_ws_layout_t* L) {
  still_ws_layout_t F;
  compute_layout(p, &F);
  const size_t es = esize(p->dtype);
  const size_t U = (size_t)p->B * p->Hq, N = p->N, d = p->d, df = p->d_f, DP = 2 * df;
  const size_t nc = (N + p->C - 1) / p->C, rows = U * N, kvrows = (size_t)p->B * p->Hkv * N;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + (bytes ? bytes : 16), 256);
    return o;
  };
  L->fwd = take(F.total);
  L->e_row = take(rows * 4);
  L->delta = take(rows * 4);
  L->ed = take(rows * 4);
  L->a = take(rows * d * es);
  L->phi_q = take(rows * DP * es);
  L->phi_k = take(rows * DP * es);
  const size_t wimg = (size_t)p->Hq * d * df * es;
  L->wqr = take(wimg);
  L->wkr = take(wimg);
  L->stq = L->stk = L->nraw = L->gq = L->dphi_k = off;   // (empty)
  L->ds = take(U * nc * DP * d * es);
  L->dz = take(U * nc * DP * 4);
  L->dfq = take(rows * df * es);
  L->dfk = take(rows * df * es);
  L->dq32 = take(rows * d * 4);
  L->dk32 = take(kvrows * d * 4);
  L->dv32 = take(kvrows * d * 4);
  L->cxq = L->cxk = off;                                 // (empty)
  // retained rows, 64 more than the forward workspace's: the last tile of 128 entries may reach past its capacity
  const size_t capt = F.cap ? (size_t)F.cap + 64 : 0;
  L->dkret = take(U * capt * d * 4);
  L->dvret = take(U * capt * d * 4);
  L->rvalid = take(U * (capt / 64) * 8 + U * capt * 4);
  L->kret = take(U * capt * d * es);
  L->vret = take(U * capt * d * es);
  L->n_pad_t = F.n_pad;
  L->cap_t = (int32_t)capt;
  L->total = off;
}

// The bytes from a tensor's first element to its last (strides are never negative).
Span strided_span(const still_params_t* p, const void* x, int64_t s_b, int64_t s_t, int64_t s_h, int H) {
  const int64_t elems = (p->B - 1) * s_b + (int64_t)(p->N - 1) * s_t + (H - 1) * s_h + p->d;
  const uintptr_t lo = reinterpret_cast<uintptr_t>(x);
  return {lo, x != nullptr ? lo + (uintptr_t)elems * esize(p->dtype) : lo};
}

still_status_t bwd_impl(const still_params_t* p, const void* q, const void* k, const void* v, const void* g,
                        const void* Wq, const void* bq, const void* Wk, const void* bk, const void* out,
                        const void* dout, const float* lse, const int32_t* sel_idx, void* dq, void* dk, void* dv,
                        void* dg, float* dWq, float* dbq, float* dWk, float* dbk, void* workspace,
                        size_t workspace_bytes, void* stream_v) {
  still_status_t st = validate_bwd_params(p);
  if (st != STILL_OK) return st;
  st = validate_strides(p, g != nullptr);
  if (st != STILL_OK) return st;
  if (!q || !k || !v || !Wq || !Wk || !out || !dout || !lse || !dq || !dk || !dv || !dWq || !dWk || !workspace)
    return fail(STILL_ERR_INVALID_ARG,
                "a required pointer (q, k, v, Wq, Wk, out, dout, lse, dq, dk, dv, dWq, dWk, workspace) is NULL");
  if ((g != nullptr) != (dg != nullptr)) return fail(STILL_ERR_INVALID_ARG, "dg must be given exactly when g is");
  if ((bq != nullptr) != (dbq != nullptr) || (bk != nullptr) != (dbk != nullptr))
    return fail(STILL_ERR_INVALID_ARG, "dbq / dbk must be given exactly when bq / bk are");
  const int B = p->B, N = p->N, d = p->d, C = p->C, Hq = p->Hq, Hkv = p->Hkv;
  const int nc = (N + C - 1) / C, ncf = N / C, U = B * Hq;
  const bool have_sel = p->lambda > 0 && ncf > 0;
  if (have_sel && sel_idx == nullptr)
    return fail(STILL_ERR_INVALID_ARG, "sel_idx (the forward pass's index lists) is NULL");
  const void* ptrs[] = {q, k, v, g, Wq, bq, Wk, bk, out, dout, lse, sel_idx, dq, dk, dv, dg, dWq, dbq, dWk, dbk, workspace};
  for (const void* x : ptrs)
    if (x != nullptr && !aligned16(x)) return fail(STILL_ERR_INVALID_ARG, "pointer %p is not 16-byte aligned", x);
  still_bwd_ws_layout_t BL;
  compute_bwd_layout(p, &BL);
  if (workspace_bytes < BL.total)
    return fail(STILL_ERR_WORKSPACE_TOO_SMALL, "workspace has %zu bytes, %zu needed", workspace_bytes, BL.total);
  still_ws_layout_t L;
  compute_layout(p, &L);

  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  unsigned char* bws = static_cast<unsigned char*>(workspace);
  unsigned char* ws = bws + BL.fwd;
  still::HeadMap map;
  fill_map(p, &map);
  const int dt = p->dtype;
  const int budget = retained_budget(p);
  hipError_t e;
  SideStream* side = nullptr;            // joined back into the caller's stream on every path
  auto join_side = [&]() -> hipError_t {
    if (side == nullptr) return hipSuccess;
    hipError_t je = hipEventRecord(side->join, side->s);
    if (je == hipSuccess) je = hipStreamWaitEvent(stream, side->join, 0);
    side = nullptr;
    return je;
  };
  auto hip_fail = [&](const char* what, hipError_t err) -> still_status_t {
    (void)join_side();
    return fail(STILL_ERR_HIP, "%s: %s", what, hipGetErrorString(err));
  };
  auto f32p = [&](size_t off) { return reinterpret_cast<float*>(bws + off); };

  // The linear branch's kernels write results while later ones still read inputs.  A caller whose gradients lie over an
  // input gets them in fp32 inside the workspace first and rounded into place after the last read.  (out, lse and the
  // weights have been read by then; dg over g is written element by element by the thread that read it.)
  const Span in_q = strided_span(p, q, p->q_sb, p->q_st, p->q_sh, Hq), in_k = strided_span(p, k, p->k_sb, p->k_st, p->k_sh, Hkv),
             in_v = strided_span(p, v, p->v_sb, p->v_st, p->v_sh, Hkv), in_g = strided_span(p, g, p->g_sb, p->g_st, p->g_sh, Hq),
             in_do = strided_span(p, dout, p->o_sb, p->o_st, p->o_sh, Hq);
  const size_t bias_bytes = (size_t)Hq * p->d_f * esize(p->dtype);
  const Span inputs[] = {in_q, in_k, in_v, in_g, in_do, flat_span(bq, bias_bytes), flat_span(bk, bias_bytes),
                         flat_span(sel_idx, (size_t)U * ncf * p->lambda * 4)};
  const Span results[] = {strided_span(p, dq, p->q_sb, p->q_st, p->q_sh, Hq), strided_span(p, dk, p->k_sb, p->k_st, p->k_sh, Hkv),
                          strided_span(p, dv, p->v_sb, p->v_st, p->v_sh, Hkv), strided_span(p, dg, p->g_sb, p->g_st, p->g_sh, Hq)};
  bool over = false;
  for (const Span& r : results)
    for (const Span& i : inputs) over = over || (meet(r, i) && !(g != nullptr && dg == g && r.lo == in_g.lo && i.lo == in_g.lo));

  // The softmax branch (row scalars, retained rows, dq, then dk and dv) and the forward pass's states need nothing of each
  // other, and the linear branch's query side and state gradient need only dq of it: two queues.  Small steps are chains
  // of launches that leave most of the chip idle (3 x 777 tokens, d = 64: 342 -> 280 us); at 16 x 1024 tokens both queues
  // fill the chip (2571 -> 2502 us).  The host pays for the events, which must hide behind the chain.  In bf16 at d = 64 that
  // takes more than 512 tokens, whatever the heads and the batch: 8 / 8 heads, C = 64, on one queue and on two, calls in a row
  // 92 / 104 us at 256 tokens, 102 / 107 at 384, 112 / 105 at 512, waited for one by one 110 / 120, 123 / 128, 133 / 132 (C = 128,
  // 512 tokens: 124 / 129; 640: 135 / 136, in a row 116 / 103).  The longer products of d = 128 (256 tokens 139 / 120,
  // waited for 154 / 150) and of fp32 (247 / 204, 266 / 239) hide them from four chunks on.  Below four chunks the linear branch
  // has the rows of one chunk at most (2 x 129 tokens, C = 128: 67 / 104).  Results that lie over lse, which dk and dv still
  // read when dq is written, take one queue after the other, as they did.
  bool over_lse = false;
  const Span in_lse = flat_span(lse, (size_t)U * N * 4);
  for (const Span& r : results) over_lse = over_lse || meet(r, in_lse);
  hipStream_t s2 = stream;
  if (nc >= 4 && (N > 512 || d == 128 || dt == STILL_F32)) side = side_stream(stream);
  if (side != nullptr) {
    if (hipEventRecord(side->fork, stream) == hipSuccess && hipStreamWaitEvent(side->s, side->fork, 0) == hipSuccess)
      s2 = side->s;
    else
      side = nullptr;
  }

  // ---- the weights in operand order, the parameter gradients (sums are added into them) cleared
  still::BwdWeightsArgs wa{Wq, Wk, ws + L.wqt, ws + L.wkf, bws + BL.wqr, bws + BL.wkr, dWq, dWk, dbq, dbk, d};
  if ((e = still::launch_bwd_weights(wa, dt, Hq, stream)) != hipSuccess) return hip_fail("bwd_weights", e);

  // ---- the forward pass's linear-attention states, rebuilt from the index lists (same kernels as the prefill)
  still::TransposeVArgs tv{v, p->v_sb, p->v_st, p->v_sh, nullptr, ws + L.vfr, N, L.n_pad, Hkv, d, C, nullptr};
  if ((e = still::launch_transpose_v(tv, dt, B, stream)) != hipSuccess) return hip_fail("transpose_v", e);
  still::KeepMaskArgs km{sel_idx, reinterpret_cast<uint32_t*>(ws + L.kmask), Hq, ncf, C, have_sel ? p->lambda : 0,
                         budget};
  if ((e = still::launch_keep_mask(km, B, stream)) != hipSuccess) return hip_fail("keep_mask", e);
  still::LaArgs la{};
  la.k = k;
  la.k_sb = p->k_sb; la.k_st = p->k_st; la.k_sh = p->k_sh;
  la.vfr = ws + L.vfr; la.wkf = ws + L.wkf; la.bk = bk;
  la.kmask = reinterpret_cast<const uint32_t*>(ws + L.kmask);
  la.map = map;
  la.N = N; la.Np = L.n_pad; la.C = C; la.Hq = Hq; la.Hkv = Hkv;
  la.nc = nc; la.ncf = ncf; la.seq_len = nullptr;
  la.seg_chunks = L.seg_chunks; la.nseg = L.nseg;
  la.seg = reinterpret_cast<float*>(ws + L.seg);
  la.snap = ws + L.snap;
  la.zsnap = reinterpret_cast<float*>(ws + L.zsnap);
  la.pimg = ws + L.pimg;
  la.zpre = reinterpret_cast<float*>(ws + L.zpre);
  la.s_final = nullptr;
  if ((e = still::launch_la_states(la, dt, d, B, stream)) != hipSuccess) return hip_fail("la_states", e);
  if ((e = still::launch_la_prefix(la, dt, d, B, stream)) != hipSuccess) return hip_fail("la_prefix", e);

  // ---- per-row scalars
  still::BwdRowArgs ra{};
  ra.out = out; ra.dout = dout; ra.o_sb = p->o_sb; ra.o_st = p->o_st; ra.o_sh = p->o_sh;
  ra.lse = lse; ra.e_row = f32p(BL.e_row); ra.delta = f32p(BL.delta); ra.ed = f32p(BL.ed);
  ra.U = U; ra.N = N; ra.Hq = Hq; ra.d = d;
  if ((e = still::launch_bwd_row_prep(ra, dt, s2)) != hipSuccess) return hip_fail("bwd_row_prep", e);

  // ---- softmax branch: dq (owned rows), dk / dv (the local span's, and the retained entries' in routing order)
  still::BwdGatherArgs ga{};
  ga.k = k; ga.v = v;
  ga.k_sb = p->k_sb; ga.k_st = p->k_st; ga.k_sh = p->k_sh;
  ga.v_sb = p->v_sb; ga.v_st = p->v_st; ga.v_sh = p->v_sh;
  ga.map = map; ga.sel = sel_idx;
  ga.nsel = have_sel ? still::retained_rows(ncf, p->lambda, budget) : 0;
  ga.sel_stride = ncf * p->lambda;
  ga.cap = BL.cap_t; ga.C = C; ga.lam = have_sel ? p->lambda : 0; ga.Hq = Hq; ga.d = d; ga.N = N;
  ga.kret = bws + BL.kret; ga.vret = bws + BL.vret;
  ga.rvalid = reinterpret_cast<unsigned long long*>(bws + BL.rvalid);
  ga.times = reinterpret_cast<int32_t*>(ga.rvalid + (size_t)U * (BL.cap_t / 64));
  if ((e = still::launch_bwd_gather(ga, dt, U, s2)) != hipSuccess) return hip_fail("bwd gather", e);
  still::BwdSaArgs sa{};
  sa.kret = ga.kret; sa.vret = ga.vret; sa.rvalid = ga.rvalid; sa.times = ga.times;
  sa.cap = BL.cap_t;
  sa.dkret = f32p(BL.dkret); sa.dvret = f32p(BL.dvret);
  sa.q = q; sa.k = k; sa.v = v; sa.dout = dout;
  sa.q_sb = p->q_sb; sa.q_st = p->q_st; sa.q_sh = p->q_sh;
  sa.k_sb = p->k_sb; sa.k_st = p->k_st; sa.k_sh = p->k_sh;
  sa.v_sb = p->v_sb; sa.v_st = p->v_st; sa.v_sh = p->v_sh;
  sa.o_sb = p->o_sb; sa.o_st = p->o_st; sa.o_sh = p->o_sh;
  sa.lse = lse; sa.delta = ra.delta;
  sa.dq32 = f32p(BL.dq32); sa.dk32 = f32p(BL.dk32); sa.dv32 = f32p(BL.dv32);
  sa.map = map;
  sa.N = N; sa.C = C; sa.lam = have_sel ? p->lambda : 0; sa.rcap = budget; sa.U = U; sa.Hq = Hq; sa.Hkv = Hkv;
  sa.n_row_tiles = (N + 127) / 128;
  sa.n_ret_tiles = (still::retained_rows(nc >= 2 ? nc - 2 : 0, sa.lam, budget) + 127) / 128;
  sa.scale = p->scale;
  if ((e = still::launch_bwd_sa_dq(sa, dt, d, s2)) != hipSuccess) return hip_fail("bwd_sparse_attention (dq)", e);
  if (side != nullptr && ((e = hipEventRecord(side->mid, s2)) != hipSuccess || (e = hipStreamWaitEvent(stream, side->mid, 0)) != hipSuccess))
    return hip_fail("side stream", e);
  if ((e = still::launch_bwd_sa_dkv(sa, dt, d, B, s2)) != hipSuccess) return hip_fail("bwd_sparse_attention (dk, dv)", e);
  if (over_lse && (e = join_side()) != hipSuccess) return hip_fail("side stream", e);

  // ---- linear branch: query side (dq, dg, and what the state gradient is made of), state gradient, key side, then the
  // parameter gradients
  still::BwdLinArgs lq{};
  lq.x = q; lq.x_sb = p->q_sb; lq.x_st = p->q_st; lq.x_sh = p->q_sh;
  lq.dout = dout; lq.o_sb = p->o_sb; lq.o_st = p->o_st; lq.o_sh = p->o_sh;
  lq.gate = g; lq.g_sb = p->g_sb; lq.g_st = p->g_st; lq.g_sh = p->g_sh; lq.gate_act = p->gate_activation != 0;
  lq.wf = wa.wqf; lq.wr = wa.wqr; lq.bias = bq;
  lq.snap = la.snap; lq.zsnap = la.zsnap; lq.pimg = la.pimg; lq.zpre = la.zpre;
  lq.e_row = ra.e_row; lq.ed = ra.ed;
  lq.a_rows = bws + BL.a; lq.phi = bws + BL.phi_q; lq.df = bws + BL.dfq;
  lq.dx32 = sa.dq32; lq.dx = dq; lq.dg = dg;
  lq.in_fp32 = over; lq.dg32 = f32p(BL.phi_k);
  lq.map = map; lq.n_units = U;
  lq.N = N; lq.C = C; lq.Hq = Hq; lq.Hkv = Hkv; lq.nc = nc; lq.ncf = ncf; lq.nseg = L.nseg; lq.seg_chunks = L.seg_chunks;
  if ((e = still::launch_bwd_lin(lq, dt, d, false, stream)) != hipSuccess) return hip_fail("bwd_lin (queries)", e);
  still::BwdRevscanArgs rs{lq.a_rows, lq.phi, ra.ed, bws + BL.ds, f32p(BL.dz), N, C, nc};
  if ((e = still::launch_bwd_revscan(rs, dt, d, U, stream)) != hipSuccess) return hip_fail("bwd_revscan", e);
  still::BwdLinArgs lk{};
  lk.x = k; lk.x_sb = p->k_sb; lk.x_st = p->k_st; lk.x_sh = p->k_sh;
  lk.v = v; lk.v_sb = p->v_sb; lk.v_st = p->v_st; lk.v_sh = p->v_sh;
  lk.wf = wa.wkf; lk.wr = wa.wkr; lk.bias = bk;
  lk.snap = rs.ds; lk.zsnap = rs.dz; lk.kmask = la.kmask;
  lk.df = bws + BL.dfk;
  lk.dx32 = sa.dk32; lk.dv32 = sa.dv32; lk.dx = dk; lk.dv = dv;
  lk.in_fp32 = over;
  lk.sel = sel_idx; lk.lam = sa.lam; lk.cap = BL.cap_t; lk.sel_stride = ga.sel_stride;
  lk.n_ret = still::retained_rows(nc >= 2 ? nc - 2 : 0, sa.lam, budget);
  if (lk.n_ret > 0) lk.dkret = sa.dkret, lk.dvret = sa.dvret;
  lk.map = map; lk.n_units = B * Hkv;
  lk.N = N; lk.C = C; lk.Hq = Hq; lk.Hkv = Hkv; lk.nc = nc; lk.ncf = ncf;
  if ((e = join_side()) != hipSuccess) return hip_fail("side stream", e);
  if ((e = still::launch_bwd_lin(lk, dt, d, true, stream)) != hipSuccess) return hip_fail("bwd_lin (keys)", e);
  still::BwdDwArgs dw{};
  dw.q = q; dw.q_sb = p->q_sb; dw.q_st = p->q_st; dw.q_sh = p->q_sh;
  dw.k = k; dw.k_sb = p->k_sb; dw.k_st = p->k_st; dw.k_sh = p->k_sh;
  dw.dfq = lq.df; dw.dfk = lk.df; dw.dwq = dWq; dw.dwk = dWk; dw.dbq = dbq; dw.dbk = dbk;
  dw.map = map; dw.B = B; dw.N = N; dw.Hq = Hq;
  if ((e = still::launch_bwd_dw(dw, dt, d, stream)) != hipSuccess) return hip_fail("bwd_dw", e);
  if (over) {
    const still::BwdRoundArgs ro[] = {{lq.dx32, dq, p->q_sb, p->q_st, p->q_sh, B, Hq, N, d},
                                      {lk.dx32, dk, p->k_sb, p->k_st, p->k_sh, B, Hkv, N, d},
                                      {lk.dv32, dv, p->v_sb, p->v_st, p->v_sh, B, Hkv, N, d},
                                      {lq.dg32, dg, p->g_sb, p->g_st, p->g_sh, B, Hq, N, d}};
    for (const still::BwdRoundArgs& r : ro)
      if (r.dst != nullptr && (e = still::launch_bwd_round(r, dt, stream)) != hipSuccess) return hip_fail("bwd_round", e);
  }
  g_err[0] = 0;
  return STILL_OK;
}

}  // namespace

extern "C" {

size_t still_bwd_workspace_bytes(const still_params_t* p) {
  if (validate_bwd_params(p) != STILL_OK) return 0;
  still_bwd_ws_layout_t L;
  compute_bwd_layout(p, &L);
  return L.total;
}

still_status_t still_bwd_workspace_layout(const still_params_t* p, still_bwd_ws_layout_t* layout) {
  if (layout == nullptr) return fail(STILL_ERR_INVALID_ARG, "layout is NULL");
  still_status_t st = validate_bwd_params(p);
  if (st != STILL_OK) return st;
  compute_bwd_layout(p, layout);
  return STILL_OK;
}

}  // extern "C"

namespace {

// What the attention map and its backward pass share: the keep mask and the weights in operand order (and, backward, the
// parameter gradients cleared), enqueued; the arguments of the map kernels.
still_status_t prepare_map(const still_params_t* p, const void* q, const void* k, const void* Wq, const void* bq,
                           const void* Wk, const void* bk, const float* lse, const int32_t* sel_idx, float* dWq,
                           float* dbq, float* dWk, float* dbk, unsigned char* bws, const still_bwd_ws_layout_t& BL,
                           hipStream_t stream, still::MapArgs* out) {
  const int N = p->N, C = p->C, Hq = p->Hq, ncf = N / C;
  still_ws_layout_t L;
  compute_layout(p, &L);
  unsigned char* ws = bws + BL.fwd;
  uint32_t* kmask = reinterpret_cast<uint32_t*>(ws + L.kmask);
  still::KeepMaskArgs km{sel_idx, kmask, Hq, ncf, C, p->lambda > 0 && ncf > 0 ? p->lambda : 0, retained_budget(p)};
  hipError_t e = still::launch_keep_mask(km, p->B, stream);
  if (e != hipSuccess) return fail(STILL_ERR_HIP, "keep_mask: %s", hipGetErrorString(e));
  still::BwdWeightsArgs wa{Wq, Wk, ws + L.wqt, ws + L.wkf, nullptr, nullptr, dWq, dWk, dbq, dbk, p->d};
  e = still::launch_bwd_weights(wa, p->dtype, Hq, stream);
  if (e != hipSuccess) return fail(STILL_ERR_HIP, "bwd_weights: %s", hipGetErrorString(e));
  still::MapArgs a{};
  a.q = q; a.k = k;
  a.q_sb = p->q_sb; a.q_st = p->q_st; a.q_sh = p->q_sh; a.k_sb = p->k_sb; a.k_st = p->k_st; a.k_sh = p->k_sh;
  a.wqf = wa.wqf; a.wkf = wa.wkf; a.bq = bq; a.bk = bk;
  a.phi_q = bws + BL.phi_q; a.phi_k = bws + BL.phi_k;
  a.kmask = kmask; a.lse = lse;
  fill_map(p, &a.map);
  a.U = p->B * Hq; a.N = N; a.C = C; a.Hq = Hq; a.nc = (N + C - 1) / C; a.ncf = ncf; a.scale = p->scale;
  *out = a;
  return STILL_OK;
}

size_t map_bwd_extra(const still_params_t* p, size_t* rowdot_off) {
  still_bwd_ws_layout_t BL;
  compute_bwd_layout(p, &BL);
  *rowdot_off = BL.total;
  return align_up(*rowdot_off + (size_t)p->B * p->Hq * p->N * 4, 256);
}

}  // namespace

extern "C" {

still_status_t still_attention_map(const still_params_t* p, const void* q, const void* k, const void* Wq,
                                   const void* bq, const void* Wk, const void* bk, const float* lse,
                                   const int32_t* sel_idx, float* map_out, void* workspace, size_t workspace_bytes,
                                   void* stream_v) {
  still_status_t st = validate_bwd_params(p);
  if (st != STILL_OK) return st;
  st = validate_strides(p, false);
  if (st != STILL_OK) return st;
  if (!q || !k || !Wq || !Wk || !lse || !map_out || !workspace)
    return fail(STILL_ERR_INVALID_ARG, "a required pointer (q, k, Wq, Wk, lse, map_out, workspace) is NULL");
  const int ncf = p->N / p->C;
  if (p->lambda > 0 && ncf > 0 && sel_idx == nullptr)
    return fail(STILL_ERR_INVALID_ARG, "sel_idx (the forward pass's index lists) is NULL");
  const void* ptrs[] = {q, k, Wq, bq, Wk, bk, lse, sel_idx, map_out, workspace};
  for (const void* x : ptrs)
    if (x != nullptr && !aligned16(x)) return fail(STILL_ERR_INVALID_ARG, "pointer %p is not 16-byte aligned", x);
  still_bwd_ws_layout_t BL;
  compute_bwd_layout(p, &BL);
  if (workspace_bytes < BL.total)
    return fail(STILL_ERR_WORKSPACE_TOO_SMALL, "workspace has %zu bytes, %zu needed", workspace_bytes, BL.total);
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  unsigned char* bws = static_cast<unsigned char*>(workspace);
  still::MapArgs a;
  st = prepare_map(p, q, k, Wq, bq, Wk, bk, lse, sel_idx, nullptr, nullptr, nullptr, nullptr, bws, BL, stream, &a);
  if (st != STILL_OK) return st;
  a.map_out = map_out;
  const hipError_t e = still::launch_map(a, p->dtype, p->d, false, stream);
  if (e != hipSuccess) return fail(STILL_ERR_HIP, "attention_map: %s", hipGetErrorString(e));
  g_err[0] = 0;
  return STILL_OK;
}

size_t still_attention_map_bwd_workspace_bytes(const still_params_t* p) {
  if (validate_bwd_params(p) != STILL_OK) return 0;
  size_t r;
  return map_bwd_extra(p, &r);
}

still_status_t still_attention_map_bwd(const still_params_t* p, const void* q, const void* k, const void* Wq,
                                       const void* bq, const void* Wk, const void* bk, const float* lse,
                                       const int32_t* sel_idx, const float* map, const float* dmap, float* dWq,
                                       float* dbq, float* dWk, float* dbk, void* workspace, size_t workspace_bytes,
                                       void* stream_v) {
  still_status_t st = validate_bwd_params(p);
  if (st != STILL_OK) return st;
  st = validate_strides(p, false);
  if (st != STILL_OK) return st;
  if (!q || !k || !Wq || !Wk || !lse || !map || !dmap || !dWq || !dWk || !workspace)
    return fail(STILL_ERR_INVALID_ARG,
                "a required pointer (q, k, Wq, Wk, lse, map, dmap, dWq, dWk, workspace) is NULL");
  if ((bq != nullptr) != (dbq != nullptr) || (bk != nullptr) != (dbk != nullptr))
    return fail(STILL_ERR_INVALID_ARG, "dbq / dbk must be given exactly when bq / bk are");
  const int ncf = p->N / p->C;
  if (p->lambda > 0 && ncf > 0 && sel_idx == nullptr)
    return fail(STILL_ERR_INVALID_ARG, "sel_idx (the forward pass's index lists) is NULL");
  const void* ptrs[] = {q, k, Wq, bq, Wk, bk, lse, sel_idx, map, dmap, dWq, dbq, dWk, dbk, workspace};
  for (const void* x : ptrs)
    if (x != nullptr && !aligned16(x)) return fail(STILL_ERR_INVALID_ARG, "pointer %p is not 16-byte aligned", x);
  size_t rowdot_off;
  const size_t need = map_bwd_extra(p, &rowdot_off);
  if (workspace_bytes < need)
    return fail(STILL_ERR_WORKSPACE_TOO_SMALL, "workspace has %zu bytes, %zu needed", workspace_bytes, need);
  still_bwd_ws_layout_t BL;
  compute_bwd_layout(p, &BL);
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  unsigned char* bws = static_cast<unsigned char*>(workspace);
  still::MapArgs a;
  st = prepare_map(p, q, k, Wq, bq, Wk, bk, lse, sel_idx, dWq, dbq, dWk, dbk, bws, BL, stream, &a);
  if (st != STILL_OK) return st;
  a.map_in = map; a.dmap = dmap;
  a.rowdot = reinterpret_cast<float*>(bws + rowdot_off);
  a.dfq = bws + BL.dfq; a.dfk = bws + BL.dfk;
  hipError_t e = still::launch_map(a, p->dtype, p->d, true, stream);
  if (e != hipSuccess) return fail(STILL_ERR_HIP, "attention_map_bwd: %s", hipGetErrorString(e));
  still::BwdDwArgs dw{};
  dw.q = q; dw.q_sb = p->q_sb; dw.q_st = p->q_st; dw.q_sh = p->q_sh;
  dw.k = k; dw.k_sb = p->k_sb; dw.k_st = p->k_st; dw.k_sh = p->k_sh;
  dw.dfq = a.dfq; dw.dfk = a.dfk; dw.dwq = dWq; dw.dwk = dWk; dw.dbq = dbq; dw.dbk = dbk;
  dw.map = a.map; dw.B = p->B; dw.N = p->N; dw.Hq = p->Hq;
  e = still::launch_bwd_dw(dw, p->dtype, p->d, stream);
  if (e != hipSuccess) return fail(STILL_ERR_HIP, "bwd_dw: %s", hipGetErrorString(e));
  g_err[0] = 0;
  return STILL_OK;
}

still_status_t still_rope_apply(const still_params_t* p, void* q, void* k, const int32_t* pos0, float base,
                                void* stream_v) {
  if (p == nullptr) return fail(STILL_ERR_INVALID_ARG, "params is NULL");
  if (p->dtype != STILL_F32 && p->dtype != STILL_BF16) return fail(STILL_ERR_INVALID_ARG, "dtype %d unknown", p->dtype);
  if (p->B < 1 || p->N < 1 || p->Hq < 1 || p->Hkv < 1) return fail(STILL_ERR_INVALID_ARG, "B, N, Hq, Hkv must be >= 1");
  if (p->d < 2 || p->d % 2 != 0) return fail(STILL_ERR_INVALID_ARG, "d = %d must be even", p->d);
  if (!(base > 1.f)) return fail(STILL_ERR_INVALID_ARG, "base must be > 1");
  if (q == nullptr && k == nullptr) return fail(STILL_ERR_INVALID_ARG, "both q and k are NULL");
  if (pos0 != nullptr && (reinterpret_cast<uintptr_t>(pos0) & 3) != 0)
    return fail(STILL_ERR_INVALID_ARG, "pos0 is not 4-byte aligned");
  const int64_t str[] = {p->q_sb, p->q_st, p->q_sh, p->k_sb, p->k_st, p->k_sh};
  for (int64_t x : str)
    if (x < 0) return fail(STILL_ERR_INVALID_ARG, "negative stride");
  if ((q != nullptr && p->q_st < p->d) || (k != nullptr && p->k_st < p->d))
    return fail(STILL_ERR_INVALID_ARG, "token stride smaller than d");
  still::RopeArgs a{q, k, p->q_sb, p->q_st, p->q_sh, p->k_sb, p->k_st, p->k_sh, pos0, log2((double)base),
                    p->B, p->N, p->Hq, p->Hkv, p->d};
  hipError_t e = still::launch_rope(a, p->dtype, static_cast<hipStream_t>(stream_v));
  if (e != hipSuccess) return fail(STILL_ERR_HIP, "rope_apply: %s", hipGetErrorString(e));
  g_err[0] = 0;
  return STILL_OK;
}

still_status_t still_hybrid_attn_bwd(const still_params_t* p, const void* q, const void* k, const void* v,
                                     const void* g, const void* Wq, const void* bq, const void* Wk, const void* bk,
                                     const void* out, const void* dout, const float* lse, const int32_t* sel_idx,
                                     void* dq, void* dk, void* dv, void* dg, float* dWq, float* dbq, float* dWk,
                                     float* dbk, void* workspace, size_t workspace_bytes, void* stream) {
  return bwd_impl(p, q, k, v, g, Wq, bq, Wk, bk, out, dout, lse, sel_idx, dq, dk, dv, dg, dWq, dbq, dWk, dbk,
                  workspace, workspace_bytes, stream);
}

}  // extern "C"
