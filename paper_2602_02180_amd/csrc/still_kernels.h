// Kernel argument blocks and host-side launchers shared by the translation units of libstill.
// Nothing here is part of the public ABI (include/still.h is).
#pragma once
#include "still_common.h"

namespace still {

struct ScoreArgs {
  const void* q;
  const void* k;
  int64_t q_sb, q_st, q_sh, k_sb, k_st, k_sh;
  HeadMap map;
  int N, C, W, lam, Hq, ncf;
  int pass_tiles; // (set by the launch) band tiles that pass through LDS at a time
  int rcap;       // budget on the retained tokens of one (batch, head): see chunk_quota()
  float scale, eps;
  float* score;   // [B, Hq, N]
  int32_t* sel;   // [B, Hq, ncf, lam] or nullptr (no selection)
  uint32_t* kmask;          // nullable, with sel: [B, Hq, ncf, C/32], bit = token selected
  const int32_t* seq_len;   // nullable, device [B]: chunks that are all padding are left empty
};

// Tokens that chunk c keeps when at most rcap tokens may be retained in total and chunks are served in order:
// lam until the budget is used up, then what is left of it, then none.  Retained row c * lam + pos therefore
// stays the row of slot pos of chunk c, and the rows in use are exactly those below min(chunks * lam, rcap).
__host__ __device__ inline int chunk_quota(int c, int lam, int rcap) {
  const int left = rcap - c * lam;
  return left >= lam ? lam : (left > 0 ? left : 0);
}
__host__ __device__ inline int retained_rows(int chunks, int lam, int rcap) {
  const int r = chunks * lam;
  return r < rcap ? r : rcap;
}
constexpr int kNoBudget = 1 << 30;
// Retained row of slot pos of chunk c, or -1 where it is none of the n_ret rows that a buffer is sure to hold.  (Under a budget
// c * lam alone leaves the buffer, whose size no longer grows with the chunks.)
__host__ __device__ inline int retained_row(int c, int lam, int pos, int n_ret) {
  const int row = c * lam + pos;
  return row < n_ret ? row : -1;
}
constexpr int kMaxEvictBudget = 4096;   // the plan and the routing step hold the retained set in LDS

// Tokens of sequence b: N for every sequence, or, for a right-padded batch, the caller's per-sequence count
// (device array, clamped to [1, N]).  Rows at and beyond it are padding: never read as keys or values by a real
// row, never written as outputs.
__device__ inline int seq_tokens(const int32_t* seq_len, int b, int N) {
  if (seq_len == nullptr) return N;
  const int n = seq_len[b];
  return n < 1 ? 1 : (n > N ? N : n);
}

struct GScoreArgs {
  const void* q;
  const void* k;
  int64_t q_sb, q_st, q_sh, k_sb, k_st, k_sh;
  HeadMap map;
  int N, Hq;
  float scale, eps;
  float* score;   // [B, Hq, N]
};

// Element offset of (token or retained row i, column x) in one head's transposed values: tiles of 64 tokens, [i / 64][x][i % 64],
// so that a tile of the sparse-attention kernel is one run of memory (like its tile of keys) and the lane offsets of its
// copies are the same for every tile.
__host__ __device__ inline int64_t value_tile_offset(int i, int x, int d) {
  return ((int64_t)(i >> 6) * d + x) * 64 + (i & 63);
}

struct TransposeVArgs {
  const void* v;
  int64_t v_sb, v_st, v_sh;
  void* vt;       // nullable [B, Hkv, Np/64, d, 64], see value_tile_offset()
  void* vfr;      // nullable: the same values in MFMA-fragment order, see vfr_offset()
  int N, Np, Hkv, d, C;
  const int32_t* seq_len;   // nullable, device [B]: see seq_tokens()
};

// Element offset of (token tau, column x) of one (batch, kv head) in the fragment-ordered copy of v that the
// linear-attention consumers load their "S += phi_k^T V" operand from: [chunk][x / 32][k-step][x % 32][lane
// group][k per lane], so that the 64 lanes of one operand load read one contiguous piece (1 KB for 2-byte types).
// KK / KPL = k per instruction / per lane of the element type's MFMA (16 / 8 for 2-byte types, 2 / 1 for fp32).
__host__ __device__ inline int64_t vfr_offset(int tau, int x, int C, int D, int KK, int KPL) {
  const int ch = tau / C, tc = tau % C;
  const int s = tc / KK, g = (tc % KK) / KPL, e = tc % KPL;
  return ((((int64_t)ch * (D / 32) + x / 32) * (C / KK) + s) * 64 + 2 * (x % 32) + g) * KPL + e;
}

struct TransposeWArgs {
  const void* w;  // [Hq, d, df]
  void* wt;       // [Hq, df, d], or (frag) the same rows in MFMA operand order, see wfrag_offset()
  int Hq, d, df;
  int frag;
};

// Element offset, inside one head's copy, of W^T[f][x] in the operand order of the key projection f^T = W^T x^T:
// [feature tile f / 32][k-step x / KK][lane = 32 g + m][k per lane], with feature 32 ft + kappa(m) in MFMA row m,
// so that the 64 lanes of one operand load read one contiguous piece.
template <typename M>
__host__ __device__ inline int wfrag_offset(int ft, int s, int lane, int d) {
  return ((ft * (d / M::KK) + s) * 64 + lane) * M::KPL;
}

// Tokens per round of the linear-attention state scan: the round's feature image [2 d_f][round] is double
// buffered in LDS, so wide features in a wide type take shorter rounds.
__host__ __device__ constexpr int la_round_tokens(int es, int d) { return es * 2 * d <= 512 ? 128 : 64; }

struct GatherArgs {
  const void* k;
  const void* v;
  int64_t k_sb, k_st, k_sh, v_sb, v_st, v_sh;
  HeadMap map;
  const int32_t* sel;  // [B, Hq, sel_stride]; the first nsel entries of each list are gathered
  int nsel, sel_stride, cap, Hq, d, N;
  int C, lam, rcap;
  const int32_t* seq_len;   // nullable, device [B]: rows of chunks beyond a sequence's full chunks are zero
  void* kret;          // [B, Hq, cap, d]
  void* vrett;         // [B, Hq, cap/64, d, 64], see value_tile_offset()
};

// Top-lambda lists -> one bit per token of every full chunk (set = kept by the softmax branch, so the token does
// NOT enter the linear state).  Entries outside their chunk are ignored (caller-supplied lists are never trusted for
// addressing); slots beyond a chunk's quota are not read.
struct KeepMaskArgs {
  const int32_t* sel;   // [B, Hq, ncf, lam], nullable when lam == 0
  uint32_t* kmask;      // [B, Hq, ncf, C/32]
  int Hq, ncf, C, lam, rcap;
};

// Element offset of (x, feature) in a state image S^T [d][2 d_f]: blocks of 32 rows x by 16 features, [x / 32][f / 16], and
// inside a block the order of an MFMA operand over features: [f / 8][x % 32, bit 2 flipped in the second half][f % 8].  An
// accumulator tile's store covers 1 KB of one block, and a consumer's copy into LDS takes a block as it stands, 64 lanes
// on 1 KB: blocks of [x % 32][f % 16] that the copy had to spread over rows cost its wave about 300 cycles per KB, a copy of
// a run about 100.  In LDS a block is then read both ways without bank conflicts (the flip is for the transposing reads).
__host__ __device__ inline int state_image_offset(int x, int f, int DP) {
  const int h = (f >> 3) & 1;
  return ((x >> 5) * (DP >> 4) + (f >> 4)) * 512 + h * 256 + ((x & 31) ^ (h << 2)) * 8 + (f & 7);
}
// A lane's 16 entries of a product "32 features from f0 (rows) x rows x (columns)" into the image of row x: one address per half of
// a block and constant offsets from it.  (With an offset per entry the fp32 instances held 16 addresses per product in
// registers: la_kernel at d = 128, C = 64 spilled 2458 values instead of 448, and a call of 2 x 2048 tokens, 32 / 8 heads, took
// 3.09 ms instead of 2.65.)
template <typename M, typename T>
__device__ __forceinline__ void store_image_tile(T* img, int x, int f0, int DP, int g, const floatx16& acc) {
  if constexpr (M::KPL == 1) {             // entry s is feature f0 + 2 s + g
    T* half[2] = {img + state_image_offset(x, f0, DP) + g, img + state_image_offset(x, f0 + 8, DP) + g};
#pragma unroll
    for (int s = 0; s < 16; ++s) half[(s >> 2) & 1][512 * (s >> 3) + ((2 * s) & 7)] = acc[s];
  } else {                                 // entries 8 s .. 8 s + 7 are features f0 + 16 s + 8 g ..
    T* p = img + state_image_offset(x, f0 + 8 * g, DP);
#pragma unroll
    for (int s = 0; s < 2; ++s) *reinterpret_cast<typename M::frag*>(p + 512 * s) = M::from_acc(acc, s);
  }
}
// The piece of an image that a slab of 64 features holds in LDS: [x / 32][f / 16 of 4], blocks as in the image.  Element i of
// the slab that starts at feature f0 lies here in the image.
__host__ __device__ inline int state_slab_source(int i, int f0, int DP) {
  return (i >> 11) * (DP >> 4) * 512 + (f0 >> 4) * 512 + (i & 2047);
}

struct LaArgs {
  const void* k;
  int64_t k_sb, k_st, k_sh;
  const void* vfr;     // [B, Hkv, Np * d]: v in fragment order (vfr_offset)
  const void* wkf;     // [Hq, df * d]: Wk^T in operand order (wfrag_offset)
  const void* bk;      // nullable [Hq, df]
  const uint32_t* kmask;  // [B, Hq, ncf, C/32]: bit = token kept by the softmax branch (see KeepMaskArgs)
  HeadMap map;
  int N, Np, C, Hq, Hkv, nc, ncf;
  const int32_t* seq_len;   // nullable, device [B]
  int seg_chunks, nseg;
  float* seg;          // [B, Hq, nseg][D*DP + DP]: every segment's total, S^T as [x][feature], then z
  void* snap;          // [B, Hq, nc][D][DP] storage type (state_image_offset): S^T summed over chunk c's own segment, through chunk c-2
  float* zsnap;        // [B, Hq, nc][DP]: z likewise
  void* pimg;          // [B, Hq, nseg][D][DP] storage type (state_image_offset): S^T through the chunk before the segment (prefix)
  float* zpre;         // [B, Hq, nseg][DP]: z likewise
  float* s_final;      // nullable [B, Hq, DP*(D+1)] as S [feature][x] then z: fp32 state through chunk (last - 2)
  const int32_t* src;  // evict policy only [B, Hq, N]: token carried by every position (-1: none); replaces kmask, and
                       //   vfr is then per QUERY head ([B, Hq, Np * d], built through the same table)
};

// Budget policy "evict the lowest score" in the prefill (still_evict.hip)
struct EvictPlanArgs {
  const float* score;      // [B, Hq, N]
  const int32_t* sel;      // [B, Hq, ncf_all, lam]: every chunk's offers (its lam highest scores)
  int32_t* src;            // [B, Hq, N]: token whose key/value a position carries into the state scan (-1: none)
  void* alive;             // [B, Hq, nc_all, AW] 64-bit words: bit j = offer j (routing order) is retained for the rows
                           //   of that chunk
  int32_t* fin_tok;        // nullable [B, Hq, M]: the set retained after the last routed step (decode hand-over)
  float* fin_score;        // [B, Hq, M]
  int32_t* fin_n;          // [B, Hq]
  const int32_t* seq_len;  // nullable, device [B]
  int N, C, lam, M, Hq, ncf_all, nc_all, AW;
};
struct VfrGatherArgs {
  const void* v;
  int64_t v_sb, v_st, v_sh;
  const int32_t* src;      // [B, Hq, N]
  void* vfr;               // [B, Hq, Np * d]
  HeadMap map;
  const int32_t* seq_len;
  int N, Np, Hq, d, C;
};
struct StateFillEvictArgs {
  const void* k;
  const void* v;
  int64_t k_sb, k_st, k_sh, v_sb, v_st, v_sh;
  const int32_t* fin_tok;
  const float* fin_score;
  const int32_t* fin_n;
  void* kret;
  void* vret;
  float* ret_score;
  int32_t* ret_tok;
  HeadMap map;
  int M, cap, Hq, d;
};
constexpr int kMaxEvictOffers = 32768;   // offers per (sequence, head) the sparse kernel's LDS mask rows hold (x 2 chunks)

// query rows per workgroup of the sparse-attention kernel (one wave per 32 rows)
constexpr int kSaRows = 128;

struct SaArgs {
  const void* q;
  const void* k;
  int64_t q_sb, q_st, q_sh, k_sb, k_st, k_sh;
  const void* vt;      // [B, Hkv, Np/64, d, 64]
  const void* kret;    // [B, Hq, cap, d]
  const void* vrett;   // [B, Hq, cap/64, d, 64]
  const void* wqt;     // [Hq, df, d]: Wq^T
  const void* bq;      // nullable [Hq, df]
  const void* g;       // nullable gate [B, N, Hq, d]
  int64_t g_sb, g_st, g_sh;
  int gate_act;        // 1: g is a pre-activation, the gate is its logistic function
  const void* snap;    // [B, Hq, nc][D][DP] in blocks (state_image_offset): see LaArgs
  const float* zsnap;  // [B, Hq, nc][DP]
  const void* pimg;    // [B, Hq, nseg][D][DP] in blocks
  const float* zpre;   // [B, Hq, nseg][DP]
  int seg_chunks, nseg;
  float* n_la_out;     // nullable [B, Hq, N, d]: the gated linear numerator of every row (inspection)
  float* d_la_out;     // nullable [B, Hq, N]
  float* lse;          // nullable [B, Hq, N]: ln(D_SA + D_LA) of every row
  void* out;
  int64_t o_sb, o_st, o_sh;
  HeadMap map;
  int N, Np, C, lam, Hq, Hkv, cap, ntiles, B_, rcap, nc;
  const int32_t* seq_len;   // nullable, device [B]
  float scale;
  const void* alive;   // evict policy only [B, Hq, nc, AW] 64-bit words: see EvictPlanArgs (the retained tiles are then
  int AW;              //   all offers, each under its chunk's mask; AW = words per row = cap / 64)
};

// Slots of a decode step's scratch, 32 per unit, d + 2 words each: the splits of the salient cache, the counters of the
// workgroups that have delivered their part (eight bytes each, for even and odd token indices), the linear terms.
constexpr int kMaxSplits = 30, kArrivalSlot = 30, kLinearSlot = 31;
struct DecArgs {
  float* S;            // [B, Hq, DP*(D+1)]
  void* kret;          // [B, Hq, cap, d]
  void* vret;
  int32_t* sel;        // [B, Hq, nchunks, lam]
  void* kring;         // [B, Hkv, R, d]
  void* vring;
  float* score;        // [B, Hq, R]
  float* part;         // [B, Hq, 32, d+2]: (m, l, acc) of every split, kArrivalSlot, kLinearSlot: (-, D_LA, N_LA)
  const void* q;       // [B, Hq, d]
  const void* k;       // [B, Hkv, d]
  const void* v;
  const void* g;       // nullable
  const void* wq;      // [Hq, d, df]
  const void* wk;
  const void* bq;      // nullable
  const void* bk;
  void* out;           // [B, Hq, d]
  HeadMap map;
  int B, Hq, Hkv, C, W, lam, cap, R, nchunks, t, nsplit, rcap;
  int shared;              // 1: the query heads of one kv head rank by their summed score (one list per group)
  int merge_apart;         // 1: the parts are merged by a launch of their own (always with shared)
  int gate_act;            // 1: g is a pre-activation, the gate is its logistic function
  int evict;               // 1: the budget is held by evicting the lowest score (ret_score, ret_tok are then kept)
  float* ret_score;        // [B, Hq, cap] score of every retained row
  int32_t* ret_tok;        // [B, Hq, cap] its token index
  const int32_t* tpos;     // nullable, device [B]: index of each sequence's new token (t is then ignored)
  int max_tokens;
  float scale, eps;
};

// Index of the new token of sequence b: the same for every sequence, or the caller's per-sequence entry.  An
// entry outside [0, max_tokens) marks a sequence that sits this step out (-1 is returned).
__device__ inline int step_index(const DecArgs& a, int b) {
  if (a.tpos == nullptr) return a.t;
  const int t = a.tpos[b];
  return (t >= 0 && t < a.max_tokens) ? t : -1;
}

// Retained rows of a decode state: one slice per (sequence, query head), or, with group-shared selection, one per
// (sequence, kv head), written by the lowest query head of the group only.
__device__ inline int64_t retained_slice(bool shared, int b, int hq, int kvh, int Hq, int Hkv) {
  return shared ? (int64_t)b * Hkv + kvh : (int64_t)b * Hq + hq;
}
__device__ inline bool writes_retained(bool shared, const HeadMap& map, int hq) {
  if (!shared) return true;
  for (int h = 0; h < hq; ++h)
    if (map.kv[h] == map.kv[hq]) return false;
  return true;
}

struct StateFillArgs {
  const void* k;
  const void* v;
  int64_t k_sb, k_st, k_sh, v_sb, v_st, v_sh;
  const float* score;      // [B, Hq, N]
  const int32_t* sel;      // [B, Hq, ncf, lam]
  HeadMap map;
  void* kret;
  void* vret;
  int32_t* sel_state;
  void* kring;
  void* vring;
  float* score_ring;
  int N, R, Hq, Hkv, d, lam, cap, ncf, nchunks, rcap, shared, C;
  int lists_only;           // 1: write the index lists of the routed chunks but no retained rows (evict policy)
  const int32_t* seq_len;   // nullable, device [B]
};

hipError_t launch_decode_step(const DecArgs& a, int dtype, int d, bool route, hipStream_t stream);
hipError_t launch_state_fill(const StateFillArgs& a, int dtype, int B, int n_routed, hipStream_t stream);
hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t stream);
hipError_t launch_score(const ScoreArgs& a, int dtype, int d, int B, int nc, hipStream_t stream);
hipError_t launch_global_score(const GScoreArgs& a, int dtype, int d, int B, hipStream_t stream);
hipError_t launch_topk_overlap(const float* sa, const float* sb, int32_t* overlap, int N, int C, int lam, int Hq,
                               int B, hipStream_t stream);
hipError_t launch_group_select(const ScoreArgs& a, int B, int Hkv, hipStream_t stream);
hipError_t launch_transpose_v(const TransposeVArgs& a, int dtype, int B, hipStream_t stream);
hipError_t launch_transpose_w(const TransposeWArgs& a, int dtype, hipStream_t stream);
hipError_t launch_gather(const GatherArgs& a, int dtype, int B, hipStream_t stream);
hipError_t launch_keep_mask(const KeepMaskArgs& a, int B, hipStream_t stream);
hipError_t launch_la_states(const LaArgs& a, int dtype, int d, int B, hipStream_t stream);
hipError_t launch_la_prefix(const LaArgs& a, int dtype, int d, int B, hipStream_t stream);
hipError_t launch_sa(const SaArgs& a, int dtype, int d, int B, hipStream_t stream);
hipError_t launch_evict_plan(const EvictPlanArgs& a, int B, hipStream_t stream);
hipError_t launch_vfr_gather(const VfrGatherArgs& a, int dtype, int B, hipStream_t stream);
hipError_t launch_state_fill_evict(const StateFillEvictArgs& a, int dtype, int B, hipStream_t stream);
size_t evict_plan_smem(int M, int lam, int AW);

// ---- backward pass (still_bwd.hip) ----
struct BwdRowArgs {
  const void* out;         // y of the forward pass, strided like dout
  const void* dout;
  int64_t o_sb, o_st, o_sh;
  const float* lse;        // [U, N]
  float* e_row;            // [U, N]: E_t = exp(-L_t)
  float* delta;            // [U, N]: dy_t . y_t
  float* ed;               // [U, N]: E_t delta_t
  int U, N, Hq, d;
};
// fp32 rows -> a strided tensor in the storage type
struct BwdRoundArgs {
  const float* src;        // [B, H, N, d]
  void* dst;
  int64_t s_b, s_t, s_h;
  int B, H, N, d;
};
// both weight matrices in the two operand orders of the linear branch, and cleared parameter gradients (each where a
// destination is given)
struct BwdWeightsArgs {
  const void* wq;          // [Hq, d, d]
  const void* wk;
  void* wqf;               // [Hq, d, d]: operand order of f^T = W^T x^T (wfrag_offset)
  void* wkf;
  void* wqr;               // nullable [Hq, d, d]: operand order of dx = df W^T
  void* wkr;
  float* dwq;              // nullable
  float* dwk;
  float* dbq;              // nullable
  float* dbk;
  int d;
};
// linear branch of one side (still_bwd_lin.hip); "q:" / "k:" = query / key side
struct BwdLinArgs {
  const void* x;           // q: q; k: k
  int64_t x_sb, x_st, x_sh;
  const void* v;           // k: v
  int64_t v_sb, v_st, v_sh;
  const void* dout;        // q
  int64_t o_sb, o_st, o_sh;
  const void* gate;        // q: nullable
  int64_t g_sb, g_st, g_sh;
  int gate_act;
  const void* wf;          // this side's weights in operand order (BwdWeightsArgs)
  const void* wr;
  const void* bias;        // nullable [Hq, d]
  const void* snap;        // q: LaArgs::snap; k: the state gradient, same layout
  const float* zsnap;
  const void* pimg;        // q: LaArgs::pimg, zpre
  const float* zpre;
  const float* e_row;      // q: [U, N]
  const float* ed;         // q: [U, N]
  const uint32_t* kmask;   // k: [B, Hq, ncf, C/32]
  void* a_rows;            // q: [U, N, d] written: A_t (tokens of chunks >= 2)
  void* phi;               // q: [U, N, 2d] written (tokens of chunks >= 2)
  void* df;                // [U, N, d] written
  float* dx32;             // the softmax branch's part: q: [U, N, d]; k: [B, Hkv, N, d]
  float* dv32;             // k
  void* dx;                // strided like x
  void* dv;                // k: strided like v
  void* dg;                // q: nullable, strided like gate
  bool in_fp32;            // the results stay fp32 (dx and dv over dx32 and dv32, dg in dg32) for a BwdRoundArgs launch
  float* dg32;             // q: [U, N, d]
  const float* dkret;      // k: nullable [U, cap, d]: the retained entries' part, entry c * lam + slot
  const float* dvret;
  const int32_t* sel;      // k: [U, sel_stride]
  HeadMap map;
  int n_units;             // q: B * Hq; k: B * Hkv
  int N, C, Hq, Hkv, nc, ncf, nseg, seg_chunks;
  int lam, cap, sel_stride;
  int n_ret;               // entries that have a gradient (some row sees them)
};
struct BwdRevscanArgs {
  const void* a_rows;      // [U, N, d]
  const void* phi;         // [U, N, 2d]
  const float* ed;         // [U, N]
  void* ds;                // [U, nc, d, 2d] storage type (state_image_offset): dS(c), chunks <= nc - 3
  float* dz;               // [U, nc, 2d]
  int N, C, nc;
};
struct BwdDwArgs {
  const void* q;
  const void* k;
  int64_t q_sb, q_st, q_sh, k_sb, k_st, k_sh;
  const void* dfq;         // [U, N, d]
  const void* dfk;
  float* dwq;              // [Hq, d, d], added into
  float* dwk;
  float* dbq;              // nullable [Hq, d], added into
  float* dbk;
  HeadMap map;
  int B, N, Hq;
  int tiles_per_block;     // set by the launcher
};
hipError_t launch_bwd_weights(const BwdWeightsArgs& a, int dtype, int Hq, hipStream_t stream);
hipError_t launch_bwd_lin(const BwdLinArgs& a, int dtype, int d, bool key, hipStream_t stream);
hipError_t launch_bwd_revscan(const BwdRevscanArgs& a, int dtype, int d, int U, hipStream_t stream);
hipError_t launch_bwd_dw(BwdDwArgs a, int dtype, int d, hipStream_t stream);
struct BwdSaArgs {
  const void* q;
  const void* k;
  const void* v;
  const void* dout;
  int64_t q_sb, q_st, q_sh, k_sb, k_st, k_sh, v_sb, v_st, v_sh, o_sb, o_st, o_sh;
  const void* kret;        // [U, cap, d]: retained keys in routing order, zero rows where no token is retained
  const void* vret;        // [U, cap, d]: retained values
  const unsigned long long* rvalid;   // [U, cap / 64]: bit = the retained entry is a token
  const int32_t* times;    // [U, cap]: entries of its chunk's list that name the entry's token; 0: no token
  const float* lse;        // [U, N]
  const float* delta;      // [U, N]
  float* dq32;             // [U, N, d]
  float* dk32;             // [B, Hkv, N, d]: the local key tiles' part
  float* dv32;
  float* dkret;            // [U, cap, d]: gradients of the retained entries, each as often as its list names the token
  float* dvret;
  HeadMap map;
  int N, cap, C, lam, rcap, U, Hq, Hkv;
  int n_row_tiles, n_ret_tiles;   // tiles of 128 rows / of 128 retained entries that some row sees
  float scale;
};
// retained keys and values of every (batch, query head) as rows, for the backward pass
struct BwdGatherArgs {
  const void* k;
  const void* v;
  int64_t k_sb, k_st, k_sh, v_sb, v_st, v_sh;
  const int32_t* sel;      // [U, sel_stride]; the first nsel entries are used
  void* kret;              // [U, cap, d]
  void* vret;
  unsigned long long* rvalid;   // [U, cap / 64]
  int32_t* times;          // [U, cap]
  HeadMap map;
  int nsel, sel_stride, cap, C, lam, Hq, d, N;
};
struct RopeArgs {
  void* q;                 // nullable [B, N, Hq, d], rotated in place
  void* k;                 // nullable [B, N, Hkv, d]
  int64_t q_sb, q_st, q_sh, k_sb, k_st, k_sh;
  const int32_t* pos0;     // nullable, device [B]: position of each sequence's token 0
  double log2_base;
  int B, N, Hq, Hkv, d;
};
hipError_t launch_rope(const RopeArgs& a, int dtype, hipStream_t stream);
hipError_t launch_bwd_row_prep(const BwdRowArgs& a, int dtype, hipStream_t stream);
hipError_t launch_bwd_round(const BwdRoundArgs& a, int dtype, hipStream_t stream);
hipError_t launch_bwd_gather(const BwdGatherArgs& a, int dtype, int U, hipStream_t stream);
hipError_t launch_bwd_sa_dq(const BwdSaArgs& a, int dtype, int d, hipStream_t stream);
hipError_t launch_bwd_sa_dkv(const BwdSaArgs& a, int dtype, int d, int B, hipStream_t stream);   // local span, then retained entries
// attention map and its backward pass (still_map.hip)
struct MapArgs {
  const void* q;
  const void* k;
  int64_t q_sb, q_st, q_sh, k_sb, k_st, k_sh;
  const void* wqf;         // [Hq, d, d]: operand order of f^T = W^T x^T (BwdWeightsArgs)
  const void* wkf;
  const void* bq;          // nullable [Hq, d]
  const void* bk;
  void* phi_q;             // [U, N, 2d] storage type
  void* phi_k;             // [U, N, 2d], zero for selected tokens
  const uint32_t* kmask;   // [U, ncf, C/32]: bit = token selected (within its chunk's quota)
  const float* lse;        // [U, N]
  float* map_out;          // forward: [U, N, N]
  const float* map_in;     // backward: the map, its gradient (at and below the diagonal)
  const float* dmap;
  float* rowdot;           // backward: [U, N], rows of chunks >= 2
  void* dfq;               // backward: [U, N, d] storage type
  void* dfk;
  HeadMap map;
  int U, N, C, Hq, nc, ncf;
  float scale;
};
hipError_t launch_map(const MapArgs& a, int dtype, int d, bool backward, hipStream_t stream);

}  // namespace still
