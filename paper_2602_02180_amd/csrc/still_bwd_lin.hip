// Backward pass of the prefill operator: the linear branch (the formulas are at the top of still_bwd.hip).
//
// One kernel serves both sides, a workgroup per 64 tokens.  Queries and keys differ in what they are multiplied with and
// not in the steps:
//   f = x W, NP-Map -> phi                              x = q, W = W_q          | x = k, W = W_k (per query head)
//   dphi = a S^T  (- coef z)                            a = A_t, S = state       | a = v, S = dS (state gradient)
//   y    = phi S                                        -> dg                    | -> dv
//   NP-Map backwards -> df;  dx = df W^T + cx x         -> dq                    | -> dk
// A key workgroup walks the query heads of its kv head and keeps dk, dv in its accumulators, so that they are written
// once, in the storage type, without atomics.  Everything in between stays on the chip: f, u, dphi in accumulators (one
// lane per token, wave pairs split the features and exchange four pairs of row statistics), phi and df in LDS.  A
// state image S^T [x][2 d_f] passes through LDS in slabs of 64 features, and one copy of a slab serves both products:
// read along its rows for phi S, down its columns (transposing LDS reads) for a S^T.
// Least traffic: the images (2 d d_f elements per chunk, four times the chunk's rows at C = 64), rows and gradients once.
// What bounds it beyond that: two workgroups per CU (registers and LDS) that alternate between products and row-wise vector
// work at one barrier per slab.  All 256 registers are in use at d = 128 and 13 (query side) / 50 (key side) values spill, 94 on
// the key side in fp32; none at d = 64 in bf16.
// Measured at 16 sequences of 1024 tokens, 32 / 8 heads, d = 128, C = 64, bf16: query side 0.465 ms, key side 0.455 ms (0.58 and
// 0.62 with loads that waited for each other and the retained entries looked up per result), state gradient 0.175 ms, parameter gradients 0.12 ms; as batched products through memory (f, u, dphi, phi S and their
// fp32 sums each written and read) 4.2 ms.
#include "still_kernels.h"
#include "still_tile.h"

namespace still {

namespace {

template <typename T, int D>
struct LinCfg {
  typedef Mma<T> M;
  static constexpr int DP = 2 * D;
  static constexpr int NS = DP / 64;                     // slabs of 64 features per state image
  static constexpr int SE = D * 64;                      // elements of a slab, and of a 64-token tile
  static constexpr int FST = D + 4;                      // row stride of the fp32 result tile
  static constexpr size_t slab_bytes = SE * sizeof(T);
  static constexpr size_t f32_bytes = 64 * FST * sizeof(float);
  static constexpr size_t work_bytes = 2 * slab_bytes > f32_bytes ? 2 * slab_bytes : f32_bytes;   // slabs, then results
  static constexpr size_t phi_bytes = 64 * DP * sizeof(T);
  static constexpr size_t smem = work_bytes + phi_bytes + DP * 4 + 2 * 64 * 4 * 4 + 64 * 4;
  static constexpr size_t key_smem(int heads) { return smem + kMaxHq + 64 * (size_t)heads; }   // + the retained entries
};

// element offset, inside one head's copy, of the operand "row x of W, contraction over features": [x / 32][k-step][lane][k
// per lane], x = 32 xt + (lane & 31)
template <typename M>
__device__ __forceinline__ int wrow_offset(int xt, int s, int lane, int d) { return ((xt * (d / M::KK) + s) * 64 + lane) * M::KPL; }

// both operand orders of both weight matrices, and the parameter gradients cleared, in one launch
template <typename T>
__global__ __launch_bounds__(256) void bwd_weights_kernel(BwdWeightsArgs a) {
  typedef Mma<T> M;
  const int h = blockIdx.y, idx = blockIdx.x * 256 + threadIdx.x, which = blockIdx.z;   // 0, 1: W_q; 2, 3: W_k
  if (idx >= a.d * a.d) return;
  const int d = a.d;
  const int64_t ho = (int64_t)h * d * d;
  const T* w = static_cast<const T*>(which < 2 ? a.wq : a.wk) + ho;
  const int e = idx % M::KPL, lane = (idx / M::KPL) % 64, blk = idx / (64 * M::KPL);
  const int s = blk % (d / M::KK), tile = blk / (d / M::KK);
  const int k = s * M::KK + (lane >> 5) * M::KPL + e;
  if ((which & 1) == 0) {
    static_cast<T*>(which == 0 ? a.wqf : a.wkf)[ho + idx] = w[(int64_t)k * d + 32 * tile + M::kappa(lane & 31)];
  } else {
    T* wr = static_cast<T*>(which == 1 ? a.wqr : a.wkr);
    float* dw = which == 1 ? a.dwq : a.dwk;
    if (wr != nullptr) wr[ho + idx] = w[(int64_t)(32 * tile + (lane & 31)) * d + k];
    if (dw != nullptr) dw[ho + idx] = 0.f;
    float* db = which == 1 ? a.dbq : a.dbk;
    if (db != nullptr && idx < d) db[(int64_t)h * d + idx] = 0.f;
  }
}

template <typename T>
__device__ __forceinline__ void load_elems(float (&x)[8], const T* p) {
  if constexpr (sizeof(T) == 2) {
    const bf16x8 v = *reinterpret_cast<const bf16x8*>(p);
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = static_cast<float>(v[e]);
  } else {
    const floatx4 u = *reinterpret_cast<const floatx4*>(p), v = *reinterpret_cast<const floatx4*>(p + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = u[e], x[4 + e] = v[e];
  }
}
template <typename T>
__device__ __forceinline__ void store_elems(T* p, const float (&x)[8]) {
  if constexpr (sizeof(T) == 2) {
    bf16x8 v;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = static_cast<bf16>(x[e]);
    *reinterpret_cast<bf16x8*>(p) = v;
  } else {
    floatx4 u, v;
#pragma unroll
    for (int e = 0; e < 4; ++e) u[e] = x[e], v[e] = x[4 + e];
    *reinterpret_cast<floatx4*>(p) = u;
    *reinterpret_cast<floatx4*>(p + 4) = v;
  }
}

// eight elements as loaded: what a loop asks for before it uses any of it
template <typename T>
struct Raw8 {
  typedef T Vec8 __attribute__((ext_vector_type(8), aligned(16)));
  Vec8 v;
  __device__ __forceinline__ void load(const T* p) { v = *reinterpret_cast<const Vec8*>(p); }
  __device__ __forceinline__ float at(int e) const { return to_f32<T>(v[e]); }
};

// IN_FP32: the results stay fp32, dx and dv over dx32 and dv32, dg in dg32.  (An instance of its own: as a run-time choice it
// cost the ordinary ones a per cent, 577 -> 582 and 619 -> 626 us at the shape above.)
template <typename T, int D, bool KEY, bool IN_FP32>
__global__ __launch_bounds__(256, 2) void bwd_lin_kernel(BwdLinArgs a) {
  typedef Mma<T> M;
  typedef LinCfg<T, D> Cf;
  typedef RowTile<T, D> RX;              // token tiles
  typedef StateSlab<T> RS;               // state slabs
  typedef RowTile<T, Cf::DP> RP;         // features of the tokens
  constexpr int DP = Cf::DP, NS = Cf::NS, NF = NS / 2, KS = D / M::KK, SK = 64 / M::KK, NX = D / 64, EPV = RX::EPV;
  static_assert(KS == SK * NX, "a slab's two products have the same number of steps");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  T* slab0 = reinterpret_cast<T*>(smem);
  T* slab1 = slab0 + Cf::SE;
  float* res = reinterpret_cast<float*>(smem);                        // fp32 results, once the slabs are done with
  T* phi = reinterpret_cast<T*>(smem + Cf::work_bytes);
  T* dfl = phi;                                                       // df, once phi is done with
  float* zl = reinterpret_cast<float*>(smem + Cf::work_bytes + Cf::phi_bytes);
  float* xch = zl + DP;                                               // [2 feature sides][64 tokens][4]
  float* cxl = xch + 2 * 64 * 4;
  uint8_t* head_of = reinterpret_cast<uint8_t*>(cxl + 64);            // (keys) the query heads of the kv head, and for each
  uint8_t* entry = head_of + kMaxHq;                                  // the slot of every token in the chunk's list, 255: none

  const int n_tiles = (a.N + 63) / 64;
  int bh, tile;                          // (batch, query head) or (batch, kv head)
  if (a.n_units % 8 == 0) {              // the tiles of a unit share an XCD (two tiles of a wide chunk read one image)
    const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
    bh = (j / n_tiles) * 8 + xcd;
    tile = j % n_tiles;
  } else {
    bh = blockIdx.x / n_tiles;
    tile = blockIdx.x % n_tiles;
  }
  const int H = KEY ? a.Hkv : a.Hq, b = bh / H, hx = bh % H;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, g = lane >> 5, rg = wave & 1, fh = wave >> 1;   // 32 tokens, half of every slab's features
  const int N = a.N, C = a.C, t0 = tile * 64, c = t0 / C;
  const int row = 32 * rg + r, t = min(t0 + row, N - 1);
  const bool full_chunk = c < a.ncf;
  // does the branch exist here: a state behind these rows / rows that see these keys
  const bool linear = KEY ? (full_chunk && c + 2 < a.nc) : c >= 2;

  const T* __restrict__ xg = static_cast<const T*>(a.x) + b * a.x_sb + hx * a.x_sh;

  floatx16 dxa[NX], ya[NX];              // results: rows = tokens (register), columns = channels (lane)
#pragma unroll
  for (int i = 0; i < NX; ++i) dxa[i] = zero16(), ya[i] = zero16();
  float cx = 0.f;
  int n_heads = 0;                       // (keys) heads walked so far
  constexpr int NE8 = 64 * D / 8 / 256;  // pieces of eight elements of a tile per thread

  for (int hi = 0; hi < (KEY ? a.Hq : 1); ++hi) {
    const int hq = KEY ? hi : hx;
    if (KEY && a.map.kv[hq] != hx) continue;
    const int64_t unit = (int64_t)b * a.Hq + hq;
    T* __restrict__ dfg = static_cast<T*>(a.df) + (unit * N + t0) * D;
    if (!linear) {                       // no gradient passes through the feature map of these tokens
      Vec16 z16;
      z16.w[0] = z16.w[1] = z16.w[2] = z16.w[3] = 0u;
      for (int i = tid; i < 64 * RX::PPR; i += 256)
        if (t0 + i / RX::PPR < N) *reinterpret_cast<Vec16*>(dfg + (int64_t)i * EPV) = z16;
      continue;
    }
    // ---- the token rows and what they are multiplied with, row by row into LDS
    // (all loads of a thread first: a loop that loads, waits and stores piece by piece took four round trips, 18 K of the 72 K
    // cycles of a query workgroup)
    {
      constexpr int NPC = 64 * RX::PPR / 256;
      const int tn = 64 * wave + fresh_lane_id();
      typedef uint32_t Piece __attribute__((ext_vector_type(4)));
      Piece xr[NPC], vr[KEY ? NPC : 1];
#pragma unroll
      for (int p = 0; p < NPC; ++p) {
        const int i = tn + 256 * p, e0 = (i % RX::PPR) * EPV, tt = min(t0 + i / RX::PPR, N - 1);
        xr[p] = *reinterpret_cast<const Piece*>(xg + (int64_t)tt * a.x_st + e0);
        if constexpr (KEY)
          vr[p] = *reinterpret_cast<const Piece*>(static_cast<const T*>(a.v) + b * a.v_sb + hx * a.v_sh + (int64_t)tt * a.v_st + e0);
      }
      if constexpr (!KEY) {              // A_t = E_t (gate_t * dy_t)
        Raw8<T> dyr[NE8], gr[NE8];
        float E[NE8];
#pragma unroll
        for (int p = 0; p < NE8; ++p) {
          const int i = tn + 256 * p, e0 = (i % (D / 8)) * 8, tt = min(t0 + i / (D / 8), N - 1);
          dyr[p].load(static_cast<const T*>(a.dout) + b * a.o_sb + (int64_t)tt * a.o_st + hx * a.o_sh + e0);
          E[p] = a.e_row[unit * N + tt];
          if (a.gate != nullptr) gr[p].load(static_cast<const T*>(a.gate) + b * a.g_sb + (int64_t)tt * a.g_st + hx * a.g_sh + e0);
        }
#pragma unroll
        for (int p = 0; p < NE8; ++p) {
          const int i = tn + 256 * p, ri = i / (D / 8), e0 = (i % (D / 8)) * 8;
          float dy[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) dy[e] = dyr[p].at(e) * E[p];
          if (a.gate != nullptr) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float g = gr[p].at(e);
              dy[e] = dyr[p].at(e) * (E[p] * (a.gate_act ? 1.f / (1.f + __expf(-g)) : g));
            }
          }
          if constexpr (sizeof(T) == 2) {
            store_elems<T>(slab1 + RX::off(ri, e0), dy);
          } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) slab1[RX::off(ri, e0 + e)] = dy[e];
          }
          if (t0 + ri < N) store_elems<T>(static_cast<T*>(a.a_rows) + (unit * N + t0 + ri) * D + e0, dy);
        }
      }
#pragma unroll
      for (int p = 0; p < NPC; ++p) {
        const int i = tn + 256 * p, at = RX::off(i / RX::PPR, (i % RX::PPR) * EPV);
        *reinterpret_cast<Piece*>(slab0 + at) = xr[p];
        if constexpr (KEY) *reinterpret_cast<Piece*>(slab1 + at) = vr[p];
      }
    }
    if constexpr (KEY) {                 // which retained entry each of the tokens is, for the results' sums
      if (a.dkret != nullptr && wave == (n_heads & 3)) {
        const int w = t0 - c * C + lane;
        const uint32_t* m = a.kmask + (unit * a.ncf + c) * (C / 32);
        int pos = 255;
        if ((m[w / 32] >> (w & 31)) & 1u) {
          const int32_t* list = a.sel + unit * a.sel_stride + c * a.lam;
          pos = __popc(m[w / 32] & ((1u << (w & 31)) - 1u));     // its rank among the list's tokens
          for (int j = 0; j < w / 32; ++j) pos += __popc(m[j]);
          if (list[pos] != t0 + lane)    // (a list with foreign or repeated entries, or in another order)
            for (pos = 0; pos < a.lam && list[pos] != t0 + lane; ++pos) {}
          if (pos == a.lam || retained_row(c, a.lam, pos, a.n_ret) < 0) pos = 255;
        }
        entry[64 * n_heads + lane] = (uint8_t)pos;
        if (lane == 0) head_of[n_heads] = (uint8_t)hq;
      }
      ++n_heads;
    }
    // the images, and z of the same states
    // (the first chunk of a segment has no local state, the first segment no prefix; never both at c >= 2)
    const T* img0 = static_cast<const T*>(a.snap) + (unit * a.nc + c) * (int64_t)(D * DP);
    const T* img1 = img0;
    int n_img = 1;
    if constexpr (!KEY) {
      const bool local = c % a.seg_chunks != 0, prefix = c >= a.seg_chunks;
      if (prefix) img1 = static_cast<const T*>(a.pimg) + (unit * a.nseg + c / a.seg_chunks) * (int64_t)(D * DP);
      if (!local) img0 = img1;
      n_img = local && prefix ? 2 : 1;
    }
    for (int i = tid; i < DP; i += 256) {
      float z = a.zsnap[(unit * a.nc + c) * DP + i];
      if constexpr (!KEY) {
        if (c >= a.seg_chunks) z += a.zpre[(unit * a.nseg + c / a.seg_chunks) * DP + i];   // (segment 0 has no prefix)
      }
      zl[i] = z;
    }
    const float coef = KEY ? 1.f : a.ed[unit * N + t];
    bool kept = false;
    if constexpr (KEY) {
      const int w = t - c * C;
      kept = (a.kmask[(unit * a.ncf + c) * (C / 32) + w / 32] >> (w & 31)) & 1u;
    }
    __syncthreads();
    typename M::frag af[KS];
    floatx16 u[NF];
    float nx2;
    {
      const T* wf = static_cast<const T*>(a.wf) + (int64_t)hq * D * D;
      typename M::frag xf[KS];
#pragma unroll
      for (int s = 0; s < KS; ++s) xf[s] = RX::along(slab0, row, s, g);
#pragma unroll
      for (int s = 0; s < KS; ++s) af[s] = RX::along(slab1, row, s, g);
#pragma unroll
      for (int j = 0; j < NF; ++j) u[j] = zero16();
      piped<typename M::frag, NF * KS, 6>(
          [&](auto I) __attribute__((always_inline)) {
            constexpr int i = decltype(I)::value;
            return M::load(wf + wfrag_offset<M>(2 * (i % NF) + fh, i / NF, lane, D));
          },
          [&](auto I, const typename M::frag& f) __attribute__((always_inline)) {
            constexpr int i = decltype(I)::value;
            u[i % NF] = M::mma(f, xf[i / NF], u[i % NF]);
          });
      float n4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < KS; ++s) n4[s & 3] = M::dot_into(xf[s], xf[s], n4[s & 3]);
      nx2 = sum32((n4[0] + n4[1]) + (n4[2] + n4[3]));
    }
    lds_barrier();                       // every wave has its fragments: the slabs may be overwritten
    // (a slab is a copy of whole blocks: 1 KB pieces, one after the other)
    auto request = [&](const T* im, int f0, T* dst) __attribute__((always_inline)) {
      const uint32_t lane_off = 16u * (uint32_t)fresh_lane_id(), base = lds_address(dst) + 1024 * wave;
      static_for<Cf::SE * (int)sizeof(T) / 4096>([&](auto J) __attribute__((always_inline)) {
        constexpr int j = decltype(J)::value;
        async_copy16_at<4096 * j>(im + state_slab_source((wave + 4 * j) * 64 * EPV, f0, DP), lane_off, base);
      });
    };
    request(img0, 0, slab0);

    // ---- NP-Map: u = f |x| / |f|, phi = [softmax(u), softmax(-u)]
    float* my = xch + (fh * 64 + row) * 4;
    const float* other = xch + ((fh ^ 1) * 64 + row) * 4;
    if (a.bias != nullptr) {
      const T* bias = static_cast<const T*>(a.bias) + (int64_t)hq * D;
#pragma unroll
      for (int j = 0; j < NF; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) u[j][i] += to_f32(bias[64 * j + 32 * fh + M::pos_of_reg(i, g)]);
    }
    float nf2 = 0.f, mx = -INFINITY, mn = INFINITY;
#pragma unroll
    for (int j = 0; j < NF; ++j)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        nf2 = fmaf(u[j][i], u[j][i], nf2);
        mx = fmaxf(mx, u[j][i]);
        mn = fminf(mn, u[j][i]);
      }
    nf2 = sum32(nf2);
    mx = max32(mx);
    mn = min32(mn);
    if (g == 0) my[0] = nf2, my[1] = mx, my[2] = mn;
    lds_barrier();
    nf2 += other[0];
    mx = fmaxf(mx, other[1]);
    mn = fminf(mn, other[2]);
    const float nx = sqrtf(nx2), nf = sqrtf(nf2);
    const float ratio = nf2 > 0.f ? nx / nf : 0.f;
    float mp = mx * ratio * kLog2e, mm = -mn * ratio * kLog2e;   // maxima of u and -u, in base-2 exponents
    float sp = 0.f, sn = 0.f;
#pragma unroll
    for (int j = 0; j < NF; ++j)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        u[j][i] *= ratio;
        sp += fast_exp2(fmaf(u[j][i], kLog2e, -mp));
        sn += fast_exp2(fmaf(u[j][i], -kLog2e, -mm));
      }
    sp = sum32(sp);
    sn = sum32(sn);
    lds_barrier();                       // (the first exchange has been read)
    if (g == 0) my[0] = sp, my[1] = sn;
    lds_barrier();
    sp += other[0];
    sn += other[1];
    const float ip = 1.f / sp, in = 1.f / sn;
#pragma unroll
    for (int j = 0; j < NF; ++j) {
      float x[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) x[i] = kept ? 0.f : fast_exp2(fmaf(u[j][i], kLog2e, -mp)) * ip;
      put_row<T, DP>(phi, row, 64 * j + 32 * fh, x, g);
#pragma unroll
      for (int i = 0; i < 16; ++i) x[i] = kept ? 0.f : fast_exp2(fmaf(u[j][i], -kLog2e, -mm)) * in;
      put_row<T, DP>(phi, row, D + 64 * j + 32 * fh, x, g);
    }

    // ---- dphi^T = S a^T (this wave's features of every slab) and y = phi S (its half of the channels)
    floatx16 dp[NS], yq[NX];
#pragma unroll
    for (int j = 0; j < NS; ++j) dp[j] = zero16();
#pragma unroll
    for (int i = 0; i < NX; ++i) yq[i] = zero16();
    const bool need_y = KEY || a.dg != nullptr;
    for (int im = 0; im < n_img; ++im) {
      static_for<NS>([&](auto J) __attribute__((always_inline)) {
        constexpr int j = decltype(J)::value;
        const T* cur = (j & 1) ? slab1 : slab0;
        T* nxt = (j & 1) ? slab0 : slab1;
        wait_async_copies();
        lds_barrier();                   // slab j is here (and phi, the first time); everybody is done with its predecessor
        if (j + 1 < NS) request(im == 0 ? img0 : img1, 64 * (j + 1), nxt);
        else if (im + 1 < n_img) request(img1, 0, nxt);
        if constexpr (!KEY && j == 0) {
          if (im == 0) {                 // the state gradient reads phi from memory
            T* pg = static_cast<T*>(a.phi) + (unit * N + t0) * DP;
#pragma unroll 2
            for (int i = tid; i < 64 * RP::PPR; i += 256) {
              const int ri = i / RP::PPR, e0 = (i % RP::PPR) * EPV;
              if (t0 + ri < N) *reinterpret_cast<Vec16*>(pg + (int64_t)ri * DP + e0) = *reinterpret_cast<const Vec16*>(phi + RP::off(ri, e0));
            }
          }
        }
        const int lane_now = fresh_lane_id(), rr = lane_now & 31, gg = lane_now >> 5;
        if (need_y) {
          // (phi's operands are read one step ahead: all of them at once would not fit the register file)
          typename M::frag pf[2];
          pf[0] = RP::along(phi, 32 * rg + rr, SK * j, gg);
          piped<typename M::frag, 2 * KS, 4>(
              [&](auto I) __attribute__((always_inline)) {
                constexpr int i = decltype(I)::value, q = i >> 1;
                if constexpr ((i & 1) == 0) return RS::down(cur, q * M::KK, 32 * fh, lane_now);
                else return RS::along(cur, fh * NX + q % NX, q / NX, rr, gg);
              },
              [&](auto I, const typename M::frag& f) __attribute__((always_inline)) {
                constexpr int i = decltype(I)::value, q = i >> 1;
                if constexpr ((i & 1) == 0) dp[j] = M::mma(f, af[q], dp[j]);
                else {
                  if constexpr (q % NX == 0 && q / NX + 1 < SK) pf[(q / NX + 1) & 1] = RP::along(phi, 32 * rg + rr, SK * j + q / NX + 1, gg);
                  if constexpr (KEY) ya[q % NX] = M::mma(pf[(q / NX) & 1], f, ya[q % NX]);
                  else yq[q % NX] = M::mma(pf[(q / NX) & 1], f, yq[q % NX]);
                }
              });
        } else {
          piped<typename M::frag, KS, 6>(
              [&](auto I) __attribute__((always_inline)) { return RS::down(cur, decltype(I)::value * M::KK, 32 * fh, lane_now); },
              [&](auto I, const typename M::frag& f) __attribute__((always_inline)) {
                dp[j] = M::mma(f, af[decltype(I)::value], dp[j]);
              });
        }
      });
    }
    lds_barrier();                       // slabs and phi are done with

    // ---- NP-Map backwards.  (The exponentials are taken again: kept across the slab loop they would not fit the register
    // file, and the empty statement keeps the compiler from doing that.)
    asm volatile("" : "+v"(mp), "+v"(mm));
    const bool dead = kept || !(nx > 0.f) || !(nf > 0.f);
    float ap = 0.f, an = 0.f;
#pragma unroll
    for (int j = 0; j < NF; ++j)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int fi = 64 * j + 32 * fh + M::pos_of_reg(i, g);
        dp[j][i] -= coef * zl[fi];
        dp[NF + j][i] -= coef * zl[D + fi];
        ap += fast_exp2(fmaf(u[j][i], kLog2e, -mp)) * ip * dp[j][i];
        an += fast_exp2(fmaf(u[j][i], -kLog2e, -mm)) * in * dp[NF + j][i];
      }
    ap = sum32(ap);
    an = sum32(an);
    if (g == 0) my[0] = ap, my[1] = an;
    if constexpr (!KEY) {
      if (need_y) {
#pragma unroll
        for (int i = 0; i < NX; ++i)
#pragma unroll
          for (int e = 0; e < 16; ++e) res[(32 * rg + c_row(e, g)) * Cf::FST + 32 * (fh * NX + i) + r] = yq[i][e];
      }
    }
    lds_barrier();
    ap += other[0];
    an += other[1];
    const float inx = nx > 0.f ? 1.f / nx : 0.f;
    float dnx = 0.f;
    if constexpr (KEY) asm volatile("" : "+v"(mp), "+v"(mm));
#pragma unroll
    for (int j = 0; j < NF; ++j)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float ep = fast_exp2(fmaf(u[j][i], kLog2e, -mp)) * ip, en = fast_exp2(fmaf(u[j][i], -kLog2e, -mm)) * in;
        dp[j][i] = ep * (dp[j][i] - ap) - en * (dp[NF + j][i] - an);
        dnx += u[j][i] * inx * dp[j][i];
      }
    dnx = sum32(dnx);
    if (g == 0) my[2] = dnx;
    if constexpr (!KEY) {                // dg = E_t dy_t * (phi_q S)_t (times the logistic function's slope)
      if (need_y) {
        const int tn = 64 * wave + fresh_lane_id();
        Raw8<T> dyr[NE8], gr[NE8];
        float E[NE8];
#pragma unroll
        for (int p = 0; p < NE8; ++p) {
          const int i = tn + 256 * p, e0 = (i % (D / 8)) * 8, tt = min(t0 + i / (D / 8), N - 1);
          dyr[p].load(static_cast<const T*>(a.dout) + b * a.o_sb + (int64_t)tt * a.o_st + hx * a.o_sh + e0);
          E[p] = a.e_row[unit * N + tt];
          if (a.gate_act) gr[p].load(static_cast<const T*>(a.gate) + b * a.g_sb + (int64_t)tt * a.g_st + hx * a.g_sh + e0);
        }
#pragma unroll
        for (int p = 0; p < NE8; ++p) {
          const int i = tn + 256 * p, ri = i / (D / 8), e0 = (i % (D / 8)) * 8, tt = t0 + ri;
          if (tt >= N) continue;
          float dy[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) dy[e] = dyr[p].at(e) * (E[p] * res[ri * Cf::FST + e0 + e]);
          if (a.gate_act) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float sg = 1.f / (1.f + __expf(-gr[p].at(e)));
              dy[e] *= sg * (1.f - sg);
            }
          }
          if constexpr (IN_FP32) store_elems<float>(a.dg32 + (unit * N + tt) * D + e0, dy);
          else store_elems<T>(static_cast<T*>(a.dg) + b * a.g_sb + (int64_t)tt * a.g_st + hx * a.g_sh + e0, dy);
        }
      }
    }
    lds_barrier();
    dnx += other[2];
    const float rt = dead ? 0.f : ratio;
    cx += dead ? 0.f : dnx * inx;
#pragma unroll
    for (int j = 0; j < NF; ++j) {
      float x[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) x[i] = dead ? 0.f : rt * (dp[j][i] - u[j][i] * inx * dnx);
      put_row<T, D>(dfl, row, 64 * j + 32 * fh, x, g);
    }
    lds_barrier();
    for (int i = tid; i < 64 * RX::PPR; i += 256) {
      const int ri = i / RX::PPR, e0 = (i % RX::PPR) * EPV;
      if (t0 + ri < N) *reinterpret_cast<Vec16*>(dfg + (int64_t)ri * D + e0) = *reinterpret_cast<const Vec16*>(dfl + RX::off(ri, e0));
    }
    {                                    // dx += df W^T
      const T* wr = static_cast<const T*>(a.wr) + (int64_t)hq * D * D;
      const int lane_now = fresh_lane_id(), rr = lane_now & 31, gg = lane_now >> 5;
      typename M::frag df[KS];
#pragma unroll
      for (int s = 0; s < KS; ++s) df[s] = RX::along(dfl, 32 * rg + rr, s, gg);
      piped<typename M::frag, NX * KS, 8>(
          [&](auto I) __attribute__((always_inline)) {
            constexpr int i = decltype(I)::value;
            return M::load(wr + wrow_offset<M>(fh * NX + i % NX, i / NX, lane_now, D));
          },
          [&](auto I, const typename M::frag& f) __attribute__((always_inline)) {
            constexpr int i = decltype(I)::value;
            dxa[i % NX] = M::mma(df[i / NX], f, dxa[i % NX]);
          });
    }
    if constexpr (KEY) lds_barrier();    // the next head reuses every buffer
  }

  // ---- results: the softmax branch's part, this branch's, and (keys) the retained entries', in the storage type
  auto emit = [&](const floatx16 (&acc)[NX], float* src, T* dst, int64_t s_b, int64_t s_t, int64_t s_h, bool with_x,
                  const float* dret) __attribute__((always_inline)) {
    if (linear) {
#pragma unroll
      for (int i = 0; i < NX; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) res[(32 * rg + c_row(e, g)) * Cf::FST + 32 * (fh * NX + i) + r] = acc[i][e];
      if (with_x && g == 0 && fh == 0) cxl[row] = cx;
      lds_barrier();
    }
    // (loads first, as above.  The retained entries: four heads at a time, every load unconditional and dropped where the head
    // does not keep the token; looked up per piece, three dependent loads per head, they took 120 K cycles of a workgroup
    // that works 45 K per head.  A load that is dropped reads the chunk's first row, so a chunk that the budget leaves
    // nothing, whose first row would lie behind the buffer, is left out)
    const int tn = 64 * wave + fresh_lane_id();
    float x[NE8][8];
    Raw8<T> xr[NE8];
#pragma unroll
    for (int p = 0; p < NE8; ++p) {
      const int i = tn + 256 * p, e0 = (i % (D / 8)) * 8, tt = min(t0 + i / (D / 8), N - 1);
      load_elems<float>(x[p], src + ((int64_t)bh * N + tt) * D + e0);
      if (with_x) xr[p].load(xg + (int64_t)tt * a.x_st + e0);
    }
    if (linear) {
#pragma unroll
      for (int p = 0; p < NE8; ++p) {
        const int i = tn + 256 * p, ri = i / (D / 8), e0 = (i % (D / 8)) * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) x[p][e] += res[ri * Cf::FST + e0 + e];
        if (with_x) {
#pragma unroll
          for (int e = 0; e < 8; ++e) x[p][e] += cxl[ri] * xr[p].at(e);
        }
      }
      const int first = KEY ? retained_row(c, a.lam, 0, a.n_ret) : -1;
      if (KEY && dret != nullptr && first >= 0) {      // (tokens that are in no state are in no retained set either)
        constexpr int HG = 4;
#pragma unroll 1
        for (int g0 = 0; g0 < n_heads; g0 += HG) {
          const float* base[HG];
#pragma unroll
          for (int u = 0; u < HG; ++u) {
            const int hq = __builtin_amdgcn_readfirstlane(head_of[min(g0 + u, n_heads - 1)]);
            base[u] = dret + (((int64_t)b * a.Hq + hq) * a.cap + first) * D;
          }
#pragma unroll
          for (int p = 0; p < NE8; ++p) {
            const int i = tn + 256 * p, ri = i / (D / 8), e0 = (i % (D / 8)) * 8;
            float xd[HG][8];
            bool on[HG];
#pragma unroll
            for (int u = 0; u < HG; ++u) {
              const int pos = entry[64 * min(g0 + u, n_heads - 1) + ri];
              on[u] = g0 + u < n_heads && pos != 255;
              load_elems<float>(xd[u], base[u] + (int64_t)(on[u] ? pos : 0) * D + e0);
            }
#pragma unroll
            for (int u = 0; u < HG; ++u)
#pragma unroll
              for (int e = 0; e < 8; ++e) x[p][e] += on[u] ? xd[u][e] : 0.f;
          }
        }
      }
    }
#pragma unroll
    for (int p = 0; p < NE8; ++p) {
      const int i = tn + 256 * p, e0 = (i % (D / 8)) * 8, tt = t0 + i / (D / 8);
      if (tt >= N) continue;
      if constexpr (IN_FP32) store_elems<float>(src + ((int64_t)bh * N + tt) * D + e0, x[p]);
      else store_elems<T>(dst + b * s_b + (int64_t)tt * s_t + hx * s_h + e0, x[p]);
    }
  };
  if (!KEY && !linear && a.dg != nullptr) {
    Vec16 z16;
    z16.w[0] = z16.w[1] = z16.w[2] = z16.w[3] = 0u;
    for (int i = tid; IN_FP32 && i < 64 * D / 4; i += 256)
      if (t0 + i / (D / 4) < N) *reinterpret_cast<Vec16*>(a.dg32 + ((int64_t)bh * N + t0) * D + 4 * i) = z16;
    for (int i = tid; !IN_FP32 && i < 64 * RX::PPR; i += 256)
      if (t0 + i / RX::PPR < N)
        *reinterpret_cast<Vec16*>(static_cast<T*>(a.dg) + b * a.g_sb + (int64_t)(t0 + i / RX::PPR) * a.g_st + hx * a.g_sh +
                                  (i % RX::PPR) * EPV) = z16;
  }
  emit(dxa, a.dx32, static_cast<T*>(a.dx), a.x_sb, a.x_st, a.x_sh, true, a.dkret);
  if constexpr (KEY) {
    lds_barrier();
    emit(ya, a.dv32, static_cast<T*>(a.dv), a.v_sb, a.v_st, a.v_sh, false, a.dvret);
  }
}

// ---------------------------------------------------------------------------------------------------------
// The state gradient as a running sum: dS(c) = sum over c' >= c + 2 of A(c')^T phi_q(c'), dz(c) likewise of the rows'
// E delta.  One workgroup owns 64 channels x BF features of one (batch, head) and walks the chunks from the last one
// down; after chunk c' its accumulators ARE dS(c' - 2), which is stored in the storage type (the layout of the
// forward states).  Token tiles are double-buffered and read down their columns on both sides.
// Bound by the images it writes (2 d d_f elements per chunk).
// ---------------------------------------------------------------------------------------------------------
template <typename T, int D>
struct RevCfg {
  static constexpr int BF = D == 128 ? 128 : 64;         // features per workgroup
  static constexpr int AE = 64 * 64, PE = 64 * BF;       // elements of a tile of A rows / of phi rows
  static constexpr size_t smem = 2 * (AE + PE) * sizeof(T) + 2 * 64 * 4;
};

template <typename T, int D>
__global__ __launch_bounds__(256, 2) void bwd_revscan_kernel(BwdRevscanArgs a) {
  typedef Mma<T> M;
  typedef RevCfg<T, D> Cf;
  constexpr int BF = Cf::BF, DP = 2 * D, SK = 64 / M::KK, NT = BF / 64;
  typedef RowTile<T, 64> RA;
  typedef RowTile<T, BF> RP;
  constexpr int EPV = RA::EPV;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  T* Al = reinterpret_cast<T*>(smem);
  T* Pl = Al + 2 * Cf::AE;
  float* wl = reinterpret_cast<float*>(Pl + 2 * Cf::PE);   // E delta of the tile's tokens
  constexpr int NXT = D / 64;
  const int unit = blockIdx.y, xt = blockIdx.x % NXT, ft = blockIdx.x / NXT;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, g = lane >> 5;
  // BF = 128: a wave owns 32 features and all 64 channels; BF = 64: 32 features and 32 channels
  const int fw = NT == 2 ? wave : wave & 1, xw = NT == 2 ? 0 : wave >> 1;
  const int N = a.N, C = a.C;
  const T* __restrict__ ag = static_cast<const T*>(a.a_rows) + (int64_t)unit * N * D + 64 * xt;
  const T* __restrict__ pg = static_cast<const T*>(a.phi) + (int64_t)unit * N * DP + BF * ft;
  const int n_tiles = (N + 63) / 64, first = 2 * (C / 64);   // chunks 0 and 1 add to nothing
  auto request = [&](int ti, int buf) __attribute__((always_inline)) {
    const int lane_now = fresh_lane_id();
    constexpr int IA = Cf::AE * (int)sizeof(T) / 4096, IP = Cf::PE * (int)sizeof(T) / 4096;
#pragma unroll
    for (int j = 0; j < IA; ++j) {
      const int piece = (wave + 4 * j) * 64 + lane_now, row = piece / RA::PPR;
      const int tok = min(ti * 64 + row, N - 1);
      async_copy16(ag + (int64_t)tok * D + ((piece % RA::PPR) ^ RA::swz(row)) * EPV,
                   lds_address(Al + buf * Cf::AE + (wave + 4 * j) * 64 * EPV));
    }
#pragma unroll
    for (int j = 0; j < IP; ++j) {
      const int piece = (wave + 4 * j) * 64 + lane_now, row = piece / RP::PPR;
      const int tok = min(ti * 64 + row, N - 1);
      async_copy16(pg + (int64_t)tok * DP + ((piece % RP::PPR) ^ RP::swz(row)) * EPV,
                   lds_address(Pl + buf * Cf::PE + (wave + 4 * j) * 64 * EPV));
    }
  };
  floatx16 acc[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) acc[j] = zero16();
  float dz0 = 0.f, dz1 = 0.f;
  // dz: thread = (two features, a quarter of the tile's tokens); BF / 2 pairs x 4 quarters
  const int pair = (wave * 16 + (lane & 15)), quarter = lane >> 4;
  auto store = [&](int c) __attribute__((always_inline)) {
    T* cp = static_cast<T*>(a.ds) + ((int64_t)unit * a.nc + c) * (int64_t)(D * DP);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int x = 64 * xt + 32 * (NT == 2 ? j : xw) + M::kappa(r), f0 = BF * ft + 32 * fw;
      store_image_tile<M>(cp, x, f0, DP, g, acc[j]);
    }
    if (xt == 0 && 2 * pair < BF) {
      float z0 = dz0 + __shfl_xor(dz0, 16, 64), z1 = dz1 + __shfl_xor(dz1, 16, 64);
      z0 += __shfl_xor(z0, 32, 64);
      z1 += __shfl_xor(z1, 32, 64);
      if (quarter == 0) {
        float* zp = a.dz + ((int64_t)unit * a.nc + c) * DP + BF * ft + 2 * pair;
        zp[0] = z0;
        zp[1] = z1;
      }
    }
  };
  if (n_tiles > first) {
    request(n_tiles - 1, 0);
    if (tid < 64) {
      const int tok = (n_tiles - 1) * 64 + tid;
      wl[tid] = tok < N ? a.ed[(int64_t)unit * N + tok] : 0.f;
    }
  }
  int buf = 0;
#pragma unroll 1
  for (int ti = n_tiles - 1; ti >= first; --ti) {
    wait_async_copies();
    lds_barrier();
    if (ti - 1 >= first) {
      request(ti - 1, buf ^ 1);
      if (tid < 64) wl[(buf ^ 1) * 64 + tid] = a.ed[(int64_t)unit * N + (ti - 1) * 64 + tid];
    }
    T* Ac = Al + buf * Cf::AE;
    const T* Pc = Pl + buf * Cf::PE;
    if (ti * 64 + 64 > N) {              // tokens past the end (the last one again) count as nothing
      for (int i = tid; i < 64 * RA::PPR; i += 256) {
        const int ri = i / RA::PPR;
        if (ti * 64 + ri >= N) {
          Vec16 z16;
          z16.w[0] = z16.w[1] = z16.w[2] = z16.w[3] = 0u;
          *reinterpret_cast<Vec16*>(Ac + RA::off(ri, (i % RA::PPR) * EPV)) = z16;
        }
      }
      lds_barrier();
    }
    const int lane_now = fresh_lane_id();
    typename M::frag pf[SK];
#pragma unroll
    for (int s = 0; s < SK; ++s) pf[s] = RP::down(Pc, s * M::KK, 32 * fw, lane_now);
    piped<typename M::frag, NT * SK, 6>(
        [&](auto I) __attribute__((always_inline)) {
          constexpr int i = decltype(I)::value;
          return RA::down(Ac, (i / NT) * M::KK, 32 * (NT == 2 ? i % NT : xw), lane_now);
        },
        [&](auto I, const typename M::frag& f) __attribute__((always_inline)) {
          constexpr int i = decltype(I)::value;
          acc[i % NT] = M::mma(pf[i / NT], f, acc[i % NT]);
        });
    if (xt == 0 && 2 * pair < BF) {
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const int tk = quarter * 16 + k;
        const T* pp = Pc + RP::off(tk, 2 * pair);
        const float w = wl[buf * 64 + tk];
        dz0 = fmaf(to_f32(pp[0]), w, dz0);
        dz1 = fmaf(to_f32(pp[1]), w, dz1);
      }
    }
    if ((ti * 64) % C == 0) store(ti * 64 / C - 2);
    buf ^= 1;
  }
}

// ---------------------------------------------------------------------------------------------------------
// dW[h] += sum over tokens of x^T df (and db[h] += sum of df): a workgroup owns one head's whole D x D matrix for a run
// of 64-token tiles (batch and sequence as one list), token tiles read down their columns on both sides, sums
// added atomically at the end.  grid.z: queries, keys.
// ---------------------------------------------------------------------------------------------------------
template <typename T, int D>
__global__ __launch_bounds__(256, 2) void bwd_dw_kernel(BwdDwArgs a) {
  typedef Mma<T> M;
  typedef RowTile<T, D> RT;
  constexpr int TE = 64 * D, EPV = RT::EPV, SK = 64 / M::KK, Q = D / 64;   // a wave owns (32 Q) x (32 Q)
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  T* Xl = reinterpret_cast<T*>(smem);
  T* Fl = Xl + 2 * TE;
  const bool key = blockIdx.z == 1;
  const int h = blockIdx.y, hx = key ? a.map.kv[h] : h;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, g = lane >> 5, xw = wave & 1, fw = wave >> 1;
  const int N = a.N, n_tiles = (N + 63) / 64;
  const int first = blockIdx.x * a.tiles_per_block, last = min(first + a.tiles_per_block, a.B * n_tiles);
  const T* xb = static_cast<const T*>(key ? a.k : a.q) + hx * (key ? a.k_sh : a.q_sh);
  const int64_t x_sb = key ? a.k_sb : a.q_sb, x_st = key ? a.k_st : a.q_st;
  const T* fb = static_cast<const T*>(key ? a.dfk : a.dfq);
  auto request = [&](int ti, int buf) __attribute__((always_inline)) {
    const int b = ti / n_tiles, t0 = (ti % n_tiles) * 64;
    const int lane_now = fresh_lane_id();
#pragma unroll
    for (int j = 0; j < TE * (int)sizeof(T) / 4096; ++j) {
      const int piece = (wave + 4 * j) * 64 + lane_now, row = piece / RT::PPR;
      const int col = ((piece % RT::PPR) ^ RT::swz(row)) * EPV, tok = min(t0 + row, N - 1);
      async_copy16(xb + b * x_sb + (int64_t)tok * x_st + col, lds_address(Xl + buf * TE + (wave + 4 * j) * 64 * EPV));
      async_copy16(fb + (((int64_t)b * a.Hq + h) * N + tok) * D + col, lds_address(Fl + buf * TE + (wave + 4 * j) * 64 * EPV));
    }
  };
  floatx16 acc[Q][Q];
#pragma unroll
  for (int i = 0; i < Q; ++i)
#pragma unroll
    for (int j = 0; j < Q; ++j) acc[i][j] = zero16();
  float* db = key ? a.dbk : a.dbq;
  float dbs = 0.f;                       // column tid % D of df, tokens tid / D, + 256 / D, ...
  if (first < last) request(first, 0);
  int buf = 0;
#pragma unroll 1
  for (int ti = first; ti < last; ++ti) {
    wait_async_copies();
    lds_barrier();
    if (ti + 1 < last) request(ti + 1, buf ^ 1);
    const T* Xc = Xl + buf * TE;
    T* Fc = Fl + buf * TE;
    const int t0 = (ti % n_tiles) * 64;
    if (t0 + 64 > N) {                   // tokens past the end (the last one again) count as nothing
      for (int i = tid; i < 64 * RT::PPR; i += 256) {
        const int ri = i / RT::PPR;
        if (t0 + ri >= N) {
          Vec16 z16;
          z16.w[0] = z16.w[1] = z16.w[2] = z16.w[3] = 0u;
          *reinterpret_cast<Vec16*>(Fc + RT::off(ri, (i % RT::PPR) * EPV)) = z16;
        }
      }
      lds_barrier();
    }
    const int lane_now = fresh_lane_id();
#pragma unroll
    for (int s = 0; s < SK; ++s) {
      typename M::frag xf[Q], ff[Q];
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        xf[i] = RT::down(Xc, s * M::KK, 32 * (xw * Q + i), lane_now);
        ff[i] = RT::down(Fc, s * M::KK, 32 * (fw * Q + i), lane_now);
      }
#pragma unroll
      for (int i = 0; i < Q; ++i)
#pragma unroll
        for (int j = 0; j < Q; ++j) acc[i][j] = M::mma(xf[i], ff[j], acc[i][j]);
    }
    if (db != nullptr) {
      for (int k = tid / D; k < 64; k += 256 / D) dbs += to_f32(Fc[RT::off(k, tid % D)]);
    }
    buf ^= 1;
  }
  float* dw = (key ? a.dwk : a.dwq) + (int64_t)h * D * D;
#pragma unroll
  for (int i = 0; i < Q; ++i)
#pragma unroll
    for (int j = 0; j < Q; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e)
        atomicAdd(dw + (int64_t)(32 * (xw * Q + i) + M::pos_of_reg(e, g)) * D + 32 * (fw * Q + j) + M::kappa(r), acc[i][j][e]);
  if (db != nullptr) atomicAdd(db + (int64_t)h * D + tid % D, dbs);
}

template <typename K>
hipError_t allow_lds(K kern, size_t smem) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
}

template <typename T, int D>
hipError_t launch_lin_t(const BwdLinArgs& a, bool key, hipStream_t s) {
  auto kern = a.in_fp32 ? (key ? bwd_lin_kernel<T, D, true, true> : bwd_lin_kernel<T, D, false, true>)
                        : (key ? bwd_lin_kernel<T, D, true, false> : bwd_lin_kernel<T, D, false, false>);
  int heads = 0;                         // of the widest group
  for (int kv = 0; kv < (key ? a.Hkv : 0); ++kv) {
    int n = 0;
    for (int h = 0; h < a.Hq; ++h) n += a.map.kv[h] == kv;
    heads = n > heads ? n : heads;
  }
  const size_t smem = key ? LinCfg<T, D>::key_smem(heads) : LinCfg<T, D>::smem;
  const hipError_t e = allow_lds(kern, smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)((a.N + 63) / 64) * a.n_units), dim3(256), smem, s, a);
  return hipGetLastError();
}

template <typename T, int D>
hipError_t launch_revscan_t(const BwdRevscanArgs& a, int U, hipStream_t s) {
  typedef RevCfg<T, D> Cf;
  const hipError_t e = allow_lds(bwd_revscan_kernel<T, D>, Cf::smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((bwd_revscan_kernel<T, D>), dim3((D / 64) * (2 * D / Cf::BF), U), dim3(256), Cf::smem, s, a);
  return hipGetLastError();
}

template <typename T, int D>
hipError_t launch_dw_t(const BwdDwArgs& a, int blocks, hipStream_t s) {
  const size_t smem = (size_t)4 * 64 * D * sizeof(T);
  const hipError_t e = allow_lds(bwd_dw_kernel<T, D>, smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((bwd_dw_kernel<T, D>), dim3(blocks, a.Hq, 2), dim3(256), smem, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_bwd_weights(const BwdWeightsArgs& a, int dtype, int Hq, hipStream_t s) {
  const dim3 grid((a.d * a.d + 255) / 256, Hq, 4);
  if (dtype == 1) hipLaunchKernelGGL(bwd_weights_kernel<bf16>, grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL(bwd_weights_kernel<float>, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_bwd_lin(const BwdLinArgs& a, int dtype, int d, bool key, hipStream_t s) {
  if (dtype == 1) return d == 128 ? launch_lin_t<bf16, 128>(a, key, s) : launch_lin_t<bf16, 64>(a, key, s);
  if (d == 64) return launch_lin_t<float, 64>(a, key, s);
  return hipErrorInvalidValue;   // fp32 is built for d = 64 only (refused by the host checks)
}

hipError_t launch_bwd_revscan(const BwdRevscanArgs& a, int dtype, int d, int U, hipStream_t s) {
  if (dtype == 1) return d == 128 ? launch_revscan_t<bf16, 128>(a, U, s) : launch_revscan_t<bf16, 64>(a, U, s);
  if (d == 64) return launch_revscan_t<float, 64>(a, U, s);
  return hipErrorInvalidValue;
}

hipError_t launch_bwd_dw(BwdDwArgs a, int dtype, int d, hipStream_t s) {
  // about four workgroups per CU over both sides: enough to hide the copies, few enough that the atomic sums (d * d_f per
  // workgroup) stay a small part of the traffic
  const int tiles = a.B * ((a.N + 63) / 64);
  a.tiles_per_block = (int)(((int64_t)tiles * a.Hq * 2 + 1023) / 1024);
  const int blocks = (tiles + a.tiles_per_block - 1) / a.tiles_per_block;
  if (dtype == 1) return d == 128 ? launch_dw_t<bf16, 128>(a, blocks, s) : launch_dw_t<bf16, 64>(a, blocks, s);
  if (d == 64) return launch_dw_t<float, 64>(a, blocks, s);
  return hipErrorInvalidValue;
}

}  // namespace still
