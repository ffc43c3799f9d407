// Backward pass of the prefill operator: the softmax branch (the formulas are at the top of still_bwd.hip).
//
// Both kernels follow the forward kernel's shape: everything is computed so that one lane owns one free index (a query
// row for dq, a key for dk and dv), P and dS stay in the accumulator registers of the product that made them and are
// the operand of the next one in place, and the operands shared by the waves of a workgroup pass through LDS as
// row-major tiles (still_tile.h), double-buffered with direct-to-LDS copies.  A tile is read along its rows for the
// products over the head dimension and down its columns (transposing LDS reads) for the products over keys or rows,
// so one copy of every tile serves both and no transposed tensor exists in memory.
//   dq  : S^T = K Q^T, dP^T = V dO^T (64 keys x 32 rows per wave), dq^T += K^T dS^T.
//   dkv : S = Q K^T, dP = dO V^T (32 rows x 32 keys per wave), dv^T += dO^T P, dk^T += Q^T dS.
// What bounds them: LDS operand bandwidth next to the matrix pipe (every product reads a fresh 1 KB fragment).
// Measured at 16 sequences of 1024 tokens, 32 / 8 heads, d = 128, C = 64, lambda = 16, bf16: dq 0.75 -> 0.24 ms, dkv of
// the local span 0.40 -> 0.16 ms, of the retained entries 0.67 -> 0.18 ms (four values spilled), against the same products with every operand
// fetched from global memory in fragment form (32 cache lines per instruction) and P, dS passed through LDS.
#include "still_kernels.h"
#include "still_tile.h"

namespace still {

namespace {

// ---- retained rows of every (batch, query head), in routing order: keys and values row by row, and one bit per entry
// (set = a token of its chunk; lists are never trusted for addressing).  Entries without a token read as zeros.
template <typename E, int D>
__global__ __launch_bounds__(256) void bwd_gather_kernel(BwdGatherArgs a) {
  __shared__ int s_tok[64];
  const int r0 = blockIdx.x * 64, unit = blockIdx.y;
  const int b = unit / a.Hq, hq = unit % a.Hq, kvh = a.map.kv[hq];
  if (threadIdx.x < 64) {
    const int e = r0 + threadIdx.x;
    int tok = e < a.nsel ? a.sel[(int64_t)unit * a.sel_stride + e] : -1;
    if (tok < 0 || tok >= a.N || tok / a.C != e / a.lam) tok = -1;
    s_tok[threadIdx.x] = tok;
    int times = 0;                       // entries of the chunk's list that name this token (more than one: the same key again)
    if (tok >= 0) {
      const int first = e / a.lam * a.lam, last = min(first + a.lam, a.nsel);
      const int32_t* list = a.sel + (int64_t)unit * a.sel_stride;
#pragma unroll 8
      for (int i = first; i < last; ++i) times += list[i] == tok;
    }
    a.times[(int64_t)unit * a.cap + e] = times;
    const unsigned long long bits = __ballot(tok >= 0);
    if (threadIdx.x == 0) a.rvalid[(int64_t)unit * (a.cap / 64) + blockIdx.x] = bits;
  }
  __syncthreads();
  constexpr int EPV = 16 / (int)sizeof(E), PPR = D / EPV;
  for (int idx = threadIdx.x; idx < 64 * PPR; idx += 256) {
    const int i = idx / PPR, x = (idx % PPR) * EPV, tok = s_tok[i];
    Vec16 kv, vv;
    kv.w[0] = kv.w[1] = kv.w[2] = kv.w[3] = 0u;
    vv = kv;
    if (tok >= 0) {
      kv = *reinterpret_cast<const Vec16*>(static_cast<const E*>(a.k) + b * a.k_sb + (int64_t)tok * a.k_st + kvh * a.k_sh + x);
      vv = *reinterpret_cast<const Vec16*>(static_cast<const E*>(a.v) + b * a.v_sb + (int64_t)tok * a.v_st + kvh * a.v_sh + x);
    }
    const int64_t o = ((int64_t)unit * a.cap + r0 + i) * D + x;
    *reinterpret_cast<Vec16*>(static_cast<E*>(a.kret) + o) = kv;
    *reinterpret_cast<Vec16*>(static_cast<E*>(a.vret) + o) = vv;
  }
}

// accumulators of a (channel x lane) product -> one fp32 row of the lane
template <typename T, int D>
__device__ __forceinline__ void store_row(float* row, const floatx16 (&acc)[D / 32], float scale, int g) {
  typedef Mma<T> M;
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      if constexpr (M::KPL == 8) {
        floatx4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = acc[dt][4 * i4 + e] * scale;
        *reinterpret_cast<floatx4*>(row + 32 * dt + M::pos_of_reg(4 * i4, g)) = x;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) row[32 * dt + M::pos_of_reg(4 * i4 + e, g)] = acc[dt][4 * i4 + e] * scale;
      }
    }
}

// ---------------------------------------------------------------------------------------------------------
// dq: one workgroup per 128 query rows of one (batch, query head), 64-key tiles (retained entries in routing order,
// then the local span), K and V tiles double-buffered.
// ---------------------------------------------------------------------------------------------------------
template <typename T, int D>
struct DqCfg {
  static constexpr int BM = 128, BN = 64, NW = 4;
  static constexpr int TE = BN * D;                                   // elements of one tile
  static constexpr int INSTR = TE * (int)sizeof(T) / 1024 / NW;       // direct-to-LDS requests per wave and tile
  static constexpr size_t smem = (size_t)4 * TE * sizeof(T);
};

template <typename T, int D>
__global__ __launch_bounds__(256, 2) void bwd_sa_dq_kernel(BwdSaArgs a) {
  typedef Mma<T> M;
  typedef RowTile<T, D> RT;
  typedef DqCfg<T, D> Cf;
  constexpr int KS = D / M::KK, DT = D / 32, SPT = M::STEPS_PER_TILE, BN = Cf::BN;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  T* Kl = reinterpret_cast<T*>(smem);
  T* Vl = Kl + 2 * Cf::TE;

  // units are dealt to the XCDs (their retained rows are re-read by every row tile), long tiles first
  int unit, tile;
  {
    const int L = blockIdx.x;
    if (a.U % 8 == 0) {
      const int xcd = L & 7, j = L >> 3;
      unit = (j / a.n_row_tiles) * 8 + xcd;
      tile = a.n_row_tiles - 1 - (j % a.n_row_tiles);
    } else {
      unit = L / a.n_row_tiles;
      tile = a.n_row_tiles - 1 - (L % a.n_row_tiles);
    }
  }
  const int b = unit / a.Hq, h = unit % a.Hq, kvh = a.map.kv[h];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, g = lane >> 5;
  const int N = a.N, C = a.C;
  const int row0 = tile * Cf::BM, q0 = row0 + 32 * wave, t = q0 + r;
  const bool active = q0 < N;
  const int cw = q0 / C;
  const int ret_w = retained_rows(cw >= 1 ? cw - 1 : 0, a.lam, a.rcap);
  const int lo_w = (cw >= 1 ? cw - 1 : 0) * C;
  const int c_first = row0 / C, last_row = min(row0 + Cf::BM, N) - 1, c_last = last_row / C;
  const int ret_max = retained_rows(c_last >= 1 ? c_last - 1 : 0, a.lam, a.rcap);
  const int loc_lo = (c_first >= 1 ? c_first - 1 : 0) * C;
  const int n_ret_tiles = (ret_max + BN - 1) / BN;
  const int n_tiles = n_ret_tiles + (last_row + 1 - loc_lo + BN - 1) / BN;

  const T* __restrict__ kloc = static_cast<const T*>(a.k) + b * a.k_sb + kvh * a.k_sh;
  const T* __restrict__ vloc = static_cast<const T*>(a.v) + b * a.v_sb + kvh * a.v_sh;
  const T* __restrict__ kret = static_cast<const T*>(a.kret) + (int64_t)unit * a.cap * D;
  const T* __restrict__ vret = static_cast<const T*>(a.vret) + (int64_t)unit * a.cap * D;
  const unsigned long long* __restrict__ rvalid = a.rvalid + (int64_t)unit * (a.cap / 64);

  auto tile_kb = [&](int ti) { return ti < n_ret_tiles ? ti * BN : loc_lo + (ti - n_ret_tiles) * BN; };
  auto request = [&](int ti) __attribute__((always_inline)) {
    const int kb = tile_kb(ti);
    const bool ret = ti < n_ret_tiles;
    T* kd = Kl + (ti & 1) * Cf::TE;
    T* vd = Vl + (ti & 1) * Cf::TE;
    const int lane_now = fresh_lane_id();
#pragma unroll
    for (int j = 0; j < Cf::INSTR; ++j) {
      const int piece = (wave + Cf::NW * j) * 64 + lane_now;
      const int row = piece / RT::PPR, col = ((piece % RT::PPR) ^ RT::swz(row)) * RT::EPV;
      const T *kp, *vp;
      if (ret) {
        kp = kret + (int64_t)(kb + row) * D + col;
        vp = vret + (int64_t)(kb + row) * D + col;
      } else {
        const int tok = min(kb + row, N - 1);      // past the end: the last token again (masked below)
        kp = kloc + (int64_t)tok * a.k_st + col;
        vp = vloc + (int64_t)tok * a.v_st + col;
      }
      async_copy16(kp, lds_address(kd + (wave + Cf::NW * j) * 64 * RT::EPV));
      async_copy16(vp, lds_address(vd + (wave + Cf::NW * j) * 64 * RT::EPV));
    }
  };

  const int tq = min(t, N - 1);
  typename M::frag qf[KS], dof[KS];
  {
    const T* qp = static_cast<const T*>(a.q) + b * a.q_sb + (int64_t)tq * a.q_st + h * a.q_sh + g * M::KPL;
    const T* dp = static_cast<const T*>(a.dout) + b * a.o_sb + (int64_t)tq * a.o_st + h * a.o_sh + g * M::KPL;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      qf[s] = M::load(qp + s * M::KK);
      dof[s] = M::load(dp + s * M::KK);
    }
  }
  const float nl2 = -a.lse[(int64_t)unit * N + tq] * kLog2e, delta = a.delta[(int64_t)unit * N + tq];
  const float sc2 = a.scale * kLog2e;
  floatx16 dq[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) dq[dt] = zero16();
  request(0);
#pragma unroll
  for (int s = 0; s < KS; ++s) asm volatile("" ::"v"(qf[s]), "v"(dof[s]));
  asm volatile("" ::"v"(nl2), "v"(delta));
  wait_async_copies();
  lds_barrier();

#pragma unroll 1
  for (int ti = 0; ti < n_tiles; ++ti) {
    if (ti + 1 < n_tiles) request(ti + 1);
    const int kb = tile_kb(ti);
    const bool ret = ti < n_ret_tiles;
    // what this wave sees of the tile (uniform): nothing, all of it, or a part
    bool live = active, full = true;
    unsigned long long bits = ~0ull;
    if (ret) {
      live = live && kb < ret_w;
      bits = rvalid[ti];
      if (ret_w - kb < 64 && ret_w > kb) bits &= (1ull << (ret_w - kb)) - 1ull;
      full = bits == ~0ull;
      live = live && bits != 0ull;
    } else {
      live = live && kb + BN - 1 >= lo_w && kb <= q0 + 31;
      full = kb >= lo_w && kb + BN - 1 <= q0;
    }
    if (live) {
      const T* Ks = Kl + (ti & 1) * Cf::TE;
      const T* Vs = Vl + (ti & 1) * Cf::TE;
      const int lane_now = fresh_lane_id(), rr = lane_now & 31, gg = lane_now >> 5;   // (addresses live in this trip only)
      typename M::frag df[2][SPT];
      // one half of the tile at a time: logits and dP of 32 keys, then their dS as operand fragments (both halves at
      // once would need 32 more registers than two waves per SIMD leave)
      static_for<2>([&](auto MT) __attribute__((always_inline)) {
        constexpr int mt = decltype(MT)::value;
        floatx16 st = zero16(), dp = zero16();
        piped<typename M::frag, 2 * KS, 6>(
            [&](auto I) __attribute__((always_inline)) {
              constexpr int i = decltype(I)::value;
              return RT::along((i & 1) ? Vs : Ks, 32 * mt + M::kappa(rr), i >> 1, gg);
            },
            [&](auto I, const typename M::frag& f) __attribute__((always_inline)) {
              constexpr int i = decltype(I)::value, s = i >> 1;
              if constexpr ((i & 1) == 0) st = M::mma(f, qf[s], st);
              else dp = M::mma(f, dof[s], dp);
            });
#pragma unroll
        for (int i = 0; i < 16; ++i) st[i] = fast_exp2(fmaf(st[i], sc2, nl2)) * (dp[i] - delta);
        if (!full) {
          const uint32_t half = (uint32_t)(mt ? bits >> 32 : bits);
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int pos = M::pos_of_reg(i, gg), key = kb + 32 * mt + pos;
            const bool vis = ret ? ((half >> pos) & 1u) != 0u : (key >= lo_w && key <= t);
            st[i] = vis ? st[i] : 0.f;
          }
        }
#pragma unroll
        for (int s = 0; s < SPT; ++s) df[mt][s] = M::from_acc(st, s);
      });
      piped<typename M::frag, 2 * SPT * DT, 6>(
          [&](auto I) __attribute__((always_inline)) {
            constexpr int i = decltype(I)::value, ms = i / DT;
            return RT::down(Ks, 32 * (ms / SPT) + (ms % SPT) * M::KK, 32 * (i % DT), lane_now);
          },
          [&](auto I, const typename M::frag& f) __attribute__((always_inline)) {
            constexpr int i = decltype(I)::value, ms = i / DT;
            dq[i % DT] = M::mma(f, df[ms / SPT][ms % SPT], dq[i % DT]);
          });
    }
    wait_async_copies();
    lds_barrier();
  }
  if (t < N) store_row<T, D>(a.dq32 + ((int64_t)unit * N + t) * D, dq, a.scale, g);
}

// ---------------------------------------------------------------------------------------------------------
// dk, dv: one workgroup per 128 keys, one wave per 32 of them (keys in registers, values in LDS: both in registers
// would not fit next to the accumulators of dk and dv), walking the 32-row tiles that see them.
// LOCAL: keys are tokens of one (batch, kv head); the workgroup walks the query heads that read this kv head one after
// the other, so the sums over the group stay in the accumulators and every row is stored once.
// !LOCAL: keys are retained entries of one (batch, query head); their rows go to a buffer in routing order, which the finishing kernel
// reads at the entries' tokens (added atomically from here they took 0.4 to 0.7 ms of the training shape's call, more
// than the products).
// ---------------------------------------------------------------------------------------------------------
template <typename T, int D>
struct DkvCfg {
  static constexpr int BK = 128, RB = 32, NW = 4;
  static constexpr int TE = RB * D;                                   // elements of one row tile
  static constexpr int INSTR = TE * (int)sizeof(T) / 1024 / NW;       // requests per wave and row tile
  static constexpr size_t smem = ((size_t)4 * TE + (size_t)BK * D) * sizeof(T) + 2 * 64 * sizeof(float);
};

template <typename T, int D, bool LOCAL>
__global__ __launch_bounds__(256, 2) void bwd_sa_dkv_kernel(BwdSaArgs a) {
  typedef Mma<T> M;
  typedef RowTile<T, D> RT;
  typedef DkvCfg<T, D> Cf;
  constexpr int KS = D / M::KK, DT = D / 32, SPT = M::STEPS_PER_TILE, RB = Cf::RB;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  T* Ql = reinterpret_cast<T*>(smem);                                 // two row tiles of q
  T* Ol = Ql + 2 * Cf::TE;                                            // two row tiles of dout
  T* Vl = Ol + 2 * Cf::TE;                                            // the workgroup's 128 value rows
  float* stats = reinterpret_cast<float*>(Vl + Cf::BK * D);           // [2][64]: lse and delta of the tile's 32 rows

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, g = lane >> 5;
  const int N = a.N, C = a.C;
  int b, kvh, h_first, ti;
  if (LOCAL) {
    ti = blockIdx.x;
    b = blockIdx.y / a.Hkv;
    kvh = blockIdx.y % a.Hkv;
    h_first = 0;
    while (h_first < a.Hq && a.map.kv[h_first] != kvh) ++h_first;
  } else {
    ti = blockIdx.x;                                                  // the first entries have the most rows
    b = blockIdx.y / a.Hq;
    h_first = blockIdx.y % a.Hq;
    kvh = a.map.kv[h_first];
  }
  const int k0 = ti * Cf::BK, kw = k0 + 32 * wave, key = kw + r;      // this lane's key (token or retained entry)
  int row_lo, row_hi;                                                 // rows that may see a key of this workgroup
  if (LOCAL) {
    row_lo = k0;
    row_hi = min(N, (min(k0 + Cf::BK, N) - 1) / C * C + 2 * C);
  } else {
    row_lo = (k0 / a.lam + 2) * C;
    row_hi = N;
  }
  const int64_t unit0 = (int64_t)b * a.Hq + h_first;                  // (!LOCAL: the unit)
  int tok;                                                            // LOCAL: token, !LOCAL: its other occurrences; -1: no key here
  const T *kp, *vbase;
  int64_t v_row;
  if (LOCAL) {
    tok = key < N ? key : -1;
    kp = static_cast<const T*>(a.k) + b * a.k_sb + (int64_t)min(key, N - 1) * a.k_st + kvh * a.k_sh;
    vbase = static_cast<const T*>(a.v) + b * a.v_sb + kvh * a.v_sh;
    v_row = a.v_st;
  } else {
    tok = a.times[unit0 * a.cap + key] - 1;
    kp = static_cast<const T*>(a.kret) + (unit0 * a.cap + key) * D;
    vbase = static_cast<const T*>(a.vret) + unit0 * a.cap * D;
    v_row = D;
  }
  const bool any_rows = LOCAL ? h_first < a.Hq : row_lo < row_hi;     // uniform
  floatx16 dk[DT], dv[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) dk[dt] = dv[dt] = zero16();

  if (any_rows) {
    // values of the wave's own keys -> LDS
#pragma unroll
    for (int j = 0; j < RB * RT::PPR / 64; ++j) {
      const int piece = j * 64 + lane, row = piece / RT::PPR, col = ((piece % RT::PPR) ^ RT::swz(row)) * RT::EPV;
      int vr = kw + row;
      if (LOCAL) vr = min(vr, N - 1);
      async_copy16(vbase + (int64_t)vr * v_row + col, lds_address(Vl + (32 * wave) * D + j * 64 * RT::EPV));
    }
    auto request = [&](int h, int r0, int buf) __attribute__((always_inline)) {
      const T* qb = static_cast<const T*>(a.q) + b * a.q_sb + h * a.q_sh;
      const T* ob = static_cast<const T*>(a.dout) + b * a.o_sb + h * a.o_sh;
      const int lane_now = fresh_lane_id();
#pragma unroll
      for (int j = 0; j < Cf::INSTR; ++j) {
        const int piece = (wave + Cf::NW * j) * 64 + lane_now;
        const int row = piece / RT::PPR, col = ((piece % RT::PPR) ^ RT::swz(row)) * RT::EPV;
        const int tr = min(r0 + row, N - 1);
        async_copy16(qb + (int64_t)tr * a.q_st + col, lds_address(Ql + buf * Cf::TE + (wave + Cf::NW * j) * 64 * RT::EPV));
        async_copy16(ob + (int64_t)tr * a.o_st + col, lds_address(Ol + buf * Cf::TE + (wave + Cf::NW * j) * 64 * RT::EPV));
      }
      if (wave == 0) {
        const int64_t o = ((int64_t)b * a.Hq + h) * N + min(r0 + (lane_now & 31), N - 1);
        async_copy4((lane_now < 32 ? a.lse : a.delta) + o, lds_address(stats + 64 * buf));
      }
    };
    typename M::frag kf[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) kf[s] = M::load(kp + g * M::KPL + s * M::KK);
    const float sc2 = a.scale * kLog2e;
    int h = h_first, r0 = row_lo, buf = 0;
    request(h, r0, 0);
#pragma unroll
    for (int s = 0; s < KS; ++s) asm volatile("" ::"v"(kf[s]));
    asm volatile("" ::"v"(tok));
    wait_async_copies();
    lds_barrier();
    while (true) {
      // the next row tile (uniform)
      int hn = h, rn = r0 + RB;
      if (rn >= row_hi) {
        rn = row_lo;
        hn = a.Hq;
        if (LOCAL)
          for (hn = h + 1; hn < a.Hq && a.map.kv[hn] != kvh; ++hn) {}
      }
      const bool more = hn < a.Hq;
      if (more) request(hn, rn, buf ^ 1);

      const int c = r0 / C, lo = (c >= 1 ? c - 1 : 0) * C;
      const int n_vis = retained_rows(c >= 1 ? c - 1 : 0, a.lam, a.rcap);
      bool live, full;
      if (LOCAL) {
        live = kw < N && kw <= r0 + RB - 1 && kw + 31 >= lo;
        full = kw >= lo && kw + 31 <= r0 && r0 + RB <= N;
      } else {
        live = kw < n_vis;
        full = kw + 32 <= n_vis && r0 + RB <= N && __all(tok >= 0);
      }
      if (live) {
        const T* Qs = Ql + buf * Cf::TE;
        const T* Os = Ol + buf * Cf::TE;
        const T* Vs = Vl + 32 * wave * D;
        floatx16 s16 = zero16(), d16 = zero16();
        struct Pair {
          typename M::frag x, y;
        };
        piped<Pair, KS, 3>(
            [&](auto I) __attribute__((always_inline)) {
              constexpr int s = decltype(I)::value;
              return Pair{RT::along(Qs, M::kappa(r), s, g), RT::along(Os, M::kappa(r), s, g)};
            },
            [&](auto I, const Pair& f) __attribute__((always_inline)) {
              constexpr int s = decltype(I)::value;
              s16 = M::mma(f.x, kf[s], s16);
              d16 = M::mma(f.y, RT::along(Vs, r, s, g), d16);
            });
        const float* ls = stats + 64 * buf;
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          float lv[4], dl[4];
          if constexpr (M::KPL == 8) {
            const floatx4 x = *reinterpret_cast<const floatx4*>(ls + M::pos_of_reg(4 * i4, g));
            const floatx4 y = *reinterpret_cast<const floatx4*>(ls + 32 + M::pos_of_reg(4 * i4, g));
#pragma unroll
            for (int e = 0; e < 4; ++e) lv[e] = x[e], dl[e] = y[e];
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              lv[e] = ls[M::pos_of_reg(4 * i4 + e, g)];
              dl[e] = ls[32 + M::pos_of_reg(4 * i4 + e, g)];
            }
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int i = 4 * i4 + e;
            float p = fast_exp2(fmaf(s16[i], sc2, -lv[e] * kLog2e));
            if (!full) {
              const int t = r0 + M::pos_of_reg(i, g);
              const bool vis = LOCAL ? (tok >= lo && tok <= t && t < N) : (tok >= 0 && key < n_vis && t < N);
              p = vis ? p : 0.f;
            }
            s16[i] = p;
            d16[i] = p * (d16[i] - dl[e]);
          }
        }
        typename M::frag pf[SPT], sf[SPT];
#pragma unroll
        for (int s = 0; s < SPT; ++s) {
          pf[s] = M::from_acc(s16, s);
          sf[s] = M::from_acc(d16, s);
        }
        piped<typename M::frag, 2 * SPT * DT, 5>(
            [&](auto I) __attribute__((always_inline)) {
              constexpr int i = decltype(I)::value, dt = (i >> 1) % DT, s = (i >> 1) / DT;
              return RT::down((i & 1) ? Qs : Os, s * M::KK, 32 * dt, lane);
            },
            [&](auto I, const typename M::frag& f) __attribute__((always_inline)) {
              constexpr int i = decltype(I)::value, dt = (i >> 1) % DT, s = (i >> 1) / DT;
              if constexpr ((i & 1) == 0) dv[dt] = M::mma(f, pf[s], dv[dt]);
              else dk[dt] = M::mma(f, sf[s], dk[dt]);
            });
      }
      wait_async_copies();
      lds_barrier();
      if (!more) break;
      h = hn;
      r0 = rn;
      buf ^= 1;
    }
  }
  if (LOCAL) {
    if (tok >= 0) {
      const int64_t o = (((int64_t)b * a.Hkv + kvh) * N + tok) * D;
      store_row<T, D>(a.dk32 + o, dk, a.scale, g);
      store_row<T, D>(a.dv32 + o, dv, 1.f, g);
    }
  } else {
    const int64_t o = (unit0 * a.cap + key) * D;   // (the capacity covers the last tile)
    const float times = (float)(tok + 1);          // equal keys have equal gradients, and one of them is added per token
    store_row<T, D>(a.dkret + o, dk, a.scale * times, g);
    store_row<T, D>(a.dvret + o, dv, times, g);
  }
}

template <typename K>
hipError_t allow_lds(K kern, size_t smem) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
}

template <typename T, int D>
hipError_t launch_dq_t(const BwdSaArgs& a, hipStream_t s) {
  auto kq = bwd_sa_dq_kernel<T, D>;
  const hipError_t e = allow_lds(kq, DqCfg<T, D>::smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kq, dim3((unsigned)a.n_row_tiles * a.U), dim3(256), (DqCfg<T, D>::smem), s, a);
  return hipGetLastError();
}

template <typename T, int D>
hipError_t launch_dkv_t(const BwdSaArgs& a, int B, hipStream_t s) {
  constexpr size_t smem = DkvCfg<T, D>::smem;
  auto kl = bwd_sa_dkv_kernel<T, D, true>;
  hipError_t e = allow_lds(kl, smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kl, dim3((a.N + 127) / 128, B * a.Hkv), dim3(256), smem, s, a);
  if ((e = hipGetLastError()) != hipSuccess || a.n_ret_tiles == 0) return e;
  auto kr = bwd_sa_dkv_kernel<T, D, false>;
  if ((e = allow_lds(kr, smem)) != hipSuccess) return e;
  hipLaunchKernelGGL(kr, dim3(a.n_ret_tiles, a.U), dim3(256), smem, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_bwd_gather(const BwdGatherArgs& a, int dtype, int U, hipStream_t s) {
  if (a.cap == 0 || a.lam <= 0) return hipSuccess;
  const dim3 grid(a.cap / 64, U);
  if (dtype == 1) {
    if (a.d == 64) hipLaunchKernelGGL((bwd_gather_kernel<uint16_t, 64>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((bwd_gather_kernel<uint16_t, 128>), grid, dim3(256), 0, s, a);
  } else {
    hipLaunchKernelGGL((bwd_gather_kernel<uint32_t, 64>), grid, dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

// (fp32 is built for d = 64 only; the host checks refuse the rest)
hipError_t launch_bwd_sa_dq(const BwdSaArgs& a, int dtype, int d, hipStream_t s) {
  if (dtype == 1) return d == 128 ? launch_dq_t<bf16, 128>(a, s) : launch_dq_t<bf16, 64>(a, s);
  return d == 64 ? launch_dq_t<float, 64>(a, s) : hipErrorInvalidValue;
}

hipError_t launch_bwd_sa_dkv(const BwdSaArgs& a, int dtype, int d, int B, hipStream_t s) {
  if (dtype == 1) return d == 128 ? launch_dkv_t<bf16, 128>(a, B, s) : launch_dkv_t<bf16, 64>(a, B, s);
  return d == 64 ? launch_dkv_t<float, 64>(a, B, s) : hipErrorInvalidValue;
}

}  // namespace still
