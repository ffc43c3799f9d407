// Attention map of the operator and its backward pass to the feature-map parameters (gfx950).
//
// A[t][j] is the weight of v_j in row t under the shared normaliser (what the first training stage of Sec. 4.1 compares
// with the teacher's softmax map): exp(scale q_t.k_j - L_t) for the local span and for selected tokens of chunks <= c-2,
// E_t phi_q(t).phi_k(j) with E_t = exp(-L_t) for the other tokens of those chunks, zero above the diagonal.  Backward,
// with q, k and the routing fixed, only the pairs of the second kind count:
//   rho_t = <dA_t, A_t>,  w_tj = (dA_tj - rho_t) E_t on those pairs,  dphi_q(t) = sum_j w_tj phi_k(j),
//   dphi_k(j) = sum_t w_tj phi_q(t),  then the NP-Map backwards to df, and dW = x^T df (still_bwd_lin.hip).
//
// Everything is bound by the N x N fp32 matrices: the map is written once, read once (rho), dA read three times (rho, and
// either side's products; the query side's second read finds it in the last-level cache).  So: one launch for the
// features of both sides, one that writes the map, one per side of the backward pass, in which w goes from dA to operand
// registers and f, u, dphi and df stay on the chip.
// Measured at 4 sequences of 1024 tokens, 32 / 8 heads, d = 128, C = 64, bf16 (forward call included): as batched products
// through memory, with w as a matrix of its own and the operands fetched 32 cache lines per instruction, 2.95 ms; now 1.12
// ms, and 0.91 with no choice per entry and no wait inside the loops' loads (features 0.06 twice; map 0.21 -> 0.19: 2.8 TB/s
// of stores; query side 0.34 -> 0.24, a third of it the row sums, which read map and gradient at 6 TB/s; key side 0.21 -> 0.125;
// parameter gradients 0.07).  What is left there is one tile in flight per workgroup and the features' trips through memory.
#include "still_kernels.h"
#include "still_tile.h"

namespace still {

namespace {

typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));   // (rows of an N x N matrix start anywhere)

template <typename T, int D>
struct MapCfg {
  typedef RowTile<T, D> RX;              // token rows
  typedef RowTile<T, 2 * D> RP;          // their features
  static constexpr int XE = 64 * D, PE = 64 * 2 * D;
  static constexpr size_t x_bytes = XE * sizeof(T), phi_bytes = PE * sizeof(T);
  static constexpr size_t xch_bytes = 2 * 64 * 4 * 4;
  static constexpr size_t phi_smem = x_bytes + phi_bytes + xch_bytes;
  static constexpr size_t map_smem = x_bytes + phi_bytes;
  static constexpr size_t bwd_smem = 2 * phi_bytes + xch_bytes + 2 * 2 * 64 * 4;   // + (rho, E) of two tiles
};

// 64 rows of W elements, from row0 on (past the end the last one again), on their way into an LDS row tile
template <typename T, int W>
__device__ __forceinline__ void request_rows(const T* base, int64_t stride, int row0, int n, T* tile, int wave) {
  typedef RowTile<T, W> RT;
  const int lane_now = fresh_lane_id();
#pragma unroll
  for (int j = 0; j < 64 * W * (int)sizeof(T) / 4096; ++j) {
    const int piece = (wave + 4 * j) * 64 + lane_now, row = piece / RT::PPR;
    const int col = ((piece % RT::PPR) ^ RT::swz(row)) * RT::EPV;
    async_copy16(base + (int64_t)min(row0 + row, n - 1) * stride + col, lds_address(tile + (wave + 4 * j) * 64 * RT::EPV));
  }
}

// The same for 64 rows that exist and lie one behind the other: a wave's copies are 4 KB apart in memory as in LDS, so one lane
// offset on a scalar base serves them all (8 rows on, bit 1 of the swizzle alternates).
template <typename T, int W>
__device__ __forceinline__ void request_run(const T* base, T* tile, int wave) {
  typedef RowTile<T, W> RT;
  constexpr int ROWS = 256 / RT::PPR;
  static_assert(ROWS == 8 || ROWS == 16, "whole periods of the swizzle, or half of one");
  const int piece = wave * 64 + fresh_lane_id(), row = piece / RT::PPR;
  const uint32_t off = (uint32_t)row * (W * sizeof(T)) + 16u * ((piece % RT::PPR) ^ RT::swz(row));
  const uint32_t dst = lds_address(tile) + 1024 * wave;
  static_for<64 * W * (int)sizeof(T) / 4096>([&](auto J) __attribute__((always_inline)) {
    constexpr int j = decltype(J)::value;
    async_copy16_at<4096 * j>(base, (ROWS == 8 && (j & 1) ? off ^ 32u : off) + 4096 * j, dst);
  });
}

// The NP-Map of 64 tokens whose rows are in LDS: wave (rg, fh) has the features 64 j + 32 fh + (0..31) of the tokens
// 32 rg + lane.  u = f |x| / |f|; the halves of phi are exp2(+-u log2 e - m) * i.
template <typename T, int D>
struct NpMap {
  typedef Mma<T> M;
  static constexpr int NF = D / 64, KS = D / M::KK;
  floatx16 u[NF];
  float nx, nf, ratio, mp, mn, ip, in;

  // (every wave has read the rows once this returns)
  __device__ __forceinline__ void forward(const T* xl, const T* wf, const T* bias, int row, int fh, int lane, float* xch) {
    typedef RowTile<T, D> RX;
    const int g = lane >> 5;
    typename M::frag xf[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) xf[s] = RX::along(xl, row, s, g);
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
    const float nx2 = sum32((n4[0] + n4[1]) + (n4[2] + n4[3]));
    if (bias != nullptr) {
#pragma unroll
      for (int j = 0; j < NF; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) u[j][i] += to_f32(bias[64 * j + 32 * fh + M::pos_of_reg(i, g)]);
    }
    float* my = xch + (fh * 64 + row) * 4;
    const float* other = xch + ((fh ^ 1) * 64 + row) * 4;
    float nf2 = 0.f, mx = -INFINITY, mi = INFINITY;
#pragma unroll
    for (int j = 0; j < NF; ++j)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        nf2 = fmaf(u[j][i], u[j][i], nf2);
        mx = fmaxf(mx, u[j][i]);
        mi = fminf(mi, u[j][i]);
      }
    nf2 = sum32(nf2);
    mx = max32(mx);
    mi = min32(mi);
    if (g == 0) my[0] = nf2, my[1] = mx, my[2] = mi;
    lds_barrier();
    nf2 += other[0];
    mx = fmaxf(mx, other[1]);
    mi = fminf(mi, other[2]);
    nx = sqrtf(nx2);
    nf = sqrtf(nf2);
    ratio = nf2 > 0.f ? nx / nf : 0.f;
    mp = mx * ratio * kLog2e;
    mn = -mi * ratio * kLog2e;
    float sp = 0.f, sn = 0.f;
#pragma unroll
    for (int j = 0; j < NF; ++j)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        u[j][i] *= ratio;
        sp += pos(j, i);
        sn += neg(j, i);
      }
    sp = sum32(sp);
    sn = sum32(sn);
    lds_barrier();                       // (the first exchange has been read)
    if (g == 0) my[0] = sp, my[1] = sn;
    lds_barrier();
    ip = 1.f / (sp + other[0]);
    in = 1.f / (sn + other[1]);
  }
  __device__ __forceinline__ float pos(int j, int i) const { return fast_exp2(fmaf(u[j][i], kLog2e, -mp)); }
  __device__ __forceinline__ float neg(int j, int i) const { return fast_exp2(fmaf(u[j][i], -kLog2e, -mn)); }
};

// does the softmax branch keep token t, of chunk c (a full one), of this (batch, query head)?
__device__ __forceinline__ bool kept_token(const uint32_t* kmask, int64_t unit, int ncf, int C, int c, int t) {
  const int w = t - c * C;
  return (kmask[(unit * ncf + c) * (C / 32) + w / 32] >> (w & 31)) & 1u;
}

// ---------------------------------------------------------------- features of both sides
template <typename T, int D>
__global__ __launch_bounds__(256) void map_phi_kernel(MapArgs a) {
  typedef MapCfg<T, D> Cf;
  typedef typename Cf::RP RP;
  typedef NpMap<T, D> Np;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  T* xl = reinterpret_cast<T*>(smem);
  T* phi = reinterpret_cast<T*>(smem + Cf::x_bytes);
  float* xch = reinterpret_cast<float*>(smem + Cf::x_bytes + Cf::phi_bytes);
  const bool key = blockIdx.y != 0;
  const int n_tiles = (a.N + 63) / 64, tile = blockIdx.x % n_tiles;
  const int64_t unit = blockIdx.x / n_tiles;
  const int b = (int)(unit / a.Hq), hq = (int)(unit % a.Hq);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 5, rg = wave & 1, fh = wave >> 1, row = 32 * rg + (lane & 31);
  const int t0 = tile * 64, t = min(t0 + row, a.N - 1), c = t0 / a.C;
  const T* x = key ? static_cast<const T*>(a.k) + b * a.k_sb + a.map.kv[hq] * a.k_sh
                   : static_cast<const T*>(a.q) + b * a.q_sb + hq * a.q_sh;
  const T* bias = static_cast<const T*>(key ? a.bk : a.bq);
  request_rows<T, D>(x, key ? a.k_st : a.q_st, t0, a.N, xl, wave);
  wait_async_copies();
  lds_barrier();
  Np np;
  np.forward(xl, static_cast<const T*>(key ? a.wkf : a.wqf) + (int64_t)hq * D * D,
             bias != nullptr ? bias + (int64_t)hq * D : nullptr, row, fh, lane, xch);
  const bool kept = key && c < a.ncf && kept_token(a.kmask, unit, a.ncf, a.C, c, t);
#pragma unroll
  for (int j = 0; j < Np::NF; ++j) {
    float p[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) p[i] = kept ? 0.f : np.pos(j, i) * np.ip;
    put_row<T, 2 * D>(phi, row, 64 * j + 32 * fh, p, g);
#pragma unroll
    for (int i = 0; i < 16; ++i) p[i] = kept ? 0.f : np.neg(j, i) * np.in;
    put_row<T, 2 * D>(phi, row, D + 64 * j + 32 * fh, p, g);
  }
  lds_barrier();
  T* dst = static_cast<T*>(key ? a.phi_k : a.phi_q) + (unit * a.N + t0) * 2 * D;
  for (int i = threadIdx.x; i < 64 * RP::PPR; i += 256) {
    const int ri = i / RP::PPR, e0 = (i % RP::PPR) * RP::EPV;
    if (t0 + ri < a.N) *reinterpret_cast<Vec16*>(dst + (int64_t)ri * 2 * D + e0) = *reinterpret_cast<const Vec16*>(phi + RP::off(ri, e0));
  }
}

// blockIdx -> (unit, tile), the tiles of a unit on one XCD (they read one side's features again and again)
__device__ __forceinline__ void unit_and_tile(int L, int U, int n_tiles, int64_t& unit, int& tile) {
  if (U % 8 == 0) {
    const int j = L >> 3;
    unit = (int64_t)(j / n_tiles) * 8 + (L & 7);
    tile = j % n_tiles;
  } else {
    unit = L / n_tiles;
    tile = L % n_tiles;
  }
}

// ---------------------------------------------------------------- the map
// One workgroup per 64 rows, whose q and phi_q stay in registers as operands; wave (rg, kh) takes 32 rows and 32 keys of
// every tile of 64.  A tile lies in one chunk and so do the rows, so which branch owns it is uniform: the local span
// needs the logits only.  Above the diagonal the rows are filled with zeros.
template <typename T, int D>
__global__ __launch_bounds__(256, 2) void attn_map_kernel(MapArgs a) {
  typedef Mma<T> M;
  typedef MapCfg<T, D> Cf;
  typedef typename Cf::RX RX;
  typedef typename Cf::RP RP;
  constexpr int KS = D / M::KK, KP = 2 * KS;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  T* Kl = reinterpret_cast<T*>(smem);
  T* Pl = reinterpret_cast<T*>(smem + Cf::x_bytes);
  const int n_tiles = (a.N + 63) / 64;
  int64_t unit;
  int rt;
  unit_and_tile(blockIdx.x, a.U, n_tiles, unit, rt);
  rt = n_tiles - 1 - rt;                 // long rows first
  const int b = (int)(unit / a.Hq), hq = (int)(unit % a.Hq), kvh = a.map.kv[hq];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, g = lane >> 5, rg = wave & 1, kh = wave >> 1;
  const int N = a.N, C = a.C, r0 = rt * 64, c = r0 / C;
  float* out = a.map_out + unit * N * (int64_t)N;
  const T* kb = static_cast<const T*>(a.k) + b * a.k_sb + kvh * a.k_sh;
  const T* pk = static_cast<const T*>(a.phi_k) + unit * N * (2 * D);
  typename M::frag qf[KS], pf[KP];
  {
    const int tr = min(r0 + 32 * rg + r, N - 1);
    const T* qp = static_cast<const T*>(a.q) + b * a.q_sb + (int64_t)tr * a.q_st + hq * a.q_sh + g * M::KPL;
    const T* pq = static_cast<const T*>(a.phi_q) + (unit * N + tr) * (2 * D) + g * M::KPL;
#pragma unroll
    for (int s = 0; s < KS; ++s) qf[s] = M::load(qp + s * M::KK);
#pragma unroll
    for (int s = 0; s < KP; ++s) pf[s] = M::load(pq + s * M::KK);
  }
  float l2[16], el[16];                  // L_t log2 e and E_t of the lane's rows
#pragma unroll
  for (int i = 0; i < 16; ++i) l2[i] = a.lse[unit * N + min(r0 + 32 * rg + c_row(i, g), N - 1)] * kLog2e;
#pragma unroll
  for (int i = 0; i < 16; ++i) el[i] = fast_exp2(-l2[i]);
  const float sc2 = a.scale * kLog2e;
#pragma unroll 1
  for (int kt = 0; kt <= rt; ++kt) {
    const int k0 = 64 * kt, cj = k0 / C;
    const bool far = cj <= c - 2;        // (chunks <= c-2 are full chunks)
    lds_barrier();                       // everybody is done with the previous tile
    request_rows<T, D>(kb, a.k_st, k0, N, Kl, wave);
    if (far) request_run<T, 2 * D>(pk + (int64_t)k0 * (2 * D), Pl, wave);
    wait_async_copies();
    lds_barrier();
    const int lane_now = fresh_lane_id(), rr = lane_now & 31, gg = lane_now >> 5;
    const int j = k0 + 32 * kh + rr;
    floatx16 s = zero16(), w = zero16();
    piped<typename M::frag, KS, 4>([&](auto I) __attribute__((always_inline)) { return RX::along(Kl, 32 * kh + rr, decltype(I)::value, gg); },
                                   [&](auto I, const typename M::frag& f) __attribute__((always_inline)) { s = M::mma(qf[decltype(I)::value], f, s); });
    bool kept = true;
    if (far) {
      piped<typename M::frag, KP, 4>([&](auto I) __attribute__((always_inline)) { return RP::along(Pl, 32 * kh + rr, decltype(I)::value, gg); },
                                     [&](auto I, const typename M::frag& f) __attribute__((always_inline)) { w = M::mma(pf[decltype(I)::value], f, w); });
      kept = kept_token(a.kmask, unit, a.ncf, C, cj, j);
    }
    // (whole tiles below the diagonal are stored without a test per entry)
    const bool inner = kt < rt && r0 + 64 <= N;
    float* op = out + (int64_t)(r0 + 32 * rg + 4 * gg) * N + j;          // row c_row(i, gg) lies 8 (i / 4) + i % 4 rows on
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float own = fast_exp2(fmaf(s[i], sc2, -l2[i])), lin = el[i] * w[i];
      s[i] = kept ? own : lin;
    }
    if (inner) {
#pragma unroll
      for (int i = 0; i < 16; ++i) op[(int64_t)(8 * (i / 4) + i % 4) * N] = s[i];
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int t = r0 + 32 * rg + c_row(i, gg);
        if (t < N && j < N) op[(int64_t)(8 * (i / 4) + i % 4) * N] = j <= t ? s[i] : 0.f;
      }
    }
  }
  const int z0 = r0 + 64, zn = N - z0;
  for (int ri = wave; ri < 64 && zn > 0; ri += 4) {
    float* p = out + (int64_t)(r0 + ri) * N + z0;   // (zn > 0: all 64 rows exist)
    for (int i = 4 * lane; i + 3 < zn; i += 256) *reinterpret_cast<floatx4u*>(p + i) = floatx4u{0.f, 0.f, 0.f, 0.f};
    if (lane < (zn & 3)) p[(zn & ~3) + lane] = 0.f;
  }
}

// ---------------------------------------------------------------- backward, one side
// A workgroup takes 64 tokens from their rows to df.  dphi^T = phi_other^T w: the other side's features pass through LDS
// in tiles of 64 tokens and are read down their columns, w comes straight from dA: on the query side a lane owns a row
// and reads 8 consecutive keys, on the key side it owns a key and the 32 lanes of a load read one piece of a row.
template <typename T, int D, bool KEY>
__global__ __launch_bounds__(256, 2) void map_bwd_kernel(MapArgs a) {
  typedef Mma<T> M;
  typedef MapCfg<T, D> Cf;
  typedef typename Cf::RX RX;
  typedef typename Cf::RP RP;
  typedef NpMap<T, D> Np;
  constexpr int NF = Np::NF, NS = 2 * NF, SK = 64 / M::KK, KPL = M::KPL;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  T* phi = reinterpret_cast<T*>(smem);   // two tiles of the other side's features
  T* xl = phi + Cf::PE;                  // the token rows, before the loop; df after it
  float* xch = reinterpret_cast<float*>(smem + 2 * Cf::phi_bytes);
  float* re = xch + 2 * 64 * 4;          // [tile parity][rho, E][64]; E = 0: no such row
  const int N = a.N, C = a.C, n_tiles = (N + 63) / 64;
  int64_t unit;
  int tile;
  unit_and_tile(blockIdx.x, a.U, n_tiles, unit, tile);
  if (!KEY) tile = n_tiles - 1 - tile;   // the long ones first
  const int b = (int)(unit / a.Hq), hq = (int)(unit % a.Hq);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, g = lane >> 5, rg = wave & 1, fh = wave >> 1, row = 32 * rg + r;
  const int t0 = tile * 64, c = t0 / C, t = min(t0 + row, N - 1);
  T* dfg = static_cast<T*>(KEY ? a.dfk : a.dfq) + (unit * N + t0) * D;
  if (KEY ? (c >= a.ncf || c + 2 >= a.nc) : c < 2) {    // these tokens are in no pair of the linear branch
    Vec16 z16;
    z16.w[0] = z16.w[1] = z16.w[2] = z16.w[3] = 0u;
    for (int i = tid; i < 64 * RX::PPR; i += 256)
      if (t0 + i / RX::PPR < N) *reinterpret_cast<Vec16*>(dfg + (int64_t)i * RX::EPV) = z16;
    return;
  }
  const int o_beg = KEY ? (c + 2) * C / 64 : 0, o_end = KEY ? n_tiles : (c - 1) * C / 64;   // tiles of the other side
  const T* po = static_cast<const T*>(KEY ? a.phi_q : a.phi_k) + unit * N * (2 * D);
  const float* dA = a.dmap + unit * N * (int64_t)N;
  const T* x = KEY ? static_cast<const T*>(a.k) + b * a.k_sb + a.map.kv[hq] * a.k_sh
                   : static_cast<const T*>(a.q) + b * a.q_sb + hq * a.q_sh;
  const T* bias = static_cast<const T*>(KEY ? a.bk : a.bq);
  request_rows<T, D>(x, KEY ? a.k_st : a.q_st, t0, N, xl, wave);
  request_rows<T, 2 * D>(po, 2 * D, 64 * o_beg, N, phi, wave);

  float rho = 0.f, E = 0.f;              // query side: of this lane's row
  if constexpr (!KEY) {                  // rho_t over the keys up to t: eight rows of a wave at a time, all their loads in flight
    constexpr int RH = 8;
    const float* A = a.map_in + unit * N * (int64_t)N;
#pragma unroll 1
    for (int r0 = 16 * wave; r0 < 16 * wave + 16; r0 += RH) {
      const int t_lo = min(t0 + r0, N - 1), full = (t_lo + 1) & ~255;   // columns all the rows have, in pieces of 256
      float acc[RH];
      const float *pa[RH], *pd[RH];
#pragma unroll
      for (int h = 0; h < RH; ++h) {
        acc[h] = 0.f;
        const int64_t o = (int64_t)min(t_lo + h, N - 1) * N;
        pa[h] = A + o;
        pd[h] = dA + o;
      }
#pragma unroll 1
      for (int j = 4 * lane; j < full; j += 256)
#pragma unroll
        for (int h = 0; h < RH; ++h) {
          const floatx4u xa = *reinterpret_cast<const floatx4u*>(pa[h] + j), xd = *reinterpret_cast<const floatx4u*>(pd[h] + j);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[h] = fmaf(xa[e], xd[e], acc[h]);
        }
      // at most 255 + RH columns are left: two steps of whole pieces whose columns past the diagonal count as nothing.  (No load
      // sits under a condition: as five steps of single columns, each tested, a row group took 18 K cycles.)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (full + 256 * q > t_lo + RH - 1) break;
        const int j = full + 256 * q + 4 * lane, jc = min(j, min(t_lo + RH - 1, N - 4));   // (rows here have more than 128 columns)
        floatx4u xa[RH], xd[RH];
#pragma unroll
        for (int h = 0; h < RH; ++h) {
          xa[h] = *reinterpret_cast<const floatx4u*>(pa[h] + jc);
          xd[h] = *reinterpret_cast<const floatx4u*>(pd[h] + jc);
        }
#pragma unroll
        for (int h = 0; h < RH; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const bool on = jc + e >= j && jc + e <= min(t_lo + h, N - 1);
            acc[h] = fmaf(on ? xa[h][e] : 0.f, on ? xd[h][e] : 0.f, acc[h]);
          }
      }
#pragma unroll
      for (int h = 0; h < RH; ++h) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) acc[h] += __shfl_xor(acc[h], o, 64);
        if (lane == 0) {
          re[r0 + h] = acc[h];
          if (t0 + r0 + h < N) a.rowdot[unit * N + t0 + r0 + h] = acc[h];
        }
      }
    }
    E = __expf(-a.lse[unit * N + t]);
  }
  wait_async_copies();
  lds_barrier();
  if constexpr (!KEY) rho = re[row];
  Np np;
  np.forward(xl, static_cast<const T*>(KEY ? a.wkf : a.wqf) + (int64_t)hq * D * D,
             bias != nullptr ? bias + (int64_t)hq * D : nullptr, row, fh, lane, xch);

  // this lane's 32 entries of dA against a tile of the other side: entry v of step v / KPL
  floatx16 d[2];
  float rho_n = 0.f, L_n = 0.f;          // key side: rho and L of row 64 ot + tid of the next tile, as loaded
  auto load_d = [&](int ot) __attribute__((always_inline)) {
    const int lane_now = fresh_lane_id(), rr = lane_now & 31, gg = lane_now >> 5;
    if constexpr (KEY) {
      const float* p = dA + (t0 + 32 * rg + rr);           // (a full chunk: the key exists)
#pragma unroll
      for (int v = 0; v < 32; ++v) {
        const int to = 64 * ot + (v / KPL) * M::KK + gg * KPL + v % KPL;
        d[v / 16][v % 16] = p[(int64_t)min(to, N - 1) * N];
      }
      if (tid < 64) {
        const int to = 64 * ot + tid;
        rho_n = a.rowdot[unit * N + min(to, N - 1)];
        L_n = a.lse[unit * N + min(to, N - 1)];   // (E = exp(-L) is taken when the tile is: here it would wait for every load above)
      }
    } else {
      const float* p = dA + (int64_t)min(t0 + 32 * rg + rr, N - 1) * N + 64 * ot + gg * KPL;   // (full chunks)
      if constexpr (KPL == 8) {
#pragma unroll
        for (int v = 0; v < 32; v += 4) {
          const floatx4u y = *reinterpret_cast<const floatx4u*>(p + (v / 8) * M::KK + v % 8);
#pragma unroll
          for (int e = 0; e < 4; ++e) d[v / 16][v % 16 + e] = y[e];
        }
      } else {
#pragma unroll
        for (int v = 0; v < 32; ++v) d[v / 16][v % 16] = p[v * M::KK];
      }
    }
  };
  floatx16 dp[NS];
#pragma unroll
  for (int j = 0; j < NS; ++j) dp[j] = zero16();
  load_d(o_beg);
#pragma unroll 1
  for (int ot = o_beg; ot < o_end; ++ot) {
    const int par = (ot - o_beg) & 1;
    if constexpr (KEY) {
      if (tid < 64) re[128 * par + tid] = rho_n, re[128 * par + 64 + tid] = 64 * ot + tid < N ? __expf(-L_n) : 0.f;
    }
    wait_async_copies();
    lds_barrier();                       // the tile and its (rho, E) are here; everybody is done with its predecessor
    typename M::frag wf[SK];
    if constexpr (KEY && KPL == 8) {     // (rows past the end weigh nothing through E = 0: no choice per entry, which would be
#pragma unroll                           // a branch and two dependent LDS reads for each of the 32)
      for (int s = 0; s < SK; ++s) {
        const float* ro = re + 128 * par + s * M::KK + g * KPL;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const floatx4 rh = *reinterpret_cast<const floatx4*>(ro + 4 * q), ev = *reinterpret_cast<const floatx4*>(ro + 64 + 4 * q);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int v = 8 * s + 4 * q + e;
            wf[s][4 * q + e] = static_cast<bf16>((d[v / 16][v % 16] - rh[e]) * ev[e]);
          }
        }
      }
    } else {
#pragma unroll
      for (int v = 0; v < 32; ++v) {
        float rv = rho, ev = E;
        if constexpr (KEY) rv = re[128 * par + v * M::KK + g], ev = re[128 * par + 64 + v * M::KK + g];
        const float wv = (d[v / 16][v % 16] - rv) * ev;
        if constexpr (KPL == 8) wf[v / KPL][v % KPL] = static_cast<bf16>(wv);
        else wf[v] = wv;
      }
    }
    if (ot + 1 < o_end) {
      load_d(ot + 1);
      T* next = phi + (par ^ 1) * Cf::PE;
      if (!KEY || 64 * (ot + 2) <= N) request_run<T, 2 * D>(po + (int64_t)64 * (ot + 1) * (2 * D), next, wave);   // (queries: full chunks)
      else request_rows<T, 2 * D>(po, 2 * D, 64 * (ot + 1), N, next, wave);
    }
    const T* cur = phi + par * Cf::PE;
    const int lane_now = fresh_lane_id();
    piped<typename M::frag, SK * NS, 6>(
        [&](auto I) __attribute__((always_inline)) {
          constexpr int i = decltype(I)::value;
          return RP::down(cur, (i / NS) * M::KK, 64 * (i % NS) + 32 * fh, lane_now);
        },
        [&](auto I, const typename M::frag& f) __attribute__((always_inline)) {
          constexpr int i = decltype(I)::value;
          dp[i % NS] = M::mma(f, wf[i / NS], dp[i % NS]);
        });
  }
  lds_barrier();                         // the tiles are done with

  // ---- NP-Map backwards.  (The exponentials are taken again: kept across the loop they would not fit the register file,
  // and the empty statement keeps the compiler from doing that.)
  asm volatile("" : "+v"(np.mp), "+v"(np.mn));
  const bool dead = !(np.nx > 0.f) || !(np.nf > 0.f) || (KEY && kept_token(a.kmask, unit, a.ncf, C, c, t));
  float* my = xch + (fh * 64 + row) * 4;
  const float* other = xch + ((fh ^ 1) * 64 + row) * 4;
  float ap = 0.f, an = 0.f;
#pragma unroll
  for (int j = 0; j < NF; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      ap += np.pos(j, i) * np.ip * dp[j][i];
      an += np.neg(j, i) * np.in * dp[NF + j][i];
    }
  ap = sum32(ap);
  an = sum32(an);
  if (g == 0) my[0] = ap, my[1] = an;
  lds_barrier();
  ap += other[0];
  an += other[1];
  const float inx = np.nx > 0.f ? 1.f / np.nx : 0.f;
  float dnx = 0.f;
#pragma unroll
  for (int j = 0; j < NF; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      dp[j][i] = np.pos(j, i) * np.ip * (dp[j][i] - ap) - np.neg(j, i) * np.in * (dp[NF + j][i] - an);
      dnx += np.u[j][i] * inx * dp[j][i];
    }
  dnx = sum32(dnx);
  if (g == 0) my[2] = dnx;
  lds_barrier();
  dnx += other[2];
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    float y[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) y[i] = dead ? 0.f : np.ratio * (dp[j][i] - np.u[j][i] * inx * dnx);
    put_row<T, D>(xl, row, 64 * j + 32 * fh, y, g);
  }
  lds_barrier();
  for (int i = tid; i < 64 * RX::PPR; i += 256) {
    const int ri = i / RX::PPR, e0 = (i % RX::PPR) * RX::EPV;
    if (t0 + ri < N) *reinterpret_cast<Vec16*>(dfg + (int64_t)ri * D + e0) = *reinterpret_cast<const Vec16*>(xl + RX::off(ri, e0));
  }
}

template <typename K>
hipError_t launch(K kern, dim3 grid, size_t smem, hipStream_t s, const MapArgs& a) {
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, grid, dim3(256), smem, s, a);
  return hipGetLastError();
}

template <typename T, int D>
hipError_t launch_map_t(const MapArgs& a, bool backward, hipStream_t s) {
  typedef MapCfg<T, D> Cf;
  const unsigned blocks = (unsigned)((a.N + 63) / 64) * (unsigned)a.U;
  hipError_t e = launch(map_phi_kernel<T, D>, dim3(blocks, 2), Cf::phi_smem, s, a);
  if (e != hipSuccess) return e;
  if (!backward) return launch(attn_map_kernel<T, D>, dim3(blocks), Cf::map_smem, s, a);
  e = launch(map_bwd_kernel<T, D, false>, dim3(blocks), Cf::bwd_smem, s, a);
  return e != hipSuccess ? e : launch(map_bwd_kernel<T, D, true>, dim3(blocks), Cf::bwd_smem, s, a);
}

}  // namespace

hipError_t launch_map(const MapArgs& a, int dtype, int d, bool backward, hipStream_t s) {
  if (dtype == 1) return d == 128 ? launch_map_t<bf16, 128>(a, backward, s) : launch_map_t<bf16, 64>(a, backward, s);
  if (d == 64) return launch_map_t<float, 64>(a, backward, s);
  return hipErrorInvalidValue;   // fp32 is built for d = 64 only (refused by the host checks)
}

}  // namespace still
