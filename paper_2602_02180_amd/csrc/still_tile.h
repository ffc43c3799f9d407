// Row-major operand tiles in LDS that serve the matrix core from both sides (gfx950).
//
// A tile holds ROWS rows (keys, queries or feature rows) of D elements, as in memory.  Read along its rows it is an
// operand whose contraction index is the row's element index (logits: q.k); read down its columns it is an operand
// whose contraction index is the row number (sums over keys or queries: dq += dS K).  The second form needs the
// elements of one column from consecutive rows in one lane; for 2-byte types the transposing LDS read of gfx950
// (ds_read_b64_tr_b16) delivers exactly that, so no transposed copy of the tensor is ever written: sixteen lanes
// address four rows of sixteen columns, four lanes per row, and lane i receives column i of the four rows.
// The 16-byte pieces of a row are XOR-ed with a function of the row number that keeps both kinds of reads free of bank
// conflicts: sixteen consecutive rows at one piece index fall on sixteen different pieces of the 256-byte bank
// width, and so do four consecutive rows at four consecutive pieces.
#pragma once
#include "still_kernels.h"

namespace still {

typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) shortx4 lds_shortx4;

template <typename T, int D>
struct RowTile {
  typedef Mma<T> M;
  static constexpr int EPV = 16 / (int)sizeof(T);   // elements per 16-byte piece
  static constexpr int PPR = D / EPV;               // pieces per row: 8 or 16 or 32
  static __device__ __forceinline__ int swz(int row) {
    if constexpr (PPR == 8) return (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
    else return ((row & 3) << 2) | ((row >> 2) & 3);
  }
  // element offset of (row, e)
  static __device__ __forceinline__ int off(int row, int e) {
    return row * D + (((e / EPV) ^ swz(row)) * EPV) + e % EPV;
  }
  // operand over the row's elements: lane r takes row `row`, k-step s
  static __device__ __forceinline__ typename M::frag along(const T* tile, int row, int s, int g) {
    return M::load(tile + off(row, s * M::KK + g * M::KPL));
  }
  // operand over rows: the lane of MFMA row m takes column c0 + kappa(m), contraction entries = rows k0 .. k0 + KK - 1
  static __device__ __forceinline__ typename M::frag down(const T* tile, int k0, int c0, int lane) {
    if constexpr (sizeof(T) == 2) {
      const int g = lane >> 5, j = (lane >> 2) & 3, b = lane & 3;
      const int col = c0 + 16 * ((lane >> 4) & 1) + 4 * (((b & 1) << 1) | (b >> 1));   // kappa swaps bits 2 and 3
      const int row = k0 + 8 * g + j;
      union {
        shortx4 h[2];
        typename M::frag f;
      } u;
      u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)(tile + off(row, col)));
      u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)(tile + off(row + 4, col)));
      return u.f;
    } else {
      return tile[off(k0 + (lane >> 5), c0 + M::kappa(lane & 31))];
    }
  }
};

// A slab of 64 features of a state image in LDS (state_image_offset: blocks of 32 rows x by 16 features in operand order), read
// over its features (rows 32 xb ..) or, transposing, over its rows x (columns = features).
template <typename T>
struct StateSlab {
  typedef Mma<T> M;
  static __device__ __forceinline__ int off(int x, int f) { return state_image_offset(x, f, 64); }
  static __device__ __forceinline__ typename M::frag along(const T* tile, int xb, int s, int r, int g) {
    return M::load(tile + xb * 2048 + off(r, s * M::KK + g * M::KPL));
  }
  static __device__ __forceinline__ typename M::frag down(const T* tile, int k0, int c0, int lane) {
    if constexpr (sizeof(T) == 2) {
      const int g = lane >> 5, j = (lane >> 2) & 3, b = lane & 3;
      const int col = 16 * ((lane >> 4) & 1) + 4 * (((b & 1) << 1) | (b >> 1));   // kappa swaps bits 2 and 3
      const T* base = tile + state_image_offset(k0, c0, 64) + state_image_offset(8 * g + j, col, 64);
      union {
        shortx4 h[2];
        typename M::frag f;
      } u;
      // (rows k0 + 8 g + j and + 4: bit 2 of the row is the second read's and the swizzle's, so the offset changes sign)
      u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)base);
      u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)(base + ((col >> 3) & 1 ? -32 : 32)));
      return u.f;
    } else {
      return tile[off(k0 + (lane >> 5), c0 + M::kappa(lane & 31))];
    }
  }
};

// one lane's 16 accumulator entries of a (feature x token) product -> its token's row of an LDS row tile, columns c0 ..
template <typename T, int W>
__device__ __forceinline__ void put_row(T* tile, int row, int c0, const float (&x)[16], int g) {
  typedef Mma<T> M;
  typedef RowTile<T, W> RT;
  if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      bf16x8 v;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = static_cast<bf16>(x[8 * s + e]);
      *reinterpret_cast<bf16x8*>(tile + RT::off(row, c0 + M::pos_of_reg(8 * s, g))) = v;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i) tile[RT::off(row, c0 + M::pos_of_reg(i, g))] = x[i];
  }
}

// N products with the streamed operand read DEPTH products ahead of its use (the scheduling barriers pin that order:
// left alone the compiler puts every read right before its product and waits for it).  a_at(IDX) reads operand IDX,
// mm(IDX, operand) issues product IDX; both get the index as a compile-time constant.
template <typename Frag, int N, int DEPTH, typename A, typename F>
__device__ __forceinline__ void piped(A&& a_at, F&& mm) {
  constexpr int DP = DEPTH < N ? DEPTH : N;
  Frag buf[DP];
  static_for<DP>([&](auto I) __attribute__((always_inline)) { buf[decltype(I)::value] = a_at(I); });
  __builtin_amdgcn_sched_barrier(0);
  static_for<N>([&](auto I) __attribute__((always_inline)) {
    constexpr int i = decltype(I)::value;
    mm(I, buf[i % DP]);
    if constexpr (i + DP < N) buf[i % DP] = a_at(std::integral_constant<int, i + DP>{});
    __builtin_amdgcn_sched_barrier(0);
  });
}

}  // namespace still
