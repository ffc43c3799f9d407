// Backward pass of the prefill operator, the routing held fixed (gfx950).
//
// What is differentiated is the output equation of Sec. 3.3, y = (N_SA + g N_LA) / (D_SA + D_LA), for the index
// lists the forward pass chose: the Top-lambda selection is a discrete decision and passes no gradient, and the
// Self-Saliency Score of Sec. 3.1 only feeds that decision.  With L_t = ln(D_SA + D_LA) (kept by the forward pass),
// delta_t = dy_t . y_t and E_t = exp(-L_t):
//   softmax branch, key j visible to row t through exp:   P_tj = exp(scale q_t.k_j - L_t)
//        dv_j += P_tj dy_t          dl_tj = P_tj (dy_t . v_j - delta_t)
//        dq_t += scale dl_tj k_j    dk_j += scale dl_tj q_t
//   linear branch, S = sum phi_k(k_j)^T v_j and z = sum phi_k(k_j) over the un-selected tokens of chunks <= c-2:
//        A_t = E_t (g_t * dy_t)                     (per channel)
//        dphi_q(t) = S A_t - E_t delta_t z          dg_t = E_t dy_t * (phi_q(t) S)
//        dS(c) = sum over the rows of chunks >= c+2 of phi_q(t)^T A_t,   dz(c) likewise of phi_q(t) E_t delta_t
//        dphi_k(j) = dS(c_j) v_j - dz(c_j)          dv_j += dS(c_j)^T phi_k(j)
//   and the NP-Map of Sec. 3.2 (f = x W + b, u = f |x| / |f|, phi = [softmax(u), softmax(-u)]) backwards:
//        du = phi+ (dphi+ - <phi+, dphi+>) - phi- (dphi- - <phi-, dphi->)
//        df = (|x| / |f|) (du - fh <fh, du>),  fh = f / |f|;   dx = df W^T + <fh, du> x / |x|;   dW = x^T df
//
// The softmax branch is in still_bwd_sa.hip, the linear branch in still_bwd_lin.hip, the attention map with its backward pass
// in still_map.hip.  Here: the per-row scalars both branches start from.  All sums are fp32; operands of the matrix core are
// in the storage type.
#include "still_kernels.h"

namespace still {

namespace {

// Every token row goes to d/8 lanes, 8 contiguous elements per lane, so that every access is a 16-byte (storage type) or
// 32-byte (fp32) vector and a row reduction is 3 or 4 exchanges inside the group.  A wave holds 64 / (d/8) rows, a
// workgroup four waves.
template <typename T>
__device__ __forceinline__ void load8_t(float (&x)[8], const T* p) {
  if constexpr (sizeof(T) == 2) {
    const bf16x8 v = *reinterpret_cast<const bf16x8*>(p);
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = static_cast<float>(v[e]);
  } else {
    const floatx4 a = *reinterpret_cast<const floatx4*>(p), b = *reinterpret_cast<const floatx4*>(p + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) { x[e] = a[e]; x[4 + e] = b[e]; }
  }
}
__device__ __forceinline__ float group_sum(float x, int lpr) {
  for (int o = lpr >> 1; o >= 1; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}
// row handled by this lane, and its first element; false when the row is past the end (whole groups drop out)
__device__ __forceinline__ bool row_of_lane(int64_t n_rows, int width, int64_t& row, int& e0, int& lpr) {
  lpr = width / 8;
  const int tid = threadIdx.x;
  row = (int64_t)blockIdx.x * (256 / lpr) + tid / lpr;
  e0 = (tid % lpr) * 8;
  return row < n_rows;
}

// delta_t = dy_t . y_t, E_t = exp(-L_t)
template <typename T>
__global__ __launch_bounds__(256) void bwd_row_prep_kernel(BwdRowArgs a) {
  int64_t row;
  int e0, lpr;
  const bool live = row_of_lane((int64_t)a.U * a.N, a.d, row, e0, lpr);
  const int64_t rowc = live ? row : 0;
  const int unit = (int)(rowc / a.N), t = (int)(rowc % a.N);
  const int b = unit / a.Hq, h = unit % a.Hq;
  const int64_t oo = b * a.o_sb + (int64_t)t * a.o_st + h * a.o_sh + e0;
  float y[8], dy[8];
  load8_t<T>(y, static_cast<const T*>(a.out) + oo);
  load8_t<T>(dy, static_cast<const T*>(a.dout) + oo);
  const float E = __expf(-a.lse[rowc]);
  float dot = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) dot += dy[e] * y[e];
  dot = group_sum(dot, lpr);
  if (!live) return;
  if (e0 == 0) {
    a.e_row[row] = E;
    a.delta[row] = dot;
    a.ed[row] = E * dot;
  }
}

// fp32 rows -> the caller's strided tensor in the storage type: the last step for results that lie over an input
template <typename T>
__global__ __launch_bounds__(256) void bwd_round_kernel(BwdRoundArgs a) {
  int64_t row;
  int e0, lpr;
  if (!row_of_lane((int64_t)a.B * a.H * a.N, a.d, row, e0, lpr)) return;
  const int t = (int)(row % a.N), bh = (int)(row / a.N);
  float x[8];
  load8_t<float>(x, a.src + row * a.d + e0);
  T* dst = static_cast<T*>(a.dst) + bh / a.H * a.s_b + (int64_t)t * a.s_t + bh % a.H * a.s_h + e0;
  __attribute__((aligned(16))) T y[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) y[e] = from_f32<T>(x[e]);
#pragma unroll
  for (int i = 0; i < (int)sizeof(y) / 16; ++i) reinterpret_cast<Vec16*>(dst)[i] = reinterpret_cast<const Vec16*>(y)[i];
}

}  // namespace

hipError_t launch_bwd_round(const BwdRoundArgs& a, int dtype, hipStream_t s) {
  const int rpb = 256 / (a.d / 8);   // rows per workgroup
  const unsigned blocks = (unsigned)(((int64_t)a.B * a.H * a.N + rpb - 1) / rpb);
  if (dtype == 1) hipLaunchKernelGGL((bwd_round_kernel<bf16>), dim3(blocks), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((bwd_round_kernel<float>), dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_bwd_row_prep(const BwdRowArgs& a, int dtype, hipStream_t s) {
  const int rpb = 256 / (a.d / 8);   // rows per workgroup
  const int blocks = (int)(((int64_t)a.U * a.N + rpb - 1) / rpb);
  if (dtype == 1) hipLaunchKernelGGL((bwd_row_prep_kernel<bf16>), dim3(blocks), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((bwd_row_prep_kernel<float>), dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace still
