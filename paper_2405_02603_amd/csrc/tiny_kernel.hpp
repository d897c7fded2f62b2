// tiny_kernel.hpp -- a whole solve in one block, for grids whose spectrum fits in LDS.
//
// A solve of 16^3 points is five launches of 3 to 7 us that keep the GPU busy for
// none of them: the launches and the passes' latency are all of its time.  Where
// S (n0 x 2 n1 x (n2 + 1) complex) fits in the LDS of a compute unit, one block
// runs the five passes there, in one launch, and S never goes to device memory.
// A thread owns a whole pencil and transforms it in registers (lengths up to 32,
// constant twiddles only), so a pass needs no exchange, only the barrier to the
// next; the axis-0 pass multiplies between its two transforms without storing
// the upper half.                                    [Section 2.2, steps 1-5]
//
// Measured (pipelined solves through the Python binding, five launches -> one;
// about 10 us is the binding's and the launch's own): 8^3 23.1 -> 10.1 us, 16^3
// float32 23.9 -> 11.5, 12x16x24 float32 23.7 -> 10.8, 16x16x32 float32 23.8 ->
// 18.2, 16^3 float64 23.8 -> 16.1; a batch of 64 16^3 127 -> 80.  What bounds it:
// the latency of one block's five passes; at 16^3 in float64 the 544 axis-0
// pencils take the 512 threads a second, nearly empty, round, and a 32-point
// pencil's registers spill 80 bytes a lane.
#pragma once

#include "solve_kernels.hpp"

namespace fsp {

struct TinyArgs {
  const ItemPtrs* items;      // table of this launch's items, or NULL (then in / out / ghat)
  const void* in[MAX_ITEMS];  // rho
  void* out[MAX_ITEMS];       // phi
  const void* ghat[MAX_ITEMS];
  const void* split;          // exp(-i pi k / n2), k in [0, n2]
  int n0, n1, n2;
  int gt;                     // column tile of the Green's octant
  long long g_k1_stride;
};

constexpr int TINY_THREADS = 512;
constexpr int TINY_LDS = 139264;  // 16^3 in float64, 16 x 16 x 32 in float32

template <typename T>
__host__ __device__ constexpr bool tiny_supported(int n0, int n1, int n2) {
  return n0 <= 16 && n1 <= 16 && n2 <= 32 && n0 * 2 * n1 * (n2 + 1) * 2 * (int)sizeof(T) <= TINY_LDS;
}

// Length-N transform of inputs whose upper half is zero (v[N / 2 ...] are set here).
template <int N, bool INV, typename T>
__device__ __forceinline__ void tiny_half_in(cx<T>* v) {
  if constexpr (32 % N == 0) {
    dft_half_in<N, INV, T>(v);
  } else {
#pragma unroll
    for (int i = N / 2; i < N; ++i) v[i] = czero<T>();
    Dft<N, INV, T>::run(v);
  }
}
// Outputs m < N / 2 of a length-N transform.
template <int N, bool INV, typename T>
__device__ __forceinline__ void tiny_half_out(cx<T>* v) {
  if constexpr (32 % N == 0)
    dft_half_out<N, INV, T>(v);
  else
    Dft<N, INV, T>::run(v);
}

// P1: rows (i0, i1) of rho to S[i0][i1][k], k <= LC = n2 (k_row_r2c's arithmetic).
template <typename T, int LC>
__device__ __forceinline__ void tiny_rows_fwd(cx<T>* S, const cx<T>* rho, const cx<T>* pp, int n0, int n1, int tid) {
  constexpr int P = LC + 1;
  for (int r = tid; r < n0 * n1; r += TINY_THREADS) {
    const int i0 = r / n1, i1 = r - i0 * n1;
    cx<T> z[LC];
#pragma unroll
    for (int j = 0; j < LC / 2; ++j) z[j] = ld_once(&rho[r * (LC / 2) + j]);
    tiny_half_in<LC, false, T>(z);
    cx<T>* out = S + (i0 * 2 * n1 + i1) * P;
#pragma unroll
    for (int k = 0; k <= LC; ++k) {
      const cx<T> A = z[k == LC ? 0 : k];
      const cx<T> B = conjg(z[k == 0 || k == LC ? 0 : LC - k]);
      const cx<T> E = {T(0.5) * (A.x + B.x), T(0.5) * (A.y + B.y)};
      const cx<T> D = {T(0.5) * (A.x - B.x), T(0.5) * (A.y - B.y)};
      const cx<T> U = cmul(pp[k], D);
      out[k] = cx<T>{E.x + U.y, E.y - U.x};
    }
  }
}

// P5: rows of S back to phi (k_row_c2r's arithmetic).
template <typename T, int LC>
__device__ __forceinline__ void tiny_rows_inv(const cx<T>* S, cx<T>* phi, const cx<T>* pp, int n0, int n1, int tid) {
  constexpr int P = LC + 1;
  for (int r = tid; r < n0 * n1; r += TINY_THREADS) {
    const int i0 = r / n1, i1 = r - i0 * n1;
    const cx<T>* in = S + (i0 * 2 * n1 + i1) * P;
    cx<T> z[LC];
#pragma unroll
    for (int n = 0; n < LC; ++n) {
      const cx<T> X1 = in[n], X2 = conjg(in[LC - n]);
      const cx<T> A = cadd(X1, X2);
      const cx<T> B = cmulc(csub(X1, X2), pp[n]);
      z[n] = {A.x - B.y, A.y + B.x};
    }
    tiny_half_out<LC, true, T>(z);
#pragma unroll
    for (int j = 0; j < LC / 2; ++j) put<true>(&phi[r * (LC / 2) + j], z[j]);
  }
}

// P2 / P4: pencils (i0, k2) along axis 1, in place; cols = n2 + 1.
template <typename T, int L, bool INV>
__device__ __forceinline__ void tiny_axis1(cx<T>* S, int n0, int cols, int tid) {
  for (int p = tid; p < n0 * cols; p += TINY_THREADS) {
    const int i0 = p / cols, k2 = p - i0 * cols;
    cx<T>* base = S + i0 * L * cols + k2;
    cx<T> v[L];
#pragma unroll
    for (int i = 0; i < (INV ? L : L / 2); ++i) v[i] = base[i * cols];
    if constexpr (INV)
      tiny_half_out<L, true, T>(v);
    else
      tiny_half_in<L, false, T>(v);
#pragma unroll
    for (int i = 0; i < (INV ? L / 2 : L); ++i) base[i * cols] = v[i];
  }
}

// P3: pencils (k1, k2) along axis 0: forward, the octant's row, inverse, in place.
template <typename T, int L>
__device__ __forceinline__ void tiny_axis0(cx<T>* S, const T* ghat, const TinyArgs& a, int tid) {
  const int cols = a.n2 + 1, l1 = 2 * a.n1, stride = l1 * cols;
  for (int p = tid; p < stride; p += TINY_THREADS) {
    const int k1 = p / cols, k2 = p - k1 * cols;
    const int k1f = k1 <= a.n1 ? k1 : l1 - k1;
    const T* g = ghat + k1f * a.g_k1_stride + (long long)(k2 / a.gt) * (L / 2 + 1) * a.gt + k2 % a.gt;
    T gv[L / 2 + 1];
#pragma unroll
    for (int k = 0; k <= L / 2; ++k) gv[k] = ld(&g[k * a.gt]);
    cx<T> v[L];
#pragma unroll
    for (int i = 0; i < L / 2; ++i) v[i] = S[i * stride + p];
    tiny_half_in<L, false, T>(v);
#pragma unroll
    for (int k = 0; k < L; ++k) v[k] = cscale(v[k], gv[k <= L / 2 ? k : L - k]);
    tiny_half_out<L, true, T>(v);
#pragma unroll
    for (int i = 0; i < L / 2; ++i) S[i * stride + p] = v[i];
  }
}

// Lengths are uniform in the block, so each pass takes one branch.
template <typename T>
__global__ __launch_bounds__(TINY_THREADS) void k_tiny_solve(TinyArgs a) {
  __shared__ cx<T> S[TINY_LDS / sizeof(cx<T>)];
  const int tid = threadIdx.x;
  const cx<T>* rho = reinterpret_cast<const cx<T>*>(a.items ? table_item(a.items, blockIdx.y).rho : a.in[blockIdx.y]);
  cx<T>* phi = reinterpret_cast<cx<T>*>(a.items ? table_item(a.items, blockIdx.y).phi : a.out[blockIdx.y]);
  const T* ghat = reinterpret_cast<const T*>(item_ghat(a));
  const cx<T>* pp = reinterpret_cast<const cx<T>*>(a.split);
  const int n0 = a.n0, n1 = a.n1, cols = a.n2 + 1;
  switch (a.n2) {
    case 8: tiny_rows_fwd<T, 8>(S, rho, pp, n0, n1, tid); break;
    case 12: tiny_rows_fwd<T, 12>(S, rho, pp, n0, n1, tid); break;
    case 16: tiny_rows_fwd<T, 16>(S, rho, pp, n0, n1, tid); break;
    case 24: tiny_rows_fwd<T, 24>(S, rho, pp, n0, n1, tid); break;
    default: tiny_rows_fwd<T, 32>(S, rho, pp, n0, n1, tid); break;
  }
  lds_barrier();
  switch (n1) {
    case 8: tiny_axis1<T, 16, false>(S, n0, cols, tid); break;
    case 12: tiny_axis1<T, 24, false>(S, n0, cols, tid); break;
    default: tiny_axis1<T, 32, false>(S, n0, cols, tid); break;
  }
  lds_barrier();
  switch (n0) {
    case 8: tiny_axis0<T, 16>(S, ghat, a, tid); break;
    case 12: tiny_axis0<T, 24>(S, ghat, a, tid); break;
    default: tiny_axis0<T, 32>(S, ghat, a, tid); break;
  }
  lds_barrier();
  switch (n1) {
    case 8: tiny_axis1<T, 16, true>(S, n0, cols, tid); break;
    case 12: tiny_axis1<T, 24, true>(S, n0, cols, tid); break;
    default: tiny_axis1<T, 32, true>(S, n0, cols, tid); break;
  }
  lds_barrier();
  switch (a.n2) {
    case 8: tiny_rows_inv<T, 8>(S, phi, pp, n0, n1, tid); break;
    case 12: tiny_rows_inv<T, 12>(S, phi, pp, n0, n1, tid); break;
    case 16: tiny_rows_inv<T, 16>(S, phi, pp, n0, n1, tid); break;
    case 24: tiny_rows_inv<T, 24>(S, phi, pp, n0, n1, tid); break;
    default: tiny_rows_inv<T, 32>(S, phi, pp, n0, n1, tid); break;
  }
}

template <typename T>
hipError_t launch_tiny(const TinyArgs& a, int items, hipStream_t s) {
  if (!tiny_supported<T>(a.n0, a.n1, a.n2)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_tiny_solve<T>, dim3(1, items), dim3(TINY_THREADS), 0, s, a);
  return hipGetLastError();
}

}  // namespace fsp
