// greens_axis.hip -- the potential's Green's transform in three axis passes (gfx950).
//
// Both routes of the potential's precompute are separable, so every axis takes
// one matrix, applied on the float64 matrix cores:
//
//   Hockney-Eastwood (Section 2.2): the DCT-I of length n + 1 of the kernel's
//     octant, Y[m] = sum_k w_k cos(pi k m / n) X[k] (w = 1 at the ends, else 2).
//   Vico-Greengard, modified (Section 2.4): the DCT-I of length 2 n + 1 of the
//     samples of eq. (3) keeping outputs m <= n, then the DCT-I of length n + 1.
//     Their product has a closed form.  With S(t) = sum over m in [-n, n) of
//     cos(m t) = sin(n t) cot(t / 2) (2 n at t = 0 mod 2 pi),
//       A[k][l] = (w_l / 2) (S(t+) + S(t-)),  t+- = pi (2 k +- l) / (2 n),
//     which is 2 n at l = 2 k and 0 at every other even l, and for odd l
//       A[k][l] = (-1)^k s_l (cot(pi (2 k + l) / 4 n) + cot(pi (l - 2 k) / 4 n)),
//       s_l = (-1)^((l - 1) / 2).
//     So an axis costs an (n + 1) x n product over the odd samples and a copy of
//     the even ones: a quarter of the products of the two transforms in turn,
//     and three passes over shrinking arrays instead of six.
//
// Folding halves the products again.  DCT-I: the even rows take the sums
// X[k] + X[n - k], the odd rows the differences.  The odd-sample matrix has
// A[n - k][2 n - l] = A[k][l]: with e_k = sum over odd l < n of
// (A[k][l] + A[n - k][l]) / 2 (X[l] + X[2 n - l]) and o_k the same with both
// signs minus, rows k and n - k are e_k + o_k and e_k - o_k.  In both cases
// two square (n / 2) x (n / 2) products remain, with n / 2 inputs each; the row
// left over (m = n, or k = n / 2) is a dot product.
//
// Axis 0 makes its inputs as it needs them (samples of eq. (3), or the kernel),
// so neither ever goes to device memory; axis 2 writes the stored octant
// (scaled, rounded once, tile-blocked) itself.
//
// A block owns CT columns of its pass (a column: one line along the contracted
// axis) and every output row.  Its sums and differences fill LDS once; its waves
// then share out the rows, each holding its 16 x 16 accumulators, and read their
// matrix operands straight into registers from an image in the operand layout
// (it stays in the L2; a fill kernel writes it, so nothing is uploaded): no
// barrier between the fill and the results.  16 columns of a long axis leave
// two blocks or more a compute unit.
//
// Measured (256^3 Vico-Greengard): samples and six contractions before 3.82 ms,
// now 1.05 ms (1.21 with two row blocks a wave and 32 columns a block); 128^3 480
// -> 134 us; Hockney-Eastwood 64^3 float64 55 -> 29 us.  What bounds it: the
// products (30 GFLOP, 0.68 ms alone) and on axis 0 the samples' float64
// arithmetic run on the same units, so one does not hide the other; with the
// library's sine and a division a sample cost 137 instructions, here about 35
// (axis 0 972 -> 729 us with the larger blocks).  Loops that fill LDS request
// eight (or compute four) inputs at a time: one at a time axis 1 took 604 us.
// Error against the transform in 80-bit arithmetic: below the six contractions'
// for Vico-Greengard (16x24x32 1.4e-16 against 2.8e-16, 64^3 3.5e-16 against
// 5.1e-16, 96x32x48 2.5e-16 against 4.5e-16), equal for Hockney-Eastwood.
//
// MFMA 16x16x4 f64 operands: lane l holds A(l % 16, l / 16) and B(l / 16, l % 16);
// D(i, j) is register i / 4 of lane j + 16 (i % 4).
#include <hip/hip_runtime.h>

#include "greens_axis.hpp"

namespace fsp {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

// cot(pi j / (4 n)) for odd j in (-4 n, 4 n), folded to [0, pi / 2] exactly
__device__ double cot_quarter(int j, int n) {
  const bool neg = j < 0;
  if (neg) j = -j;
  const bool up = j > 2 * n;
  if (up) j = 4 * n - j;
  const double x = (double)j / (double)(4 * n);
  const double c = cospi(x) / sinpi(x);
  return neg != up ? -c : c;
}

// cos(pi t / n)
__device__ double cos_pi_over(int t, int n) {
  t %= 2 * n;
  if (t > n) t = 2 * n - t;
  const bool up = 2 * t > n;
  if (up) t = n - t;
  const double c = cospi((double)t / (double)n);
  return up ? -c : c;
}

// A[k][l] of the Vico-Greengard axis, odd l
__device__ double vico_entry(int k, int l, int n) {
  const double c = cot_quarter(2 * k + l, n) + cot_quarter(l - 2 * k, n);
  return (k + (l - 1) / 2) % 2 ? -c : c;
}

// Matrix image of one axis: [step of 4 inputs][block of 16 rows][even, odd part][lane],
// then the row left over.
__global__ __launch_bounds__(256) void k_axis_image(double* out, int n, int vico) {
  const int K = n / 2, ks = (K + 3) / 4, pb = (K + 15) / 16;
  const int main = ks * pb * 128;
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= main + 4 * ks) return;
  double v = 0.0;
  if (e >= main) {
    const int i = e - main;
    if (i < K) v = vico ? vico_entry(K, 2 * i + 1, n) : (i == 0 ? 1.0 : i % 2 ? -2.0 : 2.0);
  } else {
    const int lane = e % 64, odd = (e / 64) % 2, b = (e / 128) % pb, s = e / (128 * pb);
    const int row = b * 16 + lane % 16, i = s * 4 + lane / 16;
    if (row < K && i < K) {
      if (vico) {
        const double a = vico_entry(row, 2 * i + 1, n), c = vico_entry(n - row, 2 * i + 1, n);
        v = 0.5 * (odd ? a - c : a + c);
      } else {
        v = (i == 0 ? 1.0 : 2.0) * cos_pi_over(i * (2 * row + odd), n);
      }
    }
  }
  out[e] = v;
}

// sin(pi r), |r| <= 1/2: r times the Taylor polynomial in r^2 through r^20 (the
// first term left out is below 2e-18 of the result's range).
__device__ __forceinline__ double sin_half_turn(double r) {
  // (-1)^k pi^(2 k + 1) / (2 k + 1)!
  constexpr double c[11] = {
      3.141592653589793,
      -5.16771278004997,
      2.5501640398773455,
      -0.5992645293207921,
      0.08214588661112823,
      -0.0073704309457143504,
      0.00046630280576761255,
      -2.1915353447830217e-05,
      7.952054001475513e-07,
      -2.2948428997269873e-08,
      5.392664662608129e-10};
  const double z = r * r;
  double p = c[10];
#pragma unroll
  for (int k = 9; k >= 0; --k) p = fma(p, z, c[k]);
  return r * p;
}

// A sample of eq. (3) at |k|^2 = k2: 2 sin^2(L |k| / 2) / |k|^2, with L^2 / 2 at
// 0.  sin^2 has period pi, so the argument is reduced in half turns
// (half_turns = L / (2 pi)): the remainder after the nearest whole number, one
// polynomial, no quadrants.  |k| and 1 / |k| come from one reciprocal square
// root estimate and Newton steps (the argument is never subnormal or infinite).
__device__ __forceinline__ double vico_sample(double k2, double half_turns, double at_zero) {
  const double y = __builtin_amdgcn_rsq(k2);
  double g = k2 * y, h = 0.5 * y;          // -> |k|, 1 / (2 |k|)
  const double r0 = fma(-h, g, 0.5);
  h = fma(h, r0, h);
  g = fma(g, r0, g);
  g = fma(fma(-g, g, k2), h, g);
  g = fma(fma(-g, g, k2), h, g);
  h = fma(h, fma(-h, g, 0.5), h);
  h = fma(h, fma(-h, g, 0.5), h);
  const double t = half_turns * g;
  const double q = sin_half_turn(t - rint(t)) * h;
  return k2 > 0.0 ? 8.0 * q * q : at_zero;  // 2 (s 2 h)^2
}

// Input l of a column of axis 0: a sample of eq. (3) (other = the other axes'
// part of |k|^2), or the Hockney-Eastwood kernel at the offset (the nearest
// image's on a periodic axis).
template <bool VICO>
__device__ __forceinline__ double make_input(const AxisArgs& a, int l, double other) {
  if constexpr (VICO) {
    const double kx = l * a.f[0];
    return vico_sample(kx * kx + other, a.half_turns, a.at_zero);
  } else {
    if (a.periodic & 1) l = min(l, a.n - l);
    const double x = l * a.f[0];
    const double r = sqrt(x * x + other);
    return r > 0.0 ? 1.0 / (4.0 * M_PI * r) : a.g0;
  }
}

// The tail of |k|^2 (or r^2) of column J of axis 0.
template <bool VICO>
__device__ __forceinline__ double column_tail(const AxisArgs& a, int J) {
  int l1 = J / a.p2, l2 = J - l1 * a.p2;
  if constexpr (!VICO) {
    if (a.periodic & 2) l1 = min(l1, a.n1 - l1);
    if (a.periodic & 4) l2 = min(l2, a.n2 - l2);
  }
  const double y = l1 * a.f[1], z = l2 * a.f[2];
  return y * y + z * z;
}

// VICO: the Vico-Greengard axis, else the DCT-I.  AXIS 0: inputs made here.
// AXIS 2: results go to the octant.  NMAX bounds n (the LDS array); WAVES waves
// take a 16-row block each; CG 16-column groups a block.
template <bool VICO, int AXIS, int NMAX, int WAVES, int CG>
__global__ __launch_bounds__(64 * WAVES) void k_green_axis(AxisArgs a) {
  constexpr int CT = 16 * CG, CP = CT + 1, NT = 64 * WAVES;
  __shared__ double lds[(NMAX + 1) * CP];
  __shared__ double part[NT];
  __shared__ double left[CT];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int n = a.n, K = n / 2, KS = (K + 3) / 4, PB = (K + 15) / 16;
  const int din = VICO ? 2 * n + 1 : n + 1;  // inputs along the contracted axis
  const int J0 = blockIdx.x * CT;
  // this thread's column where lanes run along columns
  const int c = t % CT, J = J0 + c;
  const bool cok = J < a.N;
  // column J's first input in memory, and the stride along the contracted axis
  auto source = [&](int J_) -> const double* {
    if constexpr (AXIS == 1) return a.x + (long long)(J_ / a.p2) * a.d1 * a.p2 + J_ % a.p2;
    return a.x + ((long long)(J_ % (a.n0 + 1)) * (a.n1 + 1) + J_ / (a.n0 + 1)) * a.p2;  // AXIS 2: J = (k1, k0)
  };
  const long long sk = AXIS == 1 ? a.p2 : 1;
  double other = 0.0;
  if constexpr (AXIS == 0) other = column_tail<VICO>(a, cok ? J : 0);
  const double* const col = AXIS == 1 ? source(cok ? J : 0) : nullptr;
  auto input = [&](int l) -> double {  // lanes along columns
    if constexpr (AXIS == 0) return make_input<VICO>(a, l, other);
    return col[l * sk];
  };

  // ---- sums at lds[i CP + c], differences at lds[(4 KS + i) CP + c], i < 4 KS
  auto put_pair = [&](int i, int cc, double u, double v) {
    lds[i * CP + cc] = u + v;
    lds[(4 * KS + i) * CP + cc] = u - v;
  };
  const int lo_step = VICO ? 2 : 1, lo_off = VICO ? 1 : 0;  // input pair i: l = lo_step i + lo_off and din - 1 - l
  // U inputs pairs (or inputs) at a time: their loads, or the chains of their
  // arithmetic, run side by side
  constexpr int U = AXIS == 0 ? 4 : 8;
  if constexpr (AXIS == 2) {  // lanes along the axis: rows are contiguous in memory
    constexpr int CW = CT / WAVES > 0 ? (CT + WAVES - 1) / WAVES : 1;  // columns a wave takes
    for (int i = lane; i < 4 * KS; i += 64) {
      const int l = i < K ? lo_step * i + lo_off : lo_off;
      double u[CW], v[CW];
#pragma unroll
      for (int w = 0; w < CW; ++w) {
        const int cc = wave + WAVES * w;
        const double* row = source(cc < CT && J0 + cc < a.N ? J0 + cc : 0);
        u[w] = row[l];
        v[w] = row[din - 1 - l];
      }
#pragma unroll
      for (int w = 0; w < CW; ++w) {
        const int cc = wave + WAVES * w;
        const bool on = i < K && J0 + cc < a.N;
        if (cc < CT) put_pair(i, cc, on ? u[w] : 0.0, on ? v[w] : 0.0);
      }
    }
  } else {
    for (int i0 = t / CT; i0 < 4 * KS; i0 += U * (NT / CT)) {
      double u[U], v[U];
#pragma unroll
      for (int w = 0; w < U; ++w) {
        const int i = i0 + w * (NT / CT);
        const int l = i < K ? lo_step * i + lo_off : lo_off;
        u[w] = input(l);
        v[w] = input(din - 1 - l);
      }
#pragma unroll
      for (int w = 0; w < U; ++w) {
        const int i = i0 + w * (NT / CT);
        const bool on = cok && i < K;
        if (i < 4 * KS) put_pair(i, c, on ? u[w] : 0.0, on ? v[w] : 0.0);
      }
    }
  }
  __syncthreads();

  // ---- the row left over: a dot product with the sums
  {
    const double* lv = a.image + (long long)KS * PB * 128;
    double s = 0.0;
#pragma unroll 4
    for (int i = t / CT; i < K; i += NT / CT) s += lv[i] * lds[i * CP + c];
    part[t] = s;
  }
  // ---- products
  v4d acc[2][CG];
#pragma unroll
  for (int o = 0; o < 2; ++o)
#pragma unroll
    for (int g = 0; g < CG; ++g) acc[o][g] = v4d{0.0, 0.0, 0.0, 0.0};
  const bool rows = wave < PB;
  if (rows) {
    const double* im = a.image + wave * 128 + lane;
    const int sstep = PB * 128;
    // operands two steps ahead of their use
    double nx[2][2];
    auto load = [&](int s, int slot) {
      const int sc = s < KS ? s : KS - 1;
#pragma unroll
      for (int o = 0; o < 2; ++o) nx[slot][o] = im[(long long)sc * sstep + o * 64];
    };
    load(0, 0);
    load(1, 1);
    const double* bl = lds + (lane / 16) * CP + lane % 16;
    double nb[2][2][CG];
    auto load_b = [&](int s, int slot) {
      const int sc = s < KS ? s : KS - 1;
#pragma unroll
      for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int g = 0; g < CG; ++g) nb[slot][o][g] = bl[(4 * sc + (o ? 4 * KS : 0)) * CP + 16 * g];
    };
    load_b(0, 0);
    auto step = [&](int s, int slot) {
      double m[2];
#pragma unroll
      for (int o = 0; o < 2; ++o) m[o] = nx[slot][o];
      load(s + 2, slot);
      load_b(s + 1, 1 - slot);
#pragma unroll
      for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int g = 0; g < CG; ++g)
          acc[o][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(m[o], nb[slot][o][g], acc[o][g], 0, 0, 0);
    };
    int s = 0;
    for (; s + 1 < KS; s += 2) {
      step(s, 0);
      step(s + 1, 1);
    }
    if (s < KS) step(s, 0);
  }
  __syncthreads();  // the sums and differences are used up; part is written
  if (t < CT) {
    double s = 0.0;
    for (int k = 0; k < NT / CT; ++k) s += part[k * CT + t];
    left[t] = s;
  }
  // ---- results at lds[m CP + c], first the terms outside the products:
  // 2 n X[2 m], or the centre input's 2 (-1)^r X[n / 2] in the even rows m = 2 r
  if constexpr (VICO) {
    const double twice = 2.0 * n;
    if constexpr (AXIS == 2) {
      constexpr int CW = (CT + WAVES - 1) / WAVES;
      for (int m = lane; m <= n; m += 64) {
        double u[CW];
#pragma unroll
        for (int w = 0; w < CW; ++w) {
          const int cc = wave + WAVES * w;
          u[w] = source(cc < CT && J0 + cc < a.N ? J0 + cc : 0)[2 * m];
        }
#pragma unroll
        for (int w = 0; w < CW; ++w) {
          const int cc = wave + WAVES * w;
          if (cc < CT) lds[m * CP + cc] = twice * u[w];
        }
      }
    } else {
      for (int m0 = t / CT; m0 <= n; m0 += U * (NT / CT)) {
        double u[U];
#pragma unroll
        for (int w = 0; w < U; ++w) u[w] = input(2 * min(m0 + w * (NT / CT), n));
#pragma unroll
        for (int w = 0; w < U; ++w) {
          const int m = m0 + w * (NT / CT);
          if (m <= n) lds[m * CP + c] = twice * u[w];
        }
      }
    }
  } else {
    double centre;
    if constexpr (AXIS == 2)
      centre = source(cok ? J : 0)[K];
    else
      centre = input(K);
    for (int m = t / CT; m <= n; m += NT / CT) lds[m * CP + c] = m % 2 ? 0.0 : (m / 2) % 2 ? -2.0 * centre : 2.0 * centre;
  }
  __syncthreads();
  if (rows) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int k = wave * 16 + lane / 16 + 4 * r;
      if (k < K) {
#pragma unroll
        for (int g = 0; g < CG; ++g) {
          const int cc = 16 * g + lane % 16;
          const double e = acc[0][g][r], o = acc[1][g][r];
          const int m0 = VICO ? k : 2 * k, m1 = VICO ? n - k : 2 * k + 1;
          lds[m0 * CP + cc] += VICO ? e + o : e;
          lds[m1 * CP + cc] += VICO ? e - o : o;
        }
      }
    }
  }
  if (t < CT) lds[(VICO ? K : n) * CP + t] += left[t];
  __syncthreads();

  // ---- out
  if constexpr (AXIS == 2) {
    // octant [k1][k2 tile][k0][tile]: a tile's rows of adjacent k0 are contiguous
    const int tile = a.tile, tiles = (n + tile) / tile;
#pragma unroll 2
    for (int e = t; e < tiles * CT * tile; e += NT) {
      const int q = e % tile, cc = (e / tile) % CT, tl = e / (tile * CT);
      const int Jc = J0 + cc, k2 = tl * tile + q;
      if (Jc >= a.N) continue;
      const int k1 = Jc / (a.n0 + 1), k0 = Jc - k1 * (a.n0 + 1);
      const double v = k2 <= n ? a.scale * lds[k2 * CP + cc] : 0.0;
      const long long at = (((long long)k1 * tiles + tl) * (a.n0 + 1) + k0) * tile + q;
      if (a.f64)
        static_cast<double*>(a.octant)[at] = v;
      else
        static_cast<float*>(a.octant)[at] = (float)v;
    }
  } else if (cok) {
    double* y = AXIS == 0 ? a.y + J : a.y + (long long)(J / a.p2) * (n + 1) * a.p2 + J % a.p2;
    const long long sm = AXIS == 0 ? a.N : a.p2;
#pragma unroll 4
    for (int m = t / CT; m <= n; m += NT / CT) y[m * sm] = lds[m * CP + c];
  }
}

// 32 columns a block reuse a matrix operand twice; 16 where 32 leave compute
// units idle, and from n = 256 on, where the LDS of 32 leaves one or two blocks a
// compute unit, whose fill and products then wait for each other (256^3
// Hockney-Eastwood 455 -> 437 us, 384^3 Vico-Greengard 4590 -> 4380, 512^3 12440
// -> 12140; 256^3 Vico-Greengard equal).
template <bool VICO, int AXIS, int NMAX, int WAVES>
hipError_t launch_size(const AxisArgs& a, hipStream_t s) {
  static_assert(16 * WAVES >= NMAX / 2, "the waves cover the rows");
  if (NMAX >= 256 || (NMAX <= 128 && a.N < 32 * 512)) {
    if constexpr (NMAX != 192)
      hipLaunchKernelGGL((k_green_axis<VICO, AXIS, NMAX, WAVES, 1>), dim3((a.N + 15) / 16), dim3(64 * WAVES), 0, s, a);
  } else {
    if constexpr (NMAX < 256)
      hipLaunchKernelGGL((k_green_axis<VICO, AXIS, NMAX, WAVES, 2>), dim3((a.N + 31) / 32), dim3(64 * WAVES), 0, s, a);
  }
  return hipGetLastError();
}

// A wave takes one 16-row block: with two, as many waves again are missing to
// hide the fill's and the samples' latency (two / one, Vico-Greengard: 256^3 1205
// / 1055 us, 384^3 5720 / 4590, 512^3 12380 / 12400).
template <bool VICO, int AXIS>
hipError_t launch_axis(const AxisArgs& a, hipStream_t s) {
  if (a.n <= 64) return launch_size<VICO, AXIS, 64, 4>(a, s);
  if (a.n <= 128) return launch_size<VICO, AXIS, 128, 4>(a, s);
  if (a.n <= 192) return launch_size<VICO, AXIS, 192, 6>(a, s);
  if (a.n <= 256) return launch_size<VICO, AXIS, 256, 8>(a, s);
  if (a.n <= 384) return launch_size<VICO, AXIS, 384, 12>(a, s);
  if (a.n <= 512) return launch_size<VICO, AXIS, 512, 16>(a, s);
  return hipErrorInvalidValue;
}

}  // namespace

size_t green_axis_image_elems(int n) {
  const size_t K = n / 2, ks = (K + 3) / 4, pb = (K + 15) / 16;
  return ks * pb * 128 + 4 * ks;
}

hipError_t green_axis_image(double* out, int n, bool vico, hipStream_t s) {
  const unsigned blocks = (unsigned)((green_axis_image_elems(n) + 255) / 256);
  hipLaunchKernelGGL(k_axis_image, dim3(blocks), dim3(256), 0, s, out, n, vico ? 1 : 0);
  return hipGetLastError();
}

hipError_t green_axis(const AxisArgs& a, bool vico, int axis, hipStream_t s) {
  // rows in blocks of 16 inputs pairs: n even; every n a plan accepts is a multiple of 4
  if (a.n < 4 || a.n % 4 != 0 || a.N < 1 || a.p2 < 1) return hipErrorInvalidValue;
  switch (axis) {
    case 0: return vico ? launch_axis<true, 0>(a, s) : launch_axis<false, 0>(a, s);
    case 1: return vico ? launch_axis<true, 1>(a, s) : launch_axis<false, 1>(a, s);
    case 2: return vico ? launch_axis<true, 2>(a, s) : launch_axis<false, 2>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fsp
