// Time-domain signals (Sec. III-F): impulse responses from the spectra (Eqs. 5-6, 9-10, 13:
// h = F^-1[H]) and received signals (Eq. 14: s = h * s_e).
//
// Impulse response of receiver m on t_n = n dt, dt = 1 / (n_t df), n < n_t:
//   h_m(t_n) = 2 df Re[ e^{-j sigma 2 pi f_lo t_n} sum_{k<F} H_m[k] e^{-j sigma 2 pi k n / n_t} ],
// so the inner sum is a length-n_t DFT of the zero-padded spectrum (sign -sigma), then a
// carrier-and-scale pass with the carrier phase reduced in FP64.  The received signal is the
// linear convolution s_m[n] = dt sum_k h_m[k] s_e[n - k] by FFT of length P (zero padding),
// spectral product and inverse FFT.
//
// Rows of up to 2^15 samples and calls of up to 2^12 are one launch each: transforms of up to 2^13 points lie in
// one workgroup's registers (16 points a thread) and are exchanged through LDS between radix-16 passes.  An impulse
// response of N = D N1 points is D such transforms, one per residue n mod D (decimation in
// frequency), padding and carrier in the same kernel; the convolution is cut into blocks (overlap-save).
// Longer rows and calls, and outputs that share memory with an input, run radix-4
// Stockham stages over global memory (plus one radix-2 stage for an odd power of two), each a streaming pass, with
// twiddles from a table, computed in FP64 and rounded to FP32; in a workgroup they stay in FP64, and a product is
// rounded once.
// Measured, both calls one after the other: 32 responses of 16,384 samples from 4,096 bins and their convolution with
// 640 samples 168 -> 20 us (bound by the one chain of passes and barriers of each workgroup; 26 us before the
// three transforms of a block shared their twiddles' first powers and formed the others by halves); error against FP64 1.26e-7 -> 1.11e-7 and 1.43e-7 -> 1.34e-7.
#include "internal.hpp"

#include <algorithm>
#include <cmath>

namespace et {

namespace {

constexpr int TB = 256;

inline unsigned tgrid(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + TB - 1) / TB, 65536)); }

// tw[m] = e^{sign j 2 pi m / N}, m < N, from FP64 sincospi rounded to FP32.
__global__ void k_twiddles(float2* __restrict__ tw, int64_t N, int sign) {
  for (int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; m < N; m += (int64_t)gridDim.x * blockDim.x) {
    double sn, cs;
    sincospi((double)sign * 2.0 * (double)m / (double)N, &sn, &cs);
    tw[m] = make_float2((float)cs, (float)sn);
  }
}

__device__ inline float2 cmulf(float2 a, float2 b) { return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
// sign j (a + j b): a quarter turn in the transform's direction
__device__ inline float2 qturn(float2 a, int sign) { return sign > 0 ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x); }

// Butterflies of one Stockham stage, sub-transforms of length Ns growing to R Ns (R = 2 or 4):
// for j < N / R with k = j % Ns, v_r = x[j + r N / R] e^{sign j 2 pi r k / (R Ns)}, then the
// R-point DFT of v, y[(j / Ns) R Ns + k + q Ns] = sum_r v_r e^{sign j 2 pi r q / R}.  After
// log2 N stages y is the DFT of the row in natural order.
template <int R>
__device__ inline void stockham_butterfly(const float2* __restrict__ x, float2* __restrict__ y, int64_t N, int64_t Ns,
                                          int64_t j, const float2* __restrict__ tw, int sign) {
  const int64_t k = j % Ns, q0 = (j / Ns) * R * Ns + k;
  const int64_t step = N / (R * Ns);   // table stride of e^{sign j 2 pi k / (R Ns)}
  if (R == 2) {
    const float2 a = x[j], b = cmulf(x[j + N / 2], tw[k * step]);
    y[q0] = make_float2(a.x + b.x, a.y + b.y);
    y[q0 + Ns] = make_float2(a.x - b.x, a.y - b.y);
  } else {
    const int64_t qN = N / 4;
    const float2 v0 = x[j];
    const float2 v1 = cmulf(x[j + qN], tw[k * step]);
    const float2 v2 = cmulf(x[j + 2 * qN], tw[2 * k * step]);
    const float2 v3 = cmulf(x[j + 3 * qN], tw[3 * k * step]);
    const float2 s02 = make_float2(v0.x + v2.x, v0.y + v2.y), d02 = make_float2(v0.x - v2.x, v0.y - v2.y);
    const float2 s13 = make_float2(v1.x + v3.x, v1.y + v3.y), d13 = qturn(make_float2(v1.x - v3.x, v1.y - v3.y), sign);
    y[q0] = make_float2(s02.x + s13.x, s02.y + s13.y);
    y[q0 + Ns] = make_float2(d02.x + d13.x, d02.y + d13.y);
    y[q0 + 2 * Ns] = make_float2(s02.x - s13.x, s02.y - s13.y);
    y[q0 + 3 * Ns] = make_float2(d02.x - d13.x, d02.y - d13.y);
  }
}

// One stage over global memory for `rows` transforms of length N.
template <int R>
__global__ void k_fft_stage(const float2* __restrict__ x, float2* __restrict__ y, int64_t rows, int64_t N, int64_t Ns,
                            const float2* __restrict__ tw, int sign) {
  const int64_t per = N / R;
  const int64_t total = rows * per;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = t / per, j = t - r * per;
    stockham_butterfly<R>(x + r * N, y + r * N, N, Ns, j, tw, sign);
  }
}

// DFT of every row (length N, a power of two) with e^{sign j 2 pi k n / N}: a holds the input;
// returns the buffer holding the result (a or b).  tw: N entries of scratch for the table.
float2* fft_rows(float2* a, float2* b, float2* tw, int64_t rows, int64_t N, int sign, hipStream_t s) {
  k_twiddles<<<tgrid(N), TB, 0, s>>>(tw, N, sign);
  float2* x = a;
  float2* y = b;
  int lg = 0;
  while ((int64_t(1) << lg) < N) ++lg;
  int64_t Ns = 1;
  if (lg & 1) {
    k_fft_stage<2><<<tgrid(rows * (N / 2)), TB, 0, s>>>(x, y, rows, N, Ns, tw, sign);
    std::swap(x, y);
    Ns = 2;
  }
  for (; Ns < N; Ns *= 4) {
    k_fft_stage<4><<<tgrid(rows * (N / 4)), TB, 0, s>>>(x, y, rows, N, Ns, tw, sign);
    std::swap(x, y);
  }
  ET_HIP(hipGetLastError());
  return x;
}

__global__ void k_pad_spectra(const float* __restrict__ H, int64_t M, int64_t F, int64_t N, float2* __restrict__ out) {
  const int64_t total = M * N;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t m = t / N, k = t - m * N;
    out[t] = k < F ? make_float2(H[(m * F + k) * 2], H[(m * F + k) * 2 + 1]) : make_float2(0.f, 0.f);
  }
}

// h[m][n] = 2 df Re(e^{-j sigma 2 pi f_lo n dt} S[m][n]); the carrier phase f_lo n dt is reduced
// to a fraction of a cycle in FP64.
__global__ void k_carrier(const float2* __restrict__ S, int64_t M, int64_t N, double f_lo_dt, int sigma, double scale,
                          float* __restrict__ h) {
  const int64_t total = M * N;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t n = t % N;
    const double cyc = f_lo_dt * (double)n;
    double sn, cs;
    sincospi(-2.0 * (double)sigma * (cyc - floor(cyc)), &sn, &cs);
    const float2 v = S[t];
    h[t] = (float)(scale * ((double)v.x * cs - (double)v.y * sn));
  }
}

// rows 0..M-1: h zero-padded to P; row M: the emitted call zero-padded to P
__global__ void k_pad_signals(const float* __restrict__ h, int64_t M, int64_t n_t, const float* __restrict__ se,
                              int64_t L, int64_t P, float2* __restrict__ out) {
  const int64_t total = (M + 1) * P;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t m = t / P, i = t - m * P;
    float v = 0.f;
    if (m < M) v = i < n_t ? h[m * n_t + i] : 0.f;
    else v = i < L ? se[i] : 0.f;
    out[t] = make_float2(v, 0.f);
  }
}

__global__ void k_spectral_product(float2* __restrict__ X, int64_t M, int64_t P) {
  const int64_t total = M * P;
  const float2* E = X + M * P;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const float2 a = X[t], b = E[t % P];
    X[t] = make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
  }
}

__global__ void k_unpack_signal(const float2* __restrict__ Y, int64_t M, int64_t P, int64_t n_out, double scale,
                                float* __restrict__ out) {
  const int64_t total = M * n_out;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t m = t / n_out, i = t - m * n_out;
    out[t] = (float)(scale * (double)Y[m * P + i].x);
  }
}

// ---- transforms in one workgroup

// A twiddle applied in FP64 and rounded once.
__device__ inline float2 twiddle(float2 v, double2 w) {
  return make_float2((float)((double)v.x * w.x - (double)v.y * w.y), (float)((double)v.x * w.y + (double)v.y * w.x));
}
// R-point DFT with e^{-j 2 pi r q / R}, natural order in and out.
template <int R>
__device__ inline void dft(float2 (&v)[R]);
template <>
__device__ inline void dft<1>(float2 (&)[1]) {}
template <>
__device__ inline void dft<2>(float2 (&v)[2]) {
  const float2 a = v[0], b = v[1];
  v[0] = make_float2(a.x + b.x, a.y + b.y);
  v[1] = make_float2(a.x - b.x, a.y - b.y);
}
template <>
__device__ inline void dft<4>(float2 (&v)[4]) {
  const float2 s02 = make_float2(v[0].x + v[2].x, v[0].y + v[2].y), d02 = make_float2(v[0].x - v[2].x, v[0].y - v[2].y);
  const float2 s13 = make_float2(v[1].x + v[3].x, v[1].y + v[3].y), d13 = qturn(make_float2(v[1].x - v[3].x, v[1].y - v[3].y), -1);
  v[0] = make_float2(s02.x + s13.x, s02.y + s13.y);
  v[1] = make_float2(d02.x + d13.x, d02.y + d13.y);
  v[2] = make_float2(s02.x - s13.x, s02.y - s13.y);
  v[3] = make_float2(d02.x - d13.x, d02.y - d13.y);
}
constexpr double COS8 = 0.92387953251128673848, SIN8 = 0.38268343236508978178, RT2 = 0.70710678118654752440;
// e^{-j 2 pi m / 16} for the products of two factors of 16
__device__ inline double2 w16(int m) {
  return m == 1 ? make_double2(COS8, -SIN8) : m == 2 ? make_double2(RT2, -RT2) : m == 3 ? make_double2(SIN8, -COS8)
       : m == 6 ? make_double2(-RT2, -RT2) : make_double2(-COS8, SIN8);   // m == 9
}
template <int R>
__device__ inline void dft(float2 (&v)[R]) {   // R = 8, 16: columns of four, then rows of R / 4
  constexpr int C = R / 4;
  float2 a[C][4];
#pragma unroll
  for (int c = 0; c < C; ++c) {
#pragma unroll
    for (int k = 0; k < 4; ++k) a[c][k] = v[c + C * k];
    dft<4>(a[c]);
#pragma unroll
    for (int k = 1; k < 4; ++k) {
      const int m = c * k * (16 / R);
      if (m == 4) a[c][k] = qturn(a[c][k], -1);
      else if (m) a[c][k] = twiddle(a[c][k], w16(m));
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    float2 b[C];
#pragma unroll
    for (int c = 0; c < C; ++c) b[c] = a[c][k];
    dft<C>(b);
#pragma unroll
    for (int q = 0; q < C; ++q) v[k + 4 * q] = b[q];
  }
}

__device__ inline double2 cmuld(double2 a, double2 b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
__device__ inline double2 cis_pi(double x) {
  double sn, cs;
  sincospi(x, &sn, &cs);
  return make_double2(cs, sn);
}

// A row of 2^LG points held by T threads: thread t has points t + T q, q < E, before and after.
template <int LG>
struct Row {
  static constexpr int N = 1 << LG, E = N < 16 ? N : 16, T = N / E;
  static constexpr int R0 = LG % 4 ? 1 << LG % 4 : E;   // radix of the first pass, the others 16
  static constexpr int LDS = N + N / 16;                // points, one in 17 left free (no two of a wave's on a bank)
};
__device__ inline int lds_at(int i) { return i + (i >> 4); }

// The first powers of a thread's twiddles, one per radix-16 pass after the first pass.
template <int LG>
struct Twiddles {
  static constexpr int P = (LG - 1) / 4;
  double2 w[P > 0 ? P : 1];
  __device__ inline explicit Twiddles(int t) {
    int Ns = Row<LG>::R0;
#pragma unroll
    for (int p = 0; p < P; ++p, Ns *= 16) w[p] = cis_pi(-2.0 * (double)(t & (Ns - 1)) / (16.0 * Ns));
  }
};

// One radix-16 pass, sub-transforms of length Ns growing to 16 Ns, then the following ones.
template <int LG, int Ns, int PASS = 0>
__device__ inline void row_passes(float2 (&v)[Row<LG>::E], float2* lds, int t, const Twiddles<LG>& tw) {
  using W = Row<LG>;
  if constexpr (Ns < W::N) {
    const int k = t & (Ns - 1);
    // powers by halves: w^r = w^(r / 2) w^(r - r / 2)
    double2 w[16];
    w[1] = tw.w[PASS];
#pragma unroll
    for (int r = 1; r < 16; ++r) {
      if (r > 1) w[r] = cmuld(w[r / 2], w[r - r / 2]);
      v[r] = twiddle(v[r], w[r]);
    }
    dft<16>(v);
    if constexpr (16 * Ns < W::N) {
      __syncthreads();
#pragma unroll
      for (int q = 0; q < 16; ++q) lds[lds_at((t - k) * 16 + k + q * Ns)] = v[q];
      __syncthreads();
#pragma unroll
      for (int q = 0; q < 16; ++q) v[q] = lds[lds_at(t + W::T * q)];
      row_passes<LG, 16 * Ns, PASS + 1>(v, lds, t, tw);
    }
  }
}

// DFT with e^{-j 2 pi k n / N} of the row in v (Stockham order; the other sign by swapping parts before and after).
template <int LG>
__device__ inline void row_fft(float2 (&v)[Row<LG>::E], float2* lds, int t, const Twiddles<LG>& tw) {
  using W = Row<LG>;
  constexpr int B = W::E / W::R0;
  float2 u[B][W::R0];
#pragma unroll
  for (int b = 0; b < B; ++b) {
#pragma unroll
    for (int r = 0; r < W::R0; ++r) u[b][r] = v[b + r * B];
    dft<W::R0>(u[b]);
  }
  if constexpr (W::N == W::R0) {
#pragma unroll
    for (int r = 0; r < W::R0; ++r) v[r] = u[0][r];
  } else {
    __syncthreads();
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
      for (int q = 0; q < W::R0; ++q) lds[lds_at((t + b * W::T) * W::R0 + q)] = u[b][q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < W::E; ++q) v[q] = lds[lds_at(t + W::T * q)];
    row_passes<LG, W::R0>(v, lds, t, tw);
  }
}

// Impulse response of row m at n = d + D n' (workgroup = (m, d)), N = D 2^LG.  With y[k] = w^{d k} sum_r x[k + r N1]
// e^{sign j 2 pi d r / D}, w = e^{sign j 2 pi / N}, the samples are the transform of y; then the carrier,
// whose phase f_lo n dt is reduced to a fraction of a cycle in FP64, its steps of D T samples by FP64 products.
template <int LG>
__global__ __launch_bounds__(Row<LG>::T) void k_impulse(const float* __restrict__ H, int F, int D, double f_lo_dt,
                                                        int sigma, double scale, float* __restrict__ h) {
  using W = Row<LG>;
  __shared__ float2 lds[W::LDS];
  const int t = threadIdx.x, d = blockIdx.x;
  const int64_t m = blockIdx.y, N = (int64_t)D << LG;
  const float* x = H + 2 * m * F;
  float2 v[W::E];
#pragma unroll
  for (int q = 0; q < W::E; ++q) {
    const int k = t + W::T * q;
    v[q] = k < F ? make_float2(x[2 * k], x[2 * k + 1]) : make_float2(0.f, 0.f);
  }
  for (int r = 1; r < D && (int64_t)r * W::N < F; ++r) {
    const double2 c = cis_pi(-2.0 * sigma * (double)(d * r % D) / (double)D);
#pragma unroll
    for (int q = 0; q < W::E; ++q) {
      const int64_t k = t + W::T * q + (int64_t)r * W::N;
      if (k < F) {
        const float2 p = twiddle(make_float2(x[2 * k], x[2 * k + 1]), c);
        v[q].x += p.x;
        v[q].y += p.y;
      }
    }
  }
  if (d > 0) {
    double2 w = cis_pi(-2.0 * sigma * (double)((int64_t)d * t) / (double)N);
    const double2 ws = cis_pi(-2.0 * sigma * (double)((int64_t)d * W::T) / (double)N);
#pragma unroll
    for (int q = 0; q < W::E; ++q) {
      v[q] = twiddle(v[q], w);
      w = cmuld(w, ws);
    }
  }
  // forward DFT for sigma = +1; the other direction with real and imaginary parts swapped
  if (sigma < 0) {
#pragma unroll
    for (int q = 0; q < W::E; ++q) v[q] = make_float2(v[q].y, v[q].x);
  }
  row_fft<LG>(v, lds, t, Twiddles<LG>(t));
  if (sigma < 0) {
#pragma unroll
    for (int q = 0; q < W::E; ++q) v[q] = make_float2(v[q].y, v[q].x);
  }
  const double c0 = f_lo_dt * (double)(d + (int64_t)D * t), cs = f_lo_dt * (double)((int64_t)D * W::T);
  double2 c = cis_pi(-2.0 * sigma * (c0 - floor(c0)));
  const double2 step = cis_pi(-2.0 * sigma * (cs - floor(cs)));
#pragma unroll
  for (int q = 0; q < W::E; ++q) {
    h[m * N + d + (int64_t)D * (t + W::T * q)] = (float)(scale * ((double)v[q].x * c.x - (double)v[q].y * c.y));
    c = cmuld(c, step);
  }
}

// Linear convolution of row m with the call (workgroup = (block b, m)): 2^LG - L + 1 samples from
// as many points of input, the wrapped L - 1 dropped.  (Two rows as real and imaginary part would halve the
// work but add the rounding of one to the other: error against FP64 2.2e-7, apart 1.6e-7, both before the products were taken in FP64.)
template <int LG>
__global__ __launch_bounds__(Row<LG>::T) void k_convolve(const float* __restrict__ h, int64_t n_t,
                                                         const float* __restrict__ se, int L, double scale,
                                                         float* __restrict__ out) {
  using W = Row<LG>;
  __shared__ float2 lds[W::LDS];
  const int t = threadIdx.x;
  const int64_t V = W::N - L + 1, n_out = n_t + L - 1, i0 = blockIdx.x * V - (L - 1), m = blockIdx.y;
  float2 e[W::E], v[W::E];
#pragma unroll
  for (int q = 0; q < W::E; ++q) {
    const int k = t + W::T * q;
    e[q] = make_float2(k < L ? se[k] : 0.f, 0.f);
  }
  const Twiddles<LG> tw(t);
  row_fft<LG>(e, lds, t, tw);
#pragma unroll
  for (int q = 0; q < W::E; ++q) {
    const int64_t i = i0 + t + W::T * q;
    v[q] = make_float2(i >= 0 && i < n_t ? h[m * n_t + i] : 0.f, 0.f);
  }
  row_fft<LG>(v, lds, t, tw);
#pragma unroll
  for (int q = 0; q < W::E; ++q) {
    const float2 p = twiddle(v[q], make_double2(e[q].x, e[q].y));
    v[q] = make_float2(p.y, p.x);   // swapped: the inverse direction
  }
  row_fft<LG>(v, lds, t, tw);
#pragma unroll
  for (int q = 0; q < W::E; ++q) {
    const int n = t + W::T * q;
    const int64_t o = i0 + n;
    if (n >= L - 1 && o < n_out) out[m * n_out + o] = (float)(scale * (double)v[q].y);
  }
}

// Points of the transforms of an impulse response of N samples (log2), -1 for the stages over global memory.  Up to
// 2^10 points a row is one workgroup; then residues of 2^10 or 2^12 points spread a row over up to eight.  At 2^16
// samples with as many bins each of 16 residues would read all of them: 64 us against the stages' 53.
int impulse_lg(int64_t N) {
  int lg = 0;
  while ((int64_t(1) << lg) < N) ++lg;
  if (lg > 15) return -1;
  return lg > 12 ? 12 : lg > 10 ? 10 : lg;
}
// Points of the blocks of a convolution with a call of L samples: at least twice the call, so that half
// of each block is new output.  2^14 points spill registers: 16 rows of 16,384 samples and a call of 6,000 took
// 96 us, the stages 90.
int convolve_lg(int64_t L) {
  int lg = 10;
  while ((int64_t(1) << lg) < 2 * L) ++lg;
  return lg <= 13 ? lg : -1;
}

inline size_t al(size_t b) { return (b + 255) / 256 * 256; }

// An output that shares memory with an input: a workgroup would write what others have yet to read, so such calls take
// the stages, which copy their inputs to the workspace first (sized for them whichever way a call goes).
bool overlap(const void* a, size_t na, const void* b, size_t nb) {
  return (uintptr_t)a < (uintptr_t)b + nb && (uintptr_t)b < (uintptr_t)a + na;
}

}  // namespace

int64_t conv_length(int64_t n_t, int64_t L) {
  int64_t P = 1;
  while (P < n_t + L - 1) P <<= 1;
  return P;
}

size_t impulse_ws_bytes(int64_t M, int64_t n_t) {
  return 2 * al(sizeof(float2) * (size_t)M * n_t) + al(sizeof(float2) * (size_t)n_t);
}

size_t signal_ws_bytes(int64_t M, int64_t n_t, int64_t L) {
  const int64_t P = conv_length(n_t, L);
  return 2 * al(sizeof(float2) * (size_t)(M + 1) * P) + al(sizeof(float2) * (size_t)P);
}

void impulse_run(int64_t M, int64_t F, double f_lo, double df, int sigma, const float* spectra, int64_t n_t, void* ws,
                 float* h, hipStream_t s) {
  const double f_lo_dt = f_lo * (1.0 / ((double)n_t * df)), scale = 2.0 * df;
  const int lg = impulse_lg(n_t);
  if (lg >= 0 && !overlap(spectra, sizeof(float) * 2 * (size_t)M * F, h, sizeof(float) * (size_t)M * n_t)) {
    const int D = (int)(n_t >> lg);
    for (int64_t m0 = 0; m0 < M; m0 += 65535) {   // (the grid's second dimension)
      const dim3 grid((unsigned)D, (unsigned)std::min<int64_t>(M - m0, 65535));
      const float* x = spectra + 2 * m0 * F;
      float* y = h + m0 * n_t;
      switch (lg) {
#define ET_ROW(LG) \
  case LG: k_impulse<LG><<<grid, Row<LG>::T, 0, s>>>(x, (int)F, D, f_lo_dt, sigma, scale, y); break
        ET_ROW(0); ET_ROW(1); ET_ROW(2); ET_ROW(3); ET_ROW(4); ET_ROW(5); ET_ROW(6); ET_ROW(7); ET_ROW(8); ET_ROW(9);
        ET_ROW(10); ET_ROW(12);
#undef ET_ROW
      }
    }
    ET_HIP(hipGetLastError());
    return;
  }
  float2* a = (float2*)ws;
  float2* b = (float2*)((char*)ws + al(sizeof(float2) * (size_t)M * n_t));
  float2* tw = (float2*)((char*)ws + 2 * al(sizeof(float2) * (size_t)M * n_t));
  k_pad_spectra<<<tgrid(M * n_t), TB, 0, s>>>(spectra, M, F, n_t, a);
  // sum_k H_k e^{-j sigma 2 pi k n / n_t}: forward DFT for sigma = +1, inverse direction for -1
  float2* S = fft_rows(a, b, tw, M, n_t, -sigma, s);
  k_carrier<<<tgrid(M * n_t), TB, 0, s>>>(S, M, n_t, f_lo_dt, sigma, scale, h);
  ET_HIP(hipGetLastError());
}

void signal_run(int64_t M, int64_t n_t, const float* h, int64_t L, const float* se, double dt, void* ws, float* out,
                hipStream_t s) {
  const int lg = convolve_lg(L);
  const size_t out_bytes = sizeof(float) * (size_t)M * (n_t + L - 1);
  if (lg >= 0 && !overlap(h, sizeof(float) * (size_t)M * n_t, out, out_bytes) &&
      !overlap(se, sizeof(float) * (size_t)L, out, out_bytes)) {
    const int64_t V = (int64_t(1) << lg) - L + 1, n_out = n_t + L - 1;
    for (int64_t m0 = 0; m0 < M; m0 += 65535) {
      const dim3 grid((unsigned)((n_out + V - 1) / V), (unsigned)std::min<int64_t>(M - m0, 65535));
      const float* x = h + m0 * n_t;
      float* y = out + m0 * n_out;
      switch (lg) {
#define ET_ROW(LG) \
  case LG: k_convolve<LG><<<grid, Row<LG>::T, 0, s>>>(x, n_t, se, (int)L, dt / (double)(1 << LG), y); break
        ET_ROW(10); ET_ROW(11); ET_ROW(12); ET_ROW(13);
#undef ET_ROW
      }
    }
    ET_HIP(hipGetLastError());
    return;
  }
  const int64_t P = conv_length(n_t, L);
  float2* a = (float2*)ws;
  float2* b = (float2*)((char*)ws + al(sizeof(float2) * (size_t)(M + 1) * P));
  float2* tw = (float2*)((char*)ws + 2 * al(sizeof(float2) * (size_t)(M + 1) * P));
  k_pad_signals<<<tgrid((M + 1) * P), TB, 0, s>>>(h, M, n_t, se, L, P, a);
  float2* X = fft_rows(a, b, tw, M + 1, P, -1, s);
  k_spectral_product<<<tgrid(M * P), TB, 0, s>>>(X, M, P);
  float2* other = X == a ? b : a;
  float2* Y = fft_rows(X, other, tw, M, P, +1, s);   // only the M product rows
  k_unpack_signal<<<tgrid(M * (n_t + L - 1)), TB, 0, s>>>(Y, M, P, n_t + L - 1, dt / (double)P, out);
  ET_HIP(hipGetLastError());
}

}  // namespace et
