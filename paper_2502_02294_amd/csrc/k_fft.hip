// FFTs for the particle-mesh Poisson solve and the initial conditions (Sec. 2.1, 2.2), with
// the spectral operators fused into the z pass.
//
// Half spectrum layout: spec[(kz * n + ky) * nh + kx], nh = n/2 + 1, kx = 0..n/2.
// Forward transforms are unnormalised; every spectral operator carries the 1/N^3 of the
// inverse.  Passes:
//   plane_forward, plane_inverse   x and y lines of a z plane (n <= 128)
//   x_r2c     rows of n reals -> n/2+1 complex (n = 256)
//   pencil<1> y lines (all (z, kx) lines of a sample, tk consecutive ones per block; n = 256)
//   pencil<2> z lines ((ky, kx) lines): forward, spectral operator, inverse, each optional,
//             and optional accumulation into the output
//   x_c2r     Hermitian extension of each row, inverse FFT, real part times a scale (n = 256).
//
// Each n-point line transform is the four-step factorisation n = N1 * N2 with both factors
// done in registers and one transpose through LDS:
//   X[k1 + N1 k2] = sum_j2 W_N2^(j2 k2) W_n^(j2 k1) sum_j1 x[j2 + N2 j1] W_N1^(j1 k1).
// Natural order "D_x": N2 threads per line, thread q holds x[q + N2 r], r < N1.
// Spectral order "D_k": N1 threads per line, thread q holds X[q + N1 r], r < N2.
// The forward transform maps D_x to D_k, the inverse D_k to D_x:
//   x[a + N2 b] = sum_k1 W_N1^(-b k1) W_n^(-a k1) sum_k2 X[k1 + N1 k2] W_N2^(-a k2).
#include <cmath>
#include <vector>

#include "dh_kernels.h"

namespace dh {

namespace {

constexpr int kFftThreads = 256;
constexpr int kMaxR = 16;

// hides how x was formed from the compiler: it is rounded before any sum it enters
__device__ __forceinline__ float opaque(float x) {
  asm volatile("" : "+v"(x));
  return x;
}

__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// cos and sin of 2 pi e / 16, e = 0..7
__device__ constexpr float kCos16[8] = {1.0f, 0.92387953251128674f, 0.70710678118654752f,
                                        0.38268343236508977f, 0.0f, -0.38268343236508977f,
                                        -0.70710678118654752f, -0.92387953251128674f};
__device__ constexpr float kSin16[8] = {0.0f, 0.38268343236508977f, 0.70710678118654752f,
                                        0.92387953251128674f, 1.0f, 0.92387953251128674f,
                                        0.70710678118654752f, 0.38268343236508977f};

// x * W_16^(+-e): forward exp(-2 pi i e / 16), inverse exp(+2 pi i e / 16); e is a constant
template <bool INV>
__device__ __forceinline__ float2 rot16(float2 x, int e) {
  if (e == 0) return x;
  if (e == 4) return INV ? make_float2(-x.y, x.x) : make_float2(x.y, -x.x);
  const float c = kCos16[e], s = INV ? kSin16[e] : -kSin16[e];
  return make_float2(x.x * c - x.y * s, x.x * s + x.y * c);
}

constexpr int bit_reverse(int i, int bits) {
  int r = 0;
  for (int b = 0; b < bits; ++b) r |= ((i >> b) & 1) << (bits - 1 - b);
  return r;
}
constexpr int log2c(int r) { return r <= 1 ? 0 : 1 + log2c(r / 2); }

// In-register R-point DFT (R = 2, 4, 8, 16) of v[0..R-1], natural order in and out: radix-2
// decimation in time after a bit-reversal permutation, twiddles as constants.
template <int R, bool INV>
__device__ __forceinline__ void dft_reg(float2 (&v)[kMaxR]) {
  constexpr int bits = log2c(R);
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const int j = bit_reverse(i, bits);
    if (j > i) {
      const float2 t = v[i];
      v[i] = v[j];
      v[j] = t;
    }
  }
#pragma unroll
  for (int m = 2; m <= R; m <<= 1) {
#pragma unroll
    for (int k = 0; k < R; k += m)
#pragma unroll
      for (int j = 0; j < m / 2; ++j) {
        const float2 t = rot16<INV>(v[k + j + m / 2], j * (16 / m));
        const float2 u = v[k + j];
        v[k + j] = cadd(u, t);
        v[k + j + m / 2] = csub(u, t);
      }
  }
}

// W_n^m (forward sign) from the half table tw[m] = exp(-2 pi i m / n), m < n/2
__device__ __forceinline__ float2 tw_full(const float2* tw, int m, int n) {
  const int h = n >> 1;
  const float2 w = tw[m & (h - 1)];
  return m < h ? w : make_float2(-w.x, -w.y);
}

// The transpose of a line transform through this line's exchange buffer ex (n floats): the
// writer thread q puts v[i] (i < NW) at [i WS + q], the reader thread q takes v[j] (j < NR)
// from [q RS + j]; real parts first, then imaginary parts, so the buffer is half the size
// of a complex one (more blocks per CU).  Element e of the buffer is at ex[e ES].  A caller
// that writes ex again needs a barrier first.
template <int NW, int WS, int NR, int RS, int ES>
__device__ __forceinline__ void exchange(float2 (&v)[kMaxR], float* ex, int q, bool writer,
                                         bool reader) {
  float re[kMaxR];
  if (writer)
#pragma unroll
    for (int i = 0; i < NW; ++i) ex[(i * WS + q) * ES] = v[i].x;
  __syncthreads();
  if (reader)
#pragma unroll
    for (int j = 0; j < NR; ++j) re[j] = ex[(q * RS + j) * ES];
  __syncthreads();
  if (writer)
#pragma unroll
    for (int i = 0; i < NW; ++i) ex[(i * WS + q) * ES] = v[i].y;
  __syncthreads();
  if (reader)
#pragma unroll
    for (int j = 0; j < NR; ++j) v[j] = make_float2(re[j], ex[(q * RS + j) * ES]);
}

// Forward line transform: D_x (thread q < N2 of the line) -> D_k (thread q < N1).
// ex: this line's exchange buffer (n floats, ES apart), tw: twiddle half table in LDS.
template <int N1, int N2, int ES = 1>
__device__ __forceinline__ void line_forward(float2 (&v)[kMaxR], float* ex, const float2* tw,
                                             int q, bool in_x, bool in_k) {
  constexpr int n = N1 * N2;
  if (in_x) {   // q = j2: DFT over j1, then W_n^(j2 k1), to [k1 * N2 + j2]
    dft_reg<N1, false>(v);
#pragma unroll
    for (int k1 = 0; k1 < N1; ++k1) v[k1] = cmul(v[k1], tw_full(tw, q * k1, n));
  }
  exchange<N1, N2, N2, N2, ES>(v, ex, q, in_x, in_k);
  if (in_k) dft_reg<N2, false>(v);   // q = k1: DFT over j2 gives X[k1 + N1 k2]
}

// Inverse line transform: D_k (thread q < N1) -> D_x (thread q < N2), unnormalised.
template <int N1, int N2, int ES = 1>
__device__ __forceinline__ void line_inverse(float2 (&v)[kMaxR], float* ex, const float2* tw,
                                             int q, bool in_x, bool in_k) {
  constexpr int n = N1 * N2;
  if (in_k) {   // q = k1: inverse DFT over k2 gives index a; times W_n^(-a k1); to [a * N1 + k1]
    dft_reg<N2, true>(v);
#pragma unroll
    for (int a = 0; a < N2; ++a) {
      const float2 w = tw_full(tw, a * q, n);
      v[a] = cmul(v[a], make_float2(w.x, -w.y));
    }
  }
  exchange<N2, N1, N1, N1, ES>(v, ex, q, in_k, in_x);
  if (in_x) dft_reg<N1, true>(v);   // q = a: inverse DFT over k1 gives x[a + N2 b]
}

__device__ __forceinline__ void load_tw(float2* sh_tw, const float2* tw, int n) {
  for (int i = threadIdx.x; i < (n >> 1); i += blockDim.x) sh_tw[i] = tw[i];
}

template <int N1, int N2>
struct Lines {
  static constexpr int n = N1 * N2;
  static constexpr int R = N1 > N2 ? N1 : N2;
  static constexpr int tk = kFftThreads / R;   // lines per block
  static constexpr int ps = n + 1;             // padded exchange stride
};

// ------------------------------------------------------------------------------- x passes
// Rows of all samples are consecutive (n^2 per sample); a block's rows lie in one sample.
// Thread t: q = t % R, row = t / R (consecutive lanes walk along the row).
template <int N1, int N2>
__global__ void __launch_bounds__(kFftThreads) x_r2c_kernel(const float* __restrict__ in,
                                                            float2* __restrict__ spec,
                                                            const float2* __restrict__ tw,
                                                            const StepScal* __restrict__ tab,
                                                            long long in_stride) {
  using L = Lines<N1, N2>;
  constexpr int n = L::n, nh = n / 2 + 1;
  __shared__ float EX[L::tk * L::ps];
  __shared__ float2 TW[n / 2];
  const long long row0 = static_cast<long long>(blockIdx.x) * L::tk;
  const long long nn = static_cast<long long>(n) * n;
  const int smp = static_cast<int>(row0 / nn);
  if (!sample_active(tab, smp)) return;
  load_tw(TW, tw, n);
  const int q = threadIdx.x % L::R, r = threadIdx.x / L::R;
  const long long row = row0 + r;
  const float* src = in + smp * in_stride + (row - smp * nn) * n;
  float2 v[kMaxR];
  const bool in_x = q < N2, in_k = q < N1;
  if (in_x)
#pragma unroll
    for (int j1 = 0; j1 < N1; ++j1) v[j1] = make_float2(src[q + N2 * j1], 0.0f);
  __syncthreads();
  line_forward<N1, N2>(v, EX + r * L::ps, TW, q, in_x, in_k);
  if (in_k)
#pragma unroll
    for (int k2 = 0; k2 < N2; ++k2) {
      const int k = q + N1 * k2;
      if (k < nh) spec[row * nh + k] = v[k2];
    }
}

template <int N1, int N2>
__global__ void __launch_bounds__(kFftThreads) x_c2r_kernel(const float2* __restrict__ spec,
                                                            float* __restrict__ out,
                                                            const float2* __restrict__ tw,
                                                            float scale,
                                                            const StepScal* __restrict__ tab,
                                                            long long out_stride) {
  using L = Lines<N1, N2>;
  constexpr int n = L::n, nh = n / 2 + 1;
  __shared__ float EX[L::tk * L::ps];
  __shared__ float2 TW[n / 2];
  const long long row0 = static_cast<long long>(blockIdx.x) * L::tk;
  const long long nn = static_cast<long long>(n) * n;
  const int smp = static_cast<int>(row0 / nn);
  if (!sample_active(tab, smp)) return;
  load_tw(TW, tw, n);
  const int q = threadIdx.x % L::R, r = threadIdx.x / L::R;
  const long long row = row0 + r;
  float2 v[kMaxR];
  const bool in_x = q < N2, in_k = q < N1;
  if (in_k)
#pragma unroll
    for (int k2 = 0; k2 < N2; ++k2) {   // Hermitian extension X[n - k] = conj(X[k])
      const int k = q + N1 * k2;
      const float2 w = spec[row * nh + (k < nh ? k : n - k)];
      v[k2] = k < nh ? w : make_float2(w.x, -w.y);
    }
  __syncthreads();
  line_inverse<N1, N2>(v, EX + r * L::ps, TW, q, in_x, in_k);
  if (in_x) {
    float* dst = out + smp * out_stride + (row - smp * nn) * n;
#pragma unroll
    for (int b = 0; b < N1; ++b) dst[q + N2 * b] = v[b].x * scale;
  }
}

// -------------------------------------------------------------------------- plane passes
// The x and y passes of one z plane in one block (n <= 128): the half spectrum of the plane (up
// to 66 KB) stays in LDS between them, and each line's exchange buffer is its own row (or the
// real parts of its own column) of it.  The transforms and their values are those of separate
// x and y passes.  Rounds of the block cover the lines; 1024 threads, since a single sample has
// only n blocks.  Latency binds it (64 of 256 CUs at 64^3), and 128^3 has half the chip; the
// gain is a launch and a round trip of the spectrum per direction.  us, forward and inverse,
// against the separate passes: 32^3 3.8 + 3.5 (6.7 + 6.4), 64^3 5.2 + 5.2 (7.5 + 7.5), 128^3
// 17.2 + 14.2 (18.1 + 15.0; 18.6 + 15.9 with 512 threads).
template <int N1, int N2>
struct Plane {
  static constexpr int n = N1 * N2, nh = n / 2 + 1;
  static constexpr int R = N1 > N2 ? N1 : N2;
  static constexpr int threads = n * R < 1024 ? n * R : 1024;
  static constexpr int tk = threads / R;                  // lines per round
  static constexpr int xrounds = n / tk;                  // n is a multiple of tk
  static constexpr int yrounds = (nh + tk - 1) / tk;
};

template <int N1, int N2>
__global__ void __launch_bounds__((Plane<N1, N2>::threads)) plane_forward_kernel(
    const float* __restrict__ in, float2* __restrict__ spec, const float2* __restrict__ tw,
    const StepScal* __restrict__ tab, long long in_stride) {
  using P = Plane<N1, N2>;
  constexpr int n = P::n, nh = P::nh;
  __shared__ float2 H[n * nh];
  __shared__ float2 TW[n / 2];
  if (!sample_active(tab, blockIdx.y)) return;
  load_tw(TW, tw, n);
  const float* src = in + blockIdx.y * in_stride + static_cast<long long>(blockIdx.x) * n * n;
  float2 v[kMaxR];
  {
    const int q = threadIdx.x % P::R, r = threadIdx.x / P::R;
    const bool in_x = q < N2, in_k = q < N1;
#pragma unroll 1
    for (int k = 0; k < P::xrounds; ++k) {
      const int row = k * P::tk + r;
      if (in_x)
#pragma unroll
        for (int j1 = 0; j1 < N1; ++j1) v[j1] = make_float2(src[row * n + q + N2 * j1], 0.0f);
      __syncthreads();
      line_forward<N1, N2>(v, reinterpret_cast<float*>(H + row * nh), TW, q, in_x, in_k);
      __syncthreads();   // the row has been read: it takes the spectrum now
      if (in_k)
#pragma unroll
        for (int k2 = 0; k2 < N2; ++k2) {
          const int kx = q + N1 * k2;
          if (kx < nh) H[row * nh + kx] = v[k2];
        }
    }
  }
  __syncthreads();
  float2* dst = spec + (static_cast<long long>(blockIdx.y) * n + blockIdx.x) * n * nh;
  {
    const int li = threadIdx.x % P::tk, q = threadIdx.x / P::tk;
#pragma unroll 1
    for (int k = 0; k < P::yrounds; ++k) {
      const int kx = k * P::tk + li;
      const bool in_x = kx < nh && q < N2, in_k = kx < nh && q < N1;
      if (in_x)
#pragma unroll
        for (int r = 0; r < N1; ++r) v[r] = H[(q + N2 * r) * nh + kx];
      __syncthreads();
      line_forward<N1, N2, 2 * nh>(v, reinterpret_cast<float*>(H + kx), TW, q, in_x, in_k);
      if (in_k)
#pragma unroll
        for (int r = 0; r < N2; ++r) dst[(q + N1 * r) * nh + kx] = v[r];
    }
  }
}

template <int N1, int N2>
__global__ void __launch_bounds__((Plane<N1, N2>::threads)) plane_inverse_kernel(
    const float2* __restrict__ spec, float* __restrict__ out, const float2* __restrict__ tw,
    float scale, const StepScal* __restrict__ tab, long long out_stride) {
  using P = Plane<N1, N2>;
  constexpr int n = P::n, nh = P::nh;
  __shared__ float2 H[n * nh];
  __shared__ float2 TW[n / 2];
  if (!sample_active(tab, blockIdx.y)) return;
  load_tw(TW, tw, n);
  const float2* src = spec + (static_cast<long long>(blockIdx.y) * n + blockIdx.x) * n * nh;
  float2 v[kMaxR];
  {
    const int li = threadIdx.x % P::tk, q = threadIdx.x / P::tk;
#pragma unroll 1
    for (int k = 0; k < P::yrounds; ++k) {
      const int kx = k * P::tk + li;
      const bool in_x = kx < nh && q < N2, in_k = kx < nh && q < N1;
      if (in_k)
#pragma unroll
        for (int r = 0; r < N2; ++r) v[r] = src[(q + N1 * r) * nh + kx];
      __syncthreads();
      line_inverse<N1, N2, 2 * nh>(v, reinterpret_cast<float*>(H + kx), TW, q, in_x, in_k);
      __syncthreads();
      if (in_x)
#pragma unroll
        for (int r = 0; r < N1; ++r) H[(q + N2 * r) * nh + kx] = v[r];
    }
  }
  __syncthreads();
  {
    const int q = threadIdx.x % P::R, r = threadIdx.x / P::R;
    const bool in_x = q < N2, in_k = q < N1;
    float* dst = out + blockIdx.y * out_stride + static_cast<long long>(blockIdx.x) * n * n;
#pragma unroll 1
    for (int k = 0; k < P::xrounds; ++k) {
      const int row = k * P::tk + r;
      if (in_k)
#pragma unroll
        for (int k2 = 0; k2 < N2; ++k2) {   // Hermitian extension X[n - k] = conj(X[k])
          const int kx = q + N1 * k2;
          const float2 w = H[row * nh + (kx < nh ? kx : n - kx)];
          v[k2] = kx < nh ? w : make_float2(w.x, -w.y);
        }
      __syncthreads();
      line_inverse<N1, N2>(v, reinterpret_cast<float*>(H + row * nh), TW, q, in_x, in_k);
      if (in_x)
#pragma unroll
        for (int b = 0; b < N1; ++b) dst[row * n + q + N2 * b] = v[b].x * scale;
    }
  }
}

// ---------------------------------------------------------------------------- line passes
struct OpArgs {
  int op;          // -1 none, kOpGreen, kOpIcHess, kOpZa, kOpZaT
  float green;     // -(3 Om / 2a) / N^3
  int axis, axis2;
  float sqrt_amp;  // sqrt(A D^2 / V_cell)
  float half_ns;   // spectral index / 2
  float om_h;      // Omega_m h
  float kphys;     // n / box: rad/cell -> h/Mpc
  float inv_n3;    // 1/N^3, times the operator's scale for kOpZa / kOpZaT
  int eh;          // transfer function: 0 BBKS, 1 Eisenstein & Hu without wiggles
  float eh_theta2, eh_alpha, eh_ks;
};

// derivative factor k_j (rad/cell) of mode (fx, fy, fz): zero on the Nyquist plane of its own
// axis (an odd derivative of the real Nyquist mode)
__device__ __forceinline__ float deriv_k(int axis, int fx, int fy, int fz, int n) {
  const int f = axis == 0 ? fx : (axis == 1 ? fy : fz);
  if (f == n / 2 || f == -n / 2) return 0.0f;
  return 6.283185307179586f / static_cast<float>(n) * static_cast<float>(f);
}

// sqrt(P(k)) / sqrt(A D^2 / V_cell) at k = kp h/Mpc: k^(n_s/2) T(k)
__device__ __forceinline__ float sqrt_shape(const OpArgs& o, float kp) {
  float t;
  if (o.eh) {
    const float x = kp * o.eh_ks;
    const float x2 = x * x;
    const float gamma = o.om_h * (o.eh_alpha + (1.0f - o.eh_alpha) / (1.0f + x2 * x2));
    const float q = kp * o.eh_theta2 / gamma;
    const float l = logf(2.0f * 2.718281828459045f + 1.8f * q);
    const float c = 14.2f + 731.0f / (1.0f + 62.5f * q);
    t = l / (l + c * q * q);
  } else {
    const float q = kp / o.om_h;
    const float q2 = 16.1f * q, q3 = 5.46f * q, q4 = 6.71f * q;
    t = logf(1.0f + 2.34f * q) / (2.34f * q) *
        powf(1.0f + 3.89f * q + q2 * q2 + q3 * q3 * q3 + (q4 * q4) * (q4 * q4), -0.25f);
  }
  return powf(kp, o.half_ns) * t;
}

__device__ __forceinline__ int signed_freq(int k, int n) { return k <= n / 2 ? k : k - n; }

// sqrt(P(k)) of mode k2 (rad/cell), and what it takes of the white-noise normalisation
__device__ __forceinline__ float mode_spectrum(const OpArgs& o, float k2) {
  return o.sqrt_amp * sqrt_shape(o, sqrtf(k2) * o.kphys);
}

__device__ __forceinline__ float mode_k2(int fx, int fy, int fz, int n) {
  const float c = 6.283185307179586f / static_cast<float>(n);
  const float ax = c * fx, ay = c * fy, az = c * fz;
  return ax * ax + ay * ay + az * az;
}

// OPK: 0 none, 1 Green's function, 2 the other operators (o.op)
template <int OPK>
__device__ __forceinline__ float2 apply_op(const OpArgs& o, int kx, int ky, int kz, int n,
                                           float2 v) {
  const int fx = kx, fy = signed_freq(ky, n), fz = signed_freq(kz, n);
  if (OPK == 0) return v;
  const float k2 = mode_k2(fx, fy, fz, n);
  if (k2 == 0.0f) return make_float2(0.0f, 0.0f);
  if (OPK == 1) {
    const float f = o.green / k2;
    return make_float2(v.x * f, v.y * f);
  }
  // initial-condition operators (derivative factors from deriv_k):
  //   kOpIcHess  k_axis k_axis2 sqrt(P(k)) / k^2 / N^3 (real): second derivative of the
  //              linear potential (its own transpose);
  //   kOpZa      i k_axis / k^2 times inv_n3 (kOpZaT: its conjugate), the displacement of a
  //              given density, scaled
  const float kj = deriv_k(o.axis, fx, fy, fz, n);
  if (o.op == kOpZa || o.op == kOpZaT) {
    const float f = kj / k2 * o.inv_n3;
    const float ff = o.op == kOpZa ? f : -f;
    return make_float2(-v.y * ff, v.x * ff);
  }
  const float f =
      kj * deriv_k(o.axis2, fx, fy, fz, n) * mode_spectrum(o, k2) / k2 * o.inv_n3;
  return make_float2(v.x * f, v.y * f);
}

// Workgroups go to the 8 XCDs (each with its own L2) round robin.  Consecutive line groups
// of a pass share cache lines (a spectrum row of nh = n/2 + 1 complex values is not line
// aligned), so each XCD takes one contiguous range of groups: block b -> group
// (b mod 8) nb/8 + b/8 when nb is a multiple of 8 (a bijection), else b.
__device__ __forceinline__ int xcd_group(int b, int nb) {
  return (nb & 7) ? b : (b & 7) * (nb >> 3) + (b >> 3);
}

// Line pass along AX (1 = y, 2 = z) over tk consecutive lines of sample blockIdx.y.  Line
// l = fixed * nh + kx (fixed = z for AX = 1, ky for AX = 2); thread t: line t % tk, q = t / tk,
// so consecutive lanes take consecutive kx.  flags: 1 forward, 2 operator, 4 inverse, 8
// accumulate into out.  Input in D_x unless the pass starts with the inverse (D_k).  The
// Green's function factor comes from the sample's step table when there is one.
template <int AX, int N1, int N2, int OPK>
// in and out may alias (in-place passes): no __restrict__ on them
__global__ void __launch_bounds__(kFftThreads) pencil_kernel(const float2* in, float2* out,
                                                             const float2* __restrict__ tw,
                                                             int flags, OpArgs op,
                                                             const StepScal* __restrict__ tab) {
  using L = Lines<N1, N2>;
  constexpr int n = L::n, nh = n / 2 + 1;
  __shared__ float EX[L::tk * L::ps];
  __shared__ float2 TW[n / 2];
  if (!sample_active(tab, blockIdx.y)) return;
  if (tab && op.op == kOpGreen) op.green = tab[blockIdx.y].green;
  const long long slab = static_cast<long long>(n) * n * nh;
  in += blockIdx.y * slab;
  out += blockIdx.y * slab;
  load_tw(TW, tw, n);
  const int li = threadIdx.x % L::tk, q = threadIdx.x / L::tk;
  const int line = xcd_group(blockIdx.x, gridDim.x) * L::tk + li;
  const bool valid = line < n * nh;
  const int fixed = line / nh, kx = line - fixed * nh;
  const long long stride = AX == 1 ? nh : static_cast<long long>(n) * nh;
  const long long base = AX == 1 ? static_cast<long long>(fixed) * n * nh + kx
                                 : static_cast<long long>(fixed) * nh + kx;
  float* ex = EX + li * L::ps;
  float2 v[kMaxR];
  const bool in_x = valid && q < N2, in_k = valid && q < N1;
  if (flags & 1) {
    if (in_x)
#pragma unroll
      for (int r = 0; r < N1; ++r) v[r] = in[base + (q + N2 * r) * stride];
    __syncthreads();
    line_forward<N1, N2>(v, ex, TW, q, in_x, in_k);
  } else {
    if (in_k)
#pragma unroll
      for (int r = 0; r < N2; ++r) v[r] = in[base + (q + N1 * r) * stride];
  }
  if ((flags & 2) && in_k) {
#pragma unroll
    for (int r = 0; r < N2; ++r) {
      const int k = q + N1 * r;
      v[r] = apply_op<OPK>(op, kx, AX == 1 ? k : fixed, AX == 1 ? fixed : k, n, v[r]);
    }
  }
  if (flags & 4) {
    __syncthreads();   // the forward pass may still read the exchange buffer
    line_inverse<N1, N2>(v, ex, TW, q, in_x, in_k);
    if (in_x)
#pragma unroll
      for (int r = 0; r < N1; ++r) {
        const long long g = base + (q + N2 * r) * stride;
        float2 w = v[r];
        if (flags & 8) w = cadd(w, out[g]);
        out[g] = w;
      }
  } else if (in_k) {
#pragma unroll
    for (int r = 0; r < N2; ++r) {
      const long long g = base + (q + N1 * r) * stride;
      float2 w = v[r];
      if (flags & 8) w = cadd(w, out[g]);
      out[g] = w;
    }
  }
}

// Zel'dovich displacement of white noise, i k_j sqrt(P(k)) / k^2 / N^3 for the three axes j, on
// the z pass: in (spectrum along x and y) forward along z, times the operator of each axis,
// inverse, into out[S][3].  full (optional, may be in): the spectrum of all three axes' input.
// What bounds a pass per axis is the spectrum's power and logarithm at every mode (95 us at
// 256^3 against 25 for a plain pass, after a forward pass of its own), so they are taken once:
// 310 -> 139 us at 256^3, 87 -> 32 at 128^3, 28 -> 12 at 16^3.
template <int N1, int N2>
__global__ void __launch_bounds__(kFftThreads) ic_disp_kernel(const float2* in, float2* full,
                                                              float2* __restrict__ out,
                                                              const float2* __restrict__ tw,
                                                              OpArgs op) {
  using L = Lines<N1, N2>;
  constexpr int n = L::n, nh = n / 2 + 1;
  __shared__ float EX[L::tk * L::ps];
  __shared__ float2 TW[n / 2];
  const long long slab = static_cast<long long>(n) * n * nh;
  in += blockIdx.y * slab;
  if (full) full += blockIdx.y * slab;
  out += blockIdx.y * 3 * slab;
  load_tw(TW, tw, n);
  const int li = threadIdx.x % L::tk, q = threadIdx.x / L::tk;
  const int line = xcd_group(blockIdx.x, gridDim.x) * L::tk + li;
  const bool valid = line < n * nh;
  const int ky = line / nh, kx = line - ky * nh;
  const long long stride = static_cast<long long>(n) * nh;
  float* ex = EX + li * L::ps;
  float2 v[kMaxR];
  float sp[kMaxR];
  const bool in_x = valid && q < N2, in_k = valid && q < N1;
  if (in_x)
#pragma unroll
    for (int r = 0; r < N1; ++r) v[r] = in[line + (q + N2 * r) * stride];
  __syncthreads();
  line_forward<N1, N2>(v, ex, TW, q, in_x, in_k);
  const int fy = signed_freq(ky, n);
  if (in_k) {
#pragma unroll
    for (int r = 0; r < N2; ++r) {
      const int kz = q + N1 * r;
      if (full) full[line + kz * stride] = v[r];
      sp[r] = mode_spectrum(op, mode_k2(kx, fy, signed_freq(kz, n), n));
    }
  }
#pragma unroll 1
  for (int axis = 0; axis < 3; ++axis) {
    float2 w[kMaxR];
    if (in_k) {
#pragma unroll
      for (int r = 0; r < N2; ++r) {
        const int fz = signed_freq(q + N1 * r, n);
        const float k2 = mode_k2(kx, fy, fz, n);
        // k = 0 has no displacement
        const float f = k2 == 0.0f ? 0.0f : deriv_k(axis, kx, fy, fz, n) * sp[r] / k2 * op.inv_n3;
        // times i f, rounded before the transform's sums
        w[r] = make_float2(opaque(-v[r].y * f), opaque(v[r].x * f));
      }
    }
    __syncthreads();   // the pass before may still read the exchange buffer
    line_inverse<N1, N2>(w, ex, TW, q, in_x, in_k);
    if (in_x)
#pragma unroll
      for (int r = 0; r < N1; ++r) out[axis * slab + line + (q + N2 * r) * stride] = w[r];
  }
}

// Adjoint of ic_disp_kernel: in[S][3] (spectra along x and y of the displacement's adjoint)
// forward along z, times the conjugate operators, summed over the axes (and with sum[S], if
// given, the spectrum of other terms; may be out), inverse along z into out[S].  (Three passes of
// forward, operator and accumulation and one of the inverse took 315 us at 256^3; this takes 173.)
template <int N1, int N2>
__global__ void __launch_bounds__(kFftThreads) ic_disp_vjp_kernel(const float2* __restrict__ in,
                                                                  const float2* sum, float2* out,
                                                                  const float2* __restrict__ tw,
                                                                  OpArgs op) {
  using L = Lines<N1, N2>;
  constexpr int n = L::n, nh = n / 2 + 1;
  __shared__ float EX[L::tk * L::ps];
  __shared__ float2 TW[n / 2];
  const long long slab = static_cast<long long>(n) * n * nh;
  in += blockIdx.y * 3 * slab;
  if (sum) sum += blockIdx.y * slab;
  out += blockIdx.y * slab;
  load_tw(TW, tw, n);
  const int li = threadIdx.x % L::tk, q = threadIdx.x / L::tk;
  const int line = xcd_group(blockIdx.x, gridDim.x) * L::tk + li;
  const bool valid = line < n * nh;
  const int ky = line / nh, kx = line - ky * nh;
  const long long stride = static_cast<long long>(n) * nh;
  float* ex = EX + li * L::ps;
  const bool in_x = valid && q < N2, in_k = valid && q < N1;
  const int fy = signed_freq(ky, n);
  float2 acc[kMaxR];
  float sp[kMaxR];
  if (in_k) {
#pragma unroll
    for (int r = 0; r < N2; ++r) {
      const int kz = q + N1 * r;
      sp[r] = mode_spectrum(op, mode_k2(kx, fy, signed_freq(kz, n), n));
      acc[r] = sum ? sum[line + kz * stride] : make_float2(0.0f, 0.0f);
    }
  }
#pragma unroll 1
  for (int axis = 0; axis < 3; ++axis) {
    float2 v[kMaxR];
    if (in_x)
#pragma unroll
      for (int r = 0; r < N1; ++r) v[r] = in[axis * slab + line + (q + N2 * r) * stride];
    __syncthreads();
    line_forward<N1, N2>(v, ex, TW, q, in_x, in_k);
    if (in_k) {
#pragma unroll
      for (int r = 0; r < N2; ++r) {
        const int fz = signed_freq(q + N1 * r, n);
        const float k2 = mode_k2(kx, fy, fz, n);
        const float f = k2 == 0.0f ? 0.0f : deriv_k(axis, kx, fy, fz, n) * sp[r] / k2 * op.inv_n3;
        acc[r] = cadd(acc[r], make_float2(v[r].y * f, -v[r].x * f));   // times -i f
      }
    }
  }
  __syncthreads();
  line_inverse<N1, N2>(acc, ex, TW, q, in_x, in_k);
  if (in_x)
#pragma unroll
    for (int r = 0; r < N1; ++r) out[line + (q + N2 * r) * stride] = acc[r];
}

template <int N1, int N2>
void ic_disp_n(hipStream_t st, const float2* in, float2* full, float2* out, const float2* tw,
               const OpArgs& op, const Batch& b) {
  using L = Lines<N1, N2>;
  constexpr int n = L::n, nh = n / 2 + 1;
  hipLaunchKernelGGL((ic_disp_kernel<N1, N2>), dim3((n * nh + L::tk - 1) / L::tk, b.S),
                     dim3(kFftThreads), 0, st, in, full, out, tw, op);
}

template <int N1, int N2>
void ic_disp_vjp_n(hipStream_t st, const float2* in, const float2* sum, float2* out,
                   const float2* tw, const OpArgs& op, const Batch& b) {
  using L = Lines<N1, N2>;
  constexpr int n = L::n, nh = n / 2 + 1;
  hipLaunchKernelGGL((ic_disp_vjp_kernel<N1, N2>), dim3((n * nh + L::tk - 1) / L::tk, b.S),
                     dim3(kFftThreads), 0, st, in, sum, out, tw, op);
}

template <int AX, int N1, int N2, int OPK>
void pencil_op(hipStream_t st, const float2* in, float2* out, const float2* tw, int flags,
               const OpArgs& op, const Batch& b) {
  using L = Lines<N1, N2>;
  constexpr int n = L::n, nh = n / 2 + 1;
  const dim3 grid((n * nh + L::tk - 1) / L::tk, b.S);
  hipLaunchKernelGGL((pencil_kernel<AX, N1, N2, OPK>), grid, dim3(kFftThreads), 0, st, in, out, tw,
                     flags, op, b.tab);
}

// z pass
template <int N1, int N2>
void pencil_n(hipStream_t st, const float2* in, float2* out, const float2* tw, int flags,
              const OpArgs& op, const Batch& b) {
  if (!(flags & 2) || op.op < 0)
    pencil_op<2, N1, N2, 0>(st, in, out, tw, flags & ~2, op, b);
  else if (op.op == kOpGreen)
    pencil_op<2, N1, N2, 1>(st, in, out, tw, flags, op, b);
  else
    pencil_op<2, N1, N2, 2>(st, in, out, tw, flags, op, b);
}

template <int N1, int N2>
void r2c_n(hipStream_t st, const float* in, float2* spec, const float2* tw, const Batch& b,
           long long in_stride) {
  using L = Lines<N1, N2>;
  const long long rows = static_cast<long long>(L::n) * L::n * b.S;
  hipLaunchKernelGGL((x_r2c_kernel<N1, N2>), dim3(static_cast<unsigned>(rows / L::tk)),
                     dim3(kFftThreads), 0, st, in, spec, tw, b.tab, in_stride);
}

template <int N1, int N2>
void c2r_n(hipStream_t st, const float2* spec, float* out, const float2* tw, float scale,
           const Batch& b, long long out_stride) {
  using L = Lines<N1, N2>;
  const long long rows = static_cast<long long>(L::n) * L::n * b.S;
  hipLaunchKernelGGL((x_c2r_kernel<N1, N2>), dim3(static_cast<unsigned>(rows / L::tk)),
                     dim3(kFftThreads), 0, st, spec, out, tw, scale, b.tab, out_stride);
}

template <int N1, int N2>
void plane_forward_n(hipStream_t st, const float* in, float2* spec, const float2* tw,
                     const Batch& b, long long in_stride) {
  hipLaunchKernelGGL((plane_forward_kernel<N1, N2>), dim3(N1 * N2, b.S),
                     dim3(Plane<N1, N2>::threads), 0, st, in, spec, tw, b.tab, in_stride);
}

template <int N1, int N2>
void plane_inverse_n(hipStream_t st, const float2* spec, float* out, const float2* tw, float scale,
                     const Batch& b, long long out_stride) {
  hipLaunchKernelGGL((plane_inverse_kernel<N1, N2>), dim3(N1 * N2, b.S),
                     dim3(Plane<N1, N2>::threads), 0, st, spec, out, tw, scale, b.tab, out_stride);
}

// n = N1 * N2 with N1 >= N2, both at most 16.  BIG: n = 256, whose planes (264 KB of half
// spectrum) exceed the LDS, so its x and y passes are separate.
#define DH_FFT_DISPATCH(n, CALL, BIG)                             \
  switch (n) {                                                    \
    case 16: CALL(4, 4); break;                                   \
    case 32: CALL(8, 4); break;                                   \
    case 64: CALL(8, 8); break;                                   \
    case 128: CALL(16, 8); break;                                 \
    case 256: BIG(16, 16); break;                                 \
    default: throw ArgError("fft: n must be a power of two in [16, 256]"); \
  }

void pencil(hipStream_t st, const float2* in, float2* out, const float2* tw, int flags,
            const OpArgs& op, const Batch& b) {
#define DH_CALL(a, c) pencil_n<a, c>(st, in, out, tw, flags, op, b)
  DH_FFT_DISPATCH(b.n, DH_CALL, DH_CALL)
#undef DH_CALL
  DH_LAUNCH_CHECK();
}

// y pass in place (flags 1 forward, 4 inverse)
template <int N1, int N2>
void y_pass(hipStream_t st, float2* spec, const float2* tw, int flags, const Batch& b) {
  OpArgs none{};
  none.op = -1;
  pencil_op<1, N1, N2, 0>(st, spec, spec, tw, flags, none, b);
}

}  // namespace

void fft_make_twiddles(int n, std::vector<float2>& tw) {
  tw.resize(n / 2);
  for (int m = 0; m < n / 2; ++m) {
    const double ang = -2.0 * M_PI * m / n;
    tw[m] = make_float2(static_cast<float>(std::cos(ang)), static_cast<float>(std::sin(ang)));
  }
}

void fft_forward_xy(hipStream_t st, const float* in, float2* spec, const float2* tw,
                    const Batch& b, long long in_stride) {
  const long long is = in_stride < 0 ? b.nc() : in_stride;
#define DH_PLANE(a, c) plane_forward_n<a, c>(st, in, spec, tw, b, is)
#define DH_PASSES(a, c)                 \
  r2c_n<a, c>(st, in, spec, tw, b, is); \
  DH_LAUNCH_CHECK();                    \
  y_pass<a, c>(st, spec, tw, 1, b)
  DH_FFT_DISPATCH(b.n, DH_PLANE, DH_PASSES)
#undef DH_PASSES
#undef DH_PLANE
  DH_LAUNCH_CHECK();
}

void fft_inverse_yx(hipStream_t st, float2* spec, float* out, const float2* tw, float scale,
                    const Batch& b, long long out_stride) {
  const long long os = out_stride < 0 ? b.nc() : out_stride;
#define DH_PLANE(a, c) plane_inverse_n<a, c>(st, spec, out, tw, scale, b, os)
#define DH_PASSES(a, c)           \
  y_pass<a, c>(st, spec, tw, 4, b); \
  DH_LAUNCH_CHECK();              \
  c2r_n<a, c>(st, spec, out, tw, scale, b, os)
  DH_FFT_DISPATCH(b.n, DH_PLANE, DH_PASSES)
#undef DH_PASSES
#undef DH_PLANE
  DH_LAUNCH_CHECK();
}

void fft_zpass_green(hipStream_t st, float2* spec, const float2* tw, const Batch& b) {
  if (!b.tab) throw ArgError("Poisson pass: step table required");
  OpArgs o{};
  o.op = kOpGreen;
  pencil(st, spec, spec, tw, 1 | 2 | 4, o, b);
}

void fft_zpass_forward(hipStream_t st, const float2* in, float2* out, const float2* tw,
                       const Batch& b) {
  OpArgs none{};
  none.op = -1;
  pencil(st, in, out, tw, 1, none, b);
}

void fft_zpass_inverse(hipStream_t st, float2* spec, const float2* tw, const Batch& b) {
  OpArgs none{};
  none.op = -1;
  pencil(st, spec, spec, tw, 4, none, b);
}

namespace {

OpArgs ic_args(const IcOp& op, int n) {
  OpArgs o{};
  o.op = op.op;
  o.axis = op.axis;
  o.axis2 = op.axis2;
  o.sqrt_amp = static_cast<float>(std::sqrt(op.amp));
  o.half_ns = static_cast<float>(0.5 * op.n_s);
  o.om_h = static_cast<float>(op.om_h);
  o.kphys = static_cast<float>(op.kphys);
  o.inv_n3 = static_cast<float>(op.scale / (static_cast<double>(n) * n * n));
  o.eh = op.eh ? 1 : 0;
  o.eh_theta2 = static_cast<float>(op.eh_theta2);
  o.eh_alpha = static_cast<float>(op.eh_alpha);
  o.eh_ks = static_cast<float>(op.eh_ks);
  return o;
}

}  // namespace

// IC operators on the z pass (see apply_op): out = op(in), forward z transform first and
// inverse after as asked
void fft_zpass_ic(hipStream_t st, const float2* in, float2* out, const float2* tw,
                  const IcOp& op, bool forward_first, bool inverse_after, bool accumulate,
                  const Batch& b) {
  const int flags = (forward_first ? 1 : 0) | 2 | (inverse_after ? 4 : 0) | (accumulate ? 8 : 0);
  pencil(st, in, out, tw, flags, ic_args(op, b.n), b);
}

void fft_zpass_disp(hipStream_t st, const float2* in, float2* full, float2* out, const float2* tw,
                    const IcOp& op, const Batch& b) {
  const OpArgs o = ic_args(op, b.n);
#define DH_CALL(a, c) ic_disp_n<a, c>(st, in, full, out, tw, o, b)
  DH_FFT_DISPATCH(b.n, DH_CALL, DH_CALL)
#undef DH_CALL
  DH_LAUNCH_CHECK();
}

void fft_zpass_disp_vjp(hipStream_t st, const float2* in, const float2* sum, float2* out,
                        const float2* tw, const IcOp& op, const Batch& b) {
  const OpArgs o = ic_args(op, b.n);
#define DH_CALL(a, c) ic_disp_vjp_n<a, c>(st, in, sum, out, tw, o, b)
  DH_FFT_DISPATCH(b.n, DH_CALL, DH_CALL)
#undef DH_CALL
  DH_LAUNCH_CHECK();
}

}  // namespace dh
