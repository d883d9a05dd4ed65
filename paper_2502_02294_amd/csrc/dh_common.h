// Internal definitions shared by the HIP translation units of libdiffhydro.
// Device math follows the paper's method; see include/diffhydro.h for the conventions.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <stdexcept>
#include <string>

#define DH_HIP(call)                                                                        \
  do {                                                                                      \
    hipError_t _e = (call);                                                                 \
    if (_e != hipSuccess)                                                                   \
      throw ::dh::HipError(std::string(#call) + ": " + hipGetErrorString(_e));              \
  } while (0)

#define DH_LAUNCH_CHECK() DH_HIP(hipGetLastError())

namespace dh {

struct HipError : std::runtime_error {
  using std::runtime_error::runtime_error;
};
struct ArgError : std::runtime_error {
  using std::runtime_error::runtime_error;
};

inline unsigned blocks_for(long long work, int threads) {
  return static_cast<unsigned>((work + threads - 1) / threads);
}

// ---------------------------------------------------------------------------------------
// Hydro: per-cell primitive recovery, flux along D and the relaxation split (Sec. 2.3.1).
// Q = (rho, m_x, m_y, m_z, Et) with m = a rho U and Et = a^2 rho E.
//   U = m/(a rho), e = Et/(a^2 rho) - U^2/2 floored at e_floor only inside the EOS,
//   p = (gamma-1) rho e, c_s = sqrt(gamma (gamma-1) e), freezing speed c = (|U_d| + c_s)/a,
//   F = (rho U_d / a, rho U_d U + p e_d, a U_d (Et/a^2 + p)),
//   F^R = (c Q + F)/2, F^L = (c Q - F)/2.
// Dual energy (NQ = 6): a sixth component S = (a^2 rho e) rho^(1-gamma), the entropy
// variable, with the flux S U_d / a; the EOS takes e = Et/(a^2 rho) - U^2/2 where that
// exceeds eta1 Et/(a^2 rho), else e_S = S rho^(gamma-2) / a^2 (the selection of Bryan et al.
// 1995 with the entropy form of Ryu et al. 1993).
// ---------------------------------------------------------------------------------------
// Reciprocal and square root on the hardware's approximate units (v_rcp_f32, v_sqrt_f32:
// within 1 ulp).  The hydro kernels take these in place of the correctly rounded division
// and square root, which expand to about ten instructions each; every operand here is a
// normal positive number (density, floored energy) or bounded away from zero (limiter
// denominator), and the error stays at the level of one FP32 rounding.
__device__ __forceinline__ float rcp_approx(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float sqrt_approx(float x) { return __builtin_amdgcn_sqrtf(x); }

// g = -grad(phi) at cell c of a periodic box of n^3 = 2^(3 lgn) cells, by two-point central
// differences: g_d = -(phi[c + e_d] - phi[c - e_d]) / 2.  The kernels over the cells take g from
// phi, one field through the cache, instead of reading it as a field of four (256^3: the source
// adjoint 402 -> 363 us, a first sweep along z 197 -> 177).
// log2 n from n^3
__device__ __forceinline__ int log2_side(long long nc) { return __builtin_ctzll(nc) / 3; }
__device__ __forceinline__ float half_difference(float up, float down) {
  return -0.5f * (up - down);
}
__device__ __forceinline__ float4 mesh_g(const float* __restrict__ phi, unsigned c, int lgn) {
  float g[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const unsigned one = 1u << (d * lgn), mask = ((1u << lgn) - 1u) << (d * lgn);
    const unsigned rest = c & ~mask;
    g[d] = half_difference(phi[rest | ((c + one) & mask)], phi[rest | ((c - one) & mask)]);
  }
  return make_float4(g[0], g[1], g[2], 0.0f);
}

// Gravity source of the gas over a half kick h (operator split): m' = m + rho g h,
// Et' = Et + h g . (m + m')/2, so the internal energy is unchanged.  One function for every
// kernel that applies or recomputes it, with every rounding spelled out (explicit FMAs, no
// contraction left to the compiler), so they all round alike wherever it is inlined.
__device__ __forceinline__ void kick_cell(float rho, const float4 g4, float h, float m[3],
                                          float& et) {
  const float g[3] = {g4.x, g4.y, g4.z};
  float de = 0.0f;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const float m0 = m[d];
    const float m1 = fmaf(__fmul_rn(rho, g[d]), h, m0);
    m[d] = m1;
    de = fmaf(__fmul_rn(0.5f, __fadd_rn(m0, m1)), g[d], de);
  }
  et = fmaf(de, h, et);
}

// Dual energy: below kDualEta1 of E the internal energy comes from the entropy; at the end of
// a step the entropy is reset from the total energy where e_E >= kDualEta2 E.
constexpr float kDualEta1 = 1e-3f;
constexpr float kDualEta2 = 0.1f;

// The dual-energy tests of one cell state Q (FP32, written on Q so that they need no a:
// a^2 rho e_E = Et - |m|^2 / (2 rho)).  Every kernel outside the sweeps that needs the
// selection takes it from here, so a cell's screening, its source term and its adjoint agree.
//   dual_total_branch: the EOS takes e_E (e_E > kDualEta1 E);
//   dual_sync_branch: the end-of-step reset of S from the total energy (e_E >= kDualEta2 E).
__device__ __forceinline__ float dual_internal(const float* q) {
  return q[4] - 0.5f * (q[1] * q[1] + q[2] * q[2] + q[3] * q[3]) / q[0];
}
__device__ __forceinline__ bool dual_total_branch(const float* q) {
  return dual_internal(q) > kDualEta1 * q[4];
}
__device__ __forceinline__ bool dual_sync_branch(const float* q) {
  return dual_internal(q) >= kDualEta2 * q[4];
}

struct HydroK {
  float a, ia, ia2;   // scale factor, 1/a, 1/a^2
  float gm1, gg1;     // gamma-1, gamma*(gamma-1)
  float efloor;
  float gm2;          // gamma-2 (the entropy's internal energy, dual energy only)
};

__host__ __device__ inline HydroK make_hydro(float a, float gamma, float efloor) {
  HydroK k;
  k.a = a;
  k.ia = 1.0f / a;
  k.ia2 = k.ia * k.ia;
  k.gm1 = gamma - 1.0f;
  k.gg1 = gamma * (gamma - 1.0f);
  k.efloor = efloor;
  k.gm2 = gamma - 2.0f;
  return k;
}

// x^y for x > 0 on the hardware's base-2 exponential and logarithm (v_exp_f32, v_log_f32:
// about one ulp each, so a relative error of a few ulp times |y log2 x|)
__device__ __forceinline__ float pow_approx(float x, float y) {
  return __builtin_amdgcn_exp2f(y * __builtin_amdgcn_logf(x));
}

// How F^R = (c Q + F)/2 or F^L = (c Q - F)/2 of a component whose flux is itself a product,
// F = x y (density, energy, entropy; the momenta's flux is a sum), is rounded.  Every FMA
// of a split is spelled out, so a cell's fluxes do not depend on where the compiler sees it.
enum SplitRound {
  kFluxRounded = 0,    // c Q exact: fma(c, Q, +-round(x y))
  kSpeedRounded = 1,   // x y exact: fma(+-x, y, round(c Q))
  kBothRounded = 2     // round(c Q) +- round(F), for the momenta too
};

// The specific internal energy before the floor, E - |U|^2/2, from et = Et / a^2: with
// E = et / rho exact inside the FMA, or (ROUNDED) rounded first.  The latter with the
// dual-energy entropy, which compares against E, and in the x adjoint (ETOT of the splits:
// there H = Et/a^2 + p, too, takes the rounded et), as those have always been rounded: in cold
// gas e is a small difference, and the last bit of it is seen in the adjoint.
template <bool ROUNDED>
__device__ __forceinline__ float total_minus_kinetic(float et, float ir, float uu) {
  return ROUNDED ? fmaf(-0.5f, uu, et * ir) : fmaf(et, ir, -0.5f * uu);
}

// a + b with both operands already rounded (never contracted with the product behind one)
__device__ __forceinline__ float add_rounded(float a, float b) {
#pragma clang fp contract(off)
  return a + b;
}

// (c q + s x y) / 2, s = +-1, with f = x y rounded
template <int ROUND>
__device__ __forceinline__ float half_split(float c, float q, float s, float f, float x, float y) {
  if (ROUND == kFluxRounded) return 0.5f * fmaf(c, q, s * f);
  if (ROUND == kSpeedRounded) return 0.5f * fmaf(s * x, y, c * q);
  return 0.5f * add_rounded(c * q, s * f);
}

template <int D, int NQ = 5, int RR = kFluxRounded, int RL = kFluxRounded, bool ETOT = false>
__device__ __forceinline__ void split_flux(const float* q, const HydroK& h, float* fr,
                                           float* fl) {
  const float rho = q[0];
  const float ir = rcp_approx(rho);
  const float u0 = q[1] * h.ia * ir, u1 = q[2] * h.ia * ir, u2 = q[3] * h.ia * ir;
  const float uu = fmaf(u2, u2, fmaf(u0, u0, u1 * u1));
  const float et = q[4] * h.ia2;
  float e = total_minus_kinetic<NQ == 6 || ETOT>(et, ir, uu);
  if (NQ == 6 && !(e > kDualEta1 * (et * ir))) e = q[5] * h.ia2 * pow_approx(rho, h.gm2);
  e = fmaxf(e, h.efloor);
  const float pe = h.gm1 * rho;
  const float p = pe * e;
  const float cs = sqrt_approx(h.gg1 * e);
  const float ud = D == 0 ? u0 : (D == 1 ? u1 : u2);
  const float c = (fabsf(ud) + cs) * h.ia;
  const float m = rho * ud;
  // F_rho = m / a, F_E = (a U_d) H with H = Et/a^2 + p, F_S = (S U_d) / a
  const float f0 = m * h.ia;
  fr[0] = half_split<RR>(c, rho, 1.0f, f0, h.ia, m);
  fl[0] = half_split<RL>(c, rho, -1.0f, f0, h.ia, m);
  const float u[3] = {u0, u1, u2};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float f = fmaf(m, u[k], D == k ? p : 0.0f);
    constexpr int mr = RR == kBothRounded ? kBothRounded : kFluxRounded;
    constexpr int ml = RL == kBothRounded ? kBothRounded : kFluxRounded;
    fr[1 + k] = half_split<mr>(c, q[1 + k], 1.0f, f, 0.0f, 0.0f);
    fl[1 + k] = half_split<ml>(c, q[1 + k], -1.0f, f, 0.0f, 0.0f);
  }
  const float au = h.a * ud, H = ETOT ? fmaf(pe, e, et) : fmaf(q[4], h.ia2, p);
  const float f4 = au * H;
  fr[4] = half_split<RR>(c, q[4], 1.0f, f4, au, H);
  fl[4] = half_split<RL>(c, q[4], -1.0f, f4, au, H);
  if (NQ == 6) {
    const float su = q[5] * ud;
    const float f5 = su * h.ia;
    fr[5] = half_split<RR>(c, q[5], 1.0f, f5, h.ia, su);
    fl[5] = half_split<RL>(c, q[5], -1.0f, f5, h.ia, su);
  }
}

// Vector-Jacobian product of the split fluxes at q: given the adjoints gR = dL/dF^R and
// gL = dL/dF^L (NQ each), returns twice dL/dq = (dF^R/dq)^T gR + (dF^L/dq)^T gL
//   = 1/2 [ c s + (dc/dq)(q . s) + (dF/dq)^T d ],  s = gR + gL, d = gR - gL
// (the callers' sums take the exact half along).
// Derivatives are those of the floored EOS (zero through e where the floor is active), of
// the branch of the dual-energy selection that the state takes, and of |U_d| with
// sign(0) = 0.  Every FMA is spelled out and none left to the compiler, so that a cell's
// adjoint is rounded alike in every visit of a walk, wherever its segment begins.
template <int D, int NQ = 5, bool ETOT = false>
__device__ __forceinline__ void split_flux_vjp(const float* q, const HydroK& h, const float* s,
                                               const float* dv, float* out) {
#pragma clang fp contract(off)
  const float rho = q[0];
  const float ir = rcp_approx(rho);
  const float iar = h.ia * ir;
  const float u[3] = {q[1] * iar, q[2] * iar, q[3] * iar};
  const float uu = fmaf(u[2], u[2], fmaf(u[0], u[0], u[1] * u[1]));
  const float ke = 0.5f * uu;
  const float et = q[4] * h.ia2;
  float eraw = total_minus_kinetic<NQ == 6 || ETOT>(et, ir, uu);
  float tot = 1.0f, rs = 0.0f;   // tot: the total energy's branch; rs = rho^(gamma-2)
  if (NQ == 6) {
    tot = eraw > kDualEta1 * (et * ir) ? 1.0f : 0.0f;
    rs = pow_approx(rho, h.gm2);
    eraw = tot > 0.0f ? eraw : q[5] * h.ia2 * rs;
  }
  // 0 where the floor is active (its derivative), 1 elsewhere; every term is computed and
  // masked, so the function has no branches
  const float live = eraw < h.efloor ? 0.0f : 1.0f;
  const float e = fmaxf(eraw, h.efloor);
  const float pe = h.gm1 * rho;
  const float p = pe * e;
  const float cs = sqrt_approx(h.gg1 * e);
  const float ud = u[D];
  const float md = q[1 + D];
  const float sgn = md > 0.0f ? 1.0f : (md < 0.0f ? -1.0f : 0.0f);
  const float c = (fabsf(ud) + cs) * h.ia;

  // derivatives of e (zero when floored); the entropy's branch: e = S rho^(gamma-2) / a^2
  const float lt = live * tot;
  float er = lt * (ke - e) * ir;
  if (NQ == 6) er = fmaf(live * (1.0f - tot) * h.gm2 * e, ir, er);
  const float liar = -lt * iar;
  float em[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) em[k] = liar * u[k];
  const float eE = lt * h.ia2 * ir;
  const float eS = NQ == 6 ? live * (1.0f - tot) * h.ia2 * rs : 0.0f;
  // pressure derivatives
  const float pr = h.gm1 * fmaf(rho, er, e);
  float pm[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) pm[k] = pe * em[k];
  const float pE = pe * eE;
  // freezing-speed derivatives
  const float cse = live > 0.0f ? 0.5f * h.gg1 * rcp_approx(cs) : 0.0f;   // cs may be 0 if floored
  const float cr = h.ia * fmaf(-fabsf(ud), ir, cse * er);
  float cm[3];
#pragma unroll
  for (int k = 0; k < 3; ++k)
    cm[k] = h.ia * (k == D ? fmaf(sgn, iar, cse * em[k]) : cse * em[k]);
  const float cE = h.ia * cse * eE;

  float qs = fmaf(q[0], s[0], q[1] * s[1]);
#pragma unroll
  for (int k = 2; k < NQ; ++k) qs = fmaf(q[k], s[k], qs);
  // (dF/dq)^T dv
  const float H = fmaf(q[4], h.ia2, p) * ir;
  const float vu = fmaf(dv[3], u[2], fmaf(dv[1], u[0], dv[2] * u[1]));
  const float va = dv[4] * h.a;
  const float W = fmaf(va, ud, dv[1 + D]);
  float jt[5];
  jt[0] = fmaf(-(va * ud), H, fmaf(-ud, vu, pr * W));
  float diag = fmaf(dv[4], H, fmaf(dv[0], h.ia2, h.ia * vu));
  if (NQ == 6) {
    // F_S = S U_d / a
    const float fs = dv[5] * q[5] * h.ia;
    jt[0] = fmaf(-(fs * ud), ir, jt[0]);
    diag = fmaf(fs, iar, diag);
  }
  const float uda = ud * h.ia;
#pragma unroll
  for (int k = 0; k < 3; ++k)
    jt[1 + k] = fmaf(pm[k], W, k == D ? fmaf(uda, dv[1 + k], diag) : uda * dv[1 + k]);
  jt[4] = fmaf(pE, W, va * ud * h.ia2);

  const float dc[5] = {cr, cm[0], cm[1], cm[2], cE};
#pragma unroll
  for (int k = 0; k < 5; ++k) out[k] = fmaf(c, s[k], dc[k] * qs) + jt[k];
  if (NQ == 6) {
    const float pS = pe * eS;
    const float cS = h.ia * cse * eS;
    out[5] = fmaf(dv[5], uda, fmaf(pS, W, fmaf(c, s[5], cS * qs)));
  }
}

// van Leer limiter (Sec. 2.3.2): phi(x, y) = (x y + |x y|) / (x + y + eps sgn(x+y)),
// eps = 1e-20, sgn(0) = +1.  The sweeps call it on half differences, phi(a/2, b/2), written
// here on the undivided differences a, b:
//   van_leer_half(a, b) = a b / (a + b + 2 eps sgn(a+b))  where a b > 0,  0 otherwise.
// Where a b > 0, |a + b| >= 2 sqrt(a b) > 0: the guard only moves the value by at most eps/2
// in absolute terms, below any FP32 flux, and is left out.  The selection on a b > 0 is the
// function itself (an FMA-contracted x y + |x y| is not exactly zero for x y < 0); both
// sides are computed and the discarded one is never read.
constexpr float kLimEps = 1e-20f;

__device__ __forceinline__ float van_leer_half(float a, float b) {
  const float ab = a * b;
  const float r = ab * rcp_approx(a + b);
  return ab > 0.0f ? r : 0.0f;
}

// Partial derivatives of van_leer_half: (b/(a+b))^2 and (a/(a+b))^2 where a b > 0; where
// a b == 0 the derivative of |a b| is taken with sign(0) = 0, which gives half the one-sided
// slopes b/(2(a+b)) and a/(2(a+b)) (the guard keeps them finite at a = b = 0); zero where
// a b < 0.
__device__ __forceinline__ void van_leer_half_d(float a, float b, float& da, float& db) {
  const float ab = a * b;
  const float s = a + b;
  const float id = rcp_approx(s + __builtin_copysignf(2.0f * kLimEps, s));
  const float hb = b * id, ha = a * id;
  // da = hb * (hb, 1/2 or 0 as a b > 0, = 0 or < 0), db likewise with ha: one product each
  // (a zero may come out as -0)
  const float k = ab < 0.0f ? 0.0f : 0.5f;
  da = hb * (ab > 0.0f ? hb : k);
  db = ha * (ab > 0.0f ? ha : k);
}

// ---------------------------------------------------------------------------------------
// Philox-4x32-10 (Salmon et al., SC'11): counter-based generator for the white noise and the
// star-formation uniforms.  Counter (cell, step, tag, 0), key (seed lo, seed hi).
// ---------------------------------------------------------------------------------------
constexpr uint32_t kTagWhite = 0x574E0000u;
constexpr uint32_t kTagStarform = 0x53460000u;
constexpr uint32_t kTagMlpSample = 0x4D4C0000u;   // training states of the learned closure

__host__ __device__ inline void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    const uint64_t p0 = static_cast<uint64_t>(0xD2511F53u) * c[0];
    const uint64_t p1 = static_cast<uint64_t>(0xCD9E8D57u) * c[2];
    const uint32_t hi0 = static_cast<uint32_t>(p0 >> 32), lo0 = static_cast<uint32_t>(p0);
    const uint32_t hi1 = static_cast<uint32_t>(p1 >> 32), lo1 = static_cast<uint32_t>(p1);
    const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
    c[0] = n0;
    c[1] = lo1;
    c[2] = n2;
    c[3] = lo0;
  }
}

// 24 random bits plus one half, times 2^-24: u in (0,1), exact in float and double.
__host__ __device__ inline double uniform_open_d(uint32_t bits) {
  return (static_cast<double>(bits >> 8) + 0.5) * (1.0 / 16777216.0);
}
__host__ __device__ inline float uniform_open_f(uint32_t bits) {
  return (static_cast<float>(bits >> 8) + 0.5f) * (1.0f / 16777216.0f);
}

}  // namespace dh
