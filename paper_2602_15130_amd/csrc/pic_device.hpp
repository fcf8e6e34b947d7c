// Device-side building blocks of the PIC/DSMC manufactured-solution step:
// simulation constants, the counter-based random stream, and the manufactured
// solution of Sec. 3 / Sec. 5.2 (FP64, with FP32 variants for the mixed form).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pic {

constexpr double kPi = 3.14159265358979323846;
constexpr float kPiF = 3.14159265358979323846f;

// Everything a kernel needs to know about the problem, derived once on the host.
// Unsigned division by a divisor d >= 1 fixed for the whole run, as one
// multiply-high and a shift (Granlund and Montgomery, PLDI 1994, the
// round-up multiplier): with s = ceil(log2 d) and
// m = floor(2^32 (2^s - d) / d) + 1, n / d = (mulhi(n, m) + n) >> s for
// every 32-bit n when the sum is formed in 64 bits.
struct DivMagic {
  uint32_t m, s;
};

__host__ __device__ inline DivMagic div_magic(uint32_t d) {
  uint32_t s = 0;
  while ((uint64_t(1) << s) < d) ++s;
  const uint64_t m = (((uint64_t(1) << s) - d) << 32) / d + 1;
  return {(uint32_t)m, s};
}

__host__ __device__ inline uint32_t div_by(DivMagic q, uint32_t n) {
  const uint64_t hi = ((uint64_t)n * q.m) >> 32;
  return (uint32_t)((hi + n) >> q.s);
}

struct SimConst {
  int family;          // 0 paper (Sec. 5.2), 1 configuration family
  int sigma_model;     // 0 polynomial (eq. sigma_ms), 1 variable hard sphere
  int n_sigma;
  int collisions, isolate, navg;
  int nc[3];
  int nn;              // nodes = cells
  DivMagic div_x, div_xy;  // division by nc[0] and by nc[0] nc[1]
  int64_t np;
  uint64_t seed;
  uint32_t rep;
  double L[3], h[3], inv_h[3], ih2[3];
  double inv_L[3], wave[3];  // 1 / L and 2 pi / L
  double qm;           // q/m, or 0 when the field does not act on the particles
  double p2f;          // 1 when the particles feed the Poisson source, else 0
  double q, eps0, T, vbar, phibar, rho_amp;
  double sigma_n[3];
  double sg_coef, sg_pow;  // VHS: sigma g = sg_coef g^sg_pow
  double sigma_ref, g_ref, omega, g_max;
  double sgmax;        // (sigma g)_max over [0, g_max]
  double sr[3];        // sigma_n vbar^(2n) / (sigma g)_max: the accept ratio in units of vbar
  double inv_vbar;     // 1 / vbar
  double pmax;         // Algorithm 1: (sigma g)_max w dt / dV
  double w, dV, dt;
  double rho_scale;    // q w / dV
  double src_half;     // w dt / (2 dV)
  double nphys;
  int poisson_op;      // field discretization: 0 7-point differences, 1 trilinear elements
  int chi_model;       // polar-angle model: 0 isotropic, 1 manufactured anisotropy, 2 VSS
  double chi_alpha;    // VSS exponent
  int coding_error;    // Sec. 5.4.1 Error 1 / Error 2 (verification studies), 0 none
  // completed steps, kept on the device for captured steps (shared by all
  // ensemble members; null when unused)
  const long long* stepc;
  double* anglog;      // scattering-angle records (chi, eps) of accepted collisions, or null
  int64_t angcap;      // records that fit
  // Ensembles: the members of one context share every size and differ only in
  // the replicate.  Member m = member0 + blockIdx.z uses replicate rep + m and
  // owns the workspace bytes starting m * mstride after member 0's.
  int member0;
  int64_t mstride;
};

// The ensemble member a workgroup works for, and a member-0 workspace pointer
// moved to that member's copy (null stays null).
__device__ inline int member_of(const SimConst& K) { return K.member0 + (int)blockIdx.z; }
template <class T>
__device__ inline T* mem(const SimConst& K, T* p) {
  return p ? (T*)((char*)p + (int64_t)member_of(K) * K.mstride) : p;
}
// The same for kernels that receive only the stride (members in blockIdx.z).
template <class T>
__device__ inline T* mem_z(int64_t mstride, T* p) {
  return p ? (T*)((char*)p + (int64_t)blockIdx.z * mstride) : p;
}

// ---------------------------------------------------------------------------
// Philox4x64-10 (Salmon et al., SC'11).  Counter layout of the random stream:
//   c0 entity (particle id or cell), c1 step, c2 tag<<56 | call<<48 | outcome,
//   c3 block; key = (seed, replicate; an ensemble member adds its index to
//   the replicate).  The N_pairs uniforms of four
//   consecutive outcomes share one block: tag NPAIRS, outcome field k / 4,
//   word k mod 4.
// ---------------------------------------------------------------------------
enum : uint64_t { kTagInit = 1, kTagColl = 2, kTagRedraw = 3, kTagNpairs = 4 };

struct U64x4 {
  uint64_t w[4];
};

// The 128-bit product of two 64-bit words from four 32 x 32 + 64 bit
// multiply-adds (v_mad_u64_u32, a quarter-rate instruction, is what a random
// block costs; high and low word taken apart need seven such multiplies).
__host__ __device__ inline void mul_wide(uint64_t a, uint64_t b, uint64_t& hi, uint64_t& lo) {
  const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32);
  const uint32_t b0 = (uint32_t)b, b1 = (uint32_t)(b >> 32);
  const uint64_t p = (uint64_t)a0 * b0;
  const uint64_t t = (uint64_t)a1 * b0 + (p >> 32);
  const uint64_t u = (uint64_t)a0 * b1 + (uint32_t)t;
  hi = (uint64_t)a1 * b1 + (t >> 32) + (u >> 32);
  lo = (u << 32) | (uint32_t)p;
}

// a ^ b ^ c, one three-input bit operation per half on the GPU.
__host__ __device__ inline uint64_t xor3(uint64_t a, uint64_t b, uint64_t c) {
#if defined(__HIP_DEVICE_COMPILE__)
  const uint32_t lo = __builtin_amdgcn_bitop3_b32((uint32_t)a, (uint32_t)b, (uint32_t)c, 0x96);
  const uint32_t hi = __builtin_amdgcn_bitop3_b32((uint32_t)(a >> 32), (uint32_t)(b >> 32),
                                                  (uint32_t)(c >> 32), 0x96);
  return ((uint64_t)hi << 32) | lo;
#else
  return a ^ b ^ c;
#endif
}

__host__ __device__ inline U64x4 philox(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3,
                                        uint64_t k0, uint64_t k1) {
  const uint64_t m0 = 0xD2E7470EE14C6C93ull, m1 = 0xCA5A826395121157ull;
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    uint64_t h0, l0, h1, l1;
    mul_wide(m0, c0, h0, l0);
    mul_wide(m1, c2, h1, l1);
    uint64_t a = xor3(h1, c1, k0), b = xor3(h0, c3, k1);
    c0 = a; c1 = l1; c2 = b; c3 = l0;
    k0 += 0x9E3779B97F4A7C15ull;
    k1 += 0xBB67AE8584CAA73Bull;
  }
  return U64x4{{c0, c1, c2, c3}};
}

__device__ inline U64x4 stream_block(const SimConst& K, uint64_t entity, uint64_t step,
                                     uint64_t tag, uint64_t call, uint64_t k, uint64_t blk) {
  return philox(entity, step, (tag << 56) | (call << 48) | k, blk, K.seed,
                (uint64_t)K.rep + (uint64_t)member_of(K));
}

// [0,1) with 53 bits, (0,1) with 52 bits + 1/2, floor(U n) exactly.
__device__ inline double unif(uint64_t w) { return (double)(w >> 11) * 0x1.0p-53; }
__device__ inline double unif_open(uint64_t w) { return ((double)(w >> 12) + 0.5) * 0x1.0p-52; }
__device__ inline float unif32(uint64_t w) { return (float)(uint32_t)(w >> 40) * 0x1.0p-24f; }
__device__ inline int index_below(uint64_t w, int n) {
  return (int)__umul64hi(w & ~0x7FFull, (uint64_t)(uint32_t)n);
}

// ---------------------------------------------------------------------------
// Safeguarded Halley iteration for a monotone CDF on [lo, hi]: F(x, dens, slope)
// gives F, its density and the density's slope, which the CDFs here have at no
// further cost, and the order three saves about half of Newton's evaluations
// (2^23 initial states 6.4 -> 1.5 ms with the paper's functions, 1.8 -> 0.9 with
// the configuration family's).
// F.done(x, step): whether the root is reached after a step of that length (the
// next one, about the cube of this one in the CDF's own length, would be below
// the rounding of x).
// ---------------------------------------------------------------------------
template <class Cdf>
__device__ inline double invert_cdf(const Cdf& F, double target, double lo, double hi, double x) {
  if (!(x > lo && x < hi)) x = 0.5 * (lo + hi);
  for (int it = 0; it < 200; ++it) {
    double dens, slope;
    const double res = F(x, dens, slope) - target;
    if (res == 0.0) break;
    if (res > 0.0) hi = x; else lo = x;
    const double den = 2.0 * dens * dens - res * slope;
    double nx = x - 2.0 * res * dens / den;
    const bool halley = dens > 0.0 && den > 0.0;
    // (before the bracket's test: at the root the step is rounding, to either side)
    if (halley && F.done(x, fabs(nx - x))) {
      x = fmin(fmax(nx, lo), hi);
      break;
    }
    if (!(halley && nx > lo && nx < hi)) nx = 0.5 * (lo + hi);
    if (nx == lo || nx == hi || fabs(nx - x) <= 4.440892098500626e-16 * fabs(nx)) {
      x = nx;
      break;
    }
    x = nx;
  }
  return x;
}

// ---------------------------------------------------------------------------
// Manufactured solution.
// ---------------------------------------------------------------------------
// What the Sec. 5.2 positions need of the time: e = exp(t / T), the phase
// shifts of y and z, and the trigonometric functions of those.
struct PaperTime {
  double e, sy, sz;              // shifts 0.15 e and e / 15
  double sin_y, cos_y, sin_z, cos_z;  // of 2 pi times the shifts
};
__device__ inline PaperTime paper_time(const SimConst& K, double t) {
  PaperTime P{};
  if (K.family == 1) return P;
  P.e = exp(t / K.T);
  P.sy = 0.15 * P.e;
  P.sz = P.e / 15.0;
  sincospi(2.0 * P.sy, &P.sin_y, &P.cos_y);
  sincospi(2.0 * P.sz, &P.sin_z, &P.cos_z);
  return P;
}

// Sec. 5.2 position densities per unit length and their CDFs from 0, as functions
// of s = x / L: density (1 + amp sin 2 pi (s + shift)) / L, CDF s + amp (c0 -
// cos 2 pi (s + shift)) / (2 pi).
struct PaperPosCdf {
  double inv_L, amp, shift, c0;
  __device__ PaperPosCdf(const SimConst& K, const PaperTime& P, int d)
      : inv_L(K.inv_L[d]),
        amp(d == 0 ? 0.2 * P.e : (d == 1 ? 0.2 : -(P.e / 6.0))),
        shift(d == 0 ? 0.0 : (d == 1 ? -P.sy : P.sz)),
        c0(d == 0 ? 1.0 : (d == 1 ? P.cos_y : P.cos_z)) {}
  __device__ double operator()(double x, double& dens, double& slope) const {
    const double s = x * inv_L;
    double sn, cs;
    sincospi(2.0 * (s + shift), &sn, &cs);
    dens = (1.0 + amp * sn) * inv_L;
    slope = 2.0 * kPi * amp * cs * inv_L * inv_L;
    return s + amp * (c0 - cs) * (0.5 / kPi);
  }
  // (a step's error is (2 pi)^2 times its cube up to amplitudes of 0.86; beyond, it and
  // the rounding of the CDF over the density grow alike: for amplitudes to 1 - 1e-7 the
  // CDF at the root is within 3e-16 of its target)
  __device__ bool done(double, double step) const { return step * inv_L <= 1e-6; }
};

// Configuration family: CDF of z given (x, y), a = A sin(2 pi x/L) sin(2 pi y/L).
struct CfgZCdf {
  double inv_L, a;
  __device__ double operator()(double z, double& dens, double& slope) const {
    const double s = z * inv_L;
    double sn, cs;
    sincospi(2.0 * s, &sn, &cs);
    dens = (1.0 + a * sn) * inv_L;
    slope = 2.0 * kPi * a * cs * inv_L * inv_L;
    return s + a * (1.0 - cs) * (0.5 / kPi);
  }
  __device__ bool done(double, double step) const { return step * inv_L <= 1e-6; }
};

// Paper velocity CDF in units of vhat: G(a) = (1 + erf a)/2 - a e^{-a^2}/sqrt(pi),
// to about 1e-16 absolute in either tail.
struct PaperGCdf {
  __device__ double operator()(double a, double& dens, double& slope) const {
    const double ea = exp(-a * a);
    dens = 1.1283791670955126 * a * a * ea;  // 2/sqrt(pi)
    slope = 2.2567583341910251 * a * (1.0 - a * a) * ea;
    return 0.5 + 0.5 * erf(a) - 0.5641895835477563 * a * ea;
  }
  __device__ bool done(double a, double step) const { return step * (1.0 + a * a) <= 1e-6 * fabs(a); }
};

__device__ inline void init_uniforms(const SimConst& K, int64_t id, double xi[6]) {
  U64x4 a = stream_block(K, (uint64_t)id, 0, kTagInit, 0, 0, 0);
  U64x4 b = stream_block(K, (uint64_t)id, 0, kTagInit, 0, 0, 1);
  for (int d = 0; d < 3; ++d) {
    xi[d] = unif_open(a.w[d]);
    xi[3 + d] = unif_open(b.w[d]);
  }
}

__device__ inline void velocity_uniforms(const SimConst& K, int64_t id, double xv[3]) {
  U64x4 b = stream_block(K, (uint64_t)id, 0, kTagInit, 0, 0, 1);
  for (int d = 0; d < 3; ++d) xv[d] = unif_open(b.w[d]);
}

__device__ inline void position_uniforms(const SimConst& K, int64_t id, double xp[3]) {
  U64x4 a = stream_block(K, (uint64_t)id, 0, kTagInit, 0, 0, 0);
  for (int d = 0; d < 3; ++d) xp[d] = unif_open(a.w[d]);
}

__device__ inline void vhat_of_t(const SimConst& K, double t, double vh[3], double vd[3]) {
  if (K.family == 1) {
    vh[0] = vh[1] = vh[2] = K.vbar;
    vd[0] = vd[1] = vd[2] = 0.0;
    return;
  }
  double u = t / K.T;
  vh[0] = (1.0 + 0.2 * sinpi(0.5 * u)) * K.vbar;
  vh[1] = (1.0 + 0.2 * cospi(u)) * K.vbar;
  vh[2] = (1.0 + 0.2 * sinpi(1.5 * u)) * K.vbar;
  vd[0] = 0.2 * (0.5 * kPi / K.T) * cospi(0.5 * u) * K.vbar;
  vd[1] = -0.2 * (kPi / K.T) * sinpi(u) * K.vbar;
  vd[2] = 0.2 * (1.5 * kPi / K.T) * cospi(1.5 * u) * K.vbar;
}

// Standard normal quantile.  The root is taken on the lower tail, Phi(-z) =
// min(xi, 1 - xi) (1 - xi is exact for xi >= 1/2), which keeps the residual
// well conditioned in both tails; starting guess Abramowitz & Stegun 26.2.23
// (|error| < 4.5e-4), then Halley steps on 0.5 erfc(-y / sqrt 2) in FP64: one or
// two, the next being below rounding once a step is under 1e-6 / (1 + y^2).
__device__ inline double normal_quantile(double xi) {
  const double pp = xi < 0.5 ? xi : 1.0 - xi;
  const double t = sqrt(-2.0 * log(pp));
  double y = -(t - (2.515517 + t * (0.802853 + t * 0.010328)) /
                       (1.0 + t * (1.432788 + t * (0.189269 + t * 0.001308))));
#pragma unroll 1
  for (int it = 0; it < 4; ++it) {
    const double f = 0.5 * erfc(-0.7071067811865476 * y) - pp;
    const double dens = 0.3989422804014327 * exp(-0.5 * y * y);
    const double dy = f / (dens + 0.5 * y * f);
    y -= dy;
    if (fabs(dy) * (1.0 + y * y) <= 1e-6) break;
  }
  return xi < 0.5 ? y : -y;
}

// Paper family: a = G^{-1}(xi), time independent (v^M = vhat(t) a).  The
// density of eq. fv is even, so G^{-1}(xi) = -G^{-1}(1 - xi): solve on the
// lower half.  The guess is within 6 %: near the centre the inverted series
// of G, in the tail G(a) ~ (|a| + 1/(2|a|)) e^{-a^2} / sqrt(pi) solved for the
// exponent twice; one to three Halley steps follow.
__device__ inline double paper_a(double xi) {
  const double pp = xi < 0.5 ? xi : 1.0 - xi;
  double a;
  if (pp > 0.2) {
    a = cbrt(2.6586807763582730 * (pp - 0.5));  // 1.5 sqrt(pi)
    const double b2 = a * a;
    a = a * (1.0 + b2 * (0.2 + b2 * 0.0771));
  } else {
    double x = sqrt(-log(pp));
    for (int it = 0; it < 2; ++it)
      x = sqrt(fmax(0.3, -log(1.7724538509055159 * pp / (x + 0.5 / x))));
    a = -x;
  }
  a = invert_cdf(PaperGCdf{}, pp, -30.0, 0.0, a);
  return xi < 0.5 ? a : -a;
}

// Velocity shape factor per component: v^M(t) = vhat(t) * shape.
__device__ inline void velocity_shape(const SimConst& K, const double xv[3], double a[3]) {
  for (int d = 0; d < 3; ++d) a[d] = (K.family == 1) ? normal_quantile(xv[d]) : paper_a(xv[d]);
}

__device__ inline void manufactured_velocity(const SimConst& K, const double a[3], double t,
                                             double v[3], double vdot[3]) {
  double vh[3], vd[3];
  vhat_of_t(K, t, vh, vd);
  for (int d = 0; d < 3; ++d) {
    v[d] = vh[d] * a[d];
    vdot[d] = vd[d] * a[d];
  }
}

__device__ inline void paper_position(const SimConst& K, const double xp[3], const PaperTime& P,
                                      const double* guess, double x[3]) {
  for (int d = 0; d < 3; ++d)
    x[d] = invert_cdf(PaperPosCdf(K, P, d), xp[d], 0.0, K.L[d], guess ? guess[d] : K.L[d] * xp[d]);
}

__device__ inline void cfg_position(const SimConst& K, const double xp[3], double x[3]) {
  x[0] = K.L[0] * xp[0];
  x[1] = K.L[1] * xp[1];
  CfgZCdf F{K.inv_L[2], K.rho_amp * sinpi(2.0 * xp[0]) * sinpi(2.0 * xp[1])};
  x[2] = invert_cdf(F, xp[2], 0.0, K.L[2], K.L[2] * xp[2]);
}

// eq. mms_sol for the positions at the time of P; `guess` speeds up the
// paper-family roots.
__device__ inline void manufactured_position(const SimConst& K, const double xp[3], const PaperTime& P,
                                             const double* guess, double x[3]) {
  if (K.family == 1) cfg_position(K, xp, x);
  else paper_position(K, xp, P, guess, x);
}
__device__ inline void manufactured_position(const SimConst& K, const double xp[3], double t,
                                             const double* guess, double x[3]) {
  manufactured_position(K, xp, paper_time(K, t), guess, x);
}

// xdot^M = -(dF/dt)/f at x^M (Sec. 3.2), dF/dt at fixed x of the Sec. 5.2 CDFs:
// amp and shift change by amp_t and shift_t, so 2 pi dF/dt = amp_t (c0 - cos) +
// 2 pi amp shift_t (sin - s0), with sin and cos at x and c0, s0 at x = 0.
__device__ inline void manufactured_xdot(const SimConst& K, const double xm[3], const PaperTime& P,
                                         double xd[3]) {
  if (K.family == 1) {
    xd[0] = xd[1] = xd[2] = 0.0;
    return;
  }
  const double rate = 1.0 / K.T;
  const double amp_t[3] = {0.2 * P.e * rate, 0.0, -(P.e / 6.0) * rate};
  const double shift_t[3] = {0.0, -P.sy * rate, P.sz * rate};
  const double s0[3] = {0.0, -P.sin_y, P.sin_z};
  for (int d = 0; d < 3; ++d) {
    const PaperPosCdf F(K, P, d);
    double sn, cs;
    sincospi(2.0 * (xm[d] * F.inv_L + F.shift), &sn, &cs);
    const double dens = (1.0 + F.amp * sn) * F.inv_L;
    const double dFdt = amp_t[d] * (F.c0 - cs) * (0.5 / kPi) + F.amp * shift_t[d] * (sn - s0[d]);
    xd[d] = -dFdt / dens;
  }
}
__device__ inline void manufactured_xdot(const SimConst& K, const double xm[3], double t,
                                         double xd[3]) {
  manufactured_xdot(K, xm, paper_time(K, t), xd);
}

// Number density f_x (eq. fx), integrating to N over the box.
__device__ inline double number_density(const SimConst& K, const double x[3], const PaperTime& P) {
  if (K.family == 1) {
    double s = sinpi(2.0 * x[0] / K.L[0]) * sinpi(2.0 * x[1] / K.L[1]) * sinpi(2.0 * x[2] / K.L[2]);
    return K.nphys / (K.L[0] * K.L[1] * K.L[2]) * (1.0 + K.rho_amp * s);
  }
  double r = K.nphys;
  for (int d = 0; d < 3; ++d) {
    double dens, slope;
    (void)PaperPosCdf(K, P, d)(x[d], dens, slope);
    r *= dens;
  }
  return r;
}

// phi^M = phibar e^{t/2T} prod sin(2 pi (x_d/L_d - c_d)), c = (1/7, 1/5, 1/3).
__device__ inline void phiM_factors(const SimConst& K, const double x[3], double s[3],
                                    double c[3]) {
  const double shift[3] = {1.0 / 7.0, 1.0 / 5.0, 1.0 / 3.0};
  for (int d = 0; d < 3; ++d) {
    double arg = 2.0 * (x[d] * K.inv_L[d] - shift[d]);
    sincospi(arg, &s[d], &c[d]);
  }
}

__device__ inline double phiM(const SimConst& K, const double x[3], double t) {
  double s[3], c[3];
  phiM_factors(K, x, s, c);
  return K.phibar * exp(0.5 * t / K.T) * s[0] * s[1] * s[2];
}

__device__ inline double lap_phiM(const SimConst& K, const double x[3], double t) {
  double k2 = 0.0;
  for (int d = 0; d < 3; ++d) k2 += K.wave[d] * K.wave[d];
  return -k2 * phiM(K, x, t);
}

__device__ inline void EM(const SimConst& K, const double x[3], double t, double E[3]) {
  double s[3], c[3];
  phiM_factors(K, x, s, c);
  double a = K.phibar * exp(0.5 * t / K.T);
  E[0] = -a * K.wave[0] * c[0] * s[1] * s[2];
  E[1] = -a * K.wave[1] * s[0] * c[1] * s[2];
  E[2] = -a * K.wave[2] * s[0] * s[1] * c[2];
}

// Cross-section models known at compile time in the fused kernels.
enum { kSigHS = 0, kSigMaxwell = 1, kSigPoly = 2 };

template <int SIG>
__device__ inline double sigma_g_t(const SimConst& K, double g) {
  if (SIG == kSigHS) return K.sg_coef * g;          // omega = 1/2: sigma constant
  if (SIG == kSigMaxwell) return K.sg_coef;         // omega = 1: sigma g constant
  double g2 = g * g, r = K.sigma_n[0];
  if (K.n_sigma > 1) r += K.sigma_n[1] * g2;
  if (K.n_sigma > 2) r += K.sigma_n[2] * (g2 * g2);
  return r;
}

// sigma(g) g.
__device__ inline double sigma_g(const SimConst& K, double g) {
  if (K.sigma_model == 1) return K.sg_coef * pow(g, K.sg_pow);
  double g2 = g * g, r = K.sigma_n[0];
  if (K.n_sigma > 1) r += K.sigma_n[1] * g2;
  if (K.n_sigma > 2) r += K.sigma_n[2] * (g2 * g2);
  return r;
}

// Hard sphere, Gaussian partners: int g (v_q - v_p) f_v = -s^2 K(l) v_p/|v_p|.
// K(l) = [(l^4 + 2l^2 - 1) erf(l/sqrt2) + 2l(l^2+1) phi_N(l)] / l^2, summed as a
// power series below l = 0.5 where the closed form cancels (eleven terms: from
// the tenth on they no longer change the rounded sum).
__device__ inline double hs_kernel(double l) {
  if (l < 0.5) {
    // erf(l/sqrt2) = sqrt(2/pi) sum a_n l^(2n+1); 2 l phi_N(l) = sqrt(2/pi) sum b_n l^(2n+1)
    // with b_n = (-1/2)^n / n!, a_n = b_n / (2n+1); K = sqrt(2/pi) sum_j c_j l^(2j-1),
    // c_j = a_{j-2} + 2 a_{j-1} - a_j + b_{j-1} + b_j.
    double bm2 = 0.0, am2 = 0.0;         // n = j-2
    double bm1 = 1.0, am1 = 1.0;         // n = j-1 (j = 1)
    double sum = 0.0, l2 = l * l, lp = l;  // l^(2j-1)
    for (int j = 1; j < 12; ++j) {
      double bj = bm1 * (-0.5) / j, aj = bj / (2.0 * j + 1.0);
      sum += (am2 + 2.0 * am1 - aj + bm1 + bj) * lp;
      am2 = am1; bm2 = bm1; am1 = aj; bm1 = bj;
      lp *= l2;
    }
    (void)bm2;
    return 0.7978845608028654 * sum;
  }
  double l2 = l * l;
  double phin = 0.3989422804014327 * exp(-0.5 * l2);
  return ((l2 * l2 + 2.0 * l2 - 1.0) * erf(0.7071067811865476 * l) + 2.0 * l * (l2 + 1.0) * phin) / l2;
}

__device__ inline void poly_source_inl(const SimConst& K, const double u[3], double t,
                                       double out[3]);
__device__ __noinline__ void poly_source(const SimConst& K, const double u[3], double t,
                                         double out[3]);

// eq. vel_change_1c integral (no prefactor) at particle velocity u and time t.
__device__ inline void source_integral(const SimConst& K, const double u[3], double t,
                                       double out[3]) {
  if (K.sigma_model == 1) {
    if (K.omega == 1.0) {
      double c = K.sigma_ref * K.g_ref;
      for (int i = 0; i < 3; ++i) out[i] = -c * u[i];
      return;
    }
    double sp = sqrt(u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
    if (sp == 0.0) {
      out[0] = out[1] = out[2] = 0.0;
      return;
    }
    double s = K.vbar;
    const double f = -K.sigma_ref * s * s * hs_kernel(sp * K.inv_vbar) / sp;
    for (int i = 0; i < 3; ++i) out[i] = f * u[i];
    return;
  }
  poly_source(K, u, t, out);
}

// Polynomial cross section (eq. sigma_ms): sum_n sigma_n f_n (eq. vel_change_3).
__device__ inline void poly_source_inl(const SimConst& K, const double u[3], double t,
                                       double out[3]) {
  double u2 = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
  double f[3][3];
  if (K.family == 0) {
    double vh[3], vd[3];
    vhat_of_t(K, t, vh, vd);
    double h2[3] = {vh[0] * vh[0], vh[1] * vh[1], vh[2] * vh[2]};
    double H = h2[0] + h2[1] + h2[2];
    double mix = h2[0] * u[0] * u[0] + h2[1] * u[1] * u[1] + h2[2] * u[2] * u[2];
    for (int i = 0; i < 3; ++i) {
      double others = h2[(i + 1) % 3] * h2[(i + 2) % 3];
      f[0][i] = -u[i];
      f[1][i] = -0.5 * (3.0 * H + 6.0 * h2[i] + 2.0 * u2) * u[i];
      f[2][i] = -0.25 * (15.0 * H * H + 36.0 * h2[i] * h2[i] + 24.0 * u2 * h2[i] + 4.0 * u2 * u2 +
                         24.0 * h2[i] * H + 12.0 * u2 * H + 24.0 * mix - 12.0 * others) * u[i];
    }
  } else {
    // symmetric product density with m2 = s^2, m4 = 3 s^4 per component
    double m2 = K.vbar * K.vbar, m4 = 3.0 * m2 * m2;
    for (int i = 0; i < 3; ++i) {
      int j = (i + 1) % 3, k = (i + 2) % 3;
      double ui2 = u[i] * u[i], uj2 = u[j] * u[j], uk2 = u[k] * u[k];
      double qj = m2 + uj2, qk = m2 + uk2;
      double s1 = qj + qk;
      double s2 = (m4 + 6.0 * uj2 * m2 + uj2 * uj2) + (m4 + 6.0 * uk2 * m2 + uk2 * uk2);
      f[0][i] = -u[i];
      f[1][i] = -u[i] * (3.0 * m2 + ui2 + s1);
      f[2][i] = -u[i] * (5.0 * m4 + 10.0 * ui2 * m2 + ui2 * ui2 + s2 + 2.0 * qj * qk +
                         2.0 * (3.0 * m2 + ui2) * s1);
    }
  }
  for (int i = 0; i < 3; ++i) {
    double r = 0.0;
    for (int n = 0; n < K.n_sigma; ++n) r += K.sigma_n[n] * f[n][i];
    out[i] = r;
  }
}

}  // namespace pic

namespace pic {
__device__ __noinline__ void poly_source(const SimConst& K, const double u[3], double t,
                                         double out[3]) {
  poly_source_inl(K, u, t, out);
}

// Source integral with the cross-section model fixed at compile time.
template <int SIG>
__device__ inline void source_integral_t(const SimConst& K, const double u[3], double t,
                                         double out[3]) {
  if (SIG == kSigMaxwell) {
    double c = K.sigma_ref * K.g_ref;
    for (int i = 0; i < 3; ++i) out[i] = -c * u[i];
  } else if (SIG == kSigHS) {
    double sp = sqrt(u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
    if (sp == 0.0) {
      out[0] = out[1] = out[2] = 0.0;
      return;
    }
    double s = K.vbar;
    const double f = -K.sigma_ref * s * s * hs_kernel(sp * K.inv_vbar) / sp;
    for (int i = 0; i < 3; ++i) out[i] = f * u[i];
  } else {
    poly_source_inl(K, u, t, out);
  }
}
}  // namespace pic
