// Device-side building blocks of the multi-channel VEGAS sample pass on
// gfx950: Philox4x32-10, the uniform -> (bin, fraction) rule, the 1-d channel
// maps, channel densities, the peak-mixture integrand and compensated sums.
//
// Method: Brass, Kilian, Reuter, arXiv:1811.09711, Sec. 3.2 (VEGAS step map,
// eq. g(x)), Sec. 3.4 (channel densities q_c = 1/phi_c'), Sec. 3.5 (eq. g(p)).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mcv {

// Hint cells per axis of a job's grids: 256 for at most 64 bins per axis,
// else 512, so that the cells stay finer than the bins (the linear map puts
// the centre +- 3 sigma on them; the log map gives M/16 cells per octave of
// |z| + 1, 8 octaves on either side of z = 0) while the tables of small
// grids stay small.  The log map's shift is 27 - log2 M.
inline int hint_cells_for_bins(int n) { return n > 64 ? 512 : 256; }
inline int hint_cell_shift(int M) { return M == 512 ? 18 : 19; }

// Read-only kernel inputs are read through the constant address space, so
// that wave-uniform reads become scalar loads.
template <typename T>
using CP = const __attribute__((address_space(4))) T*;

template <typename T>
__device__ __forceinline__ CP<T> cp(const T* p) {
  return (CP<T>)(p);
}

enum { FLAT = 0, GAUSS = 1, BW = 2 };

constexpr uint32_t kTagUnweight = 0x80000000u;

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): 10 rounds of two 32x32
// multiplies (multipliers 0xD2511F53, 0xCD9E8D57) with the key bumped by the
// Weyl constants 0x9E3779B9, 0xBB67AE85 between rounds.  Counter layout:
// (sample lo, sample hi, iteration tag, block index), key = seed.
// ---------------------------------------------------------------------------
struct U4 {
  uint32_t x, y, z, w;
};

__host__ __device__ inline U4 philox4x32_10(U4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    // each 32x32 -> 64 product as one 64-bit multiply (one v_mad_u64_u32
    // on the GPU, where separate low and high multiplies are two)
    const uint64_t p0 = (uint64_t)0xD2511F53u * c.x;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c.z;
    c = U4{(uint32_t)(p1 >> 32) ^ c.y ^ k0, (uint32_t)p1, (uint32_t)(p0 >> 32) ^ c.w ^ k1,
           (uint32_t)p0};
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return c;
}

// Words 0..nw-1 of sample i (nw <= 36).
__device__ inline void philox_words(uint64_t seed, uint64_t i, uint32_t tag, int nw,
                                    uint32_t* out) {
  for (int b = 0; 4 * b < nw; ++b) {
    const U4 r = philox4x32_10(U4{(uint32_t)i, (uint32_t)(i >> 32), tag, (uint32_t)b},
                               (uint32_t)seed, (uint32_t)(seed >> 32));
    out[4 * b + 0] = r.x;
    if (4 * b + 1 < nw) out[4 * b + 1] = r.y;
    if (4 * b + 2 < nw) out[4 * b + 2] = r.z;
    if (4 * b + 3 < nw) out[4 * b + 3] = r.w;
  }
}

// ---------------------------------------------------------------------------
// MRG32k3a streams (Sec. 4.4, eq. mrg32k3a and eq. rngstream): two
// order-three recursions modulo m1 = 2^32 - 209 and m2 = 2^32 - 22853,
// x1_n = 1403580 x1_{n-2} - 810728 x1_{n-3}, x2_n = 527612 x2_{n-1} -
// 1370589 x2_{n-3}, combined into z_n = x1_n - x2_n mod m1 (m1 in place of
// 0).  The state of a component is (x_{n-2}, x_{n-1}, x_n); jumps of 2^b
// steps are 3x3 matrices modulo m applied to it (tables built on the host).
// A call's word is floor(z 2^32 / (m1 + 1)), so the bin / fraction rule of
// the Philox words applies unchanged.  Stream, substream and offset of a
// call: see JobDev::mrg.
// ---------------------------------------------------------------------------
constexpr uint32_t kMrgM1 = 4294967087u, kMrgM2 = 4294944443u;
constexpr int kMrgEntry = 18;      // uint32 per jump entry: 3x3 for each component
constexpr int kMrgSubBase = 64;    // entries 0..63: 2^b steps; 64..127: 2^(76+b)
constexpr int kMrgTables = 128;    // jump entries before the stream starts

struct Mrg {
  uint32_t a[3], b[3];
};

// x mod m1 (x < 2^64), from 2^32 = 209 mod m1: two folds leave x < 2 m1.
__host__ __device__ inline uint32_t mrg_mod1(uint64_t x) {
  x = (x >> 32) * 209u + (uint32_t)x;
  x = (x >> 32) * 209u + (uint32_t)x;
  return (uint32_t)(x >= kMrgM1 ? x - kMrgM1 : x);
}
// x mod m2 (x < 2^64), from 2^32 = 22853 mod m2: two folds leave x < 2 m2.
__host__ __device__ inline uint32_t mrg_mod2(uint64_t x) {
  x = (x >> 32) * 22853u + (uint32_t)x;
  x = (x >> 32) * 22853u + (uint32_t)x;
  return (uint32_t)(x >= kMrgM2 ? x - kMrgM2 : x);
}

// One fold of x < 2^64 toward x mod m1 (< 210 2^32) or mod m2 (< 22854
// 2^32): the same residue, small enough that three of them sum without
// overflow before the full reduction.
__device__ inline uint64_t mrg_fold1(uint64_t x) { return (x >> 32) * 209u + (uint32_t)x; }
__device__ inline uint64_t mrg_fold2(uint64_t x) { return (x >> 32) * 22853u + (uint32_t)x; }

// s <- M s for one jump entry M (both components).
template <typename PT>
__device__ inline void mrg_apply(PT M, Mrg& s) {
  uint32_t ra[3], rb[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const uint64_t ta = mrg_fold1((uint64_t)M[3 * i] * s.a[0]) +
                        mrg_fold1((uint64_t)M[3 * i + 1] * s.a[1]) +
                        mrg_fold1((uint64_t)M[3 * i + 2] * s.a[2]);
    ra[i] = mrg_mod1(ta);
    const uint64_t tb = mrg_fold2((uint64_t)M[9 + 3 * i] * s.b[0]) +
                        mrg_fold2((uint64_t)M[9 + 3 * i + 1] * s.b[1]) +
                        mrg_fold2((uint64_t)M[9 + 3 * i + 2] * s.b[2]);
    rb[i] = mrg_mod2(tb);
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    s.a[i] = ra[i];
    s.b[i] = rb[i];
  }
}

// s <- A^(2^shift k) s with the table entries base..base+63 (A^(2^(shift+b))).
template <typename PT>
__device__ inline void mrg_jump(PT tab, int base, uint64_t k, Mrg& s) {
  for (int b = 0; k != 0; ++b, k >>= 1)
    if (k & 1) mrg_apply(tab + (size_t)(base + b) * kMrgEntry, s);
}

// One step; returns the 32-bit word of the new output.
__device__ inline uint32_t mrg_word(Mrg& s) {
  // (a12 x_{n-1} - a13 x_{n-2}) mod m1 as a12 x_{n-1} + a13 (m1 - x_{n-2})
  const uint32_t p1 = mrg_mod1((uint64_t)1403580u * s.a[1] + (uint64_t)810728u * (kMrgM1 - s.a[0]));
  s.a[0] = s.a[1];
  s.a[1] = s.a[2];
  s.a[2] = p1;
  const uint32_t p2 = mrg_mod2((uint64_t)527612u * s.b[2] + (uint64_t)1370589u * (kMrgM2 - s.b[0]));
  s.b[0] = s.b[1];
  s.b[1] = s.b[2];
  s.b[2] = p2;
  const uint32_t z = p1 > p2 ? p1 - p2 : p1 + (kMrgM1 - p2);
  // floor(z 2^32 / (m1 + 1)) with m1 + 1 = 2^32 - 208: z 2^32 / (2^32 - 208)
  // = z + 208 z / (2^32 - 208), and with 208 z = h 2^32 + l the last term's
  // floor is h + [l >= 2^32 - 208 - 208 h] (h < 208).  Exact for every z <
  // m1 (checked exhaustively against the division).
  const uint64_t t = (uint64_t)z * 208u;
  const uint32_t h = (uint32_t)(t >> 32), l = (uint32_t)t;
  return z + h + (l >= (kMrgM1 + 1u) - h * 208u ? 1u : 0u);
}

// ---------------------------------------------------------------------------
// Uniform word u -> bin j = floor(u n / 2^32) and fraction of the remainder.
// FP64: (lo + 1/2) 2^-32; FP32: (lo/2^9 + 1/2) 2^-23.  Both exact, in (0,1);
// the bin is the same integer in both precisions.
// ---------------------------------------------------------------------------
template <typename T>
struct Frac;
template <>
struct Frac<double> {
  __device__ static inline double get(uint32_t lo) { return ((double)lo + 0.5) * 0x1p-32; }
};
template <>
struct Frac<float> {
  __device__ static inline float get(uint32_t lo) {
    return ((float)(lo >> 9) + 0.5f) * 0x1p-23f;
  }
};

// ---------------------------------------------------------------------------
// Per (channel, dim) map constants, per channel density normalisation, and
// per (peak, dim) integrand constants.  Filled on the device by the set-up
// kernel in FP64 and rounded to FP32 for the mixed-precision mode.
// ---------------------------------------------------------------------------
template <typename T>
struct DimMap {
  int32_t kind;
  int32_t pad_;
  T loc;     // mu (Gauss), m (BW)
  T width;   // sigma (Gauss), Gamma (BW)
  T inv_w;   // 1/sigma (Gauss)
  T pa, qb, z;       // Gauss: Phi(a), 1 - Phi(b), Z = Phi(b) - Phi(a)
  T h, h2, ta, th;   // BW: Gamma/2, h^2, atan(-m/h), Theta = atan((1-m)/h) - ta
  T fa, fb;          // BW: atan2(h, m), atan2(h, 1-m) (distances of the ends to the poles)
  T ga, gb;          // Gauss exponent: z' = ga p + gb with z'^2 = log2(e) z^2 / 2
  float hb, hs;      // linear hint map of FP64 jobs (channels Gaussian on every axis)
  float lb, ls;      // log hint map (other channels): z = ls p + lb
};

// One table entry of an axis: a bin edge and the density of the bin that
// starts there.
template <typename T>
struct __align__(2 * sizeof(T)) Pair {
  T e, dens;
};

// Axis kinds of one channel: lin = Gaussian on every axis (its lookups use
// the linear hint map); iso = Gaussian on every axis with one width (its
// density constants take the isotropic form); bit k of gmask (bmask) marks a
// Gaussian (Breit-Wigner) axis k; the other axes are flat.
struct ChanType {
  int32_t iso;
  uint32_t gmask, bmask;
  int32_t lin;
};

// The log hint map of a flat axis, the same for every channel: z = 510 (x -
// 1/2).
constexpr float kFlatA = 510.0f, kFlatB = -255.0f;

// What the channel loop reads of one channel, in one record (stride
// chan_stride(d) bytes, one base address; as six arrays their addresses were
// spilled to vector lanes and read back, 36 lane reads per channel, and each
// array's read was waited for by itself): the masks of its Gaussian and
// Breit-Wigner axes; iso, lin (ChanType), and pair: no Gaussian axis and one
// or two Breit-Wigner ones, the others flat; the offsets ea, eb of the FP64
// skip from a partial exponent; its peak's factor of f (0: no peak of its
// shape); and, written with the allocation, the term's factor (T)alpha_c
// cnorm_c, the term bound's factor (T)alpha_c gbound_c, and alpha_c cnorm_c
// 2^s (1 + m) rounded up (the factor of the bound from looked-up densities).
// The 2d density-kernel constants of
// the axes follow: (ga, gb) on a Gaussian axis, (m, h^2) on a Breit-Wigner
// one, 0 on a flat one; for iso channels the centres m_0 .. m_{d-1}, then ga^2.
enum { kChanIso = 1, kChanLin = 2, kChanPair = 4 };
template <typename T>
struct __align__(16) ChanHead {
  uint32_t gmask, bmask;
  int16_t kind;  // kChanIso | kChanLin | kChanPair
  int16_t pad_;
  int16_t ea, eb;
  T twin, term, bound, look;
};
// Behind the constants in FP64: (m, h^2) and the log hint map's constants of a
// pair channel's Breit-Wigner axes in axis order.
struct __align__(16) PairCon {
  double c[4];
  float h[4];
};
template <typename T>
__host__ __device__ constexpr int chan_pair_at(int d) {
  return ((int)sizeof(ChanHead<T>) + 2 * d * (int)sizeof(T) + 15) & ~15;
}
template <typename T>
__host__ __device__ constexpr int chan_stride(int d) {
  return chan_pair_at<T>(d) + (sizeof(T) == 8 ? (int)sizeof(PairCon) : 0);
}

// One cell of an axis' hint map, precomputed from its p-space edges:
// J = interior edges whose cell is lower (all of them lie below any x of the
// cell); with at most one edge inside the cell, e is that edge (+inf if
// none) and the bin of x is J (density dlo) below e, J + 1 (density dhi)
// from e on.  dlo < 0 marks a cell holding two or more edges.
template <typename T>
struct __align__(4 * sizeof(T)) Cell {
  T e, dlo, dhi;
  T J;  // the start bin, stored as a value of T (exact for J < 2^24)
};

template <typename T>
struct PeakDim {
  int32_t kind;
  int32_t pad_;
  T loc, h2, ga, gb;  // BW: centre, h^2; Gauss: exponent z' = ga p + gb as in DimMap
};

// Math wrappers resolving to the device math library for each precision.
__device__ inline double m_exp(double x) { return exp(x); }
__device__ inline float m_exp(float x) { return expf(x); }
// Coefficients of the FP64 special functions (fp64_fit.py), highest power
// first.  They are read with scalar loads where they are used (fresh() hides
// where they come from): as literals the compiler kept them in vector
// registers across the pass's loop and spilled them there, 40 to 60 scratch
// reads per evaluation.
constexpr int kLog2N = 9, kErfcinvN = 26, kSinN = 7, kCosN = 8, kExp2N = 12;
__device__ const double kErfcinvTab[kLog2N + kErfcinvN] = {  // log2, then the central piece
    0.17144989425121918, 0.16862072992906546, 0.19239274586704302, 0.22195249899072644,
    0.26230819523994015, 0.32059889794090296, 0.41219858311123148, 0.5770780163555852,
    0.96179669392597555,
    5.839458082047211e-09, -8.0908977213792306e-09, -4.5087329353724268e-08, 9.8676198969758009e-08,
    8.863055592715813e-08, -4.9361783614262281e-07, 4.6807872055697208e-07, 8.4261207184972158e-07,
    -3.3435413584532678e-06, 3.7363309444613917e-06, 5.2474671433003046e-06, -2.5758430392203254e-05,
    3.2960471664389562e-05, 3.3663427339509055e-05, -0.00020245689308002459, 0.00029197778647533143,
    0.00019691980709171314, -0.0016070752518853547, 0.0026863639308647908, 0.00067461473098120062,
    -0.01281929971804836, 0.028230934696226413, -0.016552434035712049, -0.10289932479305051,
    0.88079803173219484, 1.8156662240587476};
__device__ const double kSinCosTab[kSinN + kCosN] = {
    1.589457978152985e-10, -2.5050714321896748e-08, 2.7557313359736881e-06, -0.00019841269828602579,
    0.008333333333320302, -0.16666666666666616, 1,
    -1.1353266525927744e-11, 2.0875580117542017e-09, -2.7557313080114282e-07, 2.480158728381321e-05,
    -0.0013888888888860963, 0.041666666666666449, -0.5, 1};
__device__ const double kExp2Tab[kExp2N] = {
    4.4566754636398608e-10, 7.0741945626131049e-09, 1.0178051192117847e-07, 1.3215432534254118e-06,
    1.5252733856295574e-05, 0.00015403530463727982, 0.0013333558146390351, 0.0096181291075872529,
    0.055504108664821701, 0.24022650695910158, 0.69314718055994529, 1};
__device__ __forceinline__ CP<double> fresh(const double* p) {
  asm volatile("" : "+s"(p));
  return cp(p);
}

// 2^x for x <= 1 (cut at 3e-18, about 1 ulp; below the exponent range 0, at
// minus infinity as well, where x - rint(x) would be no number).
__device__ inline double m_exp2(double x) {
  const CP<double> c = fresh(kExp2Tab);
  x = x < -4096.0 ? -4096.0 : x;  // NaN stays
  const double n = __builtin_rint(x);
  const double f = x - n;
  double P = c[0];
#pragma unroll
  for (int i = 1; i < kExp2N; ++i) P = fma(P, f, c[i]);
  return __builtin_amdgcn_ldexp(P, (int)n);
}
// FP32: the hardware exp2 (one instruction, about 1 ulp; a result below
// 2^-126 may come back as 0).  Every use is a density kernel
// 2^(-sum z'^2) <= 1, so such a result is a term at least 2^-126 below the
// peak it belongs to, which the sums of f and g cannot notice at FP32
// precision; the library exp2f spends more instructions per call only to
// return those denormals.
__device__ inline float m_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
// 1/x: exact in FP64; the hardware reciprocal (1 ulp) in FP32.
__device__ inline double m_rcp(double x) { return 1.0 / x; }
__device__ inline float m_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline float m_tan(float x) { return tanf(x); }
// FP32 erfcinv(y), 0 < y < 2, in the structure of M. Giles' erfinv
// approximation ("Approximating the erfinv function", GPU Computing Gems,
// Jade Edition, 2011): with w = -log2(y (2 - y)), erfcinv(y) = erfinv(1 - y)
// = (1 - y) P(w), P a polynomial in (w - 5) / 5 for w <= 10 (y >= 4.9e-4:
// all but a few lanes in a thousand) and in a normalised sqrt(w) for
// 10 < w <= 26; beyond (y < 7.5e-9) erfcinv_far.  Coefficients
// fitted by erfcinv_fit.py (largest relative error of the fits 2.9e-08 and
// 1.7e-08; in FP32 with the hardware log2 about 2.5e-7, median 4e-8).  The
// library function spends about 110 instructions over its three branches.
// The far tail, y < 7.5e-9 down to the smallest denormal (2 - y = 2): the same
// structure on 26 < w <= 151 (fp64_fit.py; 2e-9 of the fit).  w and its root
// carry what their rounding left over, and the centre of t its rest beyond
// FP32: at most 0.9 ulp (0.27 on average; the library's erfcinvf 2.0 and 0.45,
// without the leftovers 2.3 and 0.61).  In line: a call here, though never
// taken, made the kernels save their registers around every axis (34 spilled
// VGPRs at d = 10).
__device__ inline float erfcinv_far(float y) {
  const float v = y * 0x1p64f;
  const float e = (float)(63 - __builtin_amdgcn_frexp_expf(v));
  const float l = __builtin_amdgcn_logf(__builtin_amdgcn_frexp_mantf(v));
  const float w = e - l, wl = (e - w) - l;
  const float s = sqrtf(w), sl = (fmaf(-s, s, w) + wl) * (0.5f / s);
  const float t = ((s - 8.693612621e+00f) + (sl + 4.3184952e-07f)) * 2.781956039e-01f;
  float P = 1.396802121e-05f;
  P = fmaf(P, t, -3.095602143e-05f);
  P = fmaf(P, t, 3.235408476e-05f);
  P = fmaf(P, t, -7.128970774e-05f);
  P = fmaf(P, t, 1.744936948e-04f);
  P = fmaf(P, t, -3.016682099e-04f);
  P = fmaf(P, t, 3.495910400e-04f);
  P = fmaf(P, t, 3.016676134e-04f);
  P = fmaf(P, t, -4.534591285e-03f);
  P = fmaf(P, t, 3.017693168e+00f);
  P = fmaf(P, t, 7.108942973e+00f);
  return v == 0.0f ? INFINITY : P;
}

// CENTRAL: the caller knows that w <= 10.
template <bool CENTRAL = false>
__device__ inline float fast_erfcinv(float y) {
  const float L = __builtin_amdgcn_logf(y * (2.0f - y));  // log2, -w
  const float x = 1.0f - y;
  if (CENTRAL || L >= -10.0f) {
    const float t = fmaf(L, -0.2f, -1.0f);
    float P = -1.689334030e-05f;
    P = fmaf(P, t, 1.472581541e-04f);
    P = fmaf(P, t, -1.411730478e-04f);
    P = fmaf(P, t, -7.059459609e-04f);
    P = fmaf(P, t, 2.037662157e-03f);
    P = fmaf(P, t, -8.269816707e-04f);
    P = fmaf(P, t, -7.870274752e-03f);
    P = fmaf(P, t, 2.327191661e-02f);
    P = fmaf(P, t, -2.094532432e-02f);
    P = fmaf(P, t, -8.007366265e-02f);
    P = fmaf(P, t, 8.172793550e-01f);
    P = fmaf(P, t, 1.734757719e+00f);
    return x * P;
  }
  if (L >= -26.0f) {
    const float t = (sqrtf(-L) - 4.130648587e+00f) * 1.032662147e+00f;
    float P = 7.523363763e-06f;
    P = fmaf(P, t, -5.389624879e-05f);
    P = fmaf(P, t, 1.529154143e-04f);
    P = fmaf(P, t, -2.954300123e-04f);
    P = fmaf(P, t, 5.583441763e-04f);
    P = fmaf(P, t, -1.234308599e-03f);
    P = fmaf(P, t, 2.392615197e-03f);
    P = fmaf(P, t, 8.118207278e-01f);
    P = fmaf(P, t, 3.274039353e+00f);
    return x * P;
  }
  return erfcinv_far(y);
}
// FP64 erfcinv and log2, in the same structure (coefficients: fp64_fit.py; the
// fits are cut below 5e-17).  A central piece for w = -log2(y (2 - y)) <= 11
// (y >= 2.4e-4: all but about one lane-axis in 2000) and three pieces in
// sqrt(w) behind one branch, their coefficients read per lane; 0 < y <= 1 (the
// maps' arguments are at least the smallest denormal).  The library's
// erfcinv (and a Halley step on erfc from the FP32 value before it) spent
// about 250 instructions and the pass's registers on each axis.  Errors on the
// card against 45-digit values, ulp on average and at most: y > 0.5 0.43 and
// 1.9 (the library 0.48 and 2.0), y > 0.05 0.43 and 2.0 (0.50, 2.0), y > 2.4e-4
// 0.39 and 1.4 (0.41, 1.7), below 0.38 and 2.0 (0.48, 2.3).  The Halley step
// had 0.26 and 0.75 for y < 0.05, 0.36 and 2.3 up to 0.5 and an error of 7e-17
// however small the value beyond; over the calls of a pass, y uniform, the rms
// errors are 5.7e-17, the library's 6.4e-17 and the Halley step's 6.3e-17.
constexpr double kErfcinvW1 = 11.0;
constexpr int kErfcinvPieceN = 24;
__device__ const double kErfcinvPiece[3][kErfcinvPieceN + 2] = {  // centre, 1/half, coefficients
    {4.6583123951776999, 0.74532998322843202,
     -1.1086380178806771e-10, 8.5314266200362513e-11, 1.1768159457621137e-09, -3.259827465722147e-09,
     2.0119847879118342e-09, 1.1639619642971096e-08, -5.287517566442768e-08, 1.0914331496941178e-07,
     -3.9529159669494931e-08, -4.90894570194495e-07, 1.7433021164541841e-06, -2.975819927228338e-06,
     1.1041032389988738e-06, 9.5511633350386016e-06, -3.4482603897486704e-05, 7.3909304553016703e-05,
     -0.00012181629511168777, 0.0001799527282383712, -0.00029702458675398899, 0.00063430187633557907,
     -0.0014564631710620953, 0.0020063445487988121, 1.1272440282422962, 3.716948227966332},
    {9, 0.33333333333333331,
     -2.8525368123130821e-10, 4.0546229939122544e-10, 1.1006065715487956e-09, -1.5490385099566593e-09,
     -2.1006175675421456e-09, 2.9291320021809486e-09, 1.9649262260689024e-09, -1.8978995890107316e-09,
     -5.1685973334545114e-09, 1.2938606226043683e-08, -3.2638894957313637e-08, 1.0002834720782859e-07,
     -2.9947528703455623e-07, 8.6915250855661284e-07, -2.4601982986890966e-06, 6.7401996315247254e-06,
     -1.7617489575746311e-05, 4.2678461714130274e-05, -8.899365437713163e-05, 0.00011729837643180705,
     0.00023282738793474716, -0.003095596297196376, 2.517887937388029, 7.3661251922288393},
    {22.5, 0.095238095238095233,
     -2.3506526752021451e-09, 4.641785402277912e-09, 4.4005697389502602e-09, -7.7386916137819374e-09,
     -2.0411417674851032e-08, 3.7945844004507808e-08, -2.1884082748820938e-08, 4.6656216097020564e-08,
     -1.3846675491085614e-07, 2.5423228846803611e-07, -4.2410404863165673e-07, 7.0871841264722134e-07,
     -1.0536145477037244e-06, 1.1215274991157444e-06, 3.0239021561088597e-07, -7.1287414703839726e-06,
     3.0987099709464433e-05, -0.00010503738771968648, 0.0003219617072706045, -0.00093962051585709549,
     0.0026836974408732152, -0.0076699354856200322, 8.7644443549791156, 18.657407855140697}};

__device__ inline double erfcinv_piece(double w) {
  const double s = sqrt(w), sl = fma(-s, s, w) * (0.5 * __builtin_amdgcn_rcp(s));
  const double* c = kErfcinvPiece[s < 6.0 ? 0 : s < 12.0 ? 1 : 2];
  const double t = ((s - c[0]) + sl) * c[1];  // sl: what the root's rounding left over
  double P = c[2];
#pragma unroll 1
  for (int i = 3; i < kErfcinvPieceN + 2; ++i) P = fma(P, t, c[i]);
  return P;
}

// G values at once: the Horner chains run side by side and share their
// coefficients.  w = -log2(q) from q = m 2^e, m in [sqrt(1/2), sqrt(2)), and
// s = (m - 1) / (m + 1) by a refined reciprocal.
template <int G>
__device__ __forceinline__ void erfcinv_group(const double (&y)[G], double (&out)[G]) {
  const CP<double> c = fresh(kErfcinvTab);
  double w[G], P[G];
  {
    double s[G], z[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const double q = fma(-y[g], y[g], y[g] + y[g]);  // y (2 - y), rounded once
      double m = __builtin_amdgcn_frexp_mant(q);
      int e = __builtin_amdgcn_frexp_exp(q);
      const bool low = m < 0.70710678118654752440;
      m = low ? 2.0 * m : m;
      e = low ? e - 1 : e;
      const double f = m - 1.0, dd = m + 1.0;
      double r = __builtin_amdgcn_rcp(dd);
      r = fma(fma(-dd, r, 1.0), r, r);
      r = fma(fma(-dd, r, 1.0), r, r);
      const double s0 = f * r;
      s[g] = fma(fma(-dd, s0, f), r, s0);
      z[g] = s[g] * s[g];
      w[g] = (double)e;
      P[g] = c[0];
    }
#pragma unroll
    for (int i = 1; i < kLog2N; ++i)
#pragma unroll
      for (int g = 0; g < G; ++g) P[g] = fma(P[g], z[g], c[i]);
#pragma unroll
    for (int g = 0; g < G; ++g)
      w[g] = -fma(s[g], fma(z[g], P[g], 2.88539008177792681472), w[g]);
  }
  bool far = false;
  {
    double t[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      t[g] = fma(w[g], 2.0 / kErfcinvW1, -1.0);
      P[g] = c[kLog2N];
      far |= w[g] > kErfcinvW1;
    }
#pragma unroll
    for (int i = 1; i < kErfcinvN; ++i)
#pragma unroll
      for (int g = 0; g < G; ++g) P[g] = fma(P[g], t[g], c[kLog2N + i]);
  }
  if (far) {
#pragma unroll
    for (int g = 0; g < G; ++g)
      if (w[g] > kErfcinvW1) P[g] = erfcinv_piece(w[g]);
  }
#pragma unroll
  for (int g = 0; g < G; ++g) out[g] = fma(-y[g], P[g], P[g]);  // (1 - y) P, rounded once
}

// FP32: the central piece on every value, the others behind one branch.
template <int G>
__device__ __forceinline__ void erfcinv_group(const float (&y)[G], float (&out)[G]) {
  bool far = false;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    out[g] = fast_erfcinv<true>(y[g]);
    far |= !(__builtin_amdgcn_logf(y[g] * (2.0f - y[g])) >= -10.0f);
  }
  if (far) {
#pragma unroll
    for (int g = 0; g < G; ++g) out[g] = fast_erfcinv(y[g]);
  }
}
__device__ inline double m_erfcinv(double y) {
  const double a[1] = {y};
  double r[1];
  erfcinv_group<1>(a, r);
  return r[0];
}

// tan(a), |a| <= pi/2 in FP64 (the map's angles lie between its poles): sine
// and cosine of a, or of the distance to the pole from pi/2 in two parts, on
// [0, pi/4] (fp64_fit.py, cut below 4e-18), each as the last sum and what its
// rounding and those of r and r^2 left over, and a quotient corrected by its
// remainder: at most 0.9 ulp, 0.25 on average (0.98 and 0.25 of the library's
// tangent; without the leftovers 2.7 and 0.49).
__device__ inline double m_tan(double a) {
  const CP<double> k = fresh(kSinCosTab);
  const double b = fabs(a);
  const bool near = b > 0.78539816339744830962;
  const double h = 1.57079632679489655800 - b, lo = 6.12323399573676603587e-17;
  const double r = near ? h + lo : b;
  const double rl = near ? (h - r) + lo : 0.0;
  const double z = r * r, zl = fma(r, r, -z), rz = r * z;
  double s = k[0], c = k[kSinN];
#pragma unroll
  for (int i = 1; i < kSinN - 1; ++i) s = fma(s, z, k[i]);
#pragma unroll
  for (int i = 1; i < kCosN - 1; ++i) c = fma(c, z, k[kSinN + i]);
  // sin = r + r z s and cos = 1 + z c
  const double sh = fma(rz, s, r), ch = fma(z, c, 1.0);
  const double sl = fma(rl, ch, fma(rz, s, r - sh));
  const double cl = fma(-rl, sh, fma(c, zl, fma(z, c, 1.0 - ch)));
  const double nh = near ? ch : sh, nl = near ? cl : sl;
  const double dh = near ? sh : ch, dl = near ? sl : cl;
  double y = __builtin_amdgcn_rcp(dh);
  y = fma(fma(-dh, y, 1.0), y, y);
  y = fma(fma(-dh, y, 1.0), y, y);
  const double q = nh * y;
  const double t = fma(fma(-q, dh, nh) + fma(-q, dl, nl), y, q);
  return a < 0.0 ? -t : t;
}
__device__ inline float m_erfcinv(float x) { return fast_erfcinv(x); }

constexpr double kSqrt2 = 1.41421356237309504880;

// The upper or lower tail of a Gaussian axis: y in (0, 1] with erfcinv(y) the
// distance from the median in units of sqrt(2) sigma, and its sign.
template <typename T, typename PM>
__device__ inline T gauss_tail(PM m, T x, T xc, T& sign) {
  const T t = m->pa + x * m->z;
  const bool lower = t <= T(0.5);
  sign = lower ? -T(kSqrt2) : T(kSqrt2);
  return lower ? T(2) * t : T(2) * (m->qb + xc * m->z);
}

// Forward map p = phi(x) for one dim.  x and xc = 1 - x are both supplied so
// the upper tail keeps its relative precision.  Gauss: truncated-normal
// inverse CDF, evaluated on the tail side of the median.  BW: arctan map; in
// FP32 near either pole it is written with the distance to the pole so that
// p - m keeps its precision.  Each case picks its argument first and then makes a single
// call of the special function (lanes of a wave that take different cases
// share that call).  PM: pointer to the axis' DimMap<T> (generic or constant
// address space).
template <typename T, typename PM>
__device__ inline T map_forward(PM m, T x, T xc) {
  const int kind = m->kind;
  if (kind == GAUSS) {
    T sign;
    const T arg = gauss_tail<T>(m, x, xc, sign);
    return m->loc + m->width * (sign * m_erfcinv(arg));
  }
  if (kind == BW) {
    if constexpr (sizeof(T) == 8) return m->loc + m->h * m_tan(m->ta + x * m->th);
    const T da = m->fa + x * m->th;   // theta + pi/2
    const T db = m->fb + xc * m->th;  // pi/2 - theta
    const T quarter = T(0.78539816339744830962);
    const bool near_a = da < quarter, near_b = !near_a && db < quarter;
    const T t = m_tan(near_a ? da : near_b ? db : m->ta + x * m->th);
    if (near_a) return m->loc - m->h / t;
    if (near_b) return m->loc + m->h / t;
    return m->loc + m->h * t;
  }
  return x;
}

// Neumaier compensated accumulator in FP64.
struct Neu {
  double s, c;
  __device__ inline void add(double v) {
    const double t = s + v;
    if (fabs(s) >= fabs(v)) c += (s - t) + v;
    else c += (v - t) + s;
    s = t;
  }
};

// Sum of two compensated pairs (a.s + a.c) + (b.s + b.c) by an error-free
// TwoSum of the leading parts.
__device__ inline Neu neu_merge(Neu a, Neu b) {
  const double s = a.s + b.s;
  const double bb = s - a.s;
  const double err = (a.s - (s - bb)) + (b.s - bb);
  return Neu{s, a.c + b.c + err};
}

}  // namespace mcv
