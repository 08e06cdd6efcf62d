// Device code of the sample pass shared by the single-job kernels (single.hip)
// and the batched queue kernels (queue.hip): the kernel
// argument record, the per-call forward map and one work unit of a pass.
//
// Brass, Kilian, Reuter, arXiv:1811.09711, Sec. 3.5: for every call r_c of
// channel c, x_c = G_c^{-1}(r_c) with the VEGAS step map (Sec. 3.2, eq. g(x)),
// p = phi_c(x_c), f(p), then for every other channel c' the inverse map and the
// bin of x_c' in grid c' (eq. g(p)); the weight is w = f/g (eq. vamp-master).
// Sums of w and w^2 per channel (Sec. 3.1, eq. 4) and the per-bin sums of w^2
// along each axis (eq. 31) are accumulated for the adaptation.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <string.h>

#include "mcv_internal.h"
#include "mcv_mask.h"
#include "mcv_point.h"

namespace mcv {

namespace {

template <typename T>
struct SampleArgs {
  int d, K, n, P;
  int sT;               // per-axis table stride (entries)
  int M, mshift;        // hint cells per axis and the log map's shift
  int n_orphan;
  int off_own, off_hist, off_red, off_queue;
  uint32_t tag;         // iteration tag of trace and unweighting launches
  uint64_t seed;
  const int32_t* iter;  // sample pass: completed passes = this pass's tag
  int units;            // single-job pass: work units, and the next one to take
  int* next;
  const int64_t* start;
  const double* alpha;
  const DimMap<T>* cmap;
  const T* cnorm;
  const PeakDim<T>* pmap;
  const T* pnorm;
  const int32_t* orphans;
  const Pair<T>* xtab;   // [K][d][sT]
  const Pair<T>* ptab;   // [K][d][sT]
  const Cell<T>* ctab;   // [K][d][M]
  const char* crec;      // [K] channel records (ChanHead)
  int cstride;           // bytes of a record
  const float* hab;      // [K][d][2] hint-map constants
  const void* mco;       // channel-mask coefficients (mcv_mask.h)
  const float* mthr;     // [K rounded up to 32] channel-mask thresholds
  int fpos;              // no channel's peak has a negative weight
  double* part;
  double* hpart;
  // trace instantiation only: f, g, w of calls [tr_first, tr_first + tr_count)
  int64_t tr_first, tr_count;
  double* tr_out;        // [tr_count][3]
  int rng;               // 0 Philox4x32-10, 1 MRG32k3a streams
  const uint32_t* mrg;   // MRG32k3a jump tables and stream starts (JobDev::mrg)
  int strat;             // 0 uniform r; s >= 2 pseudo-stratified (>= s calls per box)
  const int64_t* nr;     // [K] stratified layout: boxes per axis
  const int64_t* spb;    // [K] calls per box
  const int64_t* bstart; // [K+1] box prefix
};

// Channel cc's record, and the constants behind it.
template <typename T>
__device__ __forceinline__ CP<ChanHead<T>> chan_at(const SampleArgs<T>& a, int cc) {
  return (CP<ChanHead<T>>)(cp(a.crec) + (size_t)cc * a.cstride);
}
template <typename T>
__device__ __forceinline__ CP<T> chan_con(CP<ChanHead<T>> h) {
  return (CP<T>)(h + 1);
}
template <typename T>
__device__ __forceinline__ CP<PairCon> pair_con(CP<ChanHead<T>> h, int d) {
  return (CP<PairCon>)((CP<char>)h + chan_pair_at<T>(d));
}
template <typename T, int MAXD, bool PAIR = false>
__device__ __forceinline__ T chan_r_of(CP<ChanHead<T>> h, int d, const T (&p)[MAXD]) {
  if constexpr (PAIR)
    if (h->kind & kChanPair) return pair_r<T, MAXD>(&pair_con(h, d)->c[0], h->bmask, d, p);
  return chan_r<T, MAXD>(chan_con(h), h->kind & kChanIso, h->gmask, h->bmask, d, p);
}

// Stratified sampling: bin j and fraction of one axis from the box digit b
// and the word u: r = (b + u 2^-32) / nr as the fixed-point R = b 2^32 + u
// over nr 2^32 (R n < 2^60 for nr <= 2^20, n <= 256); j = floor(R n /
// (nr 2^32)); fraction (rem + 1/2) / (nr 2^32), rem = R n - j nr 2^32 (one
// correctly rounded FP64 division); FP32 rounds it to FP32, the largest
// float below 1 if that gives 1.
template <typename T>
__device__ inline void strat_bin_frac(uint32_t b, uint32_t u, uint32_t nr, int n, uint32_t& j,
                                      T& fr) {
  const uint64_t Rn = (((uint64_t)b << 32) | u) * (uint64_t)n;
  const uint32_t hi32 = (uint32_t)(Rn >> 32);
  j = hi32 / nr;
  const uint64_t rem = ((uint64_t)(hi32 - j * nr) << 32) | (uint32_t)Rn;
  const double f = ((double)rem + 0.5) / ((double)nr * 4294967296.0);
  if constexpr (sizeof(T) == 4) {
    const float f32 = (float)f;
    fr = f32 >= 1.0f ? 0x1.fffffep-1f : f32;
  } else {
    fr = f;
  }
}

// The MRG32k3a state of the call with index i_c among channel c's calls at
// iteration tag t: stream start of c, 64 t steps in, substream i_c.
__device__ inline Mrg mrg_call_state(const uint32_t* mrg, int K_or_c, uint64_t i_c, uint32_t t) {
  CP<uint32_t> tab = cp(mrg);
  CP<uint32_t> st = tab + (size_t)kMrgTables * kMrgEntry + (size_t)K_or_c * 6;
  Mrg s{{st[0], st[1], st[2]}, {st[3], st[4], st[5]}};
  mrg_jump(tab, 0, 64ull * t, s);
  mrg_jump(tab, kMrgSubBase, i_c, s);
  return s;
}

// Cooperative copy global -> LDS in 16-byte units (both ends 16-byte aligned,
// bytes a multiple of 16).
__device__ inline void copy16(void* dst, const void* src, int bytes, int block) {
  const uint4* s = reinterpret_cast<const uint4*>(src);
  uint4* d = reinterpret_cast<uint4*>(dst);
  const int n = bytes >> 4;
  for (int t = threadIdx.x; t < n; t += block) d[t] = s[t];
}

template <int MAXD>
__device__ __forceinline__ void draw_words(uint64_t seed, uint64_t i, uint32_t tag, int d,
                                  uint32_t (&u)[MAXD]) {
#pragma unroll
  for (int b = 0; b < (MAXD + 3) / 4; ++b) {
    if (4 * b < d) {
      const U4 r = philox4x32_10(U4{(uint32_t)i, (uint32_t)(i >> 32), tag, (uint32_t)b},
                                 (uint32_t)seed, (uint32_t)(seed >> 32));
      if (4 * b + 0 < MAXD) u[4 * b + 0] = r.x;
      if (4 * b + 1 < MAXD) u[4 * b + 1] = r.y;
      if (4 * b + 2 < MAXD) u[4 * b + 2] = r.z;
      if (4 * b + 3 < MAXD) u[4 * b + 3] = r.w;
    }
  }
}

// Forward part of one call of channel c: bins, x, p = phi_c(x) and the own
// grid density prod_k 1/(n Delta) (eq. g(x)), from the channel's x-space
// (edge, density) tables ot (per-axis stride sT).  bin(k, j, fr) gives axis
// k's bin and fraction.  gauss: the channel is Gaussian on every axis (the
// same on every lane); in FP64 its axes are then mapped a few at a time, so
// that their inverse error functions run side by side.
template <typename T, int MAXD, bool GROUPED, typename Bin>
__device__ __forceinline__ T forward_axes(const Bin& bin, int d, CP<DimMap<T>> cm,
                                          const Pair<T>* ot, int sT, bool gauss, T (&p)[MAXD],
                                          uint32_t (&jpack)[(MAXD + 3) / 4]) {
  constexpr int GD = !GROUPED ? 1 : MAXD <= 4 ? MAXD : MAXD % 5 == 0 ? 5 : MAXD % 4 == 0 ? 4 : MAXD % 3 == 0 ? 3 : 1;
  static_assert(MAXD % GD == 0, "groups of whole axes");
  T own = T(1);
#pragma unroll
  for (int k = 0; k < (MAXD + 3) / 4; ++k) jpack[k] = 0u;
#pragma unroll
  for (int k0 = 0; k0 < MAXD; k0 += GD) {
    T x[GD], xc[GD];
#pragma unroll
    for (int g = 0; g < GD; ++g) {
      const int k = k0 + g;
      x[g] = xc[g] = T(0.5);
      if (k < d) {
        uint32_t j;
        T fr;
        bin(k, j, fr);
        const Pair<T> a0 = ot[k * sT + j], a1 = ot[k * sT + j + 1];
        const T w = a1.e - a0.e;
        x[g] = a0.e + fr * w;
        xc[g] = (T(1) - a1.e) + (T(1) - fr) * w;
        own *= a0.dens;
        jpack[k >> 2] |= j << (8 * (k & 3));
      }
    }
    if (GD > 1 && gauss) {
      if constexpr (GD > 1) {
        T y[GD], sign[GD], z[GD];
#pragma unroll
        for (int g = 0; g < GD; ++g) {
          y[g] = T(1);
          if (k0 + g < d) y[g] = gauss_tail<T>(cm + k0 + g, x[g], xc[g], sign[g]);
        }
        erfcinv_group<GD>(y, z);
#pragma unroll
        for (int g = 0; g < GD; ++g) {
          const int k = k0 + g;
          p[k] = T(0);
          if (k < d) p[k] = cm[k].loc + cm[k].width * (sign[g] * z[g]);
        }
      }
    } else {
#pragma unroll
      for (int g = 0; g < GD; ++g) {
        const int k = k0 + g;
        p[k] = T(0);
        if (k < d) p[k] = map_forward<T>(cm + k, x[g], xc[g]);
      }
    }
  }
  return own;
}

template <typename T, int MAXD, bool GROUPED>
__device__ inline T forward_point(const uint32_t (&u)[MAXD], int d, int n, CP<DimMap<T>> cm,
                                  const Pair<T>* ot, int sT, bool gauss, T (&p)[MAXD],
                                  uint32_t (&jpack)[(MAXD + 3) / 4]) {
  return forward_axes<T, MAXD, GROUPED>(
      [&](int k, uint32_t& j, T& fr) {
        j = __umulhi(u[k], (uint32_t)n);
        fr = Frac<T>::get(u[k] * (uint32_t)n);
      },
      d, cm, ot, sT, gauss, p, jpack);
}

// The same from given bins and fractions (stratified sampling).
template <typename T, int MAXD, bool GROUPED>
__device__ inline T forward_point_jf(const uint32_t (&jj)[MAXD], const T (&frs)[MAXD], int d,
                                     CP<DimMap<T>> cm, const Pair<T>* ot, int sT, bool gauss,
                                     T (&p)[MAXD], uint32_t (&jpack)[(MAXD + 3) / 4]) {
  return forward_axes<T, MAXD, GROUPED>(
      [&](int k, uint32_t& j, T& fr) {
        j = jj[k];
        fr = frs[k];
      },
      d, cm, ot, sT, gauss, p, jpack);
}

// ---------------------------------------------------------------------------
// Full evaluation of one call from global-memory tables (trace and
// unweighting): every other channel's bin is found, none is skipped.
// ---------------------------------------------------------------------------
// own: the call's own grid density and packed own bins (forward map done).
template <typename T, int MAXD>
__device__ __forceinline__ void eval_channels(const SampleArgs<T>& a, const double* alpha_g, int c,
                                              T own, const uint32_t (&jp)[(MAXD + 3) / 4],
                                              const T (&p)[MAXD], T& f, T& g, int32_t* bins) {
  const int d = a.d, n = a.n, K = a.K;
  CP<double> alpha = cp(alpha_g);
  CP<DimMap<T>> cmap = cp(a.cmap);
  CP<T> cnorm = cp(a.cnorm);
  CP<float> hab = cp(a.hab);
  const int sT = a.sT;
  f = T(0);
  g = T(0);
  for (int cc = 0; cc < K; ++cc) {
    const CP<ChanHead<T>> h = chan_at(a, cc);
    const T r = chan_r_of<T, MAXD>(h, d, p);
    f += h->twin * r;
    const T qd = cnorm[cc] * r;
    T Gd = T(1);
    if (cc == c) {
      Gd = own;
      if (bins)
        for (int k = 0; k < d; ++k) bins[c * d + k] = (jp[k >> 2] >> (8 * (k & 3))) & 0xFF;
    } else {
      int jb[MAXD];
      const Pair<T>* T0 = a.ptab + (size_t)cc * d * sT;
      const Cell<T>* C0 = a.ctab + (size_t)cc * d * a.M;
      Gd = h->kind & kChanLin
               ? grid_density<T, MAXD, 1, true>(T0, C0, sT, n, d, a.M, a.mshift,
                                                hab + (size_t)cc * 2 * d, p, jb)
               : grid_density<T, MAXD, 1, false>(T0, C0, sT, n, d, a.M, a.mshift,
                                                 hab + (size_t)cc * 2 * d, p, jb);
      if (bins)
        for (int k = 0; k < d; ++k) bins[cc * d + k] = jb[k];
    }
    g += (T)alpha[cc] * Gd * qd;
  }
  CP<PeakDim<T>> pmap = cp(a.pmap);
  CP<T> pnorm = cp(a.pnorm);
  CP<int32_t> orphans = cp(a.orphans);
  for (int o = 0; o < a.n_orphan; ++o) {
    const int i2 = orphans[o];
    f += pnorm[i2] * peak_r<T, MAXD>(pmap + (size_t)i2 * d, d, p);
  }
}

template <typename T, int MAXD>
__device__ __forceinline__ void eval_call(const SampleArgs<T>& a, const double* alpha_g, int c,
                                          const uint32_t (&u)[MAXD], T (&p)[MAXD], T& f, T& g,
                                          int32_t* bins /* [K][d] or null */) {
  uint32_t jp[(MAXD + 3) / 4];
  const T own = forward_point<T, MAXD, false>(u, a.d, a.n, cp(a.cmap) + (size_t)c * a.d,
                                       a.xtab + (size_t)c * a.d * a.sT, a.sT, false, p, jp);
  eval_channels<T, MAXD>(a, alpha_g, c, own, jp, p, f, g, bins);
}

// The same from given bins and fractions of the call's own grid.
template <typename T, int MAXD>
__device__ __forceinline__ void eval_call_jf(const SampleArgs<T>& a, const double* alpha_g, int c,
                                             const uint32_t (&jj)[MAXD], const T (&fr)[MAXD],
                                             T (&p)[MAXD], T& f, T& g, int32_t* bins) {
  uint32_t jp[(MAXD + 3) / 4];
  const T own = forward_point_jf<T, MAXD, false>(jj, fr, a.d, cp(a.cmap) + (size_t)c * a.d,
                                          a.xtab + (size_t)c * a.d * a.sT, a.sT, false, p, jp);
  eval_channels<T, MAXD>(a, alpha_g, c, own, jp, p, f, g, bins);
}

// Axes of the partial exponent of the all-Gaussian skip test.
constexpr int kPartial = 3;

// floor(log2 max(x, smallest normal)) for x >= 0 (the smallest normal's half
// ulp is the denormals' half spacing, so a term below it leaves 0 and every
// denormal sum unchanged).
__device__ inline int floor_log2_normal(float x) {
  return __builtin_amdgcn_frexp_expf(fmaxf(x, 0x1p-126f)) - 1;
}
__device__ inline int floor_log2_normal(double x) {
  return __builtin_amdgcn_frexp_exp(fmax(x, 0x1p-1022)) - 1;
}

__device__ inline uint64_t shfl_xor_u64(uint64_t v, int off) {
  const uint32_t lo = __shfl_xor((uint32_t)v, off);
  const uint32_t hi = __shfl_xor((uint32_t)(v >> 32), off);
  return (uint64_t)lo | ((uint64_t)hi << 32);
}

// Whether channel cc's term can change gg: terms are non-negative, so gg only
// grows, and a term below half an ulp of gg leaves it unchanged: skipping such
// a term gives the same gg as adding it.  (alpha gbound) r < gg bounds the
// term by gg 2^-25 (FP32; 2^-54 in FP64), below half an ulp.  Exactly zero
// terms are skipped as well.  The factors (T)alpha gbound and (T)alpha cnorm
// come formed with the allocation.
template <typename T, bool TB>
__device__ __forceinline__ bool term_counts(CP<ChanHead<T>> h, T r, T gg) {
  return r != T(0) && !(TB && h->bound * r < gg);
}

// Adds channel cc's term alpha G q to gg: d lookups for G.
// LAZY: crowded cells first give their largest density (an upper bound of G);
// the exact walks run only on the lanes where that bound, in the same test
// with the looked-up densities in place of the maxima, shows the term able to
// change gg.  Elsewhere the term is below half an ulp of gg, exact or not, and
// gg is unchanged.
template <typename T, int MAXD, int GROUP, bool EXACT, bool LAZY, bool PAIR>
__device__ __forceinline__ void add_term(const SampleArgs<T>& a, int cc, int d, int M, int mshift,
                                         T r, const T (&p)[MAXD], const uint32_t (&flat)[MAXD],
                                         T& gg) {
  const int n = a.n, sT = a.sT;
  const int chT = d * sT, chC = d * M;  // entries per channel table, cells per channel
  const CP<ChanHead<T>> h = chan_at(a, cc);
  GP<Pair<T>> T0 = gptr(a.ptab + (size_t)cc * chT);
  GP<Cell<T>> C0 = gptr(a.ctab + (size_t)cc * chC);
  CP<float> hab_cc = cp(a.hab) + (size_t)cc * 2 * d;
  if constexpr (PAIR) {
    if (h->kind & kChanPair) {
      const T Gd = pair_density<T, MAXD, GROUP, EXACT>(T0, C0, sT, n, d, M, mshift,
                                                       &pair_con(h, d)->h[0], h->bmask, flat, p);
      gg = fma(h->term * Gd, r, gg);
      return;
    }
  }
  const bool lin = h->kind & kChanLin;
  bool crowded = false;
  T Gd = lin ? grid_density<T, MAXD, GROUP, true, EXACT, LAZY>(T0, C0, sT, n, d, M, mshift, hab_cc,
                                                              p, nullptr, &crowded)
             : grid_density<T, MAXD, GROUP, false, EXACT, LAZY>(T0, C0, sT, n, d, M, mshift, hab_cc,
                                                               p, nullptr, &crowded);
  if (LAZY && crowded && !(h->look * r * Gd < gg))
    Gd = lin ? grid_density<T, MAXD, GROUP, true, EXACT>(T0, C0, sT, n, d, M, mshift, hab_cc, p,
                                                         nullptr)
             : grid_density<T, MAXD, GROUP, false, EXACT>(T0, C0, sT, n, d, M, mshift, hab_cc, p,
                                                          nullptr);
  gg = fma(h->term * Gd, r, gg);
}

// Every other channel's terms of one call of channel c at point p (eq. g(p)
// and the integrand's peaks): f += twin r for each channel's density kernel
// r, gg += alpha G q for the terms that can change gg (reading R25: exactly
// zero terms and, with TB, terms below half an ulp of gg are skipped, which
// leaves gg as the full sum gives it), then the peaks that share no
// channel's kernel.  GROUP hint-cell reads are issued together; EXACT: d is
// MAXD.  M, mshift: the job's hint cells per axis and the log map's shift.
// LAZY (with TB): crowded hint cells are walked only where their bound
// cannot rule the term out (see below).
template <typename T, int MAXD, int GROUP, bool EXACT, bool TB, bool LAZY = false, bool PAIR = false>
__device__ __forceinline__ void other_terms(const SampleArgs<T>& a, int c, int d, int M,
                                            int mshift, const T (&p)[MAXD], T& f, T& gg) {
  const int K = a.K;
  CP<PeakDim<T>> pmap = cp(a.pmap);
  CP<T> pnorm = cp(a.pnorm);
  CP<int32_t> orphans = cp(a.orphans);
  uint32_t flat[MAXD];
  if constexpr (PAIR) flat_cells<T, MAXD>(d, M, mshift, p, flat);
  for (int cc = 0; cc < K; ++cc) {
    if (cc == c) continue;
    const CP<ChanHead<T>> h = chan_at(a, cc);
    T r;
    if (TB && sizeof(T) == 8 && (h->kind & kChanIso)) {
      const CP<T> gab_cc = chan_con(h);
      // The exponent of the first kPartial axes bounds r from above
      // (the full sum only adds non-negative terms): when that bound
      // shows, on every lane of the wavefront, both of the channel's
      // terms below half an ulp of f and of gg, neither sum can change
      // and the wavefront skips the channel.  Otherwise the sum
      // continues in the same order, so r is the value the full
      // evaluation gives.  FP64 only: in FP32 the test cost more than
      // it saved (d = 10, 32 channels: FP32 8.2 -> 8.6 ms per 1e8 calls,
      // and 6.55 -> 7.19 ms with the later kernel; FP64 24.3 -> 23.3 ms).
      // (the sum of (p_k - m_k)^2, scaled by ga^2, as chan_r)
      const T sc = gab_cc[d];
      T gs = T(0);
#pragma unroll
      for (int k = 0; k < kPartial && k < MAXD; ++k) {
        if (k < d) {
          const T z = p[k] - gab_cc[k];
          gs = fma(z, z, gs);
        }
      }
      const int thr = max(h->ea - floor_log2_normal(f), h->eb - floor_log2_normal(gg));
      if (__all(gs * sc >= (T)thr)) continue;
#pragma unroll
      for (int k = kPartial; k < MAXD; ++k) {
        if (k < d) {
          const T z = p[k] - gab_cc[k];
          gs = fma(z, z, gs);
        }
      }
      r = m_exp2(-(gs * sc));
    } else {
      r = chan_r_of<T, MAXD, PAIR>(h, d, p);
    }
    f += h->twin * r;
    static_assert(!LAZY || TB, "the lazy walks rest on the term bound");
    if (term_counts<T, TB>(h, r, gg))
      add_term<T, MAXD, GROUP, EXACT, LAZY, PAIR>(a, cc, d, M, mshift, r, p, flat, gg);
  }
  for (int o = 0; o < a.n_orphan; ++o) {
    const int i2 = orphans[o];
    f += pnorm[i2] * peak_r<T, MAXD>(pmap + (size_t)i2 * d, d, p);
  }
}

// Lookups of one wavefront put off and done together.  A channel whose term
// counts on some lanes leaves its (lane, channel) pairs in the wavefront's LDS
// queue of 64 entries; a full queue, or the last channel, runs one entry per
// lane: the entry's lane fetches the owner's point across lanes and the
// channel's records, and leaves alpha cnorm G beside the kernel r; the owners
// then add their terms in channel order with the operation of add_term, so gg
// is the same bit for bit (a term tested against an earlier gg counts where
// it could not change the later one: adding it changes nothing).  At d = 10,
// 32 channels (24 Gaussian, 8 Breit-Wigner ridges) a wavefront needs 4.4
// channels' lookups on 11 lanes each: one pass in place of 4.4.
template <typename T>
struct WaveQueue {
  uint32_t who[64];  // owner lane, channel << 6
  T r[64], ag[64];
};

template <typename T>
__device__ __forceinline__ T lane_read(T v, int src) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(
        float, __builtin_amdgcn_ds_bpermute(src << 2, __builtin_bit_cast(int, v)));
  } else {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(src << 2, (int)(uint32_t)b);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(src << 2, (int)(uint32_t)(b >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
  }
}

template <typename T, int MAXD, int GROUP, bool EXACT>
struct PendingTerms {
  WaveQueue<T>* q;  // this wavefront's
  int nq = 0, np = 0;    // entries, channels (uniform)
  int mlo = 0, mhi = 0;  // lane i: the lanes of the queue's channel i

  __device__ __forceinline__ void push(int cc, uint64_t lanes, bool mine, T r) {
    const int lane = (int)__lane_id();
    const int pos = nq + __builtin_amdgcn_mbcnt_hi((uint32_t)(lanes >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)lanes, 0));
    if (mine) {
      q->who[pos] = (uint32_t)lane | ((uint32_t)cc << 6);
      q->r[pos] = r;
    }
    if (lane == np) {
      mlo = (int)(uint32_t)lanes;
      mhi = (int)(uint32_t)(lanes >> 32);
    }
    ++np;
    nq += __popcll(lanes);
  }

  __device__ __forceinline__ void run(const SampleArgs<T>& a, int d, int M, int mshift,
                                      const T (&p)[MAXD], T& gg) {
    if (nq == 0) return;
    const int lane = (int)__lane_id();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const bool live = lane < nq;
    const uint32_t who = live ? q->who[lane] : (uint32_t)lane;
    const T re = live ? q->r[lane] : T(0);
    const int src = (int)(who & 63u), cc = (int)(who >> 6);
    T pe[MAXD];
#pragma unroll
    for (int k = 0; k < MAXD; ++k)
      if (EXACT || k < d) pe[k] = lane_read(p[k], src);
      else pe[k] = T(0);
    const T ge = lane_read(gg, src);
    if (live) {
      const GP<ChanHead<T>> h = (GP<ChanHead<T>>)(gptr(a.crec) + (uint32_t)(cc * a.cstride));
      const T term = h->term;
      const T G = lane_density<T, MAXD, GROUP, EXACT>(gptr(a.ptab), gptr(a.ctab), gptr(a.hab), cc,
                                                      (h->kind & kChanLin) != 0, a.sT, a.n, d, M, mshift,
                                                      pe, h->look * re, ge);
      q->ag[lane] = term * G;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    int base = 0;
    for (int i = 0; i < np; ++i) {
      const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane(mlo, i);
      const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane(mhi, i);
      const int pos = base + __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0));
      const uint64_t m = ((uint64_t)hi << 32) | lo;
      if ((m >> lane) & 1ull) gg = fma(q->ag[pos], q->r[pos], gg);
      base += __popcll(m);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    nq = 0;
    np = 0;
  }
};

// The same with the channels that cannot change f or g on any lane of the
// wavefront left out up front (mcv_mask.h): f and gg enter with the call's own
// terms, both only grow from there (fpos), so a term below half an ulp of
// them now is below it when its turn comes; and with the lookups of sparse
// terms done together (PendingTerms).  Every lane of the wavefront takes part.
template <typename T, int MAXD, int GROUP, bool EXACT>
__device__ __forceinline__ void masked_terms(const SampleArgs<T>& a, int c, int d, int M,
                                             int mshift, WaveQueue<T>* queue, const T (&p)[MAXD],
                                             T& f, T& gg) {
  const int K = a.K;
  const int least = sizeof(T) == 4 ? -126 : -1022;
  const int e = a.fpos ? min(floor_log2_normal(f), floor_log2_normal(gg)) : least;
  PendingTerms<T, MAXD, GROUP, EXACT> pend{queue};
  int base = -32;  // the tile of channels that m is of
  uint32_t m = 0;
  bool last = false;
  do {
    for (;;) {
      if (m == 0) {
        base += 32;
        last = base >= K;
        if (last) break;
        m = channel_mask<MAXD, EXACT>(p, d, (float)e, a.mco, a.mthr, base >> 5);
        // the last tile's columns beyond the channels: their thresholds rule
        // them out, but not where no call of the product is a number (a call
        // without a point, as a width beyond the FP32 range gives)
        if (K - base < 32) m &= (1u << (K - base)) - 1u;
        if ((unsigned)(c - base) < 32u) m &= ~(1u << (c - base));
        continue;
      }
      const int cc = base + __builtin_ctz(m);
      const CP<ChanHead<T>> h = chan_at(a, cc);
      const T r = chan_r_of<T, MAXD>(h, d, p);
      const bool counts = term_counts<T, true>(h, r, gg);
      const uint64_t lanes = __ballot(counts);
      if (pend.nq + __popcll(lanes) > 64) break;  // run the queue, then this channel again
      m &= m - 1;
      f += h->twin * r;
      if (lanes) pend.push(cc, lanes, counts, r);
    }
    pend.run(a, d, M, mshift, p, gg);
  } while (!last);
  CP<PeakDim<T>> pmap = cp(a.pmap);
  CP<T> pnorm = cp(a.pnorm);
  CP<int32_t> orphans = cp(a.orphans);
  for (int o = 0; o < a.n_orphan; ++o) {
    const int i2 = orphans[o];
    f += pnorm[i2] * peak_r<T, MAXD>(pmap + (size_t)i2 * d, d, p);
  }
}

// ---------------------------------------------------------------------------
// The sample pass.  Every thread takes one call of the segment's channel c per
// round: draws, forward map and own grid density, then one loop over the
// other channels computes each density kernel r once; the integrand collects
// the peaks that share a channel's exponential (then the remaining peaks),
// and every channel with a non-zero density adds alpha G q to g, its grid
// density G found from the channel's hint-cell records (global memory, L2),
// with its (edge, density) table for the rare exact walks.  The segment's own
// x-space table and its per-bin sums of w^2 live in LDS.
// ---------------------------------------------------------------------------

// One work unit of a pass: unit g of the job's G units takes the calls
// [g N/G, (g+1) N/G).  BLOCK > 0: the workgroup size as a constant, else
// blockDim.x.  EXACT: the job's dimension is MAXD (no per-axis guards).
// TB: a channel's lookups are guarded by its term bound (else only exactly
// zero terms are skipped); the results are the same either way.  TRACE:
// also write f, g and w of the calls in the argument record's trace window
// (the same code path otherwise).  MT > 0: the job's hint cells per axis as
// a constant (its offsets fold into immediates).  MASK: channels left out
// by masks (mcv_mask.h).  Every thread of the workgroup calls it with the same
// unit.  staged: the channel whose own table the workgroup holds in LDS (-1:
// none, and the sums are not yet cleared).
template <typename T, int MAXD, int BLOCK, bool EXACT, bool TB, bool TRACE = false, int RNG = 0,
          int MT = 0, bool LAZY = false, bool MASK = false, bool PAIR = false>
__device__ __forceinline__ void sample_unit(const SampleArgs<T>& a, int g, int G, uint32_t tag,
                                            unsigned char* smem, int& staged) {
  static_assert(RNG == 0 || (BLOCK > 0 && (BLOCK & (BLOCK - 1)) == 0),
                "MRG32k3a substreams advance by a power-of-two workgroup");
  constexpr int GROUP = sizeof(T) == 4 ? 5 : BLOCK > 0 ? 2 : 4;
  const int block = BLOCK > 0 ? BLOCK : (int)blockDim.x;
  const int waves = block >> 6;
  Pair<T>* ownT = reinterpret_cast<Pair<T>*>(smem + a.off_own);
  double* hist = reinterpret_cast<double*>(smem + a.off_hist);
  double* red = reinterpret_cast<double*>(smem + a.off_red);
  // this wavefront's lookup queue, behind the cross-wave reduction
  WaveQueue<T>* queue = reinterpret_cast<WaveQueue<T>*>(smem + a.off_queue) + (threadIdx.x >> 6);

  const int d = EXACT ? MAXD : a.d, n = a.n, K = a.K;
  const int tid = threadIdx.x;
  CP<int64_t> start = cp(a.start);
  CP<double> alpha = cp(a.alpha);
  CP<DimMap<T>> cmap = cp(a.cmap);
  CP<T> cnorm = cp(a.cnorm);

  const int64_t ntot = start[K];
  const int64_t lo = (int64_t)g * ntot / G;
  const int64_t hi = (int64_t)(g + 1) * ntot / G;
  if (lo >= hi) return;  // uniform over the workgroup
  const int dn = d * n;
  const int sT = a.sT;
  // hint cells per axis: the constant MT (256 or 512), else the job's
  const int M = MT > 0 ? MT : a.M;
  const int mshift = MT > 0 ? (MT == 512 ? 18 : 19) : a.mshift;
  const int chT = d * sT;  // entries per channel table

  if (staged < 0)
    for (int t = tid; t < dn; t += block) hist[t] = 0.0;

  int c = 0;
  while (c < K - 1 && start[c + 1] <= lo) ++c;
  for (; c < K && start[c] < hi; ++c) {
    const int64_t s0 = start[c] > lo ? start[c] : lo;
    const int64_t s1 = start[c + 1] < hi ? start[c + 1] : hi;
    __syncthreads();
    if (staged != c) {  // uniform
      copy16(ownT, a.xtab + (size_t)c * chT, chT * (int)sizeof(Pair<T>), block);
      staged = c;
      __syncthreads();
    }

    // Per-lane sums of w and w^2 of the segment: plain FP64 sums over at
    // most kFold rounds, folded into compensated sums (little state live
    // across the channel loop).
    constexpr int kFold = 16;
    Neu S1{0.0, 0.0}, S2{0.0, 0.0};
    double q1 = 0.0, q2 = 0.0;
    int rounds = 0;
    T wmax = T(0);
    uint32_t nbad = 0u;
    const T al_c = (T)alpha[c];
    CP<DimMap<T>> cm_c = cmap + (size_t)c * d;
    const T own_norm = al_c * cnorm[c];
    const CP<ChanHead<T>> h_c = chan_at(a, c);
    // grouped axis maps in the single-job pass only: the batched kernel's 13
    // bodies would each carry both paths (its FP64 pass 2.77 -> 2.95 ms)
    const bool all_gauss = (h_c->kind & kChanLin) != 0;
    const T tw_c = h_c->twin;
    // MRG32k3a: this lane's first call of the segment is substream
    // s0 + tid - start[c] of channel c's stream; each round moves BLOCK
    // substreams on
    Mrg mst{};
    if constexpr (RNG == 1)
      mst = mrg_call_state(a.mrg, c, (uint64_t)(s0 + tid - start[c]), tag);

    for (int64_t base = s0; base < s1; base += block) {
      // The batched FP32 pass is bound by reads of hint cells that miss the L1
      // (28 KB a channel, other workgroups elsewhere); wavefronts of a workgroup
      // that start a round together read a channel's cells at about the same
      // time and share more of them.  (uniform: every thread runs every round;
      // 256 jobs, two iterations: 147.0 -> 141.9 ms; FP64 11.8 either way)
      if constexpr (BLOCK == 0 && sizeof(T) == 4) __builtin_amdgcn_s_barrier();
      const int64_t i = base + tid;
      const bool valid = i < s1;
      T p[MAXD];
      uint32_t jp[(MAXD + 3) / 4];
      T f = T(0), gg = T(1);
      // with masks every lane of a wavefront that holds a call takes part; a
      // lane beyond the segment evaluates a point that is not counted
      if (MASK ? base + (tid & ~63) < s1 : valid) {
        uint32_t u[MAXD];
        if constexpr (RNG == 1) {
          Mrg w = mst;
#pragma unroll
          for (int k = 0; k < MAXD; ++k)
            if (k < d) u[k] = mrg_word(w);
        } else {
          draw_words<MAXD>(a.seed, (uint64_t)i, tag, d, u);
        }
        const T own = forward_point<T, MAXD, (BLOCK > 0)>(u, d, n, cm_c, ownT, sT, all_gauss, p, jp);
        const T r_c = chan_r_of<T, MAXD>(h_c, d, p);
        f = tw_c * r_c;
        gg = own_norm * own * r_c;
        if constexpr (MASK)
          masked_terms<T, MAXD, GROUP, EXACT>(a, c, d, M, mshift, queue, p, f, gg);
        else
          other_terms<T, MAXD, GROUP, EXACT, TB, LAZY, PAIR>(a, c, d, M, mshift, p, f, gg);
      }
      // ---- weights and sums (FP64)
      if (valid) {
        const T wt = f / gg;
        if constexpr (TRACE) {
          if (i >= a.tr_first && i < a.tr_first + a.tr_count) {
            double* o = a.tr_out + (i - a.tr_first) * 3;
            o[0] = (double)f;
            o[1] = (double)gg;
            o[2] = (double)wt;
          }
        }
        const double w = (double)wt;
        if (!isfinite(wt)) {
          ++nbad;
        } else {
          q1 += w;
          const double w2 = w * w;
          q2 += w2;
          const T aw = fabs(wt);  // signed integrands: the largest |w|
          wmax = aw > wmax ? aw : wmax;
#pragma unroll
          for (int k = 0; k < MAXD; ++k) {
            if (k < d) {
              const int jb = (jp[k >> 2] >> (8 * (k & 3))) & 0xFF;
              __hip_atomic_fetch_add(hist + k * n + jb, w2, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_WORKGROUP);
            }
          }
        }
      }
      if constexpr (RNG == 1) {
        constexpr int kLog2Block = __builtin_ctz((unsigned)(BLOCK > 0 ? BLOCK : 1));
        mrg_apply(cp(a.mrg) + (size_t)(kMrgSubBase + kLog2Block) * kMrgEntry, mst);
      }
      if (++rounds == kFold) {  // uniform
        S1.add(q1);
        S2.add(q2);
        q1 = 0.0;
        q2 = 0.0;
        rounds = 0;
      }
    }
    S1.add(q1);
    S2.add(q2);

    // segment reduction: wavefront butterflies, then LDS across waves
    double wmax_d = (double)wmax, nbad_d = (double)nbad;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const Neu o1{__shfl_xor(S1.s, off), __shfl_xor(S1.c, off)};
      const Neu o2{__shfl_xor(S2.s, off), __shfl_xor(S2.c, off)};
      S1 = neu_merge(S1, o1);
      S2 = neu_merge(S2, o2);
      wmax_d = fmax(wmax_d, __shfl_xor(wmax_d, off));
      nbad_d += __shfl_xor(nbad_d, off);
    }
    const int wave = tid >> 6;
    if ((tid & 63) == 0) {
      red[wave * 6 + 0] = S1.s;
      red[wave * 6 + 1] = S1.c;
      red[wave * 6 + 2] = S2.s;
      red[wave * 6 + 3] = S2.c;
      red[wave * 6 + 4] = wmax_d;
      red[wave * 6 + 5] = nbad_d;
    }
    __syncthreads();
    const size_t slot = (size_t)g + (size_t)c;
    if (tid == 0) {
      Neu A{red[0], red[1]}, B{red[2], red[3]};
      double wm = red[4], nb = red[5];
      for (int w = 1; w < waves; ++w) {
        A = neu_merge(A, Neu{red[w * 6 + 0], red[w * 6 + 1]});
        B = neu_merge(B, Neu{red[w * 6 + 2], red[w * 6 + 3]});
        wm = fmax(wm, red[w * 6 + 4]);
        nb += red[w * 6 + 5];
      }
      double* r = a.part + slot * kPartStride;
      r[0] = A.s;
      r[1] = A.c;
      r[2] = B.s;
      r[3] = B.c;
      r[4] = wm;
      r[5] = nb;
    }
    for (int t = tid; t < dn; t += block) {
      a.hpart[slot * dn + t] = hist[t];
      hist[t] = 0.0;
    }
  }
}

// A wave-uniform record read with scalar loads.
template <typename S>
__device__ __forceinline__ S load_uniform(const S* p) {
  static_assert(sizeof(S) % 4 == 0, "record of whole dwords");
  S out;
  uint32_t* o = reinterpret_cast<uint32_t*>(&out);
  CP<uint32_t> q = (CP<uint32_t>)(p);
#pragma unroll
  for (int i = 0; i < (int)(sizeof(S) / 4); ++i) o[i] = q[i];
  return out;
}

// Batched pass: a persistent grid drains the work units spanning every job
// of a set.  Unit u belongs to the job jb with prefix[jb] <= u <
// prefix[jb+1] and is that job's unit u - prefix[jb] of prefix[jb+1] -
// prefix[jb]; each job's arguments (and LDS layout, after a 16-byte header
// that broadcasts the unit index) come from args[jb].  A unit's result does
// not depend on which workgroup runs it.
//
// The units, whose jobs are ordered from the costliest call to the cheapest,
// are dealt to kQueues queues in chunks (chunk i to queue i mod kQueues;
// counter[q] counts the units taken from queue q).  Workgroups are dispatched
// to the chip's 8 XCDs in turn (workgroup w on XCD w mod 8), so workgroup w
// drains queue w mod 8 first: an XCD's workgroups run a contiguous stretch of
// jobs at a time and its own L2 holds only their hint-cell tables, while every
// queue ends with cheap units.  A chunk is what an XCD runs at once, or less
// where that would leave a queue fewer than 4 chunks.  (One contiguous range
// per queue, cheapest jobs first, left the XCDs with unequal work and the
// costliest units to the end: 48 jobs FP64 14.5 ms in place of 11.8, 128 jobs
// FP64 34.8 and 28.0, serving 16 jobs 9.25 and 8.6, 256 jobs FP32 148.5 and
// 146.5.)  A workgroup whose queue is empty takes units from the next queues
// in turn, and leaves once every queue is empty.  The counters are zeroed by the
// allocation kernel before each pass.  LB: the launch bound (largest
// workgroup size); 512 leaves the compiler more registers per lane, 256 caps
// them for at least 6 (FP32; 69.1 ms on the 256-job batch, against 69.9 at 7
// and 73.0 at 8) or 4 (FP64) waves per SIMD.  TB: lookups
// guarded by the channels' term bounds.  PAIR: pair channels take their own path.
constexpr int kQueues = 8;

// One unit of a batched pass, compiled for the job's dimension: d <= 12
// exactly (no per-axis guards; the grouped hint-cell reads cover only the
// job's axes, where a 12-axis body would read 5, 10 or 15 cells for any d),
// a larger d through the generic body of the bucket MAXD.  d is uniform over
// the workgroup, and the set orders its jobs by d first, so the workgroups of one
// XCD mostly run one body at a time.
template <typename T, int MAXD, bool TB, bool PAIR>
__device__ __forceinline__ void queue_unit(const SampleArgs<T>& a, int u, int G, uint32_t tag,
                                           unsigned char* smem) {
  int staged = -1;  // the unit's job may differ from the one before
#define MCV_EXACT_CASE(D)                                         \
  case D:                                                         \
    if constexpr (D <= MAXD) {                                    \
      sample_unit<T, D, 0, true, TB, false, 0, 0, false, false, PAIR>(a, u, G, tag, smem, staged); \
      return;                                                     \
    }                                                             \
    break;
  switch (a.d) {
    MCV_EXACT_CASE(1)
    MCV_EXACT_CASE(2)
    MCV_EXACT_CASE(3)
    MCV_EXACT_CASE(4)
    MCV_EXACT_CASE(5)
    MCV_EXACT_CASE(6)
    MCV_EXACT_CASE(7)
    MCV_EXACT_CASE(8)
    MCV_EXACT_CASE(9)
    MCV_EXACT_CASE(10)
    MCV_EXACT_CASE(11)
    MCV_EXACT_CASE(12)
    default:
      break;
  }
#undef MCV_EXACT_CASE
  if constexpr (MAXD > 12) sample_unit<T, MAXD, 0, false, TB>(a, u, G, tag, smem, staged);
}

template <typename T, int MAXD, int LB, bool TB, bool PAIR>
__global__ __launch_bounds__(LB, LB == 256 ? (sizeof(T) == 4 ? 6 : 4) : 1) void k_sample_queue(
    const SampleArgs<T>* args, const int* prefix, int n_jobs, int n_units, int* counter) {
  extern __shared__ __align__(16) unsigned char smem[];
  int* bcast = reinterpret_cast<int*>(smem);
  CP<int> pf = cp(prefix);
  const int home = (int)(blockIdx.x % kQueues);
  const int chunk = max(1, min((int)gridDim.x / kQueues, n_units / (4 * kQueues)));
  int tried = 0;  // queues found empty (thread 0's view; the unit is broadcast)
  for (;;) {
    if (threadIdx.x == 0) {
      int unit = -1;
      while (tried < kQueues) {
        const int q = (home + tried) % kQueues;
        const int k = atomicAdd(counter + q, 1);
        const int64_t u = ((int64_t)(k / chunk) * kQueues + q) * chunk + k % chunk;
        if (u < n_units) {
          unit = (int)u;
          break;
        }
        ++tried;
      }
      bcast[0] = unit;
    }
    __syncthreads();
    const int u = __builtin_amdgcn_readfirstlane(bcast[0]);
    __syncthreads();
    if (u < 0) break;
    int lo = 0, hi = n_jobs;  // largest jb with prefix[jb] <= u
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (pf[mid] <= u) lo = mid;
      else hi = mid;
    }
    const int u0 = pf[lo];
    const int G = pf[lo + 1] - u0;
    const SampleArgs<T> a = load_uniform(args + lo);
    const uint32_t tag = (uint32_t)cp(a.iter)[0];
    queue_unit<T, MAXD, TB, PAIR>(a, u - u0, G, tag, smem);
  }
}

// Launch shape of the single-job kernel: 256-thread workgroups, registers
// capped for a number of waves per SIMD (d = 10, 32 channels, 24 Gaussian and
// 8 Breit-Wigner: FP32 with masks 4.10, 3.93 and 4.36 ms a pass of 1e8 at 4, 5
// and 6 waves; FP64 2.08, 1.96 and 2.4 ms a pass of 1e7 at 3, 4 and 5; FP32
// without masks 7, where its few registers allow it).  Above 12 axes fewer: 7
// without masks spilled up to 3064 registers (d = 14, 8 channels: 2.8 ms a pass
// of 2e6), and 5 with them 143 (an iteration of 2e6 calls, d = 14, 16 Gaussian
// channels: 514 us at 5, 228 at 4, 240 at 3 and 286 without masks; d = 16: 234,
// 222, 214 and 247).
template <typename T>
struct Tune {
  static constexpr int BLOCK = 256;  // one call per thread and round
};
template <typename T, int MAXD, bool MASK>
constexpr int kMinWaves =
    sizeof(T) == 8 || MAXD > 16 ? 4 : MASK ? (MAXD > 12 ? 4 : 5) : MAXD > 12 ? 5 : 7;

// Single-job pass: as many workgroups as fit the chip at once drain the
// pass's units in order, each taking the next one when it is done, so that
// units of unequal cost (the channels' calls differ by an order of magnitude)
// leave no tail longer than a unit; consecutive units mostly share a channel,
// whose own table then stays in LDS.  A unit's results do not depend on which
// workgroup runs it.  The counter is cleared by the allocation before.  RNG: 0
// Philox words, 1 MRG32k3a streams.  Lazy walks in FP32 only (d = 10, 32
// channels: FP32 6.16 -> 5.91 ms with them, FP64 22.4 -> 23.1 ms; the batched
// pass, whose channels all use the log map, 69 -> 76 ms, so it does without).
// TRACE: the same with its trace window written (the tag then comes from the
// argument record).
template <typename T>
constexpr bool kLazyWalks = sizeof(T) == 4;

template <typename T, int MAXD, int BLOCK, bool EXACT, int RNG = 0, int MT = 0,
          bool MASK = false, bool TRACE = false>
__global__ __launch_bounds__(BLOCK, (kMinWaves<T, MAXD, MASK>)) void k_sample(SampleArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int next_s;
  const uint32_t tag = TRACE ? a.tag : (uint32_t)cp(a.iter)[0];
  int staged = -1;
  for (int u = blockIdx.x; u < a.units;) {
    int next = 0;
    if (threadIdx.x == 0) next = atomicAdd(a.next, 1);  // under way while the unit runs
    sample_unit<T, MAXD, BLOCK, EXACT, true, TRACE, RNG, MT, kLazyWalks<T>, MASK>(
        a, u, a.units, tag, smem, staged);
    if (threadIdx.x == 0) next_s = next + (int)gridDim.x;
    __syncthreads();
    u = __builtin_amdgcn_readfirstlane(next_s);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Host side: argument records, LDS layouts and launch shapes.
// ---------------------------------------------------------------------------
template <typename T>
SampleArgs<T> make_args(const JobDev& j, uint32_t tag) {
  SampleArgs<T> a{};
  a.d = j.d;
  a.K = j.K;
  a.n = j.n;
  a.P = j.P;
  a.sT = j.sT;
  a.M = j.M;
  a.mshift = j.mshift;
  a.tag = tag;
  a.seed = j.seed;
  a.iter = j.iter_dev;
  a.next = j.next;
  a.start = j.start;
  a.alpha = j.alpha;
  a.orphans = j.orphans;
  a.n_orphan = j.n_orphan;
  if (sizeof(T) == 8) {
    a.cmap = reinterpret_cast<const DimMap<T>*>(j.cmap64);
    a.cnorm = reinterpret_cast<const T*>(j.cnorm64);
    a.pmap = reinterpret_cast<const PeakDim<T>*>(j.pmap64);
    a.pnorm = reinterpret_cast<const T*>(j.pnorm64);
  } else {
    a.cmap = reinterpret_cast<const DimMap<T>*>(j.cmap32);
    a.cnorm = reinterpret_cast<const T*>(j.cnorm32);
    a.pmap = reinterpret_cast<const PeakDim<T>*>(j.pmap32);
    a.pnorm = reinterpret_cast<const T*>(j.pnorm32);
  }
  a.xtab = reinterpret_cast<const Pair<T>*>(j.xtab);
  a.ptab = reinterpret_cast<const Pair<T>*>(j.ptab);
  a.ctab = reinterpret_cast<const Cell<T>*>(j.ctab);
  a.crec = j.crec;
  a.cstride = chan_stride<T>(j.d);
  a.hab = j.hab;
  a.mco = j.mco;
  a.mthr = j.mthr;
  a.fpos = j.fpos;
  a.part = j.part;
  a.hpart = j.hpart;
  a.rng = j.rng;
  a.mrg = j.mrg;
  a.strat = j.strat;
  a.nr = j.nr;
  a.spb = j.spb;
  a.bstart = j.bstart;
  return a;
}

static inline int align16(int x) { return (x + 15) & ~15; }


// LDS layout of the sample kernel from byte `base` on: the own channel's
// x-space table, the per-bin sums of w^2 and the cross-wave reduction.
// Returns the end of the layout (bytes used, base included).
template <typename T>
int lds_layout(SampleArgs<T>& a, int waves, int base = 0, bool masked = false) {
  const int chT = a.d * a.sT * (int)sizeof(Pair<T>);
  int off = base;
  a.off_own = off;
  off += align16(chT);
  a.off_hist = off;
  off += align16(a.d * a.n * 8);
  a.off_red = off;
  off += align16(waves * 6 * 8);
  a.off_queue = off;
  if (masked) off += waves * (int)sizeof(WaveQueue<T>);
  return off;
}

// Work units of one pass of n_points calls in rounds of per_round, for G
// workgroups that fit the chip at once.  A unit of r rounds costs r rounds and
// its start and end (its table, its record and bins written and summed: about
// one and a half); the workgroups run ceil(U / G) units each one after the other,
// and end about half a unit apart.  The least of ceil(U / G) (r + 3/2) + r / 2:
// for a long pass r grows as sqrt(R / G), R the pass's rounds, for a short one
// the units come out at or just under whole multiples of G.  Measured best
// (d = 10, 32 channels): r = 1 (R = 40), 2 to 3 (1300), 2 and 4 but not 3 (3900,
// G = 1024: 1302 units ran as two sets, 1.46 -> 1.60 ms for ten passes), 6 to
// 16 (39000), flat from 8 to 48 (390000).  At most the partial buffers' units.
inline int units_for(const JobDev& j, int per_round, int64_t n_points, int64_t G) {
  const int64_t R = (n_points + per_round - 1) / per_round;
  if (G < 1) G = 1;
  int64_t best = 1;
  double least = INFINITY;
  for (int64_t r = 1; r <= 4096 && (r == 1 || (r - 1) * G < R); ++r) {
    const int64_t U = (R + r - 1) / r;
    if (U > j.gmax) continue;
    const double t = (double)((U + G - 1) / G) * ((double)r + 1.5) + 0.5 * (double)r;
    if (t < least) {
      least = t;
      best = U;
    }
  }
  if (least == INFINITY) best = j.gmax;
  return (int)(best < 1 ? 1 : best);
}

// Work units and workgroups of k_sample for a pass of n_points.
template <typename T, int MAXD, bool EXACT, int RNG, int MT, bool MASK, bool TRACE = false>
Split sample_split_m(const JobDev& j, int64_t n_points) {
  constexpr int BLOCK = Tune<T>::BLOCK;
  SampleArgs<T> a = make_args<T>(j, 0);
  const int lds = lds_layout<T>(a, BLOCK / 64, 0, MASK);
  auto kern = k_sample<T, MAXD, BLOCK, EXACT, RNG, MT, MASK, TRACE>;
  if (lds > 64 * 1024 &&
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds) !=
          hipSuccess)
    return Split{0, 0};
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)kern, BLOCK, lds) !=
          hipSuccess ||
      per_cu < 1)
    return Split{0, 0};
  const int G = per_cu * j.n_cu;
  Split sp{units_for(j, BLOCK, n_points, G), G};
  if (sp.G > sp.U) sp.G = sp.U;
  return sp;
}

template <typename T, int MAXD, bool EXACT, int RNG, int MT, bool MASK>
Split launch_sample_m(const JobDev& j, int64_t n_points, hipStream_t s) {
  constexpr int BLOCK = Tune<T>::BLOCK;
  const Split sp = sample_split_m<T, MAXD, EXACT, RNG, MT, MASK>(j, n_points);
  if (sp.G < 1) return sp;
  SampleArgs<T> a = make_args<T>(j, 0);
  a.units = sp.U;
  const int lds = lds_layout<T>(a, BLOCK / 64, 0, MASK);
  hipLaunchKernelGGL((k_sample<T, MAXD, BLOCK, EXACT, RNG, MT, MASK>), dim3(sp.G),
                     dim3(BLOCK), lds, s, a);
  return sp;
}

// The trace instantiation over the trace allocation (t_start, t_alpha), split
// as k_sample splits a pass of n_points.
template <typename T, int MAXD, bool EXACT, int RNG, int MT, bool MASK>
Split launch_sample_trace_m(const JobDev& j, int64_t n_points, uint32_t tag, int64_t first,
                            int64_t count, double* out, hipStream_t s) {
  constexpr int BLOCK = Tune<T>::BLOCK;
  Split sp = sample_split_m<T, MAXD, EXACT, RNG, MT, MASK, true>(j, n_points);
  if (sp.G < 1) return sp;
  SampleArgs<T> a = make_args<T>(j, tag);
  a.units = sp.U;
  a.start = j.t_start;
  a.alpha = j.t_alpha;
  a.crec = j.t_crec;
  a.tr_first = first;
  a.tr_count = count;
  a.tr_out = out;
  const int lds = lds_layout<T>(a, BLOCK / 64, 0, MASK);
  hipLaunchKernelGGL((k_sample<T, MAXD, BLOCK, EXACT, RNG, MT, MASK, true>), dim3(sp.G),
                     dim3(BLOCK), lds, s, a);
  return sp;
}

// Calls FN<T, MAXD, EXACT, RNG, MT, MASK>(...).  The single-job pass with
// Philox words takes the job's hint cells per axis as a constant (256 or
// 512); MRG32k3a passes read it from the arguments.  MASK where the job has
// mask coefficients.
#define MCV_SAMPLE_VARIANT(FN, ...)                                                     \
  do {                                                                                  \
    constexpr bool kMask = sizeof(T) == 4 && mask_form(MAXD, EXACT).steps > 0;                           \
    if constexpr (RNG == 0) {                                                           \
      if (kMask && j.masked)                                                            \
        return j.M == 512 ? FN<T, MAXD, EXACT, RNG, 512, kMask>(__VA_ARGS__)            \
                          : FN<T, MAXD, EXACT, RNG, 256, kMask>(__VA_ARGS__);           \
      return j.M == 512 ? FN<T, MAXD, EXACT, RNG, 512, false>(__VA_ARGS__)              \
                        : FN<T, MAXD, EXACT, RNG, 256, false>(__VA_ARGS__);             \
    }                                                                                   \
    if (kMask && j.masked) return FN<T, MAXD, EXACT, RNG, 0, kMask>(__VA_ARGS__);       \
    return FN<T, MAXD, EXACT, RNG, 0, false>(__VA_ARGS__);                              \
  } while (0)

template <typename T, int MAXD, bool EXACT, int RNG = 0>
Split launch_sample_t(const JobDev& j, int64_t n_points, hipStream_t s) {
  MCV_SAMPLE_VARIANT(launch_sample_m, j, n_points, s);
}

template <typename T, int MAXD, bool EXACT, int RNG = 0>
Split launch_sample_trace_t(const JobDev& j, int64_t n_points, uint32_t tag, int64_t first,
                            int64_t count, double* out, hipStream_t s) {
  MCV_SAMPLE_VARIANT(launch_sample_trace_m, j, n_points, tag, first, count, out, s);
}
#undef MCV_SAMPLE_VARIANT


}  // namespace
}  // namespace mcv
