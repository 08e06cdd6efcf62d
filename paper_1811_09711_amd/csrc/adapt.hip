// Small device kernels around the sample pass: set-up of the map constants
// and grids, p-space edge tables, the integer channel allocation, the
// reduction of a pass, VEGAS rebinning and the channel-weight update.
//
// Brass, Kilian, Reuter, arXiv:1811.09711: Sec. 3.1 (E_N, V_N), Sec. 3.2
// (eq. g(x), eq. 30, eq. 31), Sec. 3.4 (multi-channel estimator, eq. 15 and
// the integer N_c), Sec. 3.5 (eq. g(p); the organisation of an iteration).
#include <hip/hip_runtime.h>
#include <math.h>

#include "mcv_internal.h"
#include "mcv_mask.h"
#include "mcv_point.h"

namespace mcv {

namespace {

constexpr double kInvSqrt2Pi = 0.39894228040143267794;
// sqrt(log2(e) / 2): exp(-z^2/2) = 2^(-(kExpScale z)^2)
constexpr double kExpScale = 0.84932180028801904272;
constexpr double kPi = 3.14159265358979323846;

// ---------------------------------------------------------------------------
// Set-up
// ---------------------------------------------------------------------------
template <typename T>
__device__ inline ChanHead<T>* chan_head(char* rec, int c, int d) {
  return reinterpret_cast<ChanHead<T>*>(rec + (size_t)c * chan_stride<T>(d));
}
template <typename T>
__device__ inline T* chan_constants(char* rec, int c, int d) {
  return reinterpret_cast<T*>(chan_head<T>(rec, c, d) + 1);
}

template <typename T>
__device__ inline void set_head(char* rec, int c, int d, uint32_t gmask, uint32_t bmask, int kind,
                                T twin) {
  ChanHead<T>* h = chan_head<T>(rec, c, d);
  h->gmask = gmask;
  h->bmask = bmask;
  h->kind = (int16_t)kind;
  h->twin = twin;
}
// One wavefront per channel, then one per peak: lane k takes axis k (at most
// 32), the products over the axes run in axis order across the lanes.  A
// channel's workgroup also writes its twin's factor (the norm of the peak of
// its shape), its equidistant grid (Sec. 3.2: adaptation starts from
// equidistant bins; in mixed precision rounded to FP32, which keeps them
// apart) and its weight.  The history is cleared by workgroups of its own,
// kZeroRows rows each: with 65536 rows the one wavefront of a one-channel job
// took 90 of its creation's 175 us.  One launch; as four, with a thread per
// channel or axis walking its arrays, the set-up of a 10-axis, 32-channel job
// took 110 us.
constexpr int kZeroRows = 512;
constexpr int kMaxZeroGroups = 1024;

inline int zero_groups(int max_iter) {
  const int g = max_iter / kZeroRows + (max_iter % kZeroRows ? 1 : 0);
  return g < kMaxZeroGroups ? g : kMaxZeroGroups;
}

__device__ inline double axis_product(double first, double factor, bool counts, int d) {
  double norm = first;
  for (int k = 0; k < d; ++k) {
    const double v = __shfl(factor, k);
    if (__shfl(counts ? 1 : 0, k)) norm *= v;
  }
  return norm;
}

__device__ inline double peak_norm(const JobDev& j, int i, int lane) {
  double f = 1.0;
  bool counts = false;
  if (lane < j.d) {
    const int kind = j.pkind[i * j.d + lane];
    const double w = j.pwidth[i * j.d + lane];
    counts = kind != FLAT;
    f = kind == GAUSS ? kInvSqrt2Pi / w : (0.5 * w) / kPi;
  }
  return axis_product(j.pweight[i], f, counts, j.d);
}

__global__ __launch_bounds__(64) void k_setup(JobDev j) {
  const int lane = threadIdx.x, d = j.d;
  if ((int)blockIdx.x >= j.K + j.P) {
    const int64_t g = (int64_t)blockIdx.x - (j.K + j.P), groups = (int64_t)gridDim.x - (j.K + j.P);
    for (int64_t q = g * 64 + lane; q < (int64_t)j.max_iter * kHistStride; q += groups * 64)
      j.history[q] = 0.0;
    return;
  }
  if ((int)blockIdx.x >= j.K) {
    const int i = (int)blockIdx.x - j.K;
    if (lane < d) {
      const int t = i * d + lane;
      PeakDim<double> m{};
      m.kind = j.pkind[t];
      m.loc = j.ploc[t];
      if (m.kind == GAUSS) {
        m.ga = kExpScale / j.pwidth[t];
        m.gb = -m.loc * m.ga;
      }
      if (m.kind == BW) m.h2 = 0.25 * j.pwidth[t] * j.pwidth[t];
      j.pmap64[t] = m;
      PeakDim<float> f{};
      f.kind = m.kind;
      f.loc = (float)m.loc;
      f.h2 = (float)m.h2;
      f.ga = (float)m.ga;
      f.gb = (float)m.gb;
      j.pmap32[t] = f;
    }
    const double norm = peak_norm(j, i, lane);
    if (lane == 0) {
      j.pnorm64[i] = norm;
      j.pnorm32[i] = (float)norm;
    }
    return;
  }
  const int c = blockIdx.x, t = c * d + lane;
  const bool on = lane < d;
  DimMap<double> m{};
  if (on) {
    m.kind = j.ckind[t];
    m.loc = j.cloc[t];
    m.width = j.cwidth[t];
    m.hs = (float)j.M;  // flat: the identity onto the cells
    m.hb = 0.0f;
    m.ls = kFlatA;      // flat, log map
    m.lb = kFlatB;
    if (m.kind == GAUSS) {
      const double a = (0.0 - m.loc) / m.width, b = (1.0 - m.loc) / m.width;
      m.inv_w = 1.0 / m.width;
      m.ga = kExpScale / m.width;
      m.gb = -m.loc * m.ga;
      // linear hint map: centre +- 3 sigma onto the M cells
      m.hs = (float)((double)j.M / (6.0 * m.width));
      m.hb = (float)((double)j.M * (0.5 - m.loc / (6.0 * m.width)));
      m.ls = (float)(16.0 / m.width);
      m.lb = (float)(-16.0 * m.loc / m.width);
      m.pa = 0.5 * erfc(-a / kSqrt2);
      m.qb = 0.5 * erfc(b / kSqrt2);
      m.z = (1.0 - m.qb) - m.pa;
    } else if (m.kind == BW) {
      m.h = 0.5 * m.width;
      m.h2 = m.h * m.h;
      m.ta = atan((0.0 - m.loc) / m.h);
      const double tb = atan((1.0 - m.loc) / m.h);
      m.th = tb - m.ta;
      m.fa = atan2(m.h, m.loc);
      m.fb = atan2(m.h, 1.0 - m.loc);
      m.ls = (float)(1.0 / m.h);
      m.lb = (float)(-m.loc / m.h);
    }
    j.cmap64[t] = m;
    DimMap<float> f{};
    f.kind = m.kind;
    f.loc = (float)m.loc;
    f.width = (float)m.width;
    f.inv_w = (float)m.inv_w;
    f.pa = (float)m.pa;
    f.qb = (float)m.qb;
    f.z = (float)m.z;
    f.h = (float)m.h;
    f.h2 = (float)m.h2;
    f.ta = (float)m.ta;
    f.th = (float)m.th;
    f.fa = (float)m.fa;
    f.fb = (float)m.fb;
    f.ga = (float)m.ga;
    f.gb = (float)m.gb;
    f.hb = m.hb;
    f.hs = m.hs;
    f.lb = m.lb;
    f.ls = m.ls;
    j.cmap32[t] = f;
  }
  const uint32_t gmask = (uint32_t)__ballot(on && m.kind == GAUSS);
  const uint32_t bmask = (uint32_t)__ballot(on && m.kind == BW);
  const uint32_t all = d == 32 ? ~0u : (1u << d) - 1u;
  const bool lin = gmask == all;
  // one width on every axis: the centres m_0..m_{d-1}, then ga^2, in place of
  // the density-kernel constants (ga, gb) on a Gaussian axis, (m, h^2) on a
  // Breit-Wigner one, 0 on a flat one
  const double ga0 = __shfl(m.ga, 0);
  const bool iso = lin && __ballot(on && m.ga != ga0) == 0;
  if (on) {
    const bool bw = m.kind == BW;
    auto put = [&](int at, double v64, float v32) {
      if (j.prec == 1) {
        chan_constants<float>(j.crec, c, d)[at] = v32;
        chan_constants<float>(j.t_crec, c, d)[at] = v32;
      } else {
        chan_constants<double>(j.crec, c, d)[at] = v64;
        chan_constants<double>(j.t_crec, c, d)[at] = v64;
      }
    };
    if (iso) {
      const double s2 = ga0 * ga0, v = lane == 0 ? s2 : 0.0;
      put(lane, m.loc, (float)m.loc);
      put(d + lane, v, (float)v);
    } else {
      put(2 * lane, bw ? m.loc : m.ga, bw ? (float)m.loc : (float)m.ga);
      put(2 * lane + 1, bw ? m.h2 : m.gb, bw ? (float)m.h2 : (float)m.gb);
    }
    j.hab[2 * t] = lin ? m.hs : m.ls;
    j.hab[2 * t + 1] = lin ? m.hb : m.lb;
  }
  const int nb = __popc(bmask);
  const bool pair = gmask == 0 && nb >= 1 && nb <= 2;
  if (pair && on && m.kind == BW && j.prec == 0) {
    const int i = 2 * __popc(bmask & ((1u << lane) - 1u));
    for (char* rec : {j.crec, j.t_crec}) {
      char* r = reinterpret_cast<char*>(chan_head<double>(rec, c, d));
      PairCon* pc = reinterpret_cast<PairCon*>(r + chan_pair_at<double>(d));
      pc->c[i] = m.loc;
      pc->c[i + 1] = m.h2;
      pc->h[i] = m.ls;
      pc->h[i + 1] = m.lb;
    }
  }
  const double factor = m.kind == GAUSS ? kInvSqrt2Pi / (m.width * m.z) : m.kind == BW ? m.h / m.th : 1.0;
  const double norm = axis_product(1.0, factor, on && m.kind != FLAT, d);
  const int twin = j.twin_peak[c];
  const double tn = twin >= 0 ? peak_norm(j, twin, lane) : 0.0;
  if (lane == 0) {
    j.cnorm64[c] = norm;
    j.cnorm32[c] = (float)norm;
    j.alpha[c] = 1.0 / (double)j.K;
    const ChanType ct{iso ? 1 : 0, gmask, bmask, lin ? 1 : 0};
    j.ctype[c] = ct;
    const int kind = (iso ? kChanIso : 0) | (lin ? kChanLin : 0) | (pair ? kChanPair : 0);
    for (char* rec : {j.crec, j.t_crec}) {
      if (j.prec == 1) set_head<float>(rec, c, d, gmask, bmask, kind, (float)tn);
      else set_head<double>(rec, c, d, gmask, bmask, kind, tn);
    }
  }
  const int n = j.n, ne = d * (n + 1);
  for (int q = lane; q < ne; q += 64) {
    const double e = (double)(q % (n + 1)) / (double)n;
    j.edges[(size_t)c * ne + q] = j.prec == 1 ? (double)(float)e : e;
  }
}

// Channel-mask coefficients (mcv_mask.h): thread (c, f) writes feature f of
// channel c, and thread (c, 0) the offset and factor of c's threshold.  The
// pass rules channel c out where the scaled product, less its error, shows
// S_c + e >= E_c, E_c the larger skip exponent (set_skip_exponents) raised by
// the largest Breit-Wigner factor: 2^-s (S - C + e) >= (E + eps - C) 2^-s,
// with eps the error bound below.
__global__ void k_setup_mask(JobDev j, MaskForm F) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  const int NF = 16 * F.steps;
  const int Kp = (j.K + 31) & ~31;
  if (t >= Kp * NF) return;
  const int c = t / NF, f = t - c * NF;
  double big = 0.0, sum = 0.0, lin = 0.0, C = 0.0, mine = 0.0, lb = 0.0, amin = 0.0;
  int ng = 0;
  if (c < j.K) {
    for (int k = 0; k < j.d; ++k) {
      const DimMap<double>& m = j.cmap64[(size_t)c * j.d + k];
      if (m.kind == BW) lb -= log2(m.h2);
      if (m.kind != GAUSS) continue;
      if (ng == 0 || m.ga < amin) amin = m.ga;
      ++ng;
    }
    for (int k = 0; k < j.d; ++k) {
      const DimMap<double>& m = j.cmap64[(size_t)c * j.d + k];
      if (m.kind != GAUSS) continue;
      // z' = ga q + g, with the smallest ga on every axis in the short form
      // (a width that all axes share is that one exactly)
      const double ga = F.axes > 0 ? m.ga : amin;
      const double g = F.axes > 0 ? m.gb + 0.5 * m.ga : amin * (0.5 - m.loc);
      const double A = ga * ga, B = 2.0 * ga * g;
      big = fmax(big, fmax(A, fabs(B)));
      sum += 0.25 * A + 0.5 * fabs(B) + g * g;
      lin += A + fabs(B);
      C += g * g;
      if (f == k) mine = B;
      if (F.axes > 0 ? f == F.q2 + k : f == F.q2) mine = A;
    }
  }
  int s = 0;  // scale the largest coefficient to at most 2^10
  while (s < 64 && big > ldexp(1.0, 10 + s)) ++s;
  const double sc = ldexp(1.0, -s);
  if (f == F.e) mine = 1.0;
  const int tile = c >> 5, step = f >> 4, h = (f >> 3) & 1;
  const size_t at = ((((size_t)tile * F.steps + step) * 64) + h * 32 + (c & 31)) * 8 + (f & 7);
  // the FP16 range: e's coefficient 2^-s must be a normal number
  const bool usable = (F.axes > 0 ? ng > 0 : ng == j.d) && s <= 14;
  ((_Float16*)j.mco)[at] = usable ? (_Float16)(float)(mine * sc) : (_Float16)0.0f;
  if (f == 0) {
    // Rounding of the product: q to 11 bits toward zero (2^-10 of |q| <=
    // 1/2), q^2 or their sum the same (of 1/4 an axis), the coefficients to
    // the nearest of 11 bits (2^-11), the FP32 sums (below 2^-18), and what
    // is flushed below 2^-14: at most 1.5 2^-10 of the sums of magnitudes,
    // taken as 2^-9 (the rest covers the rounding of the kernel's own
    // exponent), plus 2^-14 of the coefficients and of one per feature.
    const double eps = 0x1p-9 * sum + 0x1p-14 * lin + 2.0 * j.d * 0x1p-14 / sc + 0.5;
    const bool on = c < j.K && usable;
    j.moff[2 * c] = on ? (float)(eps - C + (lb > 0.0 ? lb : 0.0) + 1.0) : 0.0f;
    j.moff[2 * c + 1] = on ? (float)sc : 0.0f;
    if (c >= j.K) j.mthr[c] = -INFINITY;  // no such channel: always ruled out
  }
}

// Rounds one axis to FP32 and keeps it strictly increasing (forward, then
// backward) -- the mixed-precision grid.
__device__ void snap_axis32(int n, double* e) {
  e[0] = 0.0;
  e[n] = 1.0;
  for (int i = 1; i < n; ++i) {
    float f = (float)e[i];
    const float prev = (float)e[i - 1];
    if (!(f > prev)) f = nextafterf(prev, 2.0f);
    e[i] = (double)f;
  }
  for (int i = n - 1; i >= 1; --i) {
    float f = (float)e[i];
    const float next = (float)e[i + 1];
    if (!(f < next)) f = nextafterf(next, -1.0f);
    e[i] = (double)f;
  }
}

// What the passes read of one axis, from its master edges e[0..n] in LDS: the
// (edge, density) tables (eq. g(x): the density of bin j is 1/(n Delta_j)) in
// x space for the forward map and in p space, P_j = phi(X_j), for the other
// channels' bin search; the hint cells; and the axis' largest density.  Every
// thread of the workgroup takes part; P: scratch of n + 1 entries.
//
// Hint cells: for cell c of an axis, the start bin J (interior edges with a
// lower cell) and, when at most one interior edge falls into the cell, that
// edge and the densities of the bins on either side.  The cell map is
// monotone, so every edge of a lower (higher) cell lies below (above) any x
// of the cell, and the cells of the interior edges do not decrease: the edges
// below a cell and in it are two binary searches over the edges' cells.
constexpr int kAxisBlock = 256;

// Threads per axis: 256 while every axis' workgroup is resident at once (the
// hint cells are the longest loop); beyond, one wavefront, since the serial
// sums leave the others idle and eight 256-thread workgroups fill a CU (48
// jobs of up to 64 channels and 12 axes, FP64, 50 bins: 86 -> 53 us).
inline int axis_block(const JobSet& js) {
  return (int64_t)js.maxKd * js.n <= 8 * 256 ? kAxisBlock : 64;
}

template <typename T>
__device__ void axis_tables(const JobDev& j, int ax, const double* e, Pair<T>* P, uint16_t* cells,
                            double* wmax) {
  const int n = j.n, sT = j.sT, M = j.M, tid = threadIdx.x;
  const DimMap<double>* m = j.cmap64 + ax;
  Pair<T>* X = (Pair<T>*)j.xtab + (size_t)ax * sT;
  Pair<T>* Pg = (Pair<T>*)j.ptab + (size_t)ax * sT;
  const bool log_map = !j.ctype[ax / j.d].lin;  // the map the lookups of this channel use
  const float ha = j.hab[2 * ax], hb = j.hab[2 * ax + 1];
  double mx = 0.0;
  for (int i = tid; i < sT; i += blockDim.x) {
    const T dens = (i < n) ? (T)(1.0 / ((double)n * (e[i + 1] - e[i]))) : T(0);
    X[i] = Pair<T>{i <= n ? (T)e[i] : T(1), dens};
    T pe;
    if (i == 0) pe = (T)-INFINITY;
    else if (i >= n) pe = (T)INFINITY;
    else pe = (T)map_forward<double>(m, e[i], 1.0 - e[i]);
    Pg[i] = Pair<T>{pe, dens};
    if (i <= n) {
      P[i] = Pair<T>{pe, dens};
      if (i >= 1 && i < n) cells[i] = (uint16_t)hint_cell<T>(ha, hb, pe, log_map, M, j.mshift);
    }
    mx = fmax(mx, (double)dens);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
  if ((tid & 63) == 0) wmax[tid >> 6] = mx;
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < (int)blockDim.x / 64; ++w) mx = fmax(mx, wmax[w]);
    j.axmax[ax] = mx;
  }
  Cell<T>* C = (Cell<T>*)j.ctab + (size_t)ax * M;
  for (int c = tid; c < M; c += blockDim.x) {
    int lo = 1, hi = n;
    while (lo < hi) {  // first edge whose cell is >= c (n if none)
      const int mid = (lo + hi) >> 1;
      if ((int)cells[mid] < c) lo = mid + 1;
      else hi = mid;
    }
    const int lb = lo;
    hi = n;
    while (lo < hi) {  // first edge whose cell is > c
      const int mid = (lo + hi) >> 1;
      if ((int)cells[mid] <= c) lo = mid + 1;
      else hi = mid;
    }
    const int below = lb - 1, inside = lo - lb;
    Cell<T> r;
    r.J = (T)below;
    if (inside > 1) {
      // a crowded cell: the exact lookup walks from J over the bins J ..
      // J + inside; without the walk it reads dhi, the largest of their
      // densities (an upper bound), and the sign of dlo marks the cell
      T big = P[below].dens;
      for (int b = below + 1; b <= below + inside; ++b) big = big > P[b].dens ? big : P[b].dens;
      r.e = T(0);
      r.dlo = -big;
      r.dhi = big;
    } else if (inside == 0) {
      r.e = (T)INFINITY;
      r.dlo = P[below].dens;
      r.dhi = r.dlo;
    } else {
      r.e = P[lb].e;
      r.dlo = P[lb - 1].dens;
      r.dhi = P[lb].dens;
    }
    C[c] = r;
  }
}

// LDS of the per-axis kernels.
struct AxisShared {
  double es[257], out[257], m[256];
  union {
    double pre[257];        // until the new edges are placed
    Pair<double> P[257];
  };
  double wmax[kAxisBlock / 64];
  double sum;
  uint16_t cells[257];
};

// The same for every axis from the master edges as they are (set-up, a state
// loaded or injected).  One workgroup per axis; grid row y = job.
template <typename T>
__global__ __launch_bounds__(kAxisBlock) void k_tables(const JobDev* jobs) {
  __shared__ AxisShared sh;
  const JobDev& j = jobs[blockIdx.y];
  const int ax = blockIdx.x;
  if (ax >= j.K * j.d) return;  // uniform over the workgroup
  for (int i = threadIdx.x; i <= j.n; i += blockDim.x) sh.es[i] = j.edges[(size_t)ax * (j.n + 1) + i];
  __syncthreads();
  axis_tables<T>(j, ax, sh.es, reinterpret_cast<Pair<T>*>(sh.P), sh.cells, sh.wmax);
}

// Per-channel bound of the channel terms of g(p) (eq. g(p)) for the sample
// pass: gbound_c = 2^s (1 + m) cnorm_c prod_k max_j dens_kj, rounded up to
// the pass precision, with s = 25, m = 2^-16 in FP32 and s = 54, m = 2^-40 in
// FP64.  m covers the roundings of the term (at most d + 4 of the pass
// precision) and of this product, so (alpha_c gbound_c) r_c evaluated in the
// pass precision is at least 2^s times the term alpha_c cnorm_c G_c r_c as the
// pass evaluates it.  The same holds with any upper bounds of the looked-up
// densities in place of the maxima (the factor bound_factor(alpha_c cnorm_c)
// written with the allocation).
template <typename T>
__device__ T bound_factor(double g) {
  if constexpr (sizeof(T) == 4) {
    g *= 0x1p25 * (1.0 + 0x1p-16);
    float f = (float)g;
    if ((double)f < g) f = nextafterf(f, INFINITY);
    return f;
  } else {
    return g * (0x1p54 * (1.0 + 0x1p-40));
  }
}

template <typename T>
__device__ T channel_bound(const JobDev& j, int c) {
  double g = sizeof(T) == 4 ? (double)j.cnorm32[c] : j.cnorm64[c];
  for (int k = 0; k < j.d; ++k) g *= j.axmax[(size_t)c * j.d + k];
  return bound_factor<T>(g);
}

// ---------------------------------------------------------------------------
// Allocation (Sec. 3.4): N_c = floor(alpha_c N), floor min_calls, the
// remainder to the largest fractional parts (ties to the lower channel);
// N_tot = sum N_c; alpha_c = N_c / N_tot.  One wavefront per job (workgroup
// x = job), the same IEEE operations per channel as a serial host
// implementation.  Handing the remainder out one call at a time to the
// largest fraction not yet served (all served: a new round) gives channel c
// floor(rem / K) calls plus one if its rank -- the channels with a larger
// fraction, or an equal one and a lower index -- is below rem mod K; the
// kernel computes that rank per channel.  N is n_override if positive, else
// the job's own calls per pass.  to_trace:
// the result goes to the trace allocation and alpha is left alone.  Also
// writes the partial-exponent skip offsets for the resulting weights and
// resets the 8 work-queue counters of the following sample pass.
// ---------------------------------------------------------------------------
// floor(log2 x) of a positive finite x; -100000 for 0, +100000 otherwise.
__device__ inline int floor_log2(double x) {
  if (x == 0.0) return -100000;
  if (!(x > 0.0) || !isfinite(x)) return 100000;
  int e = 0;
  (void)frexp(x, &e);
  return e - 1;
}

// Exponent offsets of the partial-exponent skip (all-Gaussian channels of
// the sample pass), from the pass-precision values the pass multiplies: the
// twin factor tw (the channel's term of f is tw r) and alpha gbound (the
// term of g is at most alpha gbound r 2^-s).  With r <= 2^(1 - floor(S)) for
// a partial exponent sum S, the term of f is below 2^(ex(tw) + 3 - floor(S))
// and must be at most 2^(ex(f) - P - 1) (half an ulp, P = 24 or 53, with a
// margin of 2), so EA = ex(tw) + P + 4; likewise EB = ex(alpha) + ex(gbound)
// + 4 - s + P.  A zero twin factor never blocks the skip.  alpha: the
// allocation's channel weights the pass will use.
__device__ inline void skip_exponents(bool f32, double tw, double a, double gb, int* ea, int* eb) {
  const int P = f32 ? 24 : 53, s = f32 ? 25 : 54;
  *ea = tw == 0.0 ? -100000 : floor_log2(tw) + P + 4;
  const int la = floor_log2(a), lg = floor_log2(gb);
  *eb = (la >= 100000 || lg >= 100000) ? 100000 : la + lg + 4 - s + P;
}

// What the passes read of channel c that depends on its weight a: the factors
// of its terms in the pass precision, the skip offsets and its mask threshold.
template <typename T>
__device__ inline void set_channel_weight(const JobDev& j, char* rec, int c, double a) {
  const T cnorm = sizeof(T) == 4 ? (T)j.cnorm32[c] : (T)j.cnorm64[c];
  const T gb = channel_bound<T>(j, c);
  ChanHead<T>* h = chan_head<T>(rec, c, j.d);
  h->bound = (T)a * gb;
  h->term = (T)a * cnorm;
  h->look = bound_factor<T>(a * (double)cnorm);
  int ea, eb;
  skip_exponents(sizeof(T) == 4, (double)h->twin, (double)(T)a, (double)gb, &ea, &eb);
  h->ea = (int16_t)max(min(ea, 32000), -32000);  // beyond every exponent sum
  h->eb = (int16_t)max(min(eb, 32000), -32000);
  if (j.masked) {
    const float sc = j.moff[2 * c + 1];
    const float E = (float)(ea > eb ? ea : eb);
    j.mthr[c] = sc > 0.0f && E < 100000.0f ? (E + j.moff[2 * c]) * sc : INFINITY;
  }
}

// Stratified layout of a channel with n calls in d dimensions, at least
// s_min calls per box (Sec. 3.3): nr = the largest integer with s_min nr^d
// <= n (at most 2^20) boxes per axis, and floor(n / nr^d) calls per box.
__device__ inline void strat_layout(int64_t n, int d, int64_t s_min, int64_t* nr,
                                    int64_t* per_box, int64_t* boxes_out) {
  int64_t r = 1;
  for (;;) {
    const int64_t r1 = r + 1;
    if (r1 > ((int64_t)1 << 20)) break;
    int64_t boxes = 1;
    bool over = false;
    for (int k = 0; k < d && !over; ++k) {
      if (boxes > n / r1) over = true;
      else boxes *= r1;
    }
    if (over || boxes > n / s_min) break;
    r = r1;
  }
  int64_t boxes = 1;
  for (int k = 0; k < d; ++k) boxes *= r;
  *nr = r;
  *per_box = n / boxes;
  *boxes_out = boxes;
}

constexpr int kAllocMaxK = 1024;  // the channel limit of the interface

__global__ __launch_bounds__(64) void k_allocate(const JobDev* jobs, int64_t n_override,
                                                 int to_trace, int* counter) {
  __shared__ double frac[kAllocMaxK];
  __shared__ int64_t ncs[kAllocMaxK];
  const int tid = threadIdx.x;
  if (counter && blockIdx.x == 0 && tid < 8) counter[tid] = 0;  // the 8 unit queues
  const JobDev& j = jobs[blockIdx.x];
  const int K = j.K;
  const int64_t N = n_override > 0 ? n_override : j.n_points;
  const int64_t min_calls = j.min_calls;
  const double* alpha_in = j.alpha;
  int64_t* nc = to_trace ? j.t_nc : j.nc;
  int64_t* start = to_trace ? j.t_start : j.start;
  double* alpha_out = to_trace ? j.t_alpha : j.alpha;
  int64_t part = 0;
  for (int c = tid; c < K; c += 64) {
    const double v = alpha_in[c] * (double)N;
    const double fl = floor(v);
    int64_t b = (int64_t)fl;
    double fr = v - fl;
    if (b < min_calls) {
      b = min_calls;
      fr = -1.0;
    }
    frac[c] = fr;
    ncs[c] = b;
    part += b;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
  __syncthreads();
  const int64_t rem = N - part;  // every lane holds the sum
  if (rem > 0) {
    const int64_t q = rem / K, r = rem % K;
    for (int c = tid; c < K; c += 64) {
      const double fc = frac[c];
      int rank = 0;
      for (int c2 = 0; c2 < K; ++c2) {
        const double f2 = frac[c2];
        rank += (f2 > fc || (f2 == fc && c2 < c)) ? 1 : 0;
      }
      ncs[c] += q + (rank < r ? 1 : 0);
    }
  }
  __syncthreads();
  int64_t* nrv = to_trace ? j.t_nr : j.nr;
  int64_t* spbv = to_trace ? j.t_spb : j.spb;
  // offsets by scans of 64 channels at a time
  int64_t acc = 0, bacc = 0;
  for (int c0 = 0; c0 < K; c0 += 64) {
    const int c = c0 + tid;
    int64_t v = c < K ? ncs[c] : 0, boxes = 0;
    if (j.strat > 0) {
      // pseudo-stratified passes take whole boxes: N_c = calls per box x
      // boxes (Sec. 3.3 fixes N = s n^d; Sec. 3.4 lets N and alpha follow
      // whole numbers of calls)
      if (c < K) {
        strat_layout(v, j.d, j.strat, &nrv[c], &spbv[c], &boxes);
        v = spbv[c] * boxes;
        ncs[c] = v;
      }
      int64_t t = boxes;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const int64_t o = __shfl_up(t, off);
        if (tid >= off) t += o;
      }
      if (!to_trace && c < K) j.bstart[c + 1] = bacc + t;
      bacc += __shfl(t, 63);
    }
    int64_t t = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int64_t o = __shfl_up(t, off);
      if (tid >= off) t += o;
    }
    if (c < K) start[c + 1] = acc + t;
    acc += __shfl(t, 63);
  }
  if (tid == 0) {
    start[0] = 0;
    if (j.strat > 0 && !to_trace) j.bstart[0] = 0;
  }
  const double tot = (double)acc;
  for (int c = tid; c < K; c += 64) {
    nc[c] = ncs[c];
    alpha_out[c] = (double)ncs[c] / tot;
  }
  char* rec = to_trace ? j.t_crec : j.crec;
  for (int c = tid; c < K; c += 64) {
    const double a = (double)ncs[c] / tot;
    if (j.prec == 1) set_channel_weight<float>(j, rec, c, a);
    else set_channel_weight<double>(j, rec, c, a);
  }
}

// ---------------------------------------------------------------------------
// Finalize (Sec. 3.1 E_N and V_N per channel; Sec. 3.4 multi-channel
// estimator): the segment partials of each channel and the per-bin
// histograms, in a fixed order; deterministic.  The pass of
// a job was split into G units: from the unit prefix of a job table, or the
// single job's G.
// ---------------------------------------------------------------------------
__device__ inline int64_t seg_of(int64_t i, int G, int64_t ntot) {
  return ((i + 1) * (int64_t)G - 1) / ntot;
}

// A channel's segment slots are summed in chunks: S chunks of the channel's
// slots where it has many (S from the job's own units and channels, so that
// its sums do not depend on the other jobs), each to the chunk's first slot,
// so that a pass of many units is read by the whole chip (12207 units, 32
// channels, 1000 bins: 100 MB by 32 workgroups took 113 us).
constexpr int kChunkSlots = 24;   // slots of a chunk, at least
constexpr int kMaxChunks = 16;

__device__ __host__ inline int slot_chunks(int64_t G, int K) {
  const int64_t s = G / ((int64_t)K * kChunkSlots);
  return s < 1 ? 1 : s > kMaxChunks ? kMaxChunks : (int)s;
}

struct Slots {
  int G, S;         // units, chunks per channel
  int64_t g0, g1;   // the channel's slots are g + c, g0 <= g < g1
};

__device__ inline Slots channel_slots(const JobDev& j, int c, const int* unit_prefix, int G1) {
  Slots r;
  r.G = unit_prefix ? unit_prefix[blockIdx.y + 1] - unit_prefix[blockIdx.y] : G1;
  // the pass split the calls (or, stratified, the boxes) into G units, at most
  // one for each: with more, units between two calls of a channel would be
  // empty and leave their slots as an earlier pass wrote them
  const int64_t* st = j.strat > 0 ? j.bstart : j.start;
  const int64_t ntot = st[j.K];
  if (r.G > ntot) r.G = (int)ntot;
  r.S = slot_chunks(r.G, j.K);
  r.g0 = seg_of(st[c], r.G, ntot);
  r.g1 = seg_of(st[c + 1] - 1, r.G, ntot) + 1;
  return r;
}

__global__ __launch_bounds__(256) void k_sum_chunks(const JobDev* jobs, const int* unit_prefix,
                                                    int G1) {
  const JobDev& j = jobs[blockIdx.y];
  const int c = blockIdx.x / kMaxChunks, s = blockIdx.x % kMaxChunks;
  if (c >= j.K) return;
  const Slots sl = channel_slots(j, c, unit_prefix, G1);
  if (sl.S == 1 || s >= sl.S) return;
  const int64_t ns = sl.g1 - sl.g0;
  const int64_t a = sl.g0 + ns * s / sl.S, b = sl.g0 + ns * (s + 1) / sl.S;
  if (b - a < 2) return;
  const int dn = j.d * j.n;
  // the reads of 8 slots are issued together; the additions keep slot order
  constexpr int kAhead = 8;
  for (int t = threadIdx.x; t < dn; t += 256) {
    double* col = j.hpart + (size_t)(a + c) * dn + t;
    const int m = (int)(b - a);
    double h = 0.0;
    int g = 0;
    for (; g + kAhead <= m; g += kAhead) {
      double v[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) v[u] = col[(size_t)(g + u) * dn];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) h += v[u];
    }
    for (; g < m; ++g) h += col[(size_t)g * dn];
    col[0] = h;
  }
}

// Channel c's statistics and per-bin sums; the last workgroup of a job to
// finish its channel's statistics forms the pass's total.
constexpr int kFinBlock = 512;

__global__ __launch_bounds__(kFinBlock) void k_finalize(const JobDev* jobs,
                                                        const int* unit_prefix, int G1) {
  __shared__ double sts[kAllocMaxK][3];
  __shared__ int last_s;
  const JobDev& j = jobs[blockIdx.y];
  const int c = blockIdx.x, tid = threadIdx.x;
  if (c >= j.K) return;
  const Slots sl = channel_slots(j, c, unit_prefix, G1);
  const bool strat = j.strat > 0;
  // the records: a lane of the first wavefront takes every 64th slot, then
  // butterflies of error-free sums
  if (tid < 64) {
    Neu s1{0.0, 0.0}, s2{0.0, 0.0}, sq{0.0, 0.0};
    double wmax = 0.0, nbad = 0.0;
    for (int64_t g = sl.g0 + tid; g < sl.g1; g += 64) {
      const double* r = j.part + (size_t)(g + c) * kPartStride;
      s1.add(r[0]);
      s1.add(r[1]);
      s2.add(r[2]);
      s2.add(r[3]);
      wmax = fmax(wmax, r[4]);
      nbad += r[5];
      if (strat) sq.add(r[6]);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      s1 = neu_merge(s1, Neu{__shfl_xor(s1.s, off), __shfl_xor(s1.c, off)});
      s2 = neu_merge(s2, Neu{__shfl_xor(s2.s, off), __shfl_xor(s2.c, off)});
      if (strat) sq = neu_merge(sq, Neu{__shfl_xor(sq.s, off), __shfl_xor(sq.c, off)});
      wmax = fmax(wmax, __shfl_xor(wmax, off));
      nbad += __shfl_xor(nbad, off);
    }
    if (tid == 0) {
      const double N = (double)j.nc[c];
      const double S1 = s1.s + s1.c, S2 = s2.s + s2.c;
      const double E = S1 / N, W = S2 / N;
      double V;
      if (strat) {
        // stratified: Var(S1) = sum over boxes of m sigma_b^2, estimated by
        // m/(m-1) sum_b SSW_b with SSW_b the squared deviations of the box's
        // weights from its mean (slot word 6); V = that / N
        const double m = (double)j.spb[c];
        const double v = (m / (m - 1.0)) * (sq.s + sq.c) / N;
        V = v > 0.0 ? v : 0.0;
      } else {
        const double v = W - E * E;
        V = (j.nc[c] > 1) ? (v > 0.0 ? v : 0.0) * N / (N - 1.0) : 0.0;
      }
      double* st = j.chstats + (size_t)c * kStatStride;
      const double rec[kStatStride] = {S1, S2, wmax, nbad, E, W, V, N};
#pragma unroll
      for (int q = 0; q < kStatStride; ++q)
        __hip_atomic_store(st + q, rec[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      // The record goes past the caches by its agent-scope stores; once they
      // are complete (the wait) the ticket says so.  A release fence would
      // write back all that this XCD's L2 holds, in every workgroup.
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      const int done = __hip_atomic_fetch_add(j.ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      last_s = done == j.K - 1;
      if (last_s) __hip_atomic_store(j.ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  // the per-bin sums, rows of slots (or chunk heads) in order
  const int dn = j.d * j.n;
  const int64_t ns = sl.g1 - sl.g0;
  const int rows = sl.S > 1 ? sl.S : (int)ns;
  constexpr int kAhead = 8;
  for (int t = tid; t < dn; t += kFinBlock) {
    const double* col = j.hpart + (size_t)(sl.g0 + c) * dn + t;
    double h = 0.0;
    if (sl.S > 1) {
      // an empty chunk (fewer slots than chunks) adds nothing
      double v[kMaxChunks];
#pragma unroll
      for (int r = 0; r < kMaxChunks; ++r) {
        const int64_t p = ns * r / sl.S, q = ns * (r + 1) / sl.S;
        v[r] = r < sl.S && p < q ? col[(size_t)p * dn] : 0.0;
      }
#pragma unroll
      for (int r = 0; r < kMaxChunks; ++r) h += v[r];
    } else {
      int r = 0;
      for (; r + kAhead <= rows; r += kAhead) {
        double v[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) v[u] = col[(size_t)(r + u) * dn];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) h += v[u];
      }
      for (; r < rows; ++r) h += col[(size_t)r * dn];
    }
    j.hist[(size_t)c * dn + t] = h;
  }
  __syncthreads();
  if (!last_s) return;
  // Total estimate, error sqrt(sum_c (N_c/N)^2 V_c / N_c) and the history
  // record of the pass, at row *iter_dev, which then counts the pass.  A full
  // history is left untouched (the host rejects such a pass beforehand).  The
  // terms a channel per lane, the sums in channel order.
  const int iter = *j.iter_dev;
  if (iter < 0 || iter >= j.max_iter) return;  // uniform
  const double ntot = (double)j.start[j.K];
  double wmax = 0.0;
  for (int cc = tid; cc < j.K; cc += kFinBlock) {
    double st[kStatStride];
#pragma unroll
    for (int q = 0; q < kStatStride; ++q)
      st[q] = __hip_atomic_load(j.chstats + (size_t)cc * kStatStride + q, __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
    const double N = st[7], fr = N / ntot;
    sts[cc][0] = st[0];
    sts[cc][1] = fr * fr * st[6] / N;
    sts[cc][2] = st[3];
    wmax = fmax(wmax, st[2]);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) wmax = fmax(wmax, __shfl_xor(wmax, off));
  __shared__ double wm[kFinBlock / 64];
  if ((tid & 63) == 0) wm[tid >> 6] = wmax;
  __syncthreads();
  if (tid != 0) return;
  double e = 0.0, var = 0.0, nbad = 0.0;
#pragma unroll 8
  for (int cc = 0; cc < j.K; ++cc) {
    e += sts[cc][0];
    var += sts[cc][1];
    nbad += sts[cc][2];
  }
  for (int w = 1; w < kFinBlock / 64; ++w) wmax = fmax(wmax, wm[w]);
  double* h = j.history + (size_t)iter * kHistStride;
  h[0] = e / ntot;
  h[1] = sqrt(var);
  h[2] = ntot;
  h[3] = wmax;
  h[4] = nbad;
  *j.iter_dev = iter + 1;
}

// ---------------------------------------------------------------------------
// Channel equivalences (Sec. 3.5: the bin weights of channels that share a
// structure are combined, with a permutation of the axes and an identity,
// invert, symmetric or invariant mapping, before rebinning).  The bin
// weights are the per-bin sums of w^2 (eq. 31).  A channel named on the left
// of any equivalence (c, c', perm, mode) gets the sum of its equivalences in
// list order, from zero (its own sums enter through an entry (c, c,
// identity)); per axis k, channel c' contributes its axis perm[k] as is
// (identity), mirrored, j -> n-1-j (invert), or as the mean of both
// (symmetric); an invariant axis gets weight 1 in every bin (its grid is
// kept).  Other channels keep their own sums.  One workgroup per (channel,
// axis) of a job (grid row y = job), one bin per lane; the additions of a
// bin run in list order.
// ---------------------------------------------------------------------------
constexpr int kEqIdentity = 0, kEqInvert = 1, kEqSymmetric = 2;

__global__ void k_equivalences(const JobDev* jobs) {
  const JobDev& j = jobs[blockIdx.y];
  const int ax = blockIdx.x;
  if (j.n_eq == 0 || ax >= j.K * j.d) return;  // uniform over the workgroup
  if (*j.iter_dev >= j.adapt_passes) return;
  const int d = j.d, n = j.n, rec = 2 + 2 * d;
  const int c = ax / d, k = ax - c * d;
  bool listed = false, invariant = false;
  for (int e = 0; e < j.n_eq; ++e) {
    const int32_t* r = j.eq + (size_t)e * rec;
    if (r[0] != c) continue;
    listed = true;
    invariant |= r[2 + d + k] > kEqSymmetric;
  }
  for (int b = threadIdx.x; b < n; b += blockDim.x) {
    double w = listed ? 0.0 : j.hist[(size_t)ax * n + b];
    for (int e = 0; e < j.n_eq; ++e) {
      const int32_t* r = j.eq + (size_t)e * rec;
      if (r[0] != c) continue;
      const double* h2 = j.hist + ((size_t)r[1] * d + r[2 + k]) * n;
      const int mode = r[2 + d + k];
      if (mode == kEqIdentity) w += h2[b];
      else if (mode == kEqInvert) w += h2[n - 1 - b];
      else if (mode == kEqSymmetric) w += 0.5 * (h2[b] + h2[n - 1 - b]);
    }
    j.hist_eq[(size_t)ax * n + b] = invariant ? 1.0 : w;
  }
}

// ---------------------------------------------------------------------------
// Grid refinement (eq. 30, eq. 31), then the axis' tables: one workgroup per
// (channel, dim) of a job (grid row y = job).  The per-bin measures are
// computed in parallel; lane 0 does the ordered sums and the walk, over the
// edges staged in LDS, so that the result is the serial IEEE sequence.  One
// launch (four before: rebinning, tables, cells, bounds; each a launch and a
// pass over L2 that a small job waits for).
// ---------------------------------------------------------------------------
template <typename T>
__device__ void refine_axis(const JobDev& j, int ax, AxisShared& sh) {
  double *m = sh.m, *out = sh.out, *es = sh.es, *pre = sh.pre;
  double* om = m;  // the roots, until the weights of eq. 30 take their place
  const int n = j.n, tid = threadIdx.x;
  double* e = j.edges + (size_t)ax * (n + 1);
  const double* h = (j.n_eq > 0 ? j.hist_eq : j.hist) + (size_t)ax * n;
  for (int i = tid; i < n; i += blockDim.x) om[i] = sqrt(h[i]);
  for (int i = tid; i <= n; i += blockDim.x) es[i] = e[i];  // the walk reads LDS
  __syncthreads();
  if (tid == 0) {  // the ordered sum
    double sum = 0.0;
#pragma unroll 8
    for (int i = 0; i < n; ++i) sum += om[i];
    sh.sum = sum;
  }
  __syncthreads();
  const double sum = sh.sum;
  if (!(sum > 0.0) || !isfinite(sum)) return;  // nothing to adapt to (uniform)
  const double a = j.grid_power;
  // the per-bin weights of eq. 30 are independent: one bin per lane
  for (int i = tid; i < n; i += blockDim.x) {
    const double r = om[i] / sum;
    double v;
    if (r == 0.0) v = 0.0;
    else if (r == 1.0) v = 1.0;
    else v = pow((r - 1.0) / log(r), a);
    m[i] = v;
  }
  __syncthreads();
  // The serial walk: for new edge i, target = i M / n with M the ordered sum
  // of the m; acc runs through the ordered prefix sums S_b while m_b = 0 or
  // S_{b+1} < target, and the edge is interpolated in bin b.  Its stop is
  // the first b with S_{b+1} >= target (m_b > 0 there, S_{b+1} > S_b), else
  // n - 1: lane 0 forms the prefix sums in order, every lane finds its
  // edges' bins by bisection and interpolates with acc = S_b, the walk's
  // operands.
  if (tid == 0) {
    double acc = 0.0;
    pre[0] = 0.0;
#pragma unroll 8
    for (int i = 0; i < n; ++i) {
      acc += m[i];
      pre[i + 1] = acc;
    }
    out[0] = 0.0;
    out[n] = 1.0;
  }
  __syncthreads();
  const double M = pre[n];
  for (int i = tid + 1; i < n; i += blockDim.x) {
    const double target = ((double)i * M) / (double)n;
    int lo = 0, hi = n - 1;  // first b in [0, n - 1) with pre[b + 1] >= target, else n - 1
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (pre[mid + 1] >= target) hi = mid;
      else lo = mid + 1;
    }
    const int b = lo;
    out[i] = es[b] + ((target - pre[b]) / m[b]) * (es[b + 1] - es[b]);
  }
  __syncthreads();
  // The serial fix-ups (edges made strictly increasing forward, then
  // backward; in FP32 the edges rounded and fixed the same way) change
  // nothing when no pair violates them: every lane checks its pairs, and
  // lane 0 runs them only if some pair does.
  bool bad = false;
  for (int i = tid + 1; i < n; i += blockDim.x)
    bad |= !(out[i] > out[i - 1]) || !(out[i] < out[i + 1]);
  if (__syncthreads_or(bad)) {
    if (tid == 0) {
      for (int i = 1; i < n; ++i)
        if (!(out[i] > out[i - 1])) out[i] = nextafter(out[i - 1], 2.0);
      for (int i = n - 1; i >= 1; --i)
        if (!(out[i] < out[i + 1])) out[i] = nextafter(out[i + 1], -1.0);
    }
    __syncthreads();
  }
  if (sizeof(T) == 4) {
    bool bad32 = false;
    for (int i = tid + 1; i < n; i += blockDim.x) {
      const float f = (float)out[i];
      bad32 |= !(f > (float)out[i - 1]) || !(f < (float)out[i + 1]);
    }
    if (__syncthreads_or(bad32)) {
      if (tid == 0) snap_axis32(n, out);
    } else {
      for (int i = tid + 1; i < n; i += blockDim.x) out[i] = (double)(float)out[i];
    }
    __syncthreads();
  }
  for (int i = tid; i <= n; i += blockDim.x) e[i] = out[i];
  axis_tables<T>(j, ax, out, reinterpret_cast<Pair<T>*>(sh.P), sh.cells, sh.wmax);
}

// Channel weights, eq. 15 with omega_c = W_c (second moment of the weights):
// the powers one channel per lane, the normalising sum in channel order by
// one lane, the division per lane (the oracle's operations in its order).
__device__ void update_alpha(const JobDev& j, double* pw, double* den_s) {
  const int K = j.K, tid = threadIdx.x, block = blockDim.x;
  const double beta = j.channel_power;
  for (int c = tid; c < K; c += block) pw[c] = pow(j.chstats[c * kStatStride + 5], beta);
  __syncthreads();
  if (tid == 0) {
    double den = 0.0;
    for (int c = 0; c < K; ++c) den += j.alpha[c] * pw[c];
    *den_s = den;
  }
  __syncthreads();
  const double den = *den_s;
  if (!(den > 0.0) || !isfinite(den)) return;  // uniform
  for (int c = tid; c < K; c += block) j.alpha[c] = j.alpha[c] * pw[c] / den;
}

// One workgroup per axis (grid), and one more per job, the first, for the
// channel weights (alpha).
template <typename T>
__global__ __launch_bounds__(kAxisBlock) void k_refine(const JobDev* jobs, int grid, int alpha) {
  __shared__ union {
    AxisShared ax;
    double pw[kAllocMaxK + 1];
  } sh;
  const JobDev& j = jobs[blockIdx.y];
  if (*j.iter_dev >= j.adapt_passes) return;  // the job's last pass: grids and alpha stay
  int b = blockIdx.x;
  if (alpha) {
    if (b == 0) update_alpha(j, sh.pw, sh.pw + kAllocMaxK);
    --b;
  }
  if (b < 0 || !grid || b >= j.K * j.d) return;
  refine_axis<T>(j, b, sh.ax);
}

}  // namespace

static inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

void set_extents(JobSet& js) {
  js.maxK = js.maxKd = js.maxd = 0;
  js.has_eq = false;
  for (int i = 0; i < js.n; ++i) {
    const JobDev& j = js.host[i];
    js.has_eq |= j.n_eq > 0;
    if (j.K > js.maxK) js.maxK = j.K;
    if (j.K * j.d > js.maxKd) js.maxKd = j.K * j.d;
    if (j.d > js.maxd) js.maxd = j.d;
  }
}

void launch_setup(const JobDev& j, hipStream_t s) {
  hipLaunchKernelGGL(k_setup, dim3(j.K + j.P + zero_groups(j.max_iter)), dim3(64), 0, s, j);
  if (j.masked) {
    const MaskForm F = mask_form_of(j.d);
    hipLaunchKernelGGL(k_setup_mask, dim3(cdiv(((j.K + 31) & ~31) * 16 * F.steps, 256)), dim3(256),
                       0, s, j, F);
  }
}

void launch_tables(const JobSet& js, hipStream_t s) {
  if (js.n < 1) return;
  if (js.prec == 1)
    hipLaunchKernelGGL(k_tables<float>, dim3(js.maxKd, js.n), dim3(axis_block(js)), 0, s, js.dev);
  else
    hipLaunchKernelGGL(k_tables<double>, dim3(js.maxKd, js.n), dim3(axis_block(js)), 0, s, js.dev);
}

void launch_allocate(const JobSet& js, int64_t n_override, bool to_trace, hipStream_t s) {
  if (js.n < 1) return;
  hipLaunchKernelGGL(k_allocate, dim3(js.n), dim3(64), 0, s, js.dev, n_override,
                     to_trace ? 1 : 0, js.counter);
}

void launch_finalize(const JobSet& js, int G, hipStream_t s) {
  if (js.n < 1) return;
  int chunks = 1;
  if (js.unit_prefix) chunks = js.max_chunks;
  else chunks = slot_chunks(G, js.host[0].K);
  if (chunks > 1)
    hipLaunchKernelGGL(k_sum_chunks, dim3(js.maxK * kMaxChunks, js.n), dim3(256), 0, s, js.dev,
                       js.unit_prefix, G);
  hipLaunchKernelGGL(k_finalize, dim3(js.maxK, js.n), dim3(kFinBlock), 0, s, js.dev,
                     js.unit_prefix, G);
}

int finalize_chunks(int64_t G, int K) { return slot_chunks(G, K); }

void launch_refine(const JobSet& js, bool grid, bool alpha, hipStream_t s) {
  if (js.n < 1 || (!grid && !alpha)) return;
  if (grid && js.has_eq)
    hipLaunchKernelGGL(k_equivalences, dim3(js.maxKd, js.n), dim3(64), 0, s, js.dev);
  const dim3 g((grid ? js.maxKd : 0) + (alpha ? 1 : 0), js.n);
  if (js.prec == 1)
    hipLaunchKernelGGL(k_refine<float>, g, dim3(axis_block(js)), 0, s, js.dev, grid ? 1 : 0,
                       alpha ? 1 : 0);
  else
    hipLaunchKernelGGL(k_refine<double>, g, dim3(axis_block(js)), 0, s, js.dev, grid ? 1 : 0,
                       alpha ? 1 : 0);
}

}  // namespace mcv
