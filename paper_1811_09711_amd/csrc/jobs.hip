// Creation of one integration job's device state, shared by the single
// integrator and the batched / serving engines, plus the host-side error
// state and the combination of iterations.
//
// Brass, Kilian, Reuter, arXiv:1811.09711: Sec. 3.2 (grids start
// equidistant), Sec. 3.4 (alpha starts at 1/K), Sec. 3.5 (iterations are
// combined into the final estimate with their variances).
#include <hip/hip_runtime.h>

#include <math.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <string>
#include <unordered_map>
#include <vector>

#include "mcv_host.h"
#include "mcv_mask.h"

namespace mcv {

namespace {

thread_local std::string g_err;

// The installed allocator, and which allocator made each live block.
struct Allocator {
  mcv_alloc_fn alloc = nullptr;
  mcv_free_fn release = nullptr;
  void* ctx = nullptr;
};
std::mutex g_alloc_mu;
Allocator g_alloc;
std::unordered_map<void*, Allocator> g_blocks;

// Sub-allocation of one block: every array starts on a 256-byte boundary.
// With base == nullptr it only measures.
struct Carve {
  char* base = nullptr;
  size_t off = 0;
  template <typename T>
  void take(T*& p, size_t count) {
    off = (off + 255) & ~(size_t)255;
    p = base ? reinterpret_cast<T*>(base + off) : nullptr;
    off += (count > 0 ? count : 1) * sizeof(T);
  }
};

// The arrays uploaded from the host, in block order (the staged prefix).
void carve_inputs(JobDev& j, Carve& c) {
  const size_t d = j.d, K = j.K, P = j.P;
  c.take(j.ckind, K * d);
  c.take(j.cloc, K * d);
  c.take(j.cwidth, K * d);
  c.take(j.pkind, P * d);
  c.take(j.ploc, P * d);
  c.take(j.pwidth, P * d);
  c.take(j.pweight, P);
  c.take(j.twin_peak, K);
  c.take(j.orphans, P);
  c.take(j.iter_dev, 1);
  c.take(j.ticket, 1);
  c.take(j.self, 1);
}

void carve_state(JobDev& j, Carve& c) {
  const size_t d = j.d, K = j.K, n = j.n, P = j.P, tsz = j.prec == 1 ? 4 : 8;
  c.take(j.history, (size_t)j.max_iter * kHistStride);  // read with iter_dev, which is close before
  c.take(j.cmap64, K * d);
  c.take(j.cmap32, K * d);
  c.take(j.cnorm64, K);
  c.take(j.cnorm32, K);
  c.take(j.pmap64, P * d);
  c.take(j.pmap32, P * d);
  c.take(j.pnorm64, P);
  c.take(j.pnorm32, P);
  c.take(j.ctype, K);
  c.take(j.edges, K * d * (n + 1));  // to start: read together
  c.take(j.alpha, K);
  c.take(j.nc, K);
  c.take(j.start, K + 1);
  c.take(j.hist, K * d * n);  // and chstats: read together
  c.take(j.chstats, K * kStatStride);
  char* xt = nullptr;
  char* pt = nullptr;
  c.take(xt, K * d * (size_t)j.sT * 2 * tsz);
  c.take(pt, K * d * (size_t)j.sT * 2 * tsz);
  j.xtab = xt;
  j.ptab = pt;
  char* ct = nullptr;
  c.take(ct, K * d * (size_t)j.M * 4 * tsz);
  j.ctab = ct;
  c.take(j.axmax, K * d);
  c.take(j.next, 8);
  const size_t stride = j.prec == 1 ? chan_stride<float>(j.d) : chan_stride<double>(j.d);
  c.take(j.crec, K * stride);
  c.take(j.t_crec, K * stride);
  c.take(j.hab, K * d * 2);
  if (j.masked) {
    const size_t Kp = (K + 31) & ~(size_t)31;
    _Float16* mc = nullptr;
    c.take(mc, Kp * 16 * mask_form_of(j.d).steps);
    j.mco = mc;
    c.take(j.moff, Kp * 2);
    c.take(j.mthr, Kp);
  }
  c.take(j.t_alpha, K);
  c.take(j.t_nc, K);
  c.take(j.t_start, K + 1);
  c.take(j.nr, K);
  c.take(j.spb, K);
  c.take(j.bstart, K + 1);
  c.take(j.t_nr, K);
  c.take(j.t_spb, K);
  c.take(j.mrg, j.rng ? (size_t)kMrgTables * kMrgEntry + (K + 1) * 6 : 0);
}

// The share of (calls of one channel, another channel) pairs in which the mask
// is expected to leave the other channel out: its exponent over the first one's
// calls, taken at their centre less 2.5 times their spread towards it, reaches
// the exponents that the skip needs (32 bits, what the calls' own kernel has
// lost, the ratio of the norms).  The calls of up to 16 channels are looked at.
double masked_share(const mcv_problem* p, const MaskForm& f) {
  const int d = p->dim, K = p->n_channels, ns = std::min(K, 16);
  constexpr double kFlatSpread = 0.29;  // of a uniform variable
  std::vector<double> centre((size_t)K * d), spread(centre), bits(centre), lw(centre);
  std::vector<int> ng(K, 0);
  for (size_t i = 0; i < centre.size(); ++i) {
    const int kind = p->chan_kind[i];
    const double w = p->chan_width[i];
    centre[i] = kind == MCV_FLAT ? 0.5 : p->chan_loc[i];
    spread[i] = kind == MCV_FLAT ? kFlatSpread : std::min(kFlatSpread, kind == MCV_GAUSS ? w : 3.0 * w);
    lw[i] = kind == MCV_GAUSS ? log2(w) : 0.0;
    bits[i] = log2(kind == MCV_GAUSS ? spread[i] : kFlatSpread);
    ng[i / d] += kind == MCV_GAUSS;
  }
  int64_t hit = 0, pairs = 0;
  std::vector<double> ga(d);
  for (int c = 0; c < K; ++c) {
    const size_t cd = (size_t)c * d;
    const bool on = f.axes > 0 ? ng[c] > 0 : ng[c] == d;
    double least = INFINITY;
    for (int k = 0; k < d; ++k) {
      ga[k] = p->chan_kind[cd + k] == MCV_GAUSS ? 0.8493218 / p->chan_width[cd + k] : 0.0;
      least = std::min(least, ga[k]);
    }
    for (int i = 0; i < ns; ++i) {
      const int s = i * K / ns;
      if (s == c) continue;
      ++pairs;
      if (!on) continue;
      const size_t sd = (size_t)s * d;
      double dist = 0.0, along = 0.0, own = 0.0, need = 32.0 + 0.72 * ng[s];
      for (int k = 0; k < d; ++k) {
        if (ga[k] == 0.0) continue;
        const double a = f.axes > 0 ? ga[k] : least;
        const double x = a * (centre[sd + k] - centre[cd + k]), y = a * spread[sd + k];
        dist += x * x;
        along += x * x * y * y;
        own += y * y;
        need += bits[sd + k] - lw[cd + k];
      }
      const double away = sqrt(dist) - 2.5 * (dist > 0.0 ? sqrt(along / dist) : 0.0);
      hit += (away > 0.0 ? away * away : 0.0) + own >= need;
    }
  }
  return pairs > 0 ? (double)hit / (double)pairs : 0.0;
}

// Whether a job's passes leave channels out by masks and put sparse lookups
// off (mcv_mask.h, sample_kernel.h): in FP32 from four axes and four channels
// that the mask can bound, where 0.72 of the pairs of channels are expected
// apart.  Below four axes the channels' peaks overlap and few are left out (24
// channels: d = 2 273 us a pass with masks, 227 without; d = 3 the same).  A
// channel that is not left out goes through the queue with all its lanes,
// which costs more than its lookups at once: 48 channels, d = 10, 833333 calls:
// all Gaussian of widths 0.3 to 0.6 (share 0) 656 us with masks and 475
// without, 0.1 to 0.3 (0.1) 455 and 376, 0.05 to 0.15 (0.82) 150 and 196; a
// quarter Gaussian and the others Breit-Wigner (0.25) 1.4 times as long with
// masks, three quarters (0.75) 1.03, seven eighths (0.85) 0.86.  Of 366 jobs of
// 4 to 16 axes and 4 to 64 channels so measured, masks are slower in 10 %, by
// up to 1.3 times, where this rule takes them, and faster by more than 3 % in 4
// where it does not; in FP64 the 3-axis partial exponent does as well and the
// queue costs more registers than it saves (d = 10: 2.28 ms with masks, 1.96
// without).  The lookup queues have to fit the LDS besides what the pass needs.
bool wants_masks(const mcv_problem* p, JobDev j) {
  if (p->precision != MCV_FP32_MIXED || p->dim < 4 || p->n_channels < 4) return false;
  const MaskForm f = mask_form_of(p->dim);
  j.masked = 1;
  if (f.steps == 0 || sample_lds_bytes(j) > 160 * 1024) return false;
  int ng = 0;
  for (int c = 0; c < p->n_channels; ++c) {
    int g = 0;
    for (int k = 0; k < p->dim; ++k) g += p->chan_kind[(size_t)c * p->dim + k] == MCV_GAUSS;
    ng += f.axes > 0 ? g > 0 : g == p->dim;
  }
  return ng >= 4 && masked_share(p, f) >= 0.72;
}

// MRG32k3a jump tables and stream starts (layout: JobDev::mrg), from the
// generator's matrices by repeated squaring.
struct Mat3x2 {
  uint32_t a[9], b[9];
};

Mat3x2 mrg_mul(const Mat3x2& x, const Mat3x2& y) {
  Mat3x2 r;
  for (int i = 0; i < 3; ++i)
    for (int k = 0; k < 3; ++k) {
      uint64_t sa = 0, sb = 0;
      for (int q = 0; q < 3; ++q) {
        sa += mrg_mod1((uint64_t)x.a[3 * i + q] * y.a[3 * q + k]);
        sb += mrg_mod2((uint64_t)x.b[3 * i + q] * y.b[3 * q + k]);
      }
      r.a[3 * i + k] = mrg_mod1(sa);
      r.b[3 * i + k] = mrg_mod2(sb);
    }
  return r;
}

void mrg_vec(const Mat3x2& m, uint32_t s[6]) {
  uint32_t r[6];
  for (int i = 0; i < 3; ++i) {
    uint64_t sa = 0, sb = 0;
    for (int q = 0; q < 3; ++q) {
      sa += mrg_mod1((uint64_t)m.a[3 * i + q] * s[q]);
      sb += mrg_mod2((uint64_t)m.b[3 * i + q] * s[3 + q]);
    }
    r[i] = mrg_mod1(sa);
    r[3 + i] = mrg_mod2(sb);
  }
  for (int i = 0; i < 6; ++i) s[i] = r[i];
}

std::vector<uint32_t> mrg_host_tables(uint64_t seed, int K) {
  std::vector<Mat3x2> pw(191);  // pw[b] = A^(2^b)
  pw[0] = Mat3x2{{0, 1, 0, 0, 0, 1, kMrgM1 - 810728u, 1403580u, 0},
                 {0, 1, 0, 0, 0, 1, kMrgM2 - 1370589u, 0, 527612u}};
  for (int b = 1; b < 191; ++b) pw[b] = mrg_mul(pw[b - 1], pw[b - 1]);
  std::vector<uint32_t> out((size_t)kMrgTables * kMrgEntry + (size_t)(K + 1) * 6);
  for (int b = 0; b < 64; ++b) {
    memcpy(&out[(size_t)b * kMrgEntry], &pw[b], sizeof(Mat3x2));
    memcpy(&out[(size_t)(kMrgSubBase + b) * kMrgEntry], &pw[76 + b], sizeof(Mat3x2));
  }
  for (int c = 0; c <= K; ++c) {
    uint64_t g = 1024 * seed + (uint64_t)(c < K ? c : 1023);
    uint32_t st[6] = {12345, 12345, 12345, 12345, 12345, 12345};
    for (int b = 0; g != 0; ++b, g >>= 1)
      if (g & 1) mrg_vec(pw[127 + b], st);
    memcpy(&out[(size_t)kMrgTables * kMrgEntry + (size_t)c * 6], st, sizeof st);
  }
  return out;
}

}  // namespace

mcv_status fail(mcv_status st, const std::string& msg) {
  g_err = msg;
  return st;
}

const char* last_error() { return g_err.c_str(); }

mcv_status set_allocator(mcv_alloc_fn alloc, mcv_free_fn release, void* ctx) {
  if ((alloc == nullptr) != (release == nullptr))
    return fail(MCV_E_INVALID, "give both allocator functions, or neither");
  std::lock_guard<std::mutex> lk(g_alloc_mu);
  g_alloc = Allocator{alloc, release, ctx};
  return MCV_OK;
}

hipError_t dev_alloc(void** p, size_t bytes) {
  *p = nullptr;
  if (bytes == 0) bytes = 256;
  Allocator a;
  {
    std::lock_guard<std::mutex> lk(g_alloc_mu);
    a = g_alloc;
  }
  if (!a.alloc) {
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipSuccess) {
      std::lock_guard<std::mutex> lk(g_alloc_mu);
      g_blocks[*p] = a;
    }
    return e;
  }
  void* q = a.alloc(bytes, a.ctx);
  if (!q) return hipErrorOutOfMemory;
  std::lock_guard<std::mutex> lk(g_alloc_mu);
  g_blocks[q] = a;
  *p = q;
  return hipSuccess;
}

void dev_free(void* p) {
  if (!p) return;
  Allocator a;
  {
    std::lock_guard<std::mutex> lk(g_alloc_mu);
    auto it = g_blocks.find(p);
    if (it == g_blocks.end()) return;  // not ours
    a = it->second;
    g_blocks.erase(it);
  }
  if (!a.release) {
    (void)hipFree(p);
    return;
  }
  (void)hipDeviceSynchronize();
  a.release(p, a.ctx);
}

mcv_status validate_problem(const mcv_problem* p) {
  if (!p) return fail(MCV_E_INVALID, "problem is NULL");
  if (p->dim < 1 || p->dim > 32) return fail(MCV_E_INVALID, "dim must be in [1, 32]");
  if (p->n_bins < 1 || p->n_bins > 256) return fail(MCV_E_INVALID, "n_bins must be in [1, 256]");
  if (p->n_channels < 1 || p->n_channels > 1024)
    return fail(MCV_E_INVALID, "n_channels must be in [1, 1024]");
  if (p->n_peaks < 1 || p->n_peaks > 1024) return fail(MCV_E_INVALID, "n_peaks must be in [1, 1024]");
  if (p->precision != MCV_FP64 && p->precision != MCV_FP32_MIXED)
    return fail(MCV_E_INVALID, "precision must be MCV_FP64 or MCV_FP32_MIXED");
  if (!p->peak_kind || !p->peak_loc || !p->peak_width || !p->peak_weight || !p->chan_kind ||
      !p->chan_loc || !p->chan_width)
    return fail(MCV_E_INVALID, "a problem array is NULL");
  if (!(p->grid_power >= 0.0) || !isfinite(p->grid_power))
    return fail(MCV_E_INVALID, "grid_power must be finite and >= 0");
  if (!(p->channel_power >= 0.0) || !isfinite(p->channel_power))
    return fail(MCV_E_INVALID, "channel_power must be finite and >= 0");
  if (p->min_calls < 1) return fail(MCV_E_INVALID, "min_calls must be >= 1");
  if (p->strat < 0 || p->strat == 1 || p->strat > (1 << 20))
    return fail(MCV_E_INVALID, "strat must be 0 (uniform) or the calls per box, 2..2^20");
  if (p->rng != MCV_RNG_PHILOX && p->rng != MCV_RNG_MRG32K3A)
    return fail(MCV_E_INVALID, "rng must be MCV_RNG_PHILOX or MCV_RNG_MRG32K3A");
  if (p->rng == MCV_RNG_MRG32K3A && (p->n_channels > 1023 || p->seed >= ((uint64_t)1 << 54)))
    return fail(MCV_E_INVALID, "MRG32k3a streams need n_channels <= 1023 and seed < 2^54");
  if (p->max_iterations < 1) return fail(MCV_E_INVALID, "max_iterations must be >= 1");
  auto check = [&](const int32_t* kind, const double* loc, const double* width, int n,
                   const char* what) -> mcv_status {
    for (int i = 0; i < n * p->dim; ++i) {
      if (kind[i] != MCV_FLAT && kind[i] != MCV_GAUSS && kind[i] != MCV_BW)
        return fail(MCV_E_INVALID, std::string(what) + ": unknown kind");
      if (kind[i] == MCV_FLAT) continue;
      if (!(width[i] > 0.0) || !isfinite(width[i]))
        return fail(MCV_E_INVALID, std::string(what) + ": width must be finite and > 0");
      if (!(loc[i] >= 0.0 && loc[i] <= 1.0))
        return fail(MCV_E_INVALID, std::string(what) + ": centre must lie in [0, 1]");
    }
    return MCV_OK;
  };
  mcv_status st = check(p->peak_kind, p->peak_loc, p->peak_width, p->n_peaks, "peak");
  if (st != MCV_OK) return st;
  st = check(p->chan_kind, p->chan_loc, p->chan_width, p->n_channels, "channel");
  if (st != MCV_OK) return st;
  for (int i = 0; i < p->n_peaks; ++i)
    if (!isfinite(p->peak_weight[i])) return fail(MCV_E_INVALID, "peak weight must be finite");
  return MCV_OK;
}

mcv_status device_cus(int* device, int* n_cu) {
  hipError_t e = hipGetDevice(device);
  int ncu = 0;
  if (e == hipSuccess) e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, *device);
  if (e != hipSuccess) return fail(MCV_E_DEVICE, std::string("no HIP device: ") + hipGetErrorString(e));
  *n_cu = ncu > 0 ? ncu : 1;
  return MCV_OK;
}

size_t partial_bytes(const JobDev& j, int G) {
  const size_t slots = (size_t)G + (size_t)j.K;
  const size_t a = (slots * kPartStride * sizeof(double) + 255) & ~(size_t)255;
  return a + slots * (size_t)j.d * j.n * sizeof(double);
}

void carve_partials(JobDev& j, int G, char* base) {
  const size_t slots = (size_t)G + (size_t)j.K;
  const size_t a = (slots * kPartStride * sizeof(double) + 255) & ~(size_t)255;
  j.part = reinterpret_cast<double*>(base);
  j.hpart = reinterpret_cast<double*>(base + a);
  j.gmax = G;
}

size_t job_block_bytes(const mcv_problem* p, int gmax) {
  JobDev j;
  j.d = p->dim;
  j.K = p->n_channels;
  j.n = p->n_bins;
  j.P = p->n_peaks;
  j.prec = p->precision;
  j.sT = (j.n + 3) & ~1;
  j.M = hint_cells_for_bins(j.n);
  j.mshift = hint_cell_shift(j.M);
  j.max_iter = p->max_iterations;
  j.rng = p->rng;
  j.strat = p->strat;
  j.masked = gmax > 0 && wants_masks(p, j);
  Carve m;
  carve_inputs(j, m);
  carve_state(j, m);
  size_t total = m.off;
  if (gmax > 0) total = ((total + 255) & ~(size_t)255) + partial_bytes(j, gmax);
  return total;
}

mcv_status job_create(const mcv_problem* p, int gmax, int64_t n_points, int n_cu, hipStream_t s,
                      JobDev* out, void** block) {
  *block = nullptr;
  mcv_status st = validate_problem(p);
  if (st != MCV_OK) return st;
  JobDev j;
  j.d = p->dim;
  j.K = p->n_channels;
  j.n = p->n_bins;
  j.P = p->n_peaks;
  j.prec = p->precision;
  j.npow2 = 1;
  while (j.npow2 < j.n) j.npow2 <<= 1;
  j.sT = (j.n + 3) & ~1;  // entries 0..n+1, even
  j.M = hint_cells_for_bins(j.n);
  j.mshift = hint_cell_shift(j.M);
  j.n_cu = n_cu;
  j.seed = p->seed;
  j.grid_power = p->grid_power;
  j.channel_power = p->channel_power;
  j.min_calls = p->min_calls;
  j.max_iter = p->max_iterations;
  j.n_points = n_points;
  j.rng = p->rng;
  j.strat = p->strat;
  j.masked = gmax > 0 && wants_masks(p, j);
  if (sample_lds_bytes(j) > 160 * 1024)
    return fail(MCV_E_INVALID, "dim * n_bins too large for the LDS of one workgroup");
  const size_t d = j.d, K = j.K, P = j.P;

  // channels whose map has the exact shape of a peak share that peak's
  // exponential; each peak is claimed by at most one channel
  std::vector<int32_t> twin(K, -1), orphan;
  {
    std::vector<char> taken(P, 0);
    for (size_t c = 0; c < K; ++c)
      for (size_t i = 0; i < P && twin[c] < 0; ++i) {
        if (taken[i]) continue;
        bool same = true;
        for (size_t k = 0; k < d && same; ++k) {
          const size_t a = c * d + k, b = i * d + k;
          if (p->chan_kind[a] != p->peak_kind[b]) same = false;
          else if (p->chan_kind[a] != MCV_FLAT &&
                   (p->chan_loc[a] != p->peak_loc[b] || p->chan_width[a] != p->peak_width[b]))
            same = false;
        }
        if (same) {
          twin[c] = (int32_t)i;
          taken[i] = 1;
        }
      }
    for (size_t i = 0; i < P; ++i)
      if (!taken[i]) orphan.push_back((int32_t)i);
  }
  j.n_orphan = (int)orphan.size();
  for (size_t c = 0; c < K; ++c)
    if (twin[c] >= 0 && p->peak_weight[twin[c]] < 0.0) j.fpos = 0;

  // measure, allocate, carve
  Carve m;
  carve_inputs(j, m);
  const size_t staged = m.off;
  carve_state(j, m);
  size_t total = m.off;
  size_t part_off = 0;
  if (gmax > 0) {
    part_off = (total + 255) & ~(size_t)255;
    total = part_off + partial_bytes(j, gmax);
  }
  void* dev = nullptr;
  hipError_t e = dev_alloc(&dev, total);
  if (e != hipSuccess) return fail(MCV_E_NOMEM, std::string("job block: ") + hipGetErrorString(e));
  Carve c;
  c.base = static_cast<char*>(dev);
  carve_inputs(j, c);
  carve_state(j, c);
  if (gmax > 0) carve_partials(j, gmax, static_cast<char*>(dev) + part_off);

  // stage the inputs in the block's own layout: one upload
  std::vector<char> stage(staged, 0);
  JobDev h = j;
  Carve hc;
  hc.base = stage.data();
  carve_inputs(h, hc);
  memcpy(h.ckind, p->chan_kind, K * d * sizeof(int32_t));
  memcpy(h.cloc, p->chan_loc, K * d * sizeof(double));
  memcpy(h.cwidth, p->chan_width, K * d * sizeof(double));
  memcpy(h.pkind, p->peak_kind, P * d * sizeof(int32_t));
  memcpy(h.ploc, p->peak_loc, P * d * sizeof(double));
  memcpy(h.pwidth, p->peak_width, P * d * sizeof(double));
  memcpy(h.pweight, p->peak_weight, P * sizeof(double));
  memcpy(h.twin_peak, twin.data(), K * sizeof(int32_t));
  if (!orphan.empty()) memcpy(h.orphans, orphan.data(), orphan.size() * sizeof(int32_t));
  *h.iter_dev = 0;
  *h.ticket = 0;
  memcpy(h.self, &j, sizeof(JobDev));

  e = hipMemcpyAsync(dev, stage.data(), staged, hipMemcpyHostToDevice, s);
  std::vector<uint32_t> mrg_tab;
  if (e == hipSuccess && j.rng) {
    mrg_tab = mrg_host_tables(j.seed, j.K);
    e = hipMemcpyAsync(j.mrg, mrg_tab.data(), mrg_tab.size() * sizeof(uint32_t),
                       hipMemcpyHostToDevice, s);
  }
  if (e == hipSuccess) {
    launch_setup(j, s);
    launch_tables(single_set(j), s);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipStreamSynchronize(s);  // stage and j are read until here
  if (e != hipSuccess) {
    dev_free(dev);
    return fail(MCV_E_DEVICE, std::string("job set-up: ") + hipGetErrorString(e));
  }
  *out = j;
  *block = dev;
  return MCV_OK;
}

void HostRead::reserve(size_t bytes) {
  if (hipHostMalloc(&pin, bytes, hipHostMallocDefault) == hipSuccess) {
    cap = bytes;
  } else {
    (void)hipGetLastError();
    pin = nullptr;
  }
}

void HostRead::release() {
  if (pin) hipHostFree(pin);
  pin = nullptr;
  cap = 0;
}

mcv_status HostRead::read(const HostSeg* seg, int n, hipStream_t s) {
  constexpr size_t kGap = 4096;  // a copy's start costs as much as some 100 KB of it
  std::vector<HostSeg> run;      // neighbours joined: dst = offset in the buffer
  size_t sum = 0;
  for (int i = 0; i < n; ++i) {
    if (!seg[i].dst || seg[i].bytes == 0) continue;
    const char* p = static_cast<const char*>(seg[i].src);
    if (!run.empty()) {
      HostSeg& r = run.back();
      const char* e = static_cast<const char*>(r.src) + r.bytes;
      if (p >= e && (size_t)(p - e) <= kGap) {
        sum += (size_t)(p - e) + seg[i].bytes;
        r.bytes = (size_t)(p - static_cast<const char*>(r.src)) + seg[i].bytes;
        continue;
      }
    }
    run.push_back(HostSeg{nullptr, p, seg[i].bytes});
    sum += seg[i].bytes;
  }
  std::unique_lock<std::mutex> lk(mu, std::defer_lock);
  char small[kReadSmall];
  char* buf = nullptr;
  if (sum <= cap) {
    lk.lock();
    buf = static_cast<char*>(pin);
  } else if (sum <= kReadSmall) {
    buf = small;
  }
  if (!buf) {
    for (int i = 0; i < n; ++i)
      if (seg[i].dst && seg[i].bytes)
        MCV_HIP(hipMemcpyAsync(seg[i].dst, seg[i].src, seg[i].bytes, hipMemcpyDeviceToHost, s));
    MCV_HIP(hipStreamSynchronize(s));
    return MCV_OK;
  }
  size_t off = 0;
  hipError_t e = hipSuccess;
  for (HostSeg& r : run) {
    r.dst = buf + off;
    off += r.bytes;
    if (e == hipSuccess) e = hipMemcpyAsync(r.dst, r.src, r.bytes, hipMemcpyDeviceToHost, s);
  }
  const hipError_t e2 = hipStreamSynchronize(s);  // also after an error: buf must be idle
  MCV_HIP(e);
  MCV_HIP(e2);
  for (int i = 0; i < n; ++i) {
    if (!seg[i].dst || seg[i].bytes == 0) continue;
    const char* p = static_cast<const char*>(seg[i].src);
    for (const HostSeg& r : run) {
      const char* b = static_cast<const char*>(r.src);
      if (p >= b && p + seg[i].bytes <= b + r.bytes) {
        memcpy(seg[i].dst, static_cast<const char*>(r.dst) + (p - b), seg[i].bytes);
        break;
      }
    }
  }
  return MCV_OK;
}

void state_segs(const JobDev& j, double* edges, double* alpha, int64_t* alloc, HostSeg (&seg)[4]) {
  seg[0] = HostSeg{edges, j.edges, (size_t)j.K * j.d * (j.n + 1) * sizeof(double)};
  seg[1] = HostSeg{alpha, j.alpha, j.K * sizeof(double)};
  seg[2] = HostSeg{alloc, j.nc, j.K * sizeof(int64_t)};
  seg[3] = HostSeg{alloc ? alloc + j.K : nullptr, j.start + j.K, sizeof(int64_t)};
}

size_t state_read_bytes(const JobDev& j) {
  const size_t st = (const char*)(j.start + j.K + 1) - (const char*)j.edges;
  const size_t ps = (const char*)(j.chstats + (size_t)j.K * kStatStride) - (const char*)j.hist;
  return st > ps ? st : ps;
}

void combine_history(const double* hist, int n, int first, mcv_summary* out) {
  double sw = 0.0, swe = 0.0, zsum = 0.0, npts = 0.0, nbad = 0.0;
  int nz = 0, used = 0;
  for (int t = first; t < n; ++t) {
    const double* r = &hist[(size_t)t * kHistStride];
    ++used;
    npts += r[2];
    nbad += r[4];
    if (r[1] == 0.0) {
      zsum += r[0];
      ++nz;
    } else {
      sw += 1.0 / (r[1] * r[1]);
      swe += r[0] / (r[1] * r[1]);
    }
  }
  memset(out, 0, sizeof *out);
  out->n_iter_used = used;
  out->n_points = (int64_t)npts;
  out->n_bad = (int64_t)nbad;
  out->w_max = hist[(size_t)(n - 1) * kHistStride + 3];
  if (nz > 0) {
    out->integral = zsum / nz;
    return;
  }
  const double mean = swe / sw;
  double chi2 = 0.0;
  for (int t = first; t < n; ++t) {
    const double* r = &hist[(size_t)t * kHistStride];
    chi2 += (r[0] - mean) * (r[0] - mean) / (r[1] * r[1]);
  }
  out->integral = mean;
  out->error = 1.0 / sqrt(sw);
  out->chi2_ndf = used > 1 ? chi2 / (used - 1) : 0.0;
}

}  // namespace mcv
