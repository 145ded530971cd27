// filter.hpp -- particle-filter kernels on gfx950: noise draws, observation
// and likelihood, weights / ESS / tempering, systematic resampling, gathers.
#pragma once

#include "device.hpp"

namespace sch {

// dW[p][n][q] = sqrt(dt) z, one Philox block per (particle, step, mode pair).
static __global__ void k_draw_increments(uint64_t seed, uint32_t step0, uint32_t tag, uint32_t word3,
                                  int n_particles, int n_steps, int n_modes, double sdt,
                                  double* dW) {
  const int n_pairs = (n_modes + 1) / 2;
  const int64_t total = static_cast<int64_t>(n_particles) * n_steps * n_pairs;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < total;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int kk = static_cast<int>(i % n_pairs);
    const int64_t pn = i / n_pairs;
    const int n = static_cast<int>(pn % n_steps);
    const int p = static_cast<int>(pn / n_steps);
    double z0, z1;
    normal2(seed, static_cast<uint32_t>(p), step0 + static_cast<uint32_t>(n),
            static_cast<uint32_t>(kk) | (tag << 24), word3, z0, z1);
    double* row = dW + pn * n_modes;
    row[2 * kk] = sdt * z0;
    if (2 * kk + 1 < n_modes) row[2 * kk + 1] = sdt * z1;
  }
}

// Raw Philox blocks: out[i] = philox(ctr[i], seed).
static __global__ void k_philox_blocks(uint64_t seed, int n, const uint32_t* ctr, uint32_t* out) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const Ctr4 r = philox10(Ctr4{{ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3]}}, seed);
#pragma unroll
    for (int k = 0; k < 4; ++k) out[4 * i + k] = r.w[k];
  }
}

// Random numbers of n_jitter pCN moves (section 3.1.2): zeta[j][p][n][q] =
// sqrt(dt) z with z from the PCN-tagged block (p, step0 + n, pair | tag << 24,
// word3 | j), and the acceptance uniform vacc[j][p] from the ACCEPT-tagged
// block (p, cycle, tag << 24, word3 | j).
static __global__ void k_draw_pcn(uint64_t seed, uint32_t step0, uint32_t cycle, uint32_t word3,
                           int n_jitter, int n_particles, int n_steps, int n_modes, double sdt,
                           double* zeta, double* vacc) {
  const int n_pairs = (n_modes + 1) / 2;
  const int64_t per = static_cast<int64_t>(n_particles) * n_steps * n_pairs;
  const int64_t total = per * n_jitter;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < total;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int j = static_cast<int>(i / per);
    const int64_t r = i - j * per;
    const int kk = static_cast<int>(r % n_pairs);
    const int64_t pn = r / n_pairs;
    const int n = static_cast<int>(pn % n_steps);
    const int p = static_cast<int>(pn / n_steps);
    const uint32_t w3 = word3 | static_cast<uint32_t>(j);
    double z0, z1;
    normal2(seed, static_cast<uint32_t>(p), step0 + static_cast<uint32_t>(n),
            static_cast<uint32_t>(kk) | (SCH_TAG_PCN << 24), w3, z0, z1);
    double* row = zeta + (static_cast<int64_t>(j) * n_particles * n_steps + pn) * n_modes;
    row[2 * kk] = sdt * z0;
    if (2 * kk + 1 < n_modes) row[2 * kk + 1] = sdt * z1;
    if (n == 0 && kk == 0)
      vacc[static_cast<int64_t>(j) * n_particles + p] =
          uniform1(seed, static_cast<uint32_t>(p), cycle, SCH_TAG_ACCEPT << 24, w3);
  }
}

// One uniform in [0,1) into a device scalar.
static __global__ void k_draw_uniform(uint64_t seed, uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                               double* out) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *out = uniform1(seed, c0, c1, c2, c3);
}

// P1 point evaluation at x_j = j L / n_obs, one wavefront per particle.
__device__ __forceinline__ double p1_at(const double* u, int nx, int n_obs, int j) {
  const int64_t num = static_cast<int64_t>(j) * nx;
  const int e = static_cast<int>(num / n_obs);
  const double r = static_cast<double>(num % n_obs) / static_cast<double>(n_obs);
  const int e1 = e + 1 == nx ? 0 : e + 1;
  return (1.0 - r) * u[e] + r * u[e1];
}

static __global__ void __launch_bounds__(kWave) k_observe(int nx, int n_obs, const double* u,
                                                   double* out) {
  const int p = blockIdx.x;
  const double* up = u + static_cast<size_t>(p) * nx;
  for (int j = threadIdx.x; j < n_obs; j += kWave)
    out[static_cast<size_t>(p) * n_obs + j] = p1_at(up, nx, n_obs, j);
}

static __global__ void __launch_bounds__(kWave) k_loglik(int nx, int n_obs, const double* u,
                                                  const double* y, const double* sigma,
                                                  double* phi) {
  const int p = blockIdx.x;
  const double* up = u + static_cast<size_t>(p) * nx;
  double acc = 0.0;
  for (int j = threadIdx.x; j < n_obs; j += kWave) {
    const double e = (p1_at(up, nx, n_obs, j) - y[j]) / sigma[j];
    acc += e * e;
  }
  acc = wave_sum(acc);
  if (threadIdx.x == 0) {
    const double v = 0.5 * acc;
    phi[p] = isfinite(v) ? v : INFINITY;
  }
}

// ---------------------------------------------------------------------------
// Weights, ESS and adaptive tempering in one workgroup of kTB threads.
// ---------------------------------------------------------------------------
constexpr int kTB = 1024;

struct TemperLds {
  alignas(16) double red[2][kTB / kWave][2];  // double buffered
};

// Maxima (MAX) or sums of a and b over the workgroup; slot alternates between
// calls, so that one barrier is enough.  Every lane reads one of the 16
// wavefronts' pairs and the row of 16 lanes joins them: reading all of them in
// every lane took the LDS longer than the exponentials took.
template <bool MAX>
__device__ __forceinline__ void tb_reduce2(double& a, double& b, int& slot, TemperLds& L) {
  static_assert(kTB / kWave == 16, "a row of lanes");
  a = MAX ? wave_max(a) : wave_sum(a);
  b = MAX ? wave_max(b) : wave_sum(b);
  const int lane = threadIdx.x & (kWave - 1);
  if (lane == 0) {
    L.red[slot][threadIdx.x / kWave][0] = a;
    L.red[slot][threadIdx.x / kWave][1] = b;
  }
  __syncthreads();
  a = L.red[slot][lane & 15][0];
  b = L.red[slot][lane & 15][1];
#define SCH_STEP(N)                                                            \
  {                                                                            \
    const double x = dpp_f64z<kDppRowRor + N>(a), y = dpp_f64z<kDppRowRor + N>(b); \
    a = MAX ? fmax(a, x) : a + x;                                              \
    b = MAX ? fmax(b, y) : b + y;                                              \
  }
  SCH_STEP(8)
  SCH_STEP(4)
  SCH_STEP(2)
  SCH_STEP(1)
#undef SCH_STEP
  slot ^= 1;
}

// exponent s_p = extra_p - beta phi_p (a NaN or -inf exponent gives weight 0)
__device__ __forceinline__ double log_weight(double phi, double extra, double beta) {
  double s;
  if (beta == 0.0)
    s = extra;
  else if (isnan(phi))
    s = -INFINITY;
  else
    s = extra - beta * phi;
  return isnan(s) ? -INFINITY : s;
}

// -beta phi - smax with the product rounded by itself, as it is in smax and in
// the weights: fused, the exponents would keep the product's remainder (up to
// 7e-9 at phi = 1e8) that the others have dropped, and the weights would not
// add up to 1.  (__dmul_rn and __dsub_rn are plain operators in HIP, which the
// compiler contracts.)
__device__ __forceinline__ double exponent_below(double beta, double phi, double smax) {
#pragma clang fp contract(off)
  const double s = -beta * phi;
  return s - smax;
}

// exp(x) for x <= 0 and NaN: x = k ln 2 + r with |r| <= ln 2 / 2 (Cody and Waite's
// reduction), the Taylor polynomial to r^13 (cut off at 5e-18), and 2^k.  k of at
// most 1155 times ln 2's first part (20 trailing zero bits) is exact.  Over 4
// million points it errs by 1.36e-16 at most, the device library's exp by 1.38e-16
// (root mean square 4.9e-17 both).
__device__ __forceinline__ double exp_neg(double x) {
  constexpr double kLn2Hi = 0x1.62e42feep-1, kLn2Lo = 0x1.a39ef35793c76p-33;
  x = x < -800.0 ? -800.0 : x;
  const double k = rint(x * 1.4426950408889634);
  const double r = fma(-k, kLn2Lo, fma(-k, kLn2Hi, x));
  double p = 1.0 / 6227020800.0;
  p = fma(p, r, 1.0 / 479001600.0);
  p = fma(p, r, 1.0 / 39916800.0);
  p = fma(p, r, 1.0 / 3628800.0);
  p = fma(p, r, 1.0 / 362880.0);
  p = fma(p, r, 1.0 / 40320.0);
  p = fma(p, r, 1.0 / 5040.0);
  p = fma(p, r, 1.0 / 720.0);
  p = fma(p, r, 1.0 / 120.0);
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  p = fma(p, r, 1.0);
  p = fma(p, r, 1.0);
  return ldexp(p, static_cast<int>(k));
}

// Body of k_temper for one workgroup of kTB threads (also used per
// instance by the batched runner).  The ESS is evaluated n_bisect + 2 times
// one after the other, so what counts is the time of one: the particles' phi
// (and extra) stay in registers, kTK a thread (any more are read each time);
// without extra the largest exponent needs no reduction, it is that of the
// smallest phi (-beta phi rounds monotonically; of the largest for beta < 0);
// and the two sums take one barrier.  With a bisection's weights, resampling
// and 2048 rows of 2048 gathered: 178 us before, 101 now.
constexpr int kTK = 8;
template <bool EXTRA>
__device__ __forceinline__ void temper_run(int n, const double* phi, const double* extra,
                                           double* theta_io, double thr, int n_bisect,
                                           double* dtheta_out, double* w, double* logw_out,
                                           double* ess_out, TemperLds& L) {
  const int t = threadIdx.x;
  const double theta = *theta_io;
  const double rem = 1.0 - theta;
  double rp[kTK], rx[kTK], rq[kTK];
#pragma unroll
  for (int k = 0; k < kTK; ++k) {
    const int p = t + k * kTB;
    rp[k] = p < n ? phi[p] : 0.0;
    rx[k] = EXTRA && p < n ? extra[p] : 0.0;
    rq[k] = p < n && !isnan(rp[k]) ? rp[k] : INFINITY;
  }
  // f(particle, phi, extra) over the thread's particles, in order
  auto each = [&](auto f) {
#pragma unroll
    for (int k = 0; k < kTK; ++k)
      if (k * kTB < n && t + k * kTB < n) f(t + k * kTB, rp[k], rx[k]);
    for (int p = t + kTK * kTB; p < n; p += kTB) f(p, phi[p], EXTRA ? extra[p] : 0.0);
  };
  int slot = 0;
  double least = INFINITY, most = -INFINITY;  // phi, without extra
  if constexpr (!EXTRA) {
    double a = -INFINITY, b = -INFINITY;
    each([&](int, double f, double) {
      a = fmax(a, -f);
      b = fmax(b, f);
    });
    tb_reduce2<true>(a, b, slot, L);
    least = -a;
    most = b;
  }
  // ESS at beta; also the max exponent and the sum of exp(s - smax)
  double smax, tot;
  auto ess_at = [&](double beta) {
    if constexpr (EXTRA) {
      double mx = -INFINITY, unused = -INFINITY;
      each([&](int, double f, double x) { mx = fmax(mx, log_weight(f, x, beta)); });
      tb_reduce2<true>(mx, unused, slot, L);
      smax = mx;
    } else {
      smax = log_weight(beta < 0.0 ? most : least, 0.0, beta);
    }
    if (!(smax > -INFINITY)) {
      tot = 0.0;
      return 0.0;
    }
    double s1 = 0.0, s2 = 0.0;
    if (!EXTRA && beta > 0.0 && fabs(smax) < INFINITY) {
      // (rq: phi with +infinity, weight 0, where there is none)
#pragma unroll
      for (int k = 0; k < kTK; ++k) {
        if (k * kTB >= n) break;
        const double e = exp_neg(fmax(exponent_below(beta, rq[k], smax), -800.0));
        s1 += e;
        s2 = fma(e, e, s2);
      }
      for (int p = t + kTK * kTB; p < n; p += kTB) {
        const double e = exp_neg(log_weight(phi[p], 0.0, beta) - smax);
        s1 += e;
        s2 += e * e;
      }
    } else {
      each([&](int, double f, double x) {
        const double e = exp_neg(log_weight(f, x, beta) - smax);
        s1 += e;
        s2 += e * e;
      });
    }
    tb_reduce2<false>(s1, s2, slot, L);
    tot = s1;
    return s1 * s1 / s2;
  };
  double e = ess_at(rem);
  double pick = rem;
  if (n_bisect > 0 && !(e >= thr)) {
    double lo = 0.0, hi = rem;
    for (int k = 0; k < n_bisect; ++k) {
      const double mid = 0.5 * (lo + hi);
      const double em = ess_at(mid);
      if (em >= thr)
        lo = mid;
      else
        hi = mid;
    }
    pick = lo > 0.0 ? lo : hi;
    e = ess_at(pick);
  }
  const bool dead = !(smax > -INFINITY);
  const double ltot = dead ? 0.0 : log(tot);
  each([&](int p, double f, double x) {
    const double s = log_weight(f, x, pick);
    w[p] = dead ? 0.0 : exp_neg(s - smax) / tot;
    if (logw_out) logw_out[p] = dead ? -INFINITY : (s - smax) - ltot;
  });
  __syncthreads();  // every thread has read *theta_io
  if (t == 0) {
    *dtheta_out = pick;
    *ess_out = e;
    *theta_io = (pick == rem) ? 1.0 : theta + pick;
  }
}

__device__ __forceinline__ void temper_body(int n, const double* phi, const double* extra, double* theta_io,
                            double thr, int n_bisect, double* dtheta_out, double* w,
                            double* logw_out, double* ess_out, TemperLds& L) {
  if (extra)
    temper_run<true>(n, phi, extra, theta_io, thr, n_bisect, dtheta_out, w, logw_out, ess_out, L);
  else
    temper_run<false>(n, phi, extra, theta_io, thr, n_bisect, dtheta_out, w, logw_out, ess_out,
                      L);
}

static __global__ void __launch_bounds__(kTB) k_temper(int n, const double* phi, const double* extra,
                                                double* theta_io, double thr, int n_bisect,
                                                double* dtheta_out, double* w, double* logw_out,
                                                double* ess_out) {
  __shared__ TemperLds L;
  temper_body(n, phi, extra, theta_io, thr, n_bisect, dtheta_out, w, logw_out, ess_out, L);
}

// ---------------------------------------------------------------------------
// Integer-exact systematic resampling in one workgroup of kTB threads.
// cum (workspace, uint64 [n]) receives the prefix sums of the quantised weights.
// ---------------------------------------------------------------------------
constexpr int kCumLds = 8192;
struct ResampleLds {
  double red[kTB / kWave];
  unsigned long long part[kTB / kWave];
  int flag;
  unsigned long long cum[kCumLds];
};

// T_j = ((j + u0) * Q) / n, each operation rounded once (no contraction).
__device__ __forceinline__ double systematic_point(int j, double u0, double Q, int n) {
  double t = __dadd_rn(static_cast<double>(j), u0);
  t = __dmul_rn(t, Q);
  return __ddiv_rn(t, static_cast<double>(n));
}

// Body of k_resample for one workgroup of kTB threads (also used per
// instance by the batched runner).
__device__ __forceinline__ void resample_body(int n, const double* w, const double* u0p, const double* cond_ess,
                              double cond_thr, int* idx, int* degenerate,
                              unsigned long long* cum, ResampleLds& L) {
  const int t = threadIdx.x;
  if (cond_ess && *cond_ess >= cond_thr) {
    for (int j = t; j < n; j += kTB) idx[j] = j;
    return;
  }
  // max weight and validity
  double mx = 0.0;
  int bad = 0;
  for (int p = t; p < n; p += kTB) {
    const double v = w[p];
    if (!(v >= 0.0) || isinf(v)) bad = 1;
    mx = fmax(mx, v);
  }
  mx = wave_max(mx);
  bad = wave_or(bad);
  if (t == 0) L.flag = 0;
  __syncthreads();
  if ((t & (kWave - 1)) == 0) {
    L.red[t / kWave] = mx;
    if (bad) atomicOr(&L.flag, 1);
  }
  __syncthreads();
  double wmax = L.red[0];
  for (int i = 1; i < kTB / kWave; ++i) wmax = fmax(wmax, L.red[i]);
  if (L.flag || !(wmax > 0.0)) {
    for (int j = t; j < n; j += kTB) idx[j] = j;
    if (t == 0 && degenerate) *degenerate = 1;
    return;
  }
  int e;
  frexp(wmax, &e);
  int b = 0;
  while ((1LL << b) < n) ++b;
  const int sh = 51 - b - e;
  // contiguous block of particles per thread: local sums, then a scan of the
  // per-thread totals
  const int per = (n + kTB - 1) / kTB;
  const int lo = t * per, hi = min(n, lo + per);
  unsigned long long s = 0;
  for (int p = lo; p < hi; ++p) s += static_cast<unsigned long long>(floor(ldexp(w[p], sh)));
  // inclusive over the wavefront, then the totals of the wavefronts before
  unsigned long long inc = s;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const unsigned long long x = __shfl_up(inc, d);
    inc += (t & (kWave - 1)) >= d ? x : 0ull;
  }
  if ((t & (kWave - 1)) == kWave - 1) L.part[t / kWave] = inc;
  __syncthreads();
  unsigned long long run = inc - s, Qi = 0ull;
#pragma unroll
  for (int i = 0; i < kTB / kWave; ++i) {
    run += i < t / kWave ? L.part[i] : 0ull;
    Qi += L.part[i];
  }
  // the searches below read them at random: from LDS where they fit
  const bool in_lds = n <= kCumLds;
  for (int p = lo; p < hi; ++p) {
    run += static_cast<unsigned long long>(floor(ldexp(w[p], sh)));
    if (in_lds)
      L.cum[p] = run;
    else
      cum[p] = run;
  }
  __threadfence_block();
  __syncthreads();
  if (Qi == 0ull) {
    for (int j = t; j < n; j += kTB) idx[j] = j;
    if (t == 0 && degenerate) *degenerate = 1;
    return;
  }
  const double Q = static_cast<double>(Qi);
  const double u0 = *u0p;
  auto search = [&](auto at) {
    for (int j = t; j < n; j += kTB) {
      const double T = systematic_point(j, u0, Q, n);
      // first p with cum[p] > T
      int a = 0, c = n;
      while (a < c) {
        const int mid = (a + c) >> 1;
        if (static_cast<double>(at(mid)) > T)
          c = mid;
        else
          a = mid + 1;
      }
      idx[j] = a < n ? a : n - 1;
    }
  };
  if (in_lds)
    search([&](int i) { return L.cum[i]; });
  else
    search([&](int i) { return cum[i]; });
}

static __global__ void __launch_bounds__(kTB) k_resample(int n, const double* w, const double* u0p,
                                                  const double* cond_ess, double cond_thr,
                                                  int* idx, int* degenerate,
                                                  unsigned long long* cum) {
  __shared__ ResampleLds L;
  resample_body(n, w, u0p, cond_ess, cond_thr, idx, degenerate, cum, L);
}

// Whether rows are read and written 16 bytes a lane.
__host__ __device__ inline bool rows_in_pairs(const double* src, const double* dst,
                                              int64_t row_len) {
  return ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst) |
           static_cast<uintptr_t>(8 * row_len)) & 15) == 0;
}

// dst[j][:] = src[idx[j]][:], 16 bytes a lane where the rows allow
static __global__ void k_gather(int n_rows, int64_t row_len, const int* idx, const double* src,
                         double* dst) {
  const int j = blockIdx.y;
  const int r = idx[j];
  if (r < 0 || r >= n_rows) return;  // out-of-range index: row left untouched
  const double* s = src + static_cast<int64_t>(r) * row_len;
  double* d = dst + static_cast<int64_t>(j) * row_len;
  const int64_t i0 = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x,
                step = static_cast<int64_t>(gridDim.x) * blockDim.x;
  if (rows_in_pairs(src, dst, row_len)) {
    typedef double d2 __attribute__((ext_vector_type(2)));
    for (int64_t i = i0; i < row_len / 2; i += step)
      reinterpret_cast<d2*>(d)[i] = reinterpret_cast<const d2*>(s)[i];
    return;
  }
  for (int64_t i = i0; i < row_len; i += step) d[i] = s[i];
}

// Rows of up to eight fields resampled in place, one launch where a gather and
// a copy back of each took two: a workgroup owns kGatherCols columns (a cache
// line of a row) of a field, reads all their rows into LDS and then writes
// them.  Rows that stay are left alone, as are those of an index out of range.
//
// Up to kGatherRows rows fit 64 KB, two workgroups a compute unit (six fields,
// one launch / gathers and copies: 256 nodes, 512 rows 16 / 37 us; 4096 nodes
// 61 / 68 us; with 768 rows, one workgroup a unit, 138 / 80 us).  Each row is a
// stream of its own, so that beside many rows the fields have to stay in the
// last-level cache: at 200 to 512 rows the lines cross between 280 and 400 MB
// (512 rows, 240 MB 173 / 200 us, 280 MB 232 / 221 us, 369 MB 355 / 272 us; 256
// rows, 250 MB 119 / 195 us, 350 MB 249 / 259 us, 450 MB 366 / 339 us); at 64 and
// 128 rows not at all (128 rows, 250 MB 98 / 203 us, 1.2 GB 683 / 971 us).
constexpr int kGatherRows = 512, kGatherCols = 16;
constexpr int kGatherFewRows = 128;
constexpr int64_t kGatherBytes = int64_t(256) << 20;
struct GatherSet {
  int n, n_fields, first[9];  // first block of each field
  double* p[8];
  int64_t len[8];
};
static __global__ void __launch_bounds__(256) k_gather_rows(const GatherSet G, const int* idx) {
  extern __shared__ double rows[];
  int f = 0;
  while (f + 1 < G.n_fields && static_cast<int>(blockIdx.x) >= G.first[f + 1]) ++f;
  double* p = G.p[f];
  const int64_t len = G.len[f];
  const int c = threadIdx.x % kGatherCols;
  const int64_t col = static_cast<int64_t>(blockIdx.x - G.first[f]) * kGatherCols + c;
  const bool in = col < len;
#pragma unroll 4
  for (int j = threadIdx.x / kGatherCols; j < G.n; j += 256 / kGatherCols) {
    const int r = idx[j];
    if (in && r != j && r >= 0 && r < G.n) rows[j * kGatherCols + c] = p[r * len + col];
  }
  __syncthreads();
#pragma unroll 4
  for (int j = threadIdx.x / kGatherCols; j < G.n; j += 256 / kGatherCols) {
    const int r = idx[j];
    if (in && r != j && r >= 0 && r < G.n) p[j * len + col] = rows[j * kGatherCols + c];
  }
}

// ---------------------------------------------------------------------------
// Ensemble statistics of section 4 (EMRE, RB, RES) against a truth row.
// ---------------------------------------------------------------------------
// mean[i] = (1/n) sum_p u[p][i]
static __global__ void k_ens_mean(int n, int nx, const double* u, double* mean) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nx; i += gridDim.x * blockDim.x) {
    double acc = 0.0;
    for (int p = 0; p < n; ++p) acc += u[static_cast<size_t>(p) * nx + i];
    mean[i] = acc / n;
  }
}

// Per particle (one wavefront each): |ua - u_p|^2 and |u_p - mean|^2.
static __global__ void __launch_bounds__(kWave) k_ens_norms(int nx, const double* u, const double* ua,
                                                     const double* mean, double* sq) {
  const int p = blockIdx.x;
  const double* up = u + static_cast<size_t>(p) * nx;
  double a = 0.0, b = 0.0;
  for (int i = threadIdx.x; i < nx; i += kWave) {
    const double d = ua[i] - up[i], e = up[i] - mean[i];
    a = fma(d, d, a);
    b = fma(e, e, b);
  }
  a = wave_sum(a);
  b = wave_sum(b);
  if (threadIdx.x == 0) {
    sq[2 * p] = a;
    sq[2 * p + 1] = b;
  }
}

// out = (EMRE, RB, RES) from the per-particle squares (one wavefront).
static __global__ void __launch_bounds__(kWave) k_ens_final(int n, int nx, const double* ua,
                                                     const double* mean, const double* sq,
                                                     double* out) {
  double na = 0.0, nb = 0.0, se = 0.0, ss = 0.0;
  for (int i = threadIdx.x; i < nx; i += kWave) {
    const double d = ua[i] - mean[i];
    na = fma(ua[i], ua[i], na);
    nb = fma(d, d, nb);
  }
  for (int p = threadIdx.x; p < n; p += kWave) {
    se += sqrt(sq[2 * p]);
    ss += sqrt(sq[2 * p + 1]);
  }
  na = wave_sum(na);
  nb = wave_sum(nb);
  se = wave_sum(se);
  ss = wave_sum(ss);
  if (threadIdx.x == 0) {
    const double nrm = sqrt(na);
    out[0] = se / n / nrm;
    out[1] = sqrt(nb) / nrm;
    out[2] = n > 1 ? ss / (n - 1) / nrm : 0.0;
  }
}

// A particle whose window failed (status != SCH_OK) gets phi = +inf: zero
// weight, so the next resampling replaces it.
static __global__ void k_mask_failed(int n, const int* status, double* phi) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && status[i] != SCH_OK) phi[i] = INFINITY;
}

static __global__ void k_fill(double* p, double v, int64_t n) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    p[i] = v;
}

// *out += sum of a[0 .. n) (one workgroup of 256 threads).
static __global__ void __launch_bounds__(256) k_sum_i32_u64(int n, const int* a,
                                                     unsigned long long* out) {
  __shared__ unsigned long long part[256];
  unsigned long long s = 0;
  for (int i = threadIdx.x; i < n; i += 256) s += static_cast<unsigned long long>(a[i]);
  part[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (static_cast<int>(threadIdx.x) < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out += part[0];
}

static __global__ void k_zero_u64(unsigned long long* p, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0ull;
}

}  // namespace sch
