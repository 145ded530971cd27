// device.hpp -- device building blocks for the gfx950 SCH particle-filter
// kernels: the counter-based generator, wavefront/workgroup reductions, and
// the workgroup-wide solver for periodic (cyclic) tridiagonal systems.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sch.h"

namespace sch {

constexpr int kWave = 64;

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror & Shaw, SC'11): per round, the words at
// positions 0 and 2 are multiplied by two fixed odd constants; the new word 0
// is hi(M1*c2) ^ c1 ^ k0, word 1 is lo(M1*c2), word 2 is hi(M0*c0) ^ c3 ^ k1,
// word 3 is lo(M0*c0); the 2x32-bit key advances by a Weyl increment after
// each round.
// ---------------------------------------------------------------------------
struct Ctr4 {
  uint32_t w[4];
};

__device__ __forceinline__ Ctr4 philox10(Ctr4 c, uint64_t seed) {
  constexpr uint32_t kMulA = 0xD2511F53u, kMulB = 0xCD9E8D57u;
  constexpr uint32_t kWeylA = 0x9E3779B9u, kWeylB = 0xBB67AE85u;
  uint32_t ka = static_cast<uint32_t>(seed), kb = static_cast<uint32_t>(seed >> 32);
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    // both halves of a product from one multiplication
    const uint64_t a = static_cast<uint64_t>(kMulA) * c.w[0];
    const uint64_t b = static_cast<uint64_t>(kMulB) * c.w[2];
    Ctr4 n;
    n.w[0] = static_cast<uint32_t>(b >> 32) ^ c.w[1] ^ ka;
    n.w[1] = static_cast<uint32_t>(b);
    n.w[2] = static_cast<uint32_t>(a >> 32) ^ c.w[3] ^ kb;
    n.w[3] = static_cast<uint32_t>(a);
    c = n;
    ka += kWeylA;
    kb += kWeylB;
  }
  return c;
}

// 53 high bits of (hi:lo) as an exact double in [0, 1).
__device__ __forceinline__ double unit_double(uint32_t hi, uint32_t lo) {
  return fma(static_cast<double>(hi), 0x1.0p-32, static_cast<double>(lo >> 11) * 0x1.0p-53);
}

// 1/x: the hardware estimate (relative error about 5e-8 on gfx950) and one
// Newton step, which squares that error (at most about 11 ulp, 2e-15
// relative).
__device__ __forceinline__ double rcp64(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  return fma(r, fma(-x, r, 1.0), r);
}

// The two factors of a Box-Muller pair.  The device library's log, sqrt and
// sincos cover all arguments (330 instructions a pair, with branches for
// reductions that never happen here); these cover the ones that do, from the
// plain series, in about 100.  Together with the single multiplication of
// philox10 they took the jitter with the Matern-type noise, which draws a pair
// for every two nodes, steps and moves, from 18.4 to 17.4 ms at 4096 nodes and
// 1024 particles.  Over 4 million points the radius errs by 1.17e-16 at most (the
// library's: 1.66e-16), sine and cosine by 1.9e-16 (6.9e-16, with the angle
// rounded before).
//
// sqrt(-2 log v) for v = k 2^-53 in (0, 1].  v = 2^e m with m in [0.707, 1.414),
// log m = 2 atanh(s), s = (m - 1) / (m + 1), |s| <= 0.172: the series to s^19
// is cut off at 3e-17 of it.
__device__ __forceinline__ double box_radius(double v) {
  double m = __builtin_amdgcn_frexp_mant(v);  // [0.5, 1)
  int e = __builtin_amdgcn_frexp_exp(v);
  const bool low = m < 0.70710678118654752;
  m = low ? m + m : m;
  e = low ? e - 1 : e;
  const double f = m - 1.0, d = 2.0 + f, r = rcp64(d);
  double s = f * r;
  s = fma(fma(-s, d, f), r, s);
  const double z = s * s;
  double p = 1.0 / 19.0;
  p = fma(p, z, 1.0 / 17.0);
  p = fma(p, z, 1.0 / 15.0);
  p = fma(p, z, 1.0 / 13.0);
  p = fma(p, z, 1.0 / 11.0);
  p = fma(p, z, 1.0 / 9.0);
  p = fma(p, z, 1.0 / 7.0);
  p = fma(p, z, 1.0 / 5.0);
  p = fma(p, z, 1.0 / 3.0);
  // ln 2 in two parts (Cody and Waite), the first with 20 trailing zero bits: its
  // products with the exponent (at most 53) are exact.  2 s = f - s f takes f,
  // which is exact, out of the series: what is rounded on the way is a sixth of
  // the sum at most, and the sum's own rounding is kept (lo).
  constexpr double kLn2Hi = 0x1.62e42feep-1, kLn2Lo = 0x1.a39ef35793c76p-33;
  const double k = static_cast<double>(e);
  const double a = fma(k, kLn2Hi, f), b = fma(s, fma(-2.0 * z, p, f), -k * kLn2Lo);
  const double l = a - b, lo = (a - l) - b;
  // sqrt(x) by the coupled iteration for sqrt and its half reciprocal, lo in its
  // last residual; x = 0 (v = 1) has no reciprocal
  const double x = -2.0 * l, y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double q = fma(-h, g, 0.5);
  g = fma(g, q, g);
  h = fma(h, q, h);
  g = fma(fma(-2.0, lo, fma(-g, g, x)), h, g);
  return v < 1.0 ? g : 0.0;
}

// sin and cos of 2 pi u for u = k 2^-53 in [0, 1): the nearest quarter turn is
// taken off exactly, and |2 pi r| <= pi / 4 goes into the Taylor polynomials to
// the 17th and 16th power (cut off at 6e-20 and 2e-18).
__device__ __forceinline__ void turn_sincos(double u, double& sn, double& cs) {
  const double qd = rint(4.0 * u);
  const int n = static_cast<int>(qd);
  const double x = 6.283185307179586 * fma(-0.25, qd, u), w = x * x;
  double a = 1.0 / 355687428096000.0;
  a = fma(a, w, -1.0 / 1307674368000.0);
  a = fma(a, w, 1.0 / 6227020800.0);
  a = fma(a, w, -1.0 / 39916800.0);
  a = fma(a, w, 1.0 / 362880.0);
  a = fma(a, w, -1.0 / 5040.0);
  a = fma(a, w, 1.0 / 120.0);
  a = fma(a, w, -1.0 / 6.0);
  const double s = fma(x * w, a, x);
  double b = 1.0 / 20922789888000.0;
  b = fma(b, w, -1.0 / 87178291200.0);
  b = fma(b, w, 1.0 / 479001600.0);
  b = fma(b, w, -1.0 / 3628800.0);
  b = fma(b, w, 1.0 / 40320.0);
  b = fma(b, w, -1.0 / 720.0);
  b = fma(b, w, 1.0 / 24.0);
  const double c = fma(w * w, b, fma(-0.5, w, 1.0));
  sn = (n & 1) ? c : s;
  cs = (n & 1) ? s : c;
  sn = (n & 2) ? -sn : sn;
  cs = ((n + 1) & 2) ? -cs : cs;
}

// Two standard normals from one Philox block (Box-Muller on 1 - u1 in (0,1]).
__device__ __forceinline__ void normal2(uint64_t seed, uint32_t c0, uint32_t c1, uint32_t c2,
                                        uint32_t c3, double& z0, double& z1) {
  const Ctr4 r = philox10(Ctr4{{c0, c1, c2, c3}}, seed);
  const double rad = box_radius(1.0 - unit_double(r.w[0], r.w[1]));
  double sn, cs;
  turn_sincos(unit_double(r.w[2], r.w[3]), sn, cs);
  z0 = rad * cs;
  z1 = rad * sn;
}

__device__ __forceinline__ double uniform1(uint64_t seed, uint32_t c0, uint32_t c1, uint32_t c2,
                                           uint32_t c3) {
  const Ctr4 r = philox10(Ctr4{{c0, c1, c2, c3}}, seed);
  return unit_double(r.w[0], r.w[1]);
}

// ---------------------------------------------------------------------------
// Cross-lane moves without LDS: DPP row shifts (a lane reads lane l -/+ d of
// its 16-lane row, or keeps `old` where no such lane exists), whole-wave
// shifts by one, and readlane broadcasts into scalar registers.
// ---------------------------------------------------------------------------
constexpr int kDppRowShr = 0x110, kDppRowShl = 0x100, kDppRowRor = 0x120, kDppWaveShr1 = 0x138,
              kDppWaveShl1 = 0x130;

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double src, double old) {
  const int lo = __builtin_amdgcn_update_dpp(__double2loint(old), __double2loint(src), CTRL, 0xf,
                                             0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(__double2hiint(old), __double2hiint(src), CTRL, 0xf,
                                             0xf, false);
  return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ __forceinline__ int dpp_i32(int src, int old) {
  return __builtin_amdgcn_update_dpp(old, src, CTRL, 0xf, 0xf, false);
}
// The same with bound control: lanes without a source lane read 0 (no old
// value, so no register copy ahead of the move).
template <int CTRL>
__device__ __forceinline__ double dpp_f64z(double src) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(src), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(src), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
// Row broadcast into the rows selected by ROWS; the other rows' results are
// undefined (callers read only lanes of the selected rows afterwards).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64b(double src) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(src), CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(src), CTRL, ROWS, 0xf, false);
  return __hiloint2double(hi, lo);
}
// The value of the lane before / after, around the wavefront's ends.
__device__ __forceinline__ double wave_prev(double v) { return dpp_f64z<0x13C>(v); }
__device__ __forceinline__ double wave_next(double v) { return dpp_f64z<0x134>(v); }
// lane must be wave-uniform
__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

// ---------------------------------------------------------------------------
// Wave reductions (every lane receives the result): inclusive prefix within
// each row by row shifts, then the four row results from lanes 15, 31, 47, 63.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_f64z<kDppRowShr + 1>(v);
  v += dpp_f64z<kDppRowShr + 2>(v);
  v += dpp_f64z<kDppRowShr + 4>(v);
  v += dpp_f64z<kDppRowShr + 8>(v);
  return (readlane_f64(v, 15) + readlane_f64(v, 31)) + (readlane_f64(v, 47) + readlane_f64(v, 63));
}
// max of two doubles as one v_max_f64: fmax() would first canonicalise
// operands that arrive through lane moves (two more instructions each); the
// operands here are results of arithmetic, never signalling NaNs.
__device__ __forceinline__ double vmax(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
// max(acc, |x|) as one v_max_f64 with the absolute-value source modifier (for
// accumulating the growth of an elimination; a NaN x leaves acc unchanged).
__device__ __forceinline__ double vmax_abs(double acc, double x) {
  double r;
  asm("v_max_f64 %0, %1, |%2|" : "=v"(r) : "v"(acc), "v"(x));
  return r;
}
// (of nonnegative values: lanes without a partner take 0).  After the row
// steps, lane 15 of each row is broadcast into the next row and lane 31 into
// rows 2 and 3, so lane 63 holds the wave's maximum.
constexpr int kDppRowBcast15 = 0x142, kDppRowBcast31 = 0x143;
__device__ __forceinline__ double wave_max(double v) {
  v = vmax(v, dpp_f64z<kDppRowShr + 1>(v));
  v = vmax(v, dpp_f64z<kDppRowShr + 2>(v));
  v = vmax(v, dpp_f64z<kDppRowShr + 4>(v));
  v = vmax(v, dpp_f64z<kDppRowShr + 8>(v));
  v = vmax(v, dpp_f64b<kDppRowBcast15, 0xa>(v));
  v = vmax(v, dpp_f64b<kDppRowBcast31, 0xc>(v));
  return readlane_f64(v, 63);
}
// In lane 63: the maximum over the wave of the high words of nonnegative
// doubles, each raised by one unit where the low word is not zero: the high
// word of an upper bound, within a relative 2^-20, of the wave's maximum.  The
// 32-bit maximum fuses with the lane moves, one instruction a step.
__device__ __forceinline__ uint32_t wave_max_word(double v) {
  uint32_t h = static_cast<uint32_t>(__double2hiint(v)) + (__double2loint(v) != 0 ? 1u : 0u);
#define SCH_STEP(CTRL, ROWS)                                                                 \
  h = max(h, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(h), CTRL, \
                                                               ROWS, 0xf, false)));
  SCH_STEP(kDppRowShr + 1, 0xf)
  SCH_STEP(kDppRowShr + 2, 0xf)
  SCH_STEP(kDppRowShr + 4, 0xf)
  SCH_STEP(kDppRowShr + 8, 0xf)
  SCH_STEP(kDppRowBcast15, 0xa)
  SCH_STEP(kDppRowBcast31, 0xc)
#undef SCH_STEP
  return h;
}
__device__ __forceinline__ int wave_or(int v) {
  v |= dpp_i32<kDppRowShr + 1>(v, 0);
  v |= dpp_i32<kDppRowShr + 2>(v, 0);
  v |= dpp_i32<kDppRowShr + 4>(v, 0);
  v |= dpp_i32<kDppRowShr + 8>(v, 0);
  return __builtin_amdgcn_readlane(v, 15) | __builtin_amdgcn_readlane(v, 31) |
         __builtin_amdgcn_readlane(v, 47) | __builtin_amdgcn_readlane(v, 63);
}

// ---------------------------------------------------------------------------
// Shared memory of the row solver for a workgroup of NT threads (NT a power
// of two, 64..512).  Values cross lanes of one wavefront by DPP and
// ds_bpermute; only what crosses wavefronts goes through LDS.
// ---------------------------------------------------------------------------
template <int NT>
struct RowLds {
  static constexpr int W = NT / kWave;
  // interface equations (A, B, C, R), one per chunk (on one wavefront they stay
  // in its lanes)
  alignas(16) double eq[4][NT > kWave ? NT : 2];
  double etail[3][W];          // last-row spike values of each wavefront's last chunk
  double edge[2][W][6];        // wavefront edge values of halo exchanges, double buffered
  double red[W];               // workgroup sums
  // per-wavefront records of solve_helm(), double buffered: the scans' totals,
  // the factor of the wavefront's rows (ragged grids), and the reduction that
  // rides along
  double hrec[2][W][2];
  double hmul[2][W];
  double hscale[2][W];
  uint32_t hword[2][W];
  // lane factors of solve_helm() on full grids: [0] the model's operator,
  // [1] the Matern-type noise's
  double tab[2][3][kWave];
};

// A row of the periodic mesh is split over the NT threads of a workgroup:
// thread t owns the `cnt` consecutive rows starting at `start`, held in
// register slots 0..cnt-1 (PMAX slots in total).  FULL means cnt == PMAX for
// every thread.
struct Chunk {
  int start, cnt;
};

template <int NT>
__device__ __forceinline__ Chunk chunk_of(int nx, int t) {
  const int base = nx / NT, rem = nx % NT;
  Chunk c;
  c.cnt = base + (t < rem ? 1 : 0);
  c.start = t * base + (t < rem ? t : rem);
  return c;
}

// Rows every chunk holds: chunk_of deals nx / NT or nx / NT + 1 rows, and the
// tiles (tile_for) take 6 slots only when nx > 4 NT, 8 when nx > 6 NT, 12 when
// nx > 8 NT, 16 when nx > 12 NT, and always nx >= NT; the host refuses a tile
// that breaks this.  Slots below kMinRows are live in every chunk, so the masks
// of ragged chunks start there (compile-time true below it).
template <int PMAX>
inline constexpr int kMinRows = PMAX >= 12 ? PMAX - 4 : PMAX >= 6 ? PMAX - 2 : 1;
template <int PMAX, bool FULL>
__device__ __forceinline__ bool slot_live(int j, int cnt) {
  return FULL || j < kMinRows<PMAX> || j < cnt;
}
// slot j is the chunk's last live one
template <int PMAX, bool FULL>
__device__ __forceinline__ bool slot_last(int j, int cnt) {
  return FULL ? j == PMAX - 1 : (j >= kMinRows<PMAX> - 1 && j == cnt - 1);
}

// Value of slot j's left / right neighbour given the halo values.
template <int PMAX, bool FULL>
__device__ __forceinline__ double left_of(const double (&v)[PMAX], int j, double hl) {
  return j == 0 ? hl : v[j > 0 ? j - 1 : 0];
}
template <int PMAX, bool FULL>
__device__ __forceinline__ double right_of(const double (&v)[PMAX], int j, int cnt, double hr) {
  return slot_last<PMAX, FULL>(j, cnt) ? hr : v[j + 1 < PMAX ? j + 1 : PMAX - 1];
}

// Value in the chunk's last active slot.  For ragged chunks a sum of masked
// terms: a select chain over the slots is turned by the compiler into a
// dynamic register index, which moves the whole array to scratch memory.
template <int PMAX, bool FULL>
__device__ __forceinline__ double last_of(const double (&v)[PMAX], int cnt) {
  if (FULL) return v[PMAX - 1];
  double r = 0.0;
#pragma unroll
  for (int j = kMinRows<PMAX> - 1; j < PMAX; ++j) r = fma(j == cnt - 1 ? 1.0 : 0.0, v[j], r);
  return r;
}

// ds_bpermute of a double: every lane reads `v` of lane `src` (0..63).
__device__ __forceinline__ double bperm_f64(double v, int src) {
  const int lo = __builtin_amdgcn_ds_bpermute(src << 2, __double2loint(v));
  const int hi = __builtin_amdgcn_ds_bpermute(src << 2, __double2hiint(v));
  return __hiloint2double(hi, lo);
}

// Periodic neighbour exchange of K values per thread: thread t receives
// last[i] of thread t-1 in fromL[i] and first[i] of thread t+1 in fromR[i]
// (indices mod NT).  Inside a wavefront by whole-wave DPP shifts; the
// wavefront ends go through LDS (one barrier) or, for a single wavefront,
// through readlane.  The edge buffers alternate between calls (hs toggles),
// so a buffer is rewritten only after the barrier of the exchange in between.
template <int NT, int K>
__device__ __forceinline__ void exchange(const double (&first)[K], const double (&last)[K],
                                         double (&fromL)[K], double (&fromR)[K], RowLds<NT>& L,
                                         int t, int& hs) {
  constexpr int W = NT / kWave;
  static_assert(K <= 3, "at most three values per exchange");
  const int lane = t & (kWave - 1);
#pragma unroll
  for (int i = 0; i < K; ++i) {
    fromL[i] = dpp_f64z<kDppWaveShr1>(last[i]);
    fromR[i] = dpp_f64z<kDppWaveShl1>(first[i]);
  }
  if constexpr (W == 1) {
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const double wl = readlane_f64(last[i], kWave - 1), wr = readlane_f64(first[i], 0);
      fromL[i] = lane == 0 ? wl : fromL[i];
      fromR[i] = lane == kWave - 1 ? wr : fromR[i];
    }
  } else {
    const int w = t / kWave;
    if (lane == kWave - 1) {
#pragma unroll
      for (int i = 0; i < K; ++i) L.edge[hs][w][2 * i + 1] = last[i];
    }
    if (lane == 0) {
#pragma unroll
      for (int i = 0; i < K; ++i) L.edge[hs][w][2 * i] = first[i];
    }
    __syncthreads();
    const int wl = (w + W - 1) & (W - 1), wr = (w + 1) & (W - 1);
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const double a = L.edge[hs][wl][2 * i + 1], b = L.edge[hs][wr][2 * i];
      fromL[i] = lane == 0 ? a : fromL[i];
      fromR[i] = lane == kWave - 1 ? b : fromR[i];
    }
    hs ^= 1;
  }
}

// Left and right neighbours of the chunk (periodic).
template <int PMAX, int NT, bool FULL>
__device__ __forceinline__ void halo(const double (&v)[PMAX], int cnt, RowLds<NT>& L, int t,
                                     double& hl, double& hr, int& hs) {
  const double f[1] = {v[0]}, l[1] = {last_of<PMAX, FULL>(v, cnt)};
  double a[1], b[1];
  exchange<NT, 1>(f, l, a, b, L, t, hs);
  hl = a[0];
  hr = b[0];
}

// Partition elimination of the rows 1..E-1 of a run of E consecutive rows
// whose first unknown z_0 and whose successor z_E (the next run's z_0) are
// kept: on exit z_j = y[j] + g[j] z_0 + k[j] z_E for j = 1..E-1.  The
// coefficient arrays are indexed by the run's rows.
// `grow` receives the running maximum of the eliminated super-diagonal
// |c'_j| = |C_j / pivot_j| (see cyclic_solve).
template <int E>
__device__ __forceinline__ void spike_eliminate(const double (&A)[E], const double (&B)[E],
                                                const double (&C)[E], const double (&R)[E],
                                                double (&y)[E], double (&g)[E], double (&k)[E],
                                                double& grow) {
  double cp[E];
  double cprev = 0.0, yprev = 0.0, gprev = 1.0;
#pragma unroll
  for (int j = 1; j < E; ++j) {
    const double inv = rcp64(j == 1 ? B[j] : B[j] - A[j] * cprev);
    cp[j] = C[j] * inv;
    grow = vmax_abs(grow, cp[j]);
    y[j] = (j == 1 ? R[j] : R[j] - A[j] * yprev) * inv;
    g[j] = (j == 1 ? -A[j] : -A[j] * gprev) * inv;
    cprev = cp[j];
    yprev = y[j];
    gprev = g[j];
  }
  double yn = 0.0, gn = 0.0, kn = 1.0;
#pragma unroll
  for (int j = E - 1; j >= 1; --j) {
    y[j] = y[j] - cp[j] * yn;
    g[j] = g[j] - cp[j] * gn;
    k[j] = -cp[j] * kn;
    yn = y[j];
    gn = g[j];
    kn = k[j];
  }
}

// The interface equations A s_prev + B s + C s_next = R are close to diagonal
// where chunks are long: a coupling falls by a factor per row (0.41 at the
// 4096-node workloads, so 5e-7 over 16 rows).  Where every |A| + |C| is below
// eps |B|, K sweeps s <- (R - A s_prev - C s_next) / B from s = R / B leave an
// error below eps^(K+1) of the largest unknown within K + 1 equations; these
// bounds give 2^-57, a sixteenth of the rounding of the result.  (2^-60, from
// which on the reduction follows couplings, changed no error against 64 bits and
// cost the windows and the adjoint 1%.)
constexpr double kSweep2 = 0x1.0p-19, kSweep4 = 3.4e-4, kSweep6 = 3.4e-3;
// Sweeps that the wavefront's equations s + a s_prev + c s_next = z take; 0 if
// six are not enough.
__device__ __forceinline__ int sweeps_for(double a, double c) {
  const double e = fabs(a) + fabs(c);
  if (!__any(!(e <= kSweep2))) return 2;
  if (!__any(!(e <= kSweep4))) return 4;
  return __any(!(e <= kSweep6)) ? 0 : 6;
}

// Whether a pivot is 16 times smaller than a coupling of its equation, or more
// (where the rows are diagonally dominant none is smaller at all): eliminating
// with it would drown the neighbours.  On the high words of what is there
// before the reciprocal: compared in FP64, or taken from the quotients, it cost
// the adjoint and the forecast 2%.
__device__ __forceinline__ bool drowns(double pivot, double a, double c) {
  const auto word = [](double v) {
    return static_cast<uint32_t>(__double2hiint(v)) & 0x7fffffffu;
  };
  return max(word(a), word(c)) >= word(pivot) + 0x400000u;
}
__device__ __forceinline__ double nan_if(bool bad, double v) {
  return bad ? __hiloint2double(0x7ff80000, __double2loint(v)) : v;
}

// The same system over the 64 lanes of one wavefront, lane l holding equation
// l (periodic): sweeps where they suffice, cyclic reduction levels (which
// square the couplings and double the distance d of the coupled lanes) until
// they do.  The first level moves its values by lane rotations; the farther
// ones by ds_bpermute.  Returns s of the lane.
__device__ __forceinline__ double interface_wave(double A, double B, double C, double R,
                                                 int lane) {
  auto level = [&](auto prev, auto next) {
    const double Am = prev(A), Bm = prev(B), Cm = prev(C), Rm = prev(R);
    const double Ap = next(A), Bp = next(B), Cp = next(C), Rp = next(R);
    const double q1 = A * rcp64(Bm), q2 = C * rcp64(Bp);
    A = -q1 * Am;
    B = B - q1 * Cm - q2 * Ap;
    C = -q2 * Cp;
    R = R - q1 * Rm - q2 * Rp;
  };
  double s = 0.0;
  // true, with s set, if the couplings are small enough for sweeps
  auto sweep = [&](auto prev, auto next) {
    const double e = fabs(A) + fabs(C), b = fabs(B);
    if (__any(!(e <= kSweep4 * b))) return false;
    const bool four = __any(!(e <= kSweep2 * b));
    const double inv = rcp64(B), a = A * inv, c = C * inv, z = R * inv;
    s = z;
#pragma unroll
    for (int k = 0; k < 2; ++k) s = fma(-a, prev(s), fma(-c, next(s), z));
    if (four) {
#pragma unroll
      for (int k = 0; k < 2; ++k) s = fma(-a, prev(s), fma(-c, next(s), z));
    }
    return true;
  };
  {
    auto prev = [](double v) { return wave_prev(v); };
    auto next = [](double v) { return wave_next(v); };
    if (sweep(prev, next)) return s;
    level(prev, next);
  }
#pragma unroll 1
  for (int d = 2; d < kWave; d <<= 1) {
    const int lm = (lane - d) & (kWave - 1), lp = (lane + d) & (kWave - 1);
    auto prev = [&](double v) { return bperm_f64(v, lm); };
    auto next = [&](double v) { return bperm_f64(v, lp); };
    if (sweep(prev, next)) return s;
    level(prev, next);
  }
  // after every level each equation couples s_l to itself only
  return R * rcp64(A + B + C);
}

// Solve of the periodic tridiagonal interface system of the NT chunks,
//   A_t s_{t-1} + B_t s_t + C_t s_{t+1} = R_t   (t mod NT),
// redundantly by every wavefront: lane l holds the E = NT/64 consecutive
// equations E l .. E l + E - 1 in eA..eR, eliminates all but the first by
// the partition method, and the 64 remaining equations (one per lane,
// periodic) are solved by interface_wave().  Returns, for the calling thread
// t = 64 w + lane, s_t, s_{t+1} and s_{t-1}.  For NT > 64 where couplings are
// too strong for sweeps across the chunks themselves (short chunks, large
// dv).
template <int NT>
__device__ __forceinline__ void interface_solve(const double (&eA)[NT / kWave],
                                                const double (&eB)[NT / kWave],
                                                const double (&eC)[NT / kWave],
                                                const double (&eR)[NT / kWave], int t, double& s,
                                                double& snext, double& sprev, double& grow) {
  constexpr int E = NT / kWave;
  static_assert(E > 1, "several wavefronts");
  const int lane = t & (kWave - 1);
  double y[E], g[E], k[E];
  y[0] = 0.0;
  g[0] = 1.0;
  k[0] = 0.0;
  spike_eliminate<E>(eA, eB, eC, eR, y, g, k, grow);
  // run tails: the last unknown in terms of (z_0, z_E); first interior row
  const double yT = y[E - 1], gT = g[E - 1], kT = k[E - 1];
  const double y1 = y[1], g1 = g[1], k1 = k[1];
  // tails of lane l-1 (periodic over the 64 lanes)
  double pY = dpp_f64z<kDppWaveShr1>(yT), pG = dpp_f64z<kDppWaveShr1>(gT),
         pK = dpp_f64z<kDppWaveShr1>(kT);
  {
    const double wy = readlane_f64(yT, kWave - 1), wg = readlane_f64(gT, kWave - 1),
                 wk = readlane_f64(kT, kWave - 1);
    pY = lane == 0 ? wy : pY;
    pG = lane == 0 ? wg : pG;
    pK = lane == 0 ? wk : pK;
  }
  const double A = eA[0] * pG;
  const double B = fma(eA[0], pK, fma(eC[0], g1, eB[0]));
  const double C = eC[0] * k1;
  const double R = fma(-eA[0], pY, fma(-eC[0], y1, eR[0]));
  const double z = interface_wave(A, B, C, R, lane);
  // the run's unknowns
  const double zn = [&] {
    const double v = dpp_f64z<kDppWaveShl1>(z), w0 = readlane_f64(z, 0);
    return lane == kWave - 1 ? w0 : v;
  }();
  double zr[E];
  zr[0] = z;
#pragma unroll
  for (int e = 1; e < E; ++e) zr[e] = fma(k[e], zn, fma(g[e], z, y[e]));
  // thread t = 64 w + lane owns unknown t, held by lane t / E, slot lane % E
  const int wu = __builtin_amdgcn_readfirstlane(t / kWave);
  const int src = (kWave / E) * wu + lane / E;
  double sv = bperm_f64(zr[0], src);
#pragma unroll
  for (int e = 1; e < E; ++e) {
    const double v = bperm_f64(zr[e], src);
    sv = (lane % E) == e ? v : sv;
  }
  s = sv;
  {
    const double v = dpp_f64z<kDppWaveShl1>(sv);
    const double w = readlane_f64(zr[0], ((kWave / E) * (wu + 1)) & (kWave - 1));
    snext = lane == kWave - 1 ? w : v;
  }
  {
    const double v = dpp_f64z<kDppWaveShr1>(sv);
    const double w = readlane_f64(zr[E - 1], ((kWave / E) * wu + kWave - 1) & (kWave - 1));
    sprev = lane == 0 ? w : v;
  }
}

// Workgroup solve of the periodic tridiagonal system
//     a_i x_{i-1} + b_i x_i + c_i x_{i+1} = d_i   (indices mod nx)
// distributed as chunks of rows per thread.  Partition method: the first row
// of every chunk is an interface unknown s_t; each thread eliminates its
// remaining rows by Thomas' algorithm into x_j = y_j + g_j s_t + k_j s_{t+1}
// (two spike columns), the interface rows form a periodic tridiagonal system
// of NT unknowns, solved behind one barrier by a few sweeps of every wavefront
// over its own unknowns and its neighbours' halves, or by interface_solve()
// where the couplings are too strong for that (above about 0.2), and the chunk
// is recombined.  row(j, a, b, c) returns the coefficients of local slot j and
// d(j) its right-hand side (both evaluated once per slot).  xl and xr receive
// the solution at the row before the chunk and the row after it (the halo of
// x, from the interface values, without another exchange).
//
// The pivots' reciprocals (rcp64) do not exclude small ones: an elimination
// that meets them grows its eliminated super-diagonal, which is measured.
// No pivoting.  The mass and Helmholtz matrices are symmetric positive
// definite and diagonally dominant.  A row of the implicit-midpoint matrix,
// (o - v_-, d + v_+ - v_-, o + v_+) with o = h/6 - mu dt/(2h),
// d = 2h/3 + mu dt/h (so d + 2o = h) and v_-+ = dv_{i-+1}/4, is diagonally
// dominant whenever |dv| / 4 <= |o| everywhere and, for o < 0, the
// compression dv_{i-1} - dv_{i+1} stays below 2h; without pivoting the LU
// factors then satisfy |L||U| <= 3|A|.  Outside that range (steep or very
// large dv) the elimination can still be accurate, and its growth is
// measured instead: row j of |L||U| is bounded by |A|'s row plus
// 2 |a_j| |c'_{j-1}|, c'_j = c_j / pivot_j the eliminated super-diagonal, so
// the solution's error grows about like max |c'| times the unit roundoff
// (near-zero pivots of a compressive saw-tooth dv: max |c'| = 250 gives a
// relative error of 1e-14, 2.5e5 gives 6e-13, 2.5e8 gives 6e-10).  `grow`
// receives the running maximum of |c'_j| over the chunk's rows and
// interface_solve()'s eliminations, and callers reject a system whose growth
// exceeds kMaxGrowth = 2^16 (errors below about 1e-12).
constexpr double kMaxGrowth = 65536.0;
#ifndef SCH_SWEEP_FENCE
#define SCH_SWEEP_FENCE 4
#endif
template <int PMAX, int NT, bool FULL, class RowF, class DF>
__device__ __forceinline__ void cyclic_solve(RowF row, DF d, double (&x)[PMAX], int cnt,
                                             RowLds<NT>& L, int t, double& xl, double& xr,
                                             double& grow) {
  static_assert(PMAX >= 2, "need at least two rows per thread");
  constexpr int W = NT / kWave;
  const int lane = t & (kWave - 1);
  double cp[PMAX], g[PMAX];
  // forward elimination over the interior slots 1..cnt-1; inactive slots
  // (j >= cnt) are given c' = -1, y' = g' = 0 so the back sweep passes the
  // right-spike seed (k = 1) and zeros through them unchanged.
  double cprev = 0.0, yprev = 0.0, gprev = 1.0;
#pragma unroll
  for (int j = 1; j < PMAX; ++j) {
    double a, b, c;
    row(j, a, b, c);
    // slot 1 starts the recurrences (c' = y' = 0, g' = 1 before it)
    const double inv = rcp64(j == 1 ? b : b - a * cprev);
    double cj = c * inv, yj = (j == 1 ? d(j) : d(j) - a * yprev) * inv,
           gj = (j == 1 ? -a : -a * gprev) * inv;
    if (!slot_live<PMAX, FULL>(j, cnt)) {
      cj = -1.0;
      yj = 0.0;
      gj = 0.0;
    }
    grow = vmax_abs(grow, cj);
    cp[j] = cj;
    x[j] = yj;
    g[j] = gj;
    cprev = cj;
    yprev = yj;
    gprev = gj;
    // bound the scheduler's look-ahead: rows hoisted from far ahead of the
    // recurrence would each hold four registers pairs
    if (j % SCH_SWEEP_FENCE == 0) __builtin_amdgcn_sched_barrier(0);
  }
  // back substitution for y and both spikes; the right spike k_j is the
  // running product of -c'_i over i = j..PMAX-1 and is rebuilt when needed
  double yn = 0.0, gn = 0.0, kn = 1.0;
  double yL = 0.0, gL = 1.0, kL = 0.0;  // last row of the chunk (the interface if cnt == 1)
#pragma unroll
  for (int j = PMAX - 1; j >= 1; --j) {
    const double yj = x[j] - cp[j] * yn;
    const double gj = g[j] - cp[j] * gn;
    const double kj = -cp[j] * kn;
    x[j] = yj;
    g[j] = gj;
    yn = yj;
    gn = gj;
    kn = kj;
    if (!FULL && slot_last<PMAX, FULL>(j, cnt)) {
      yL = yj;
      gL = gj;
      kL = kj;
    }
    if (FULL && j == PMAX - 1) {
      yL = yj;
      gL = gj;
      kL = kj;
    }
  }
  // interface equation of chunk t: a0 x_{-1} + b0 s_t + c0 x_1 = d0 with
  // x_{-1} = ypl + gpl s_{t-1} + kpl s_t (thread t-1's last row) and
  // x_1 = yn + gn s_t + kn s_{t+1}
  double ypl = dpp_f64z<kDppWaveShr1>(yL), gpl = dpp_f64z<kDppWaveShr1>(gL),
         kpl = dpp_f64z<kDppWaveShr1>(kL);
  double a0, b0, c0;
  row(0, a0, b0, c0);
  const double Bp = fma(c0, gn, b0), Rp = fma(-c0, yn, d(0)), C = c0 * kn;
  double s, snext, sprev;
  if constexpr (W == 1) {
    const double wy = readlane_f64(yL, kWave - 1), wg = readlane_f64(gL, kWave - 1),
                 wk = readlane_f64(kL, kWave - 1);
    ypl = lane == 0 ? wy : ypl;
    gpl = lane == 0 ? wg : gpl;
    kpl = lane == 0 ? wk : kpl;
    s = interface_wave(a0 * gpl, fma(a0, kpl, Bp), C, fma(-a0, ypl, Rp), lane);
    snext = wave_next(s);
    sprev = wave_prev(s);
  } else {
    // the equation of each wavefront's first chunk goes to LDS without its
    // left-tail terms (A holds a0); the reader completes it from L.etail
    const int w = t / kWave;
    const bool firstlane = lane == 0;
    L.eq[0][t] = firstlane ? a0 : a0 * gpl;
    L.eq[1][t] = firstlane ? Bp : fma(a0, kpl, Bp);
    L.eq[2][t] = C;
    L.eq[3][t] = firstlane ? Rp : fma(-a0, ypl, Rp);
    if (lane == kWave - 1) {
      L.etail[0][w] = yL;
      L.etail[1][w] = gL;
      L.etail[2][w] = kL;
    }
    __syncthreads();
    // Each wavefront takes its own equations and 32 on either side, lane l the
    // two from 64 w - 32 + 2 l on (with two wavefronts that is the whole
    // ring).  The odd ones are eliminated, which squares the couplings, and
    // the 64 even ones swept; what is wrong at the window's ends stays out of
    // the sweeps' reach of the unknowns taken (lanes 15..48).
    typedef double d2 __attribute__((ext_vector_type(2)));
    const int wp = (w + W - 1) & (W - 1);
    const int n0 = (kWave * w + NT - 32 + 2 * lane) & (NT - 1);
    d2 eA = *reinterpret_cast<const d2*>(&L.eq[0][n0]), eB = *reinterpret_cast<const d2*>(&L.eq[1][n0]);
    const d2 eC = *reinterpret_cast<const d2*>(&L.eq[2][n0]);
    d2 eR = *reinterpret_cast<const d2*>(&L.eq[3][n0]);
    {
      const int q = lane < 32 ? wp : w;
      const double ty = L.etail[0][q], tg = L.etail[1][q], tk = L.etail[2][q];
      if ((lane & 31) == 16) {  // the first equations of this wavefront and the next
        eB.x = fma(eA.x, tk, eB.x);
        eR.x = fma(-eA.x, ty, eR.x);
        eA.x *= tg;
      }
      if (firstlane) {
        ypl = ty;
        gpl = tg;
        kpl = tk;
      }
    }
    //
    // This eliminates in another order than interface_solve(), which measures
    // its growth; its own is bounded instead: a pivot that drowns() the
    // neighbours makes them not a number, which sweeps_for() refuses, and the
    // system is left to interface_solve().  (Even couplings of 3e5 cost 1e-8 of
    // the solution where that one errs by 1e-13, and it may not meet at all an
    // odd pivot that would have to be refused here.)
    const double i1 = nan_if(drowns(eB.y, eA.y, eC.y), rcp64(eB.y));
    const double y = eR.y * i1, g1 = -eA.y * i1, k1 = -eC.y * i1;
    double a, c, z;
    {
      const double py = wave_prev(y), pg = wave_prev(g1), pk = wave_prev(k1);
      const double inv = rcp64(fma(eA.x, pk, fma(eC.x, g1, eB.x)));
      a = eA.x * pg * inv;
      c = eC.x * k1 * inv;
      z = fma(-eA.x, py, fma(-eC.x, y, eR.x)) * inv;
    }
    double v = z;
    int sweeps = sweeps_for(a, c);
    bool swept = sweeps != 0;
    if (swept) {
#pragma unroll 1
      for (; sweeps > 0; sweeps -= 2) {
#pragma unroll
        for (int i = 0; i < 2; ++i) v = fma(-a, wave_prev(v), fma(-c, wave_next(v), z));
      }
    } else {
      // one level of cyclic reduction: the couplings squared again, to the
      // lanes two away
      a = nan_if(drowns(1.0, a, c), a);
      const double am = wave_prev(a), cm = wave_prev(c), zm = wave_prev(z);
      const double ap = wave_next(a), cpn = wave_next(c), zp = wave_next(z);
      const double inv = rcp64(fma(-a, cm, fma(-c, ap, 1.0)));
      z = fma(-a, zm, fma(-c, zp, z)) * inv;
      a = -a * am * inv;
      c = -c * cpn * inv;
      v = z;
      sweeps = sweeps_for(a, c);
      swept = sweeps != 0;
#pragma unroll 1
      for (; sweeps > 0; --sweeps)
        v = fma(-a, wave_prev(wave_prev(v)), fma(-c, wave_next(wave_next(v)), z));
    }
    if (swept) {
      const double o = fma(k1, wave_next(v), fma(g1, v, y));  // the odd unknowns
      const int src = 16 + lane / 2;
      const double se = bperm_f64(v, src), so = bperm_f64(o, src);
      s = (lane & 1) ? so : se;
      const double sl = readlane_f64(o, 15), sr = readlane_f64(v, 48);
      sprev = wave_prev(s);
      snext = wave_next(s);
      sprev = firstlane ? sl : sprev;
      snext = lane == kWave - 1 ? sr : snext;
    } else {
      double fA[W], fB[W], fC[W], fR[W];
#pragma unroll
      for (int e = 0; e < W; ++e) {
        fA[e] = L.eq[0][W * lane + e];
        fB[e] = L.eq[1][W * lane + e];
        fC[e] = L.eq[2][W * lane + e];
        fR[e] = L.eq[3][W * lane + e];
      }
      {
        // equation W*lane is the first of a wavefront when (W*lane) % 64 == 0
        const int wq = ((W * lane) / kWave + W - 1) & (W - 1);
        const double ty = L.etail[0][wq], tg = L.etail[1][wq], tk = L.etail[2][wq];
        const bool first = ((W * lane) & (kWave - 1)) == 0;
        const double a1 = fA[0];
        fA[0] = first ? a1 * tg : fA[0];
        fB[0] = first ? fma(a1, tk, fB[0]) : fB[0];
        fR[0] = first ? fma(-a1, ty, fR[0]) : fR[0];
      }
      interface_solve<NT>(fA, fB, fC, fR, t, s, snext, sprev, grow);
    }
  }
  // last row of chunk t-1: y + g s_{t-1} + k s_t with its tail values
  xl = fma(kpl, s, fma(gpl, sprev, ypl));
  xr = snext;
  x[0] = s;
  double kr = 1.0;
#pragma unroll
  for (int j = PMAX - 1; j >= 1; --j) {
    kr *= -cp[j];
    x[j] = x[j] + g[j] * s + kr * snext;
  }
}

// The same for the constant symmetric positive definite systems (no growth
// to watch).
template <int PMAX, int NT, bool FULL, class RowF, class DF>
__device__ __forceinline__ void cyclic_solve(RowF row, DF d, double (&x)[PMAX], int cnt,
                                             RowLds<NT>& L, int t, double& xl, double& xr) {
  double grow = 0.0;
  cyclic_solve<PMAX, NT, FULL>(row, d, x, cnt, L, t, xl, xr, grow);
}

template <int NT>
__device__ __forceinline__ double block_sum(double a, RowLds<NT>& L, int t) {
  a = wave_sum(a);
  if ((t & (kWave - 1)) == 0) L.red[t / kWave] = a;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < NT / kWave; ++i) s += L.red[i];
  __syncthreads();
  return s;
}

}  // namespace sch
