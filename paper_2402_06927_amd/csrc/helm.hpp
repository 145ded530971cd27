// helm.hpp -- workgroup solve of the constant periodic Helmholtz system
// H u = f (or H u = M f), H = d I + o (S + S^{-1}) (S the cyclic shift; d = 2h/3 + 2 alpha^2/h,
// o = h/6 - alpha^2/h from the first line of eq. fde1), in one barrier.
//
// H factors as kappa (1 - r S)(1 - r S^{-1}) with r the root of modulus < 1 of
// r^2 + (d/o) r + 1 = 0 and kappa = -o/r, so
//   H^{-1} f = (F+ + F- - f) / (kappa (1 - r^2)),
// where F+ and F- are the periodic solutions of the first-order recurrences
// F+_i = f_i + r F+_{i-1} and F-_i = f_i + r F-_{i+1}.  Both recurrences are
// linear scans: each thread scans its chunk, the chunk carries are combined
// across lanes by DPP row shifts and readlane and across wavefronts through
// one LDS record per wavefront; the carry into a wavefront is the sum over all
// wavefronts' totals in cyclic order, its own the farthest, over 1 - r^N.  The
// record also carries a reduction (HelmRed), so a caller can fold a workgroup
// maximum into the same barrier.
#pragma once

#include "device.hpp"

namespace sch {

struct HelmConst {
  double r, coef;   // root and 1/(kappa (1 - r^2)), kappa = -o / r
  double rN1;       // 1/(1 - r^nx)
  double rb, rb1;   // r^base, r^(base+1): multipliers of chunks of base / base+1 rows
  int base;         // nx / NT
  double ho, hd;    // off-diagonal and diagonal of H
  double iho;       // 1 / ho
  // The mass matrix M (rows h/6, 2h/3, h/6) lies in the span of I and H:
  // M = beta H + gamma I with beta = (h/6) / ho, gamma = 2h/3 - beta hd, so
  // H^{-1} M f = beta f + gamma H^{-1} f = mg (F+ + F-) + mf f with
  // mg = gamma coef and mf = beta - gamma coef (the scan form below).
  double mg, mf;
  double mh6, mh23;  // h/6 and 2h/3
  double pwt[65];  // rb^e for e = 0..64: the lane scans' factors on full grids
};

// Composition of affine carries: apply (m1, c1) then (m2, c2).
__device__ __forceinline__ void compose(double m1, double c1, double m2, double c2, double& m,
                                        double& c) {
  m = m1 * m2;
  c = fma(m2, c1, c2);
}

// Inclusive affine scan inside each 16-lane row: CTRL = row shift right
// (forward: compose the lanes to the left first) or left (backward: the
// lanes to the right first).
template <int CTRL>
__device__ __forceinline__ void scan_rows(double& m, double& c) {
#pragma unroll
  for (int d = 1; d < 16; d <<= 1) {
    double pm, pc;
    if (d == 1) { pm = dpp_f64<CTRL + 1>(m, 1.0); pc = dpp_f64z<CTRL + 1>(c); }
    else if (d == 2) { pm = dpp_f64<CTRL + 2>(m, 1.0); pc = dpp_f64z<CTRL + 2>(c); }
    else if (d == 4) { pm = dpp_f64<CTRL + 4>(m, 1.0); pc = dpp_f64z<CTRL + 4>(c); }
    else { pm = dpp_f64<CTRL + 8>(m, 1.0); pc = dpp_f64z<CTRL + 8>(c); }
    compose(pm, pc, m, c, m, c);
  }
}

// Lane factors of the scans on full grids, where every chunk has PMAX rows and
// the factor of any run of e chunks is rb^e: [0] joins the odd rows of 16
// lanes to the row before, [1] the upper 32 lanes to the lower, [2] the lane's
// distance from the wavefront's first.  The backward scans read the same
// tables mirrored.  In LDS, because in registers they are 12 a thread for the
// whole kernel, and the kernels have none to spare.
__device__ __forceinline__ void helm_table(const HelmConst& K, double (&tab)[3][kWave], int t) {
  if (t < kWave) {
    tab[0][t] = (t & 16) ? K.pwt[(t & 15) + 1] : 0.0;
    tab[1][t] = t >= 32 ? K.pwt[t - 31] : 0.0;
    tab[2][t] = K.pwt[t];
  }
}

// Reduction that rides on a solve's barrier: in, the thread's share of the
// change (and of the scale, on the first iteration, when `first`) and whether
// its elimination failed; out, the workgroup's word, the same in every
// thread: kUnstable if an elimination failed anywhere, at least kNonfinite if
// the right-hand side holds a value that is not finite, else the high word of
// an upper bound within 2^-20 of the maximum change; and the maximum scale.
struct HelmRed {
  double diff, scale;
  bool bad, first;
  uint32_t word;
};
constexpr uint32_t kUnstable = 0xffffffffu, kNonfinite = 0x7ff00000u;

// MASS: u = H^{-1} M f instead of H^{-1} f, with fl, fr the values of f at
// the nodes bordering the chunk (for the bordering values of u).  tab: the
// operator's lane factors (helm_table; read on full grids).
//
// Per chunk and direction one scan for the carry out of it, the lanes' scan of
// those carries, the wavefronts' totals through LDS behind one barrier, and
// the scan again from the carry into the chunk.  What bounds it is the number
// of vector instructions (about 65 besides the rows' own on full grids, 150
// when the records were scanned across lanes with their maxima and the rows of
// 16 lanes joined by selects), so the periodic sum over the wavefronts is a
// plain Horner sum that every lane forms for itself from the records, read
// from LDS in the wavefront's own rotation.
template <int PMAX, int NT, bool FULL, bool MASS = false, bool RED = false>
__device__ __forceinline__ void solve_helm(const HelmConst& K, const double (&tab)[3][kWave],
                                           const double (&f)[PMAX], double (&u)[PMAX], double& uL,
                                           double& uR, int cnt, RowLds<NT>& L, int slot, int t,
                                           HelmRed& R, double fl = 0.0, double fr = 0.0) {
  constexpr int W = NT / kWave;
  const int lane = t & (kWave - 1), wv = t / kWave;
  const double r = K.r;
  // carries out of the chunk: the local forward scan at its last node and
  // the local backward scan at its first node
  double fc = f[0], bc = FULL ? f[PMAX - 1] : 0.0;
#pragma unroll
  for (int j = 1; j < PMAX; ++j) fc = slot_live<PMAX, FULL>(j, cnt) ? fma(r, fc, f[j]) : fc;
#pragma unroll
  for (int j = FULL ? PMAX - 2 : PMAX - 1; j >= 0; --j) bc = slot_live<PMAX, FULL>(j, cnt) ? fma(r, bc, f[j]) : bc;
  uint32_t word = 0;
  if constexpr (RED) word = wave_max_word(R.diff);
  // inclusive scans over the wavefront, then the exclusive carries (xf*, xb*)
  double xfm, xfc, xbm, xbc, tm;
  if constexpr (FULL) {
    const double rb = K.rb, rb2 = K.pwt[2], rb4 = K.pwt[4], rb8 = K.pwt[8];
    const int ml = kWave - 1 - lane;
    const double a1 = tab[0][lane], a2 = tab[1][lane], b1 = tab[0][ml], b2 = tab[1][ml];
    xfm = tab[2][lane];
    xbm = tab[2][ml];
    tm = K.pwt[64];
    fc = fma(rb, dpp_f64z<kDppRowShr + 1>(fc), fc);
    bc = fma(rb, dpp_f64z<kDppRowShl + 1>(bc), bc);
    fc = fma(rb2, dpp_f64z<kDppRowShr + 2>(fc), fc);
    bc = fma(rb2, dpp_f64z<kDppRowShl + 2>(bc), bc);
    fc = fma(rb4, dpp_f64z<kDppRowShr + 4>(fc), fc);
    bc = fma(rb4, dpp_f64z<kDppRowShl + 4>(bc), bc);
    fc = fma(rb8, dpp_f64z<kDppRowShr + 8>(fc), fc);
    bc = fma(rb8, dpp_f64z<kDppRowShl + 8>(bc), bc);
    // rows of 16 in pairs, then halves (the factors of the lanes that take
    // nothing are 0; there is no backward broadcast, so its sources go
    // through scalar registers)
    const double h0 = readlane_f64(bc, 16), h2 = readlane_f64(bc, 48);
    fc = fma(a1, dpp_f64z<kDppRowBcast15>(fc), fc);
    bc = fma(b1, lane < 32 ? h0 : h2, bc);
    const double h1 = readlane_f64(bc, 32);
    fc = fma(a2, dpp_f64z<kDppRowBcast31>(fc), fc);
    bc = fma(b2, h1, bc);
  } else {
    // Hillis-Steele steps inside each 16-lane row by DPP row shifts (identity
    // where the row has no partner), then the rows are joined with the row
    // results read from the row ends into scalar registers.
    const double mth = cnt == K.base ? K.rb : K.rb1;
    const int row = lane >> 4;
    double fm = mth, bm = mth;
    scan_rows<kDppRowShr>(fm, fc);
    scan_rows<kDppRowShl>(bm, bc);
    {
      const double r0m = readlane_f64(fm, 15), r0c = readlane_f64(fc, 15);
      const double r1m = readlane_f64(fm, 31), r1c = readlane_f64(fc, 31);
      const double r2m = readlane_f64(fm, 47), r2c = readlane_f64(fc, 47);
      double p2m, p2c, p3m, p3c;
      compose(r0m, r0c, r1m, r1c, p2m, p2c);
      compose(p2m, p2c, r2m, r2c, p3m, p3c);
      const double pm = row == 0 ? 1.0 : row == 1 ? r0m : row == 2 ? p2m : p3m;
      const double pc = row == 0 ? 0.0 : row == 1 ? r0c : row == 2 ? p2c : p3c;
      compose(pm, pc, fm, fc, fm, fc);
      const double t1m = readlane_f64(bm, 16), t1c = readlane_f64(bc, 16);
      const double t2m = readlane_f64(bm, 32), t2c = readlane_f64(bc, 32);
      const double t3m = readlane_f64(bm, 48), t3c = readlane_f64(bc, 48);
      double h1m, h1c, h0m, h0c;
      compose(t3m, t3c, t2m, t2c, h1m, h1c);
      compose(h1m, h1c, t1m, t1c, h0m, h0c);
      const double hm = row == 3 ? 1.0 : row == 2 ? t3m : row == 1 ? h1m : h0m;
      const double hc = row == 3 ? 0.0 : row == 2 ? t3c : row == 1 ? h1c : h0c;
      compose(hm, hc, bm, bc, bm, bc);
    }
    // exclusive factors within the wavefront (identity at the ends)
    xfm = dpp_f64<kDppWaveShr1>(fm, 1.0);
    xbm = dpp_f64<kDppWaveShl1>(bm, 1.0);
    tm = fm;  // lane 63: the wavefront's
  }
  xfc = dpp_f64z<kDppWaveShr1>(fc);
  xbc = dpp_f64z<kDppWaveShl1>(bc);
  if constexpr (RED) {
    // the wavefront's forward total (lane 63) is finite iff every f_j is
    word = fabs(fc) <= 1.7976931348623157e308 ? word : kNonfinite;
    if (__any(R.bad)) word = kUnstable;
  }
  double scale = 0.0;
  if (RED && R.first) scale = wave_max(R.scale);
  // carries into the wavefront: the periodic sums over all wavefronts' totals,
  // farthest (its own) first, over 1 - r^N
  double cf, cb;
  if constexpr (W == 1) {
    cf = readlane_f64(fc, kWave - 1);
    cb = readlane_f64(bc, 0);
    if constexpr (RED) {
      R.word = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(word), kWave - 1));
      R.scale = scale;
    }
  } else {
    if (lane == kWave - 1) {
      L.hrec[slot][wv][0] = fc;
      if constexpr (!FULL) L.hmul[slot][wv] = tm;
      if constexpr (RED) {
        L.hword[slot][wv] = word;
        if (R.first) L.hscale[slot][wv] = scale;
      }
    }
    if (lane == 0) L.hrec[slot][wv][1] = bc;
    __syncthreads();
    const int w0 = __builtin_amdgcn_readfirstlane(wv);
    double rf[W], rbk[W], rm[W];
#pragma unroll
    for (int i = 0; i < W; ++i) {
      const int v = (w0 + i) & (W - 1);
      rf[i] = L.hrec[slot][v][0];
      rbk[i] = L.hrec[slot][v][1];
      rm[i] = FULL ? tm : L.hmul[slot][v];
    }
    if constexpr (RED) {
      uint32_t m = L.hword[slot][0];
#pragma unroll
      for (int i = 1; i < W; ++i) m = max(m, L.hword[slot][i]);
      R.word = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(m)));
      if (R.first) {
        R.scale = L.hscale[slot][0];
#pragma unroll
        for (int i = 1; i < W; ++i) R.scale = vmax(R.scale, L.hscale[slot][i]);
      }
    }
    cf = rf[0];
    cb = rbk[0];
#pragma unroll
    for (int i = 1; i < W; ++i) {
      cf = fma(rm[i], cf, rf[i]);
      cb = fma(rm[W - i], cb, rbk[W - i]);
    }
  }
  // thread-exclusive carries, at the nodes bordering the chunk
  const double Ep = fma(xfm, cf * K.rN1, xfc);
  const double Em = fma(xbm, cb * K.rN1, xbc);
  // the global scans inside the chunk, rerun from the carries into it:
  // F+_j = f_j + r F+_{j-1} from F+_{start-1} = Ep, F-_j = f_j + r F-_{j+1}
  // from F-_{end+1} = Em; u_j = coef (F+_j + F-_j - f_j)
  double acc = Ep;
#pragma unroll
  for (int j = 0; j < PMAX; ++j) {
    acc = slot_live<PMAX, FULL>(j, cnt) ? fma(r, acc, f[j]) : acc;
    u[j] = MASS ? acc : acc - f[j];
  }
  acc = Em;
#pragma unroll
  for (int j = PMAX - 1; j >= 0; --j) {
    acc = slot_live<PMAX, FULL>(j, cnt) ? fma(r, acc, f[j]) : acc;
    u[j] = MASS ? fma(K.mg, u[j] + acc, K.mf * f[j]) : K.coef * (u[j] + acc);
  }
  // bordering values from the Helmholtz rows of the first and last node,
  // o u_{i-1} + d u_i + o u_{i+1} = g_i with g = f, or g = M f (MASS)
  // (meaningful for chunks of >= 2 rows)
  const int last = FULL ? PMAX - 1 : cnt - 1;
  double ul = u[PMAX - 1], ulm = u[PMAX - 2], fla = f[PMAX - 1], flm = f[PMAX - 2];
  if (!FULL) {
#pragma unroll
    for (int j = 1; j < PMAX; ++j)
      if (j >= kMinRows<PMAX> - 1 && j == last) {
        ul = u[j];
        ulm = u[j - 1];
        fla = f[j];
        flm = f[j - 1];
      }
  }
  const double g0 = MASS ? fma(K.mh6, fl + f[1], K.mh23 * f[0]) : f[0];
  const double gl = MASS ? fma(K.mh6, flm + fr, K.mh23 * fla) : fla;
  const double iho = K.iho;
  uL = (g0 - K.hd * u[0] - K.ho * u[1]) * iho;
  uR = (gl - K.hd * ul - K.ho * ulm) * iho;
}

// The same without a reduction.
template <int PMAX, int NT, bool FULL, bool MASS = false>
__device__ __forceinline__ void solve_helm(const HelmConst& K, const double (&tab)[3][kWave],
                                           const double (&f)[PMAX], double (&u)[PMAX], double& uL,
                                           double& uR, int cnt, RowLds<NT>& L, int slot, int t,
                                           double fl = 0.0, double fr = 0.0) {
  HelmRed none{};
  solve_helm<PMAX, NT, FULL, MASS, false>(K, tab, f, u, uL, uR, cnt, L, slot, t, none, fl, fr);
}

}  // namespace sch
