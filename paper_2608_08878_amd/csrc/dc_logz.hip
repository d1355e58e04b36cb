// Exact log-partition of the size-B subset law and the log-probability of a
// kept set (App. C, policy-gradient derivation for Gumbel-top-B), gfx950.
//
// For the scores s_i of one unit's L rows and r_i = s_i / tau:
//   log Z(s, B, tau) = log sum over size-B subsets a of exp(sum_{i in a} r_i)
//                    = log e_B(exp(r_1), ..., exp(r_L)),
// e_B the elementary symmetric polynomial of degree B, and
//   log pi(a | s) = sum_{i in a} r_i - log Z.
//
// Design.  e_B is a Poisson-binomial probability in disguise: for any t, with
// p_i = exp(r_i - t) / (1 + exp(r_i - t)),
//   e_B(exp r) = exp(B t) prod_i (1 + exp(r_i - t)) P(S = B),
// S the number of successes of L independent trials of probabilities p_i.
// t is chosen so that E[S] is close to B; P(S = B) is then of the order of
// 1 / sigma, sigma^2 = sum p_i (1 - p_i), and comes from the characteristic
// function by the trapezoidal rule over M nodes w_k = 2 pi k / M,
//   P(S = B) = (1 / M) sum_k exp(-i w_k B) prod_i (1 + p_i (exp(i w_k) - 1)),
// which is exact up to the aliases P(S = B + n M).  Two tail bounds say how many
// nodes matter: M = 10 + sqrt(100 + 60 sigma^2) past the offset |E[S] - B|
// makes the aliases less than e^-30 (Bernstein), and |phi(w)| <=
// exp(-sigma^2 (1 - cos w)) leaves out the nodes below e^-30: 10 to 13 of them
// for a large sigma, 21 at most (sigma^2 = 15).  The work is about L times 11
// node factors instead of the L K updates of the defining recursion, K =
// min(B, L - B).  Everything but the choice of t is binary64 and no term
// cancels: the node sum's rounding is absolute, about 1e-15 of its zeroth term,
// which is at least a tenth of the sum; log Z is good to about 1e-13 of its terms.
//
// One workgroup per unit, a thread taking every NT-th row.  What bounds it: vector
// instructions, nearly all binary64 (their rate equals that of binary32 here): in the
// call below the vector units issue in 202 k of 258 k cycles (counters); the rest is
// the serial order of statistics, search, coefficients and nodes.  Four rows at a time become the polynomial 1 + e_1 z + .. + e_4 z^4
// in z = exp(i w) - 1, so a row costs a node three operations instead of six;
// the coefficients of up to 4096 rows go through LDS and each wave takes them
// through three nodes at a time, whose powers of z sit in its registers.  (With
// the nodes' products of all rows in every thread's registers instead, the
// kernel spills at four waves per SIMD.)
// Measured (2048 units, L = 8193, B = 2048, tau = 1, standard normal scores):
// 109 us a call (2 steps of the search for t, 11 nodes); the L K recursion in this
// kernel's place, 117 M updates of seven instructions a unit, took 6390 us.  Error
// of log Z against binary64: 6e-16 relative (the binary32 recursion: 2e-10).
//
// The search for t starts at the scores' mean and takes 2-3 Newton steps where the
// scores have one scale (up to 16 for a spread of thousands).  Where no row lies near
// the mean, or Newton does not arrive, search() goes on: from the mean of the rows on
// B's side, then from the order statistics, whose bracket holds at any spread.
// Measured (the call above, 64 rows of every unit masked with float32's lowest value,
// -1e9, -1e4): 142 us each; Newton and bisection alone 2310 (without arriving), 311, 135.
// B t enters the result only by the rows that the sum over x > 0 does not already
// count, so a t in the middle of a wide gap costs no digits.
//
// Two to eight rows kept or evicted: e_K itself, the rows' factors 1 + w z multiplied
// up as far as z^8 (KF fused multiply-adds a row; every term is positive).  Where the K
// rows lie so far apart that the product underflows, the factors q + p z behind t.
// Measured (2048 units, K = 2 and 8): 1025 rows 13 and 19 us, 8193 rows 33 and 39; by
// the nodes above 41 and 43, 110 and 118; by the recursion in binary32 14 and 25, 74 and
// 97.  (That one was also faster for nine rows and more of very short units: 2048 units
// of 65 rows, 16 of them, 13 us against 33 here; of 257 rows 33 and 36.)
//
// One row kept or one row evicted (K = 1, the steady step) is a logsumexp over
// the rows and skips all this.
// Measured (2048 units of 2049 rows): 18-22 us, all of it latency (33 MB are
// read); with one wave per unit it took 47 us.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dc_device.hpp"
#include "dc_kernels.hpp"

#pragma clang fp contract(off)

namespace dc {

namespace {

constexpr int BAND = 4096;               // see logz_ws_bytes
constexpr int CHUNK = 4096;              // rows whose coefficients are in LDS together (32 KB)
constexpr int NGRP = 4;                  // node groups (one wave each, or several with parts of the rows)
constexpr int NPG = 6;                   // nodes of a group, in threes
constexpr int NMAX = NGRP * NPG;         // nodes at most (the bounds above give 21)
constexpr int KR = 8;                    // rows a thread keeps in registers
constexpr int NEWTON = 24;               // steps of the search for t from a mean of the scores (2-3 usual)
constexpr int HALVINGS = 64;             // and from the order statistics
constexpr double MASK_R = 1e4;           // -r of a row that the sum over all rows would lose digits to
constexpr double PI = 0x1.921fb54442d18p+1;

// Sizes of unit u (ragged caches and per-unit budgets: per unit).
struct UnitDims {
  int L, B, nk;
};

__device__ __forceinline__ UnitDims unit_dims(const LogzArgs& a, int u) {
  UnitDims d;
  // device values clamped to the host's bounds (rows [1, L], budgets [1, B])
  const int n = a.unit_len ? a.unit_len[u] + a.len_add : a.L;
  d.L = n < 1 ? 1 : n > a.L ? a.L : n;
  d.B = a.budgets ? (a.budgets[u] < 1 ? 1 : a.budgets[u] > a.B ? a.B : a.budgets[u]) : a.B;
  d.nk = d.B < d.L ? d.B : d.L;
  return d;
}

// e^x for x <= 0 in binary64: x = k ln 2 + f (Cody-Waite), |f| <= ln 2 / 2, the
// exponential series to f^12 / 12! (the next term is below 2^-52).
__device__ __forceinline__ double exp_neg(double x) {
  x = __builtin_fmax(x, -800.0);
  const double k = __builtin_rint(x * 0x1.71547652b82fep+0);
  const double f = __builtin_fma(k, -0x1.a39ef35793c76p-33, __builtin_fma(k, -0x1.62e42fee00000p-1, x));
  double y = 1.0 / 479001600.0;
  y = __builtin_fma(y, f, 1.0 / 39916800.0);
  y = __builtin_fma(y, f, 1.0 / 3628800.0);
  y = __builtin_fma(y, f, 1.0 / 362880.0);
  y = __builtin_fma(y, f, 1.0 / 40320.0);
  y = __builtin_fma(y, f, 1.0 / 5040.0);
  y = __builtin_fma(y, f, 1.0 / 720.0);
  y = __builtin_fma(y, f, 1.0 / 120.0);
  y = __builtin_fma(y, f, 1.0 / 24.0);
  y = __builtin_fma(y, f, 1.0 / 6.0);
  y = __builtin_fma(y, f, 0.5);
  y = __builtin_fma(y, f, 1.0);
  y = __builtin_fma(y, f, 1.0);
  return __builtin_amdgcn_ldexp(y, (int)k);
}

// float32 values (no NaN) as integers of the same order, and back
__device__ __forceinline__ uint32_t order_key(float x) {
  const uint32_t b = __float_as_uint(x);
  return b ^ ((b >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}
__device__ __forceinline__ float order_value(uint32_t k) {
  return __uint_as_float(k ^ ((k >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}

struct Add {
  __device__ double operator()(double x, double y) const { return x + y; }
};
struct Max {
  __device__ double operator()(double x, double y) const { return x > y ? x : y; }
};

template <int CTRL>
__device__ __forceinline__ double dppd(double x) {
  return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xF, 0xF, true),
                          __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ double lane_of(double x, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l),
                          __builtin_amdgcn_readlane(__double2loint(x), l));
}

// Over the wave, uniform result: the 16 lanes of a row by DPP moves (the LDS
// pipe, which lane shuffles share, was what a steady step waited for), then the
// four rows in order.
template <typename Op>
__device__ __forceinline__ double wave_red(double x, Op op) {
  x = op(x, dppd<DPP_XOR1>(x));
  x = op(x, dppd<DPP_XOR2>(x));
  x = op(x, dppd<DPP_HALF_MIRROR>(x));
  x = op(x, dppd<DPP_MIRROR>(x));
  return op(op(op(lane_of(x, 0), lane_of(x, 16)), lane_of(x, 32)), lane_of(x, 48));
}

// Block reductions of N values (fixed order: the lanes' butterfly, then the
// waves in order); every thread receives the results.  buf: N * NT / 64 doubles.
template <int NT, int N, typename Op>
__device__ __forceinline__ void block_red(double (&x)[N], Op op, double* buf) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int j = 0; j < N; ++j) x[j] = wave_red(x[j], op);
  __syncthreads();                       // the readers of an earlier reduction are done
  if (lane == 0)
#pragma unroll
    for (int j = 0; j < N; ++j) buf[j * NW + wave] = x[j];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < N; ++j) {
    double v = buf[j * NW];
    for (int w = 1; w < NW; ++w) v = op(v, buf[j * NW + w]);
    x[j] = v;
  }
}

// E[S] and its variance at t (relative to ref), with binary32 weights.
template <int NT>
__device__ __forceinline__ void moments(const float* s, int L, double itau, double ref, double t, double* red,
                                        double& mean, double& var) {
  float pm = 0.0f, pv = 0.0f;
#pragma unroll 8
  for (int i = threadIdx.x; i < L; i += NT) {
    const double y = (double)s[i] * itau - ref;
    const float x = fminf(fmaxf((float)(y - t), -80.0f), 80.0f);
    const float e = __builtin_amdgcn_exp2f(-fabsf(x) * 1.44269504088896340736f);
    const float q = __builtin_amdgcn_rcpf(1.0f + e);
    const float w = e * q;
    pm += x >= 0.0f ? q : w;
    pv = __builtin_fmaf(w, q, pv);
  }
  double v[2] = {(double)pm, (double)pv};
  block_red<NT, 2>(v, Add(), red);
  mean = v[0];
  var = v[1];
}
__device__ __forceinline__ bool close_to(double mean, double var, int B) {
  return fabs(mean - B) <= 0.25 * sqrt(var + 0.25);
}
__device__ __forceinline__ double newton(double t, double mean, double var, double lb, int L) {
  double m = mean > 1e-30 ? mean : 1e-30;
  m = m < L * (1.0 - 1e-7) ? m : L * (1.0 - 1e-7);
  return t + (log(m / (L - m)) - lb) * m * (1.0 - m / L) / (var > 1e-30 ? var : 1e-30);
}

struct Search {
  double ref, t, mean, var;
  bool found;
};

// The search for t where the scores have several scales (rows masked with a large
// finite value, say), so that Newton from their mean does not arrive: E[S] is `mean`
// at t, relative to mx.  Ends with |E[S] - B| as close_to asks (found), at any spread.
template <int NT>
__device__ __forceinline__ Search search(const float* s, int L, int B, double itau, double mx, double mn,
                                         double t, double mean, double* red) {
  Search r = {mx, t, mean, 0.0, false};
  double lo = mn - mx - 50.0, hi = 50.0, rl = -INFINITY, rh = INFINITY;
  const double lb = log((double)B / (double)(L - B));
  bool halve = false;
  for (int it = 0; !r.found && it < NEWTON + HALVINGS; ++it) {
    if (r.mean > B) lo = r.t;
    else hi = r.t;
    double next = r.t;
    if (it == 0 || (it == 1 && r.var < 1e-6 * fabs(r.mean - B))) {
      // the start again, from the mean of the rows on B's side of t (and of where
      // that leads, once: masked rows are one group)
      if (r.mean > B) rl = mx + r.t;
      else rh = mx + r.t;
      double n[3] = {0.0, 0.0, 0.0};      // rows in (rl, rh], their sum, rows above rh
#pragma unroll 4
      for (int i = threadIdx.x; i < L; i += NT) {
        const double x = (double)s[i] * itau;
        const bool in = x > rl && x <= rh;
        n[0] += in ? 1.0 : 0.0;
        n[1] += in ? x : 0.0;
        n[2] += x > rh ? 1.0 : 0.0;
      }
      block_red<NT, 3>(n, Add(), red);
      next = n[1] / n[0] - mx - log(((double)B - n[2]) / (n[0] + n[2] - (double)B));
      next = next > lo && next < hi ? next : 0.5 * (lo + hi);
    } else if (!halve && it < NEWTON) {
      next = newton(r.t, r.mean, r.var, lb, L);
      next = next > lo && next < hi ? next : 0.5 * (lo + hi);
    }
    if (!halve && next == r.t) {
      // Many scales, or ties so far from the largest that t cannot be stated between
      // them: from the order statistics.  s_(B), the B-th largest score, is the
      // largest value that at least B scores reach: two bits of its key a pass.
      uint32_t key = 0;
      for (int sh = 30; sh >= 0; sh -= 2) {
        int c1 = 0, c2 = 0, c3 = 0;
#pragma unroll 4
        for (int i = threadIdx.x; i < L; i += NT) {
          const uint32_t k = order_key(s[i]);
          c1 += k >= (key | 1u << sh) ? 1 : 0;
          c2 += k >= (key | 2u << sh) ? 1 : 0;
          c3 += k >= (key | 3u << sh) ? 1 : 0;
        }
        double n[3] = {(double)c1, (double)c2, (double)c3};
        block_red<NT, 3>(n, Add(), red);
        key |= (n[2] >= B ? 3u : n[1] >= B ? 2u : n[0] >= B ? 1u : 0u) << sh;
      }
      // relative to r_(B): E[S] <= B - 1 + (L - B + 1) e^-t, so t is at most
      // log(L - B + 1); and at r_(B+1) - x, E[S] >= (B + 1)(1 - e^-x), so it is at
      // least r_(B+1) - r_(B) - log(B + 1).  The middle of a wide gap between the two
      // is close enough, and a narrow bracket is halved: about 15 times at most.
      double n[1] = {0.0};
      float below = -INFINITY;
      for (int i = threadIdx.x; i < L; i += NT) {
        const float x = s[i];
        const bool in = order_key(x) >= key;
        n[0] += in ? 1.0 : 0.0;
        below = in ? below : fmaxf(below, x);
      }
      block_red<NT, 1>(n, Add(), red);
      double b[1] = {(double)below};
      block_red<NT, 1>(b, Max(), red);
      r.ref = (double)order_value(key) * itau;
      lo = (n[0] > B ? 0.0 : b[0] * itau - r.ref) - log((double)B + 1.0) - 1.0;
      hi = log((double)(L - B) + 1.0) + 1.0;
      halve = true;
    }
    r.t = halve ? 0.5 * (lo + hi) : next;
    moments<NT>(s, L, itau, r.ref, r.t, red, r.mean, r.var);
    r.found = close_to(r.mean, r.var, B);
  }
  return r;
}

// (re, im) of the product of two complex numbers
struct Cplx {
  double re, im;
};
__device__ __forceinline__ Cplx cmul(const Cplx& x, const Cplx& y) {
  return {__builtin_fma(x.re, y.re, -(x.im * y.im)), __builtin_fma(x.re, y.im, x.im * y.re)};
}

// e = e o of two polynomials, up to z^KF
template <int KF>
__device__ __forceinline__ void poly_mul(double (&e)[KF + 1], const double (&o)[KF + 1]) {
#pragma unroll
  for (int j = KF; j >= 0; --j) {
    double v = e[j] * o[0];
#pragma unroll
    for (int i = 0; i < j; ++i) v = __builtin_fma(e[i], o[j - i], v);
    e[j] = v;
  }
}

// The product over the block of the threads' polynomials (fixed order), for every
// thread; buf: (KF + 1) NT / 64 doubles.
template <int NT, int KF>
__device__ __forceinline__ void poly_red(double (&e)[KF + 1], double* buf) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double o[KF + 1];
#define DC_STEP(CTRL)                                    \
  _Pragma("unroll") for (int j = 0; j <= KF; ++j) o[j] = dppd<CTRL>(e[j]); \
  poly_mul<KF>(e, o);
  DC_STEP(DPP_XOR1)
  DC_STEP(DPP_XOR2)
  DC_STEP(DPP_HALF_MIRROR)
  DC_STEP(DPP_MIRROR)
#undef DC_STEP
  // the four rows of lanes, then the waves (a wave's lanes past NW repeat its last)
  double r[KF + 1];
#pragma unroll
  for (int j = 0; j <= KF; ++j) r[j] = lane_of(e[j], 0);
#pragma unroll
  for (int q = 16; q < 64; q += 16) {
#pragma unroll
    for (int j = 0; j <= KF; ++j) o[j] = lane_of(e[j], q);
    poly_mul<KF>(r, o);
  }
  __syncthreads();
  if (lane == 0)
#pragma unroll
    for (int j = 0; j <= KF; ++j) buf[wave * (KF + 1) + j] = r[j];
  __syncthreads();
#pragma unroll
  for (int j = 0; j <= KF; ++j) e[j] = buf[j];
  for (int w = 1; w < NW; ++w) {
#pragma unroll
    for (int j = 0; j <= KF; ++j) o[j] = buf[w * (KF + 1) + j];
    poly_mul<KF>(e, o);
  }
}

// KF = 0: any budgets.  KF = 1: at most one row is kept or evicted in every unit (the
// host knows), 4 and 8: two to KF of them; the characteristic function's registers and
// LDS are left out.
template <int NT, int KF>
__global__ void __launch_bounds__(NT, 4) logz_kernel(LogzArgs a) {
  constexpr int NW = NT / 64;
  constexpr bool ONE = KF == 1;
  __shared__ double red[3 * NW];
  __shared__ double zpow[NMAX][8];        // z, z^2, z^3, z^4 of every node
  __shared__ double2 co[2][CHUNK / 4];
  __shared__ double part[NW / NGRP][NMAX][2];
  __shared__ double term[NMAX];
  const int u = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const UnitDims d = unit_dims(a, u);
  const int L = d.L, B = d.B;
  const float* s = a.scores + (size_t)u * a.L;
  const int32_t* kept = a.kept ? a.kept + (size_t)u * a.nk : nullptr;
  const double itau = 1.0 / (double)a.tau;

  // statistics: sums of r over the rows and over the kept rows, its range
  // (the kept rows first: their scores then wait for one load, not two)
  double sum = 0.0, ks = 0.0, bad = 0.0;
  float smx = -INFINITY, smn = INFINITY;  // (tau > 0: the range of s gives that of r)
  if (kept) {
#pragma unroll 8
    for (int t = tid; t < d.nk; t += NT) {
      const int idx = kept[t];
      const bool in = idx >= 0 && idx < L;
      if (!in) bad = 1.0;
      ks += in ? (double)s[in ? idx : 0] * itau : 0.0;
    }
  }
  double mx, mn;
  // the first KR rows of a thread stay in registers (eight rows' loads in flight)
  float keep[KR];
#pragma unroll
  for (int j = 0; j < KR; ++j) keep[j] = s[tid + j * NT < L ? tid + j * NT : L - 1];
  auto row = [&](float x) {
    sum += (double)x * itau;
    smx = fmaxf(smx, x);
    smn = fminf(smn, x);
  };
#pragma unroll
  for (int j = 0; j < KR; ++j)
    if (tid + j * NT < L) row(keep[j]);
#pragma unroll 8
  for (int i = tid + KR * NT; i < L; i += NT) row(s[i]);
  {
    double v[3] = {sum, ks, bad};
    block_red<NT, 3>(v, Add(), red);
    sum = v[0];
    ks = v[1];
    bad = v[2];
    double m[2] = {(double)smx, -(double)smn};
    block_red<NT, 2>(m, Max(), red);
    mx = m[0] * itau;
    mn = -m[1] * itau;
  }
  auto finish = [&](double logz) {
    if (tid) return;
    const double logp = B >= L ? 0.0 : ks - logz;
    if (a.logz) a.logz[u] = logz;
    if (a.logp) a.logp[u] = logp;
  };
  // a kept index outside the row, or a score that is not finite (finite ones
  // sum to less than 2^300)
  if (bad != 0.0 || !isfinite(sum)) {
    if (tid == 0) {
      if (a.logz) a.logz[u] = __builtin_nan("");
      if (a.logp) a.logp[u] = __builtin_nan("");
    }
    return;
  }
  if (B >= L) {                           // one subset: the whole cache
    finish(sum);
    return;
  }
  if (ONE || (KF == 0 && (B == 1 || L - B == 1))) {
    // one row kept: log sum e^r; one row evicted: sum r + log sum e^-r
    const bool one = B == 1;
    const double c = one ? mx : -mn;
    double e[1] = {0.0};
    auto add = [&](float x) {
      const double r = (double)x * itau;
      e[0] += exp_neg((one ? r : -r) - c);
    };
#pragma unroll
    for (int j = 0; j < KR; ++j)
      if (tid + j * NT < L) add(keep[j]);
#pragma unroll 2
    for (int i = tid + KR * NT; i < L; i += NT) add(s[i]);
    block_red<NT, 1>(e, Add(), red);
    if (!one && c > MASK_R) {
      // a masked row is far larger than the rows that count: sum r without one
      // smallest r, as a sum over the others
      double v[2] = {0.0, 0.0};             // sum of r, number of rows above mn
      for (int i = tid; i < L; i += NT) {
        const double r = (double)s[i] * itau;
        v[0] += r > mn ? r : 0.0;
        v[1] += r > mn ? 1.0 : 0.0;
      }
      block_red<NT, 2>(v, Add(), red);
      finish(v[0] + ((double)(L - 1) - v[1]) * mn + log(e[0]));
      return;
    }
    finish((one ? 0.0 : sum) + c + log(e[0]));
    return;
  }
  if constexpr (KF > 1) {
    // few rows kept or few evicted: e_K of the weights relative to the largest, by
    // multiplying up the rows' factors 1 + w z as far as z^KF
    __shared__ double buf[(KF + 1) * NW];
    const bool neg = L - B < B;
    const int K = neg ? L - B : B;
    const double c = neg ? -mn : mx;
    double e[KF + 1] = {1.0};
    auto kth = [&]() {
      double v = 0.0;                       // (a sum: a chosen element would put e in memory)
#pragma unroll
      for (int j = 2; j <= KF; ++j) v = __builtin_fma(K == j ? 1.0 : 0.0, e[j], v);
      return v;
    };
    auto add = [&](float x) {
      const double r = (double)x * itau, w = exp_neg((neg ? -r : r) - c);
#pragma unroll
      for (int j = KF; j > 0; --j) e[j] = __builtin_fma(w, e[j - 1], e[j]);
    };
#pragma unroll
    for (int j = 0; j < KR; ++j)
      if (tid + j * NT < L) add(keep[j]);
#pragma unroll 2
    for (int i = tid + KR * NT; i < L; i += NT) add(s[i]);
    poly_red<NT, KF>(e, buf);
    if (kth() > 1e-250 && !(neg && c > MASK_R)) {
      finish((neg ? sum : 0.0) + K * c + log(kth()));
      return;
    }
    // the K rows are far from the largest, or a sum over masked rows would lose
    // digits: the factors q + p z of the trials behind t
    Search f = {mx, sum / L - mx - log((double)B / (double)(L - B)), 0.0, 0.0, false};
    moments<NT>(s, L, itau, mx, f.t, red, f.mean, f.var);
    f.found = close_to(f.mean, f.var, B);
    if (!f.found) f = search<NT>(s, L, B, itau, mx, mn, f.t, f.mean, red);
#pragma unroll
    for (int j = 0; j <= KF; ++j) e[j] = j == 0 ? 1.0 : 0.0;
    double v[3] = {0.0, 0.0, 0.0};        // sum of r over x > 0, of log(1 + e^-|x|), rows with x > 0
    for (int i = tid; i < L; i += NT) {
      const double r = (double)s[i] * itau, x = (r - f.ref) - f.t;
      const double g = exp_neg(-fabs(x)), hi = 1.0 / (1.0 + g), lo = g * hi;
      const double w1 = (x >= 0.0) == neg ? lo : hi, w0 = (x >= 0.0) == neg ? hi : lo;
#pragma unroll
      for (int j = KF; j > 0; --j) e[j] = __builtin_fma(w1, e[j - 1], w0 * e[j]);
      e[0] *= w0;
      v[0] += x > 0.0 ? r : 0.0;
      v[1] += log(1.0 + g);
      v[2] += x > 0.0 ? 1.0 : 0.0;
    }
    poly_red<NT, KF>(e, buf);
    block_red<NT, 3>(v, Add(), red);
    const bool ok = f.found && kth() > 0.0;
    finish(ok ? v[0] + ((double)B - v[2]) * (f.ref + f.t) + v[1] + log(kth()) : __builtin_nan(""));
    return;
  }
  if constexpr (KF == 0) {

  // t, relative to ref: E[S] within a quarter of a standard deviation of B is
  // enough, so binary32 weights do.  Newton on logit(E[S] / L), exact in one step
  // for equal scores, inside a bracket that bisection halves.
  double ref = mx, mean, var;
  double lo = mn - mx - 50.0, hi = 50.0;
  const double lb = log((double)B / (double)(L - B));
  double t = sum / L - mx - lb;
  t = t > lo && t < hi ? t : 0.5 * (lo + hi);
  bool found = false;
  for (int it = 0;; ++it) {
    moments<NT>(s, L, itau, ref, t, red, mean, var);
    found = close_to(mean, var, B);
    if (found || it >= NEWTON || (it == 0 && var < 1e-6 * fabs(mean - B))) break;
    if (mean > B) lo = t;
    else hi = t;
    const double next = newton(t, mean, var, lb, L);
    t = next > lo && next < hi ? next : 0.5 * (lo + hi);
  }
  if (!found) {
    const Search r = search<NT>(s, L, B, itau, mx, mn, t, mean, red);
    found = r.found;
    ref = r.ref;
    t = r.t;
    mean = r.mean;
    var = r.var;
  }

  // nodes (M odd: they come in conjugate pairs around the zeroth)
  const double reach = fabs(mean - B) + 11.0 + sqrt(100.0 + 60.0 * (var * 1.01 + 0.05));
  const int M = 2 * (int)ceil(0.5 * reach) + 1;
  int N = (M - 1) / 2;
  const double cut = 30.0 / (var * 0.99 + 1e-30);         // 1 - cos of the last node that matters
  if (cut < 2.0) {
    const int n = (int)ceil(acos(1.0 - cut) * M / (2.0 * PI));
    N = n < N ? n : N;
  }
  found = found && N <= NMAX;
  N = N < NMAX ? N : NMAX;
  if (tid < NMAX) {
    const double h = PI * (double)(tid + 1) / (double)M;   // half the node's angle
    const double sh = sin(h), ch = cos(h);
    const Cplx z = {-2.0 * sh * sh, 2.0 * sh * ch};        // exp(i w) - 1 without cancellation
    const Cplx z2 = cmul(z, z), z3 = cmul(z2, z), z4 = cmul(z2, z2);
    double* q = zpow[tid];
    q[0] = z.re;
    q[1] = z.im;
    q[2] = z2.re;
    q[3] = z2.im;
    q[4] = z3.re;
    q[5] = z3.im;
    q[6] = z4.re;
    q[7] = z4.im;
  }
  __syncthreads();

  // Chunks of rows: every thread turns groups of four rows into coefficients in
  // LDS, then every wave takes them through its nodes (node group wave mod
  // NGRP, its part of the groups where there are more waves than node groups).
  constexpr int PARTS = NW / NGRP;
  const int ng = wave % NGRP, rp = wave / NGRP;
  Cplx acc[NPG];
#pragma unroll
  for (int k = 0; k < NPG; ++k) acc[k] = {1.0, 0.0};
  double base = 0.0, prod = 1.0;          // sum of r over x > 0, product of 1 + e^-|x| <= 2
  int npos = 0;                           // rows with x > 0
  const int nch = (L + CHUNK - 1) / CHUNK;
  const int G4 = (L + 4 * nch - 1) / (4 * nch);            // groups of a chunk (<= CHUNK / 4)
  for (int c0 = 0; c0 < L; c0 += 4 * G4) {
    for (int g = tid; g < G4; g += NT) {
      float v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {       // rows c0 + g + j G4: coalesced over the threads
        const int i = c0 + g + j * G4;
        v[j] = s[i < L ? i : L - 1];
      }
      double p[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bool ok = c0 + g + j * G4 < L;
        const double r = (double)v[j] * itau, x = (r - ref) - t;
        const double e = exp_neg(-fabs(x)), w = 1.0 + e;
        double q = __builtin_amdgcn_rcp(w);                // 1 / w, w in [1, 2]: two Newton steps
        q = __builtin_fma(__builtin_fma(-w, q, 1.0), q, q);
        q = __builtin_fma(__builtin_fma(-w, q, 1.0), q, q);
        p[j] = !ok ? 0.0 : x >= 0.0 ? q : e * q;
        const bool pos = ok && x > 0.0;
        base += pos ? r : 0.0;
        npos += pos ? 1 : 0;
        prod *= ok ? w : 1.0;
      }
      const double a1 = p[0] + p[1], a2 = p[0] * p[1], b1 = p[2] + p[3], b2 = p[2] * p[3];
      co[0][g] = make_double2(a1 + b1, __builtin_fma(a1, b1, a2 + b2));
      co[1][g] = make_double2(__builtin_fma(a2, b1, a1 * b2), a2 * b2);
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < NPG / 3; ++h) {
      const int k0 = 3 * (h * NGRP + ng);      // threes dealt over the node groups
      if (k0 < N) {
        double z[3][8];
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
          for (int j = 0; j < 8; ++j) z[k][j] = zpow[k0 + k][j];
        for (int g = rp * 64 + lane; g < G4; g += PARTS * 64) {
          const double2 e12 = co[0][g], e34 = co[1][g];
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            Cplx f;
            f.re = __builtin_fma(e12.x, z[k][0], 1.0);
            f.im = e12.x * z[k][1];
            f.re = __builtin_fma(e12.y, z[k][2], f.re);
            f.im = __builtin_fma(e12.y, z[k][3], f.im);
            f.re = __builtin_fma(e34.x, z[k][4], f.re);
            f.im = __builtin_fma(e34.x, z[k][5], f.im);
            f.re = __builtin_fma(e34.y, z[k][6], f.re);
            f.im = __builtin_fma(e34.y, z[k][7], f.im);
            acc[3 * h + k] = cmul(acc[3 * h + k], f);
          }
        }
      }
    }
    __syncthreads();                      // the coefficients are read
  }
  // the product over the lanes, then over the wave's parts in order
#pragma unroll
  for (int k = 0; k < NPG; ++k) {
    const int node = 3 * (k / 3 * NGRP + ng) + k % 3;
    if (node < N) {
      Cplx c = acc[k];
      c = cmul(c, {dppd<DPP_XOR1>(c.re), dppd<DPP_XOR1>(c.im)});
      c = cmul(c, {dppd<DPP_XOR2>(c.re), dppd<DPP_XOR2>(c.im)});
      c = cmul(c, {dppd<DPP_HALF_MIRROR>(c.re), dppd<DPP_HALF_MIRROR>(c.im)});
      c = cmul(c, {dppd<DPP_MIRROR>(c.re), dppd<DPP_MIRROR>(c.im)});
      Cplx r = {lane_of(c.re, 0), lane_of(c.im, 0)};
#pragma unroll
      for (int q = 16; q < 64; q += 16) r = cmul(r, {lane_of(c.re, q), lane_of(c.im, q)});
      c = r;
      if (lane == 0) {
        part[rp][node][0] = c.re;
        part[rp][node][1] = c.im;
      }
    }
  }
  __syncthreads();
  if (tid < N) {
    Cplx c = {part[0][tid][0], part[0][tid][1]};
    for (int w = 1; w < PARTS; ++w) c = cmul(c, {part[w][tid][0], part[w][tid][1]});
    // times exp(-i w_k B), k B reduced modulo M; the real part
    const double th = 2.0 * PI * (double)(int)(((int64_t)(tid + 1) * B) % M) / (double)M;
    term[tid] = __builtin_fma(c.re, cos(th), c.im * sin(th));
  }
  double v[3] = {base, log(prod), (double)npos};
  block_red<NT, 3>(v, Add(), red);        // (its barriers also publish term)
  if (tid == 0) {
    double ps = 1.0;
    for (int k = 0; k < N; ++k) ps = ps + 2.0 * term[k];
    // (a search without its end or a node sum that is no probability: neither occurs)
    const bool ok = found && ps > 0.0;
    // B t + sum max(x, 0), without the t that every row above it shares (in the
    // middle of a gap t may be far larger than the rows that count)
    finish(ok ? v[0] + ((double)B - v[2]) * (ref + t) + v[1] + log(ps / (double)M) : __builtin_nan(""));
  }
  }
}

}  // namespace

// Callers size and pass this workspace when min(B, L - B) > BAND (part of the
// entry points' contract); the kernel needs none.
size_t logz_ws_bytes(int units, int L, int B) {
  const int K = B >= L ? 0 : (B < L - B ? B : L - B);
  return K > BAND ? (size_t)units * L * (sizeof(float) + sizeof(int)) : 0;
}

int launch_logz(const LogzArgs& a, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  const bool uniform = !a.unit_len && !a.budgets;
  const int K = a.L - a.B < a.B ? a.L - a.B : a.B;
  // At most one unit per CU: 1024 threads each, so that a unit's rows go by faster
  // (256 units of 8193 rows 30.6 us; 257 in 256 threads each 34.4 us); beyond, a
  // CU holds one such workgroup at a time (511 units 68 us, in 256 threads 37 us).
  const bool wide = a.units <= 256;
  auto launch = [&](auto kern, int nt) {
    hipLaunchKernelGGL(kern, dim3(a.units), dim3(nt), 0, s, a);
  };
  // (the polynomials of 2-8 rows spill at 1024 threads: 8 units of 8193 rows, 8 evicted,
  // 20 us, 300 units in 256 threads each 14)
  if (uniform && K <= 1 && wide) launch(logz_kernel<1024, 1>, 1024);
  else if (uniform && K <= 1) launch(logz_kernel<256, 1>, 256);
  else if (uniform && K <= 4) launch(logz_kernel<256, 4>, 256);
  else if (uniform && K <= 8) launch(logz_kernel<256, 8>, 256);
  else if (wide) launch(logz_kernel<1024, 0>, 1024);
  else launch(logz_kernel<256, 0>, 256);
  return (int)hipGetLastError();
}

}  // namespace dc
