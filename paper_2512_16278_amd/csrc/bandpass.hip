// ArPLS bandpass normalisation (Sec. 3.1; its parameters lam, ratio and
// itermax are those of Sec. 4.5): for each beam and sub-interval, the channel
// means y_j = S_b(k, j) / L (the sums of Eq. 1 over the sub-interval) are
// fitted by asymmetrically reweighted penalised least squares (Baek et al.
// 2015): with D the second-difference operator, solve (W + lam D^T D) z = W y,
// take the residuals d = y - z, the mean m and sample standard deviation s
// (ddof 1) of the negative ones, the weights w' = 1 / (1 + exp(2 (d - (2 s -
// m)) / s)), and repeat with W = diag(w') until ||w - w'|| / ||w|| < ratio
// (that pass's z is kept) or itermax passes. The baseline z is the bandpass
// that Sec. 3.1 subtracts from every sample of the channel.
//
// One workgroup per (beam, sub-interval) system. The matrix is pentadiagonal
// and positive definite; a sequential factorisation along the channels has
// only the systems as parallelism (190 threads for ten sub-intervals of 19
// beams), so the channels are cut into T chunks, one per thread, and the
// unknowns are eliminated in nested order (any symmetric order is backward
// stable for a positive definite matrix):
//  - each thread eliminates its chunk's rows but the last two (LDL^T with the
//    fill towards the two rows before the chunk), all threads at once;
//  - what remains couples each chunk's last two rows to the next chunk's: a
//    block tridiagonal system of T blocks of 2 x 2, reduced in LDS by log2 T
//    levels of cyclic reduction (every second block eliminated per level) and
//    solved back the same way;
//  - each thread substitutes back inside its chunk;
//  - after the last pass (after every pass for a large lam) one more solve, of
//    that pass's residual, takes the rounding of the elimination out of z (error
//    against an extended-precision solve 4.3e-12 of the spectrum, 7.7e-12
//    without; a sequential FP64 Cholesky has 6.4e-12).
// Rows past the last channel are unit rows (w = 1, y = 0, no coupling).
// Bound: latency of the dependent FP64 steps (one reciprocal per row of a
// chunk, log2 T levels each way). 190 systems of 4096 channels, two passes: 44 us,
// against 6811 us with one thread per system and a sequential Cholesky.
#include <hip/hip_runtime.h>
#include <math.h>

#include "internal.h"

namespace rfi {
namespace {

constexpr int kVecs = 7;          // doubles of workspace per channel and system (M = 0: six
                                  // vectors of at most 7/6 of the channels; else unused)
constexpr int kMinRows = 4;       // rows per chunk: at least two interior ones
constexpr int kLdsVecs = 9;       // doubles per block of the reduced system
constexpr double kRefineLam = 1e6;   // from here on every pass is refined: see launch_arpls

struct BpArgs {
  int nbeam, nsub, nchan, itermax;
  int m;                  // rows per chunk
  double lam, ratio;
  const int32_t* sum_x;   // rows layout: sum_x[b][k * nchan + j]
  const int32_t* count;   // [nsub]
  double* z;              // out [nbeam][ncell]
  int32_t* passes;        // out [nsub][nbeam] or NULL
  double* ws;             // 6 vectors of T * m doubles per system (M = 0 only)
};

// A chunk's vector: registers, or element i of thread t at [i * T + t] of the
// workspace (M = 0, chunks too long for registers).
template <int T, int M>
struct Vec {
  double v[M];
  __device__ __forceinline__ explicit Vec(double*) {}
  __device__ __forceinline__ double& operator[](int i) { return v[i]; }
};
template <int T>
struct Vec<T, 0> {
  double* p;
  __device__ __forceinline__ explicit Vec(double* base) : p(base) {}
  __device__ __forceinline__ double& operator[](int i) { return p[(size_t)i * T]; }
};

// 1 / x to full FP64 precision (the hardware estimate and two Newton steps);
// x is a pivot: positive and normal
__device__ __forceinline__ double rcp2(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  return fma(r, fma(-x, r, 1.0), r);
}

// Row i of D^T D: diagonal, first and second super-diagonal. D has rows r = 0
// .. F - 3 with 1, -2, 1 at columns r, r + 1, r + 2; row i of D^T D collects
// the rows r = i - 2, i - 1, i that exist (none past the last channel).
struct Dtd {
  double d0, d1, d2;
};
__device__ __forceinline__ Dtd dtd_row(int i, int F) {
  const double a = (i >= 2 && i <= F - 1) ? 1.0 : 0.0;
  const double b = (i >= 1 && i <= F - 2) ? 1.0 : 0.0;
  const double c = (i >= 0 && i <= F - 3) ? 1.0 : 0.0;
  return {a + 4.0 * b + c, -2.0 * (b + c), c};
}

__device__ __forceinline__ double bp_wave_sum(double x) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o);
  return x;
}

// Sum over the workgroup, the same bits in every thread.
template <int T>
__device__ __forceinline__ double bp_sum(double x, double* red) {
  x = bp_wave_sum(x);
  if constexpr (T == 64) return x;
  __syncthreads();                       // red may still be read by an earlier call
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < T / 64; ++w) s += red[w];
  return s;
}

// Symmetric positive definite 2 x 2 block (a b; b d) as L D L^T.
struct Sym2 {
  double ia, l, id;       // 1 / a, b / a, 1 / (d - b^2 / a)
  __device__ __forceinline__ Sym2(double a, double b, double d) {
    ia = rcp2(a);
    l = b * ia;
    id = rcp2(fma(-l, b, d));
  }
  // (x0, x1) <- block^-1 (x0, x1)
  __device__ __forceinline__ void solve(double& x0, double& x1) const {
    x1 = fma(-l, x0, x1) * id;
    x0 = fma(-l, x1, x0 * ia);
  }
};

// padded LDS position of channel j of the staged spectrum / baseline: threads
// reading consecutive chunks do not meet in one bank
__device__ __forceinline__ int pos(int j) { return j + (j >> 4); }

// R: every pass's z is refined, not only the last one's
template <int T, int M, bool R>
__global__ __launch_bounds__(T) void arpls_kernel(BpArgs a) {
  extern __shared__ __attribute__((aligned(16))) double lds[];
  __shared__ double red[T / 64];
  const int t = threadIdx.x;
  const int sys = blockIdx.x;
  const int b = sys % a.nbeam, k = sys / a.nbeam;
  const int F = a.nchan;
  const int m = M ? M : a.m;
  constexpr int kU = M ? M : 1;           // unrolling of the loops over a chunk
  const int64_t ncell = (int64_t)a.nsub * F;
  const double L = (double)a.count[k];
  const int32_t* sx = a.sum_x + (int64_t)b * ncell + (int64_t)k * F;
  double* zo = a.z + (int64_t)b * ncell + (int64_t)k * F;
  if (F < 3) {
    for (int j = t; j < F; j += T) zo[j] = (double)sx[j] / L;
    if (a.passes && t == 0) a.passes[k * a.nbeam + b] = 0;
    return;
  }
  const size_t vs = (size_t)T * m;
  double* wsys = M ? nullptr : a.ws + (size_t)sys * 6 * vs + t;
  Vec<T, M> y(wsys), w(wsys + (M ? 0 : vs)), l1(wsys + (M ? 0 : 2 * vs)),
      l2(wsys + (M ? 0 : 3 * vs)), di(wsys + (M ? 0 : 4 * vs)), x(wsys + (M ? 0 : 5 * vs));
  const int s0 = t * m;                   // the chunk's first row
  // the spectrum (channel means), through LDS so that the loads are coalesced
  if constexpr (M > 0) {
    int32_t* st = (int32_t*)lds;
    for (int j = t; j < F; j += T) st[pos(j)] = sx[j];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < M; ++i) y[i] = s0 + i < F ? (double)st[pos(s0 + i)] / L : 0.0;
  } else {
    for (int i = 0; i < m; ++i) y[i] = s0 + i < F ? (double)sx[s0 + i] / L : 0.0;
  }
#pragma unroll
  for (int i = 0; i < m; ++i) {
    w[i] = 1.0;
    x[i] = y[i];
  }

  // reduced system, level by level: level l has Tn >> l blocks at offset
  // 2 Tn - (2 Tn >> l); arrays A (3: a, b, d), E (4: coupling to the block
  // before, row-major), r (2), each of 2 T doubles. Tn (a power of two) covers the
  // chunks that hold channels; the others' unit rows couple to nothing and their
  // solution is not read (3 channels: no level instead of six).
  int Tn = 1;
  while (Tn * m < F) Tn <<= 1;
  auto arr = [&](int v) { return lds + (size_t)v * 2 * T; };
  double *Aa = arr(0), *Ab = arr(1), *Ad = arr(2), *E0 = arr(3), *E1 = arr(4), *E2 = arr(5),
         *E3 = arr(6), *R0 = arr(7), *R1 = arr(8);

  // solves A x = rhs, rhs given in x: W y, or (fix) the residual of the solution
  // before, which takes that one's rounding out
  int passes = 0;
  bool fix = false;
  for (;;) {
    __syncthreads();     // the staged spectrum / the last pass's solution has been read
    // coupling of this chunk's first two rows to the two rows before it
    const Dtd cp = dtd_row(s0 - 2, F), cq = dtd_row(s0 - 1, F);
    const double f0 = t ? a.lam * cp.d2 : 0.0, g0 = t ? a.lam * cq.d1 : 0.0;
    const double g1 = t ? a.lam * cq.d2 : 0.0;
    // interior rows 0 .. m - 3; *p: row i - 1, *q: row i - 2
    double l1p = 0.0, Bp = 0.0, cpv = 0.0, l2p = 0.0, l2q = 0.0, cqv = 0.0;
    double fp = 0.0, fq = 0.0, gp = 0.0, gq = 0.0, up = 0.0, uq = 0.0;
    double Spp = 0.0, Spq = 0.0, Sqq = 0.0, sp = 0.0, sq = 0.0;
#pragma unroll
    for (int i = 0; i < m - 2; ++i) {
      const Dtd c = dtd_row(s0 + i, F);
      const double cc = a.lam * c.d2;
      const double D = fma(-l2q, cqv, fma(-l1p, Bp, fma(a.lam, c.d0, w[i])));
      const double B = fma(-l1p, cpv, a.lam * c.d1);
      const double f = fma(-l2q, fq, fma(-l1p, fp, i == 0 ? f0 : 0.0));
      const double g = fma(-l2q, gq, fma(-l1p, gp, i == 0 ? g0 : (i == 1 ? g1 : 0.0)));
      const double u = fma(-l2q, uq, fma(-l1p, up, x[i]));
      const double inv = rcp2(D);
      l1[i] = B * inv;
      l2[i] = cc * inv;
      di[i] = inv;
      const double lf = f * inv, lg = g * inv;
      Spp = fma(lf, f, Spp);
      Spq = fma(lf, g, Spq);
      Sqq = fma(lg, g, Sqq);
      sp = fma(lf, u, sp);
      sq = fma(lg, u, sq);
      l2q = l2p;
      l2p = cc * inv;
      cqv = cpv;
      cpv = cc;
      l1p = B * inv;
      Bp = B;
      fq = fp;
      fp = f;
      gq = gp;
      gp = g;
      uq = up;
      up = u;
    }
    // the chunk's last two rows (not eliminated) and their coupling to the
    // two before the chunk
    {
      const Dtd c = dtd_row(s0 + m - 2, F), e = dtd_row(s0 + m - 1, F);
      Aa[t] = fma(-l2q, cqv, fma(-l1p, Bp, fma(a.lam, c.d0, w[m - 2])));
      Ab[t] = fma(-l1p, cpv, a.lam * c.d1);
      Ad[t] = fma(-l2p, cpv, fma(a.lam, e.d0, w[m - 1]));
      E0[t] = fma(-l2q, fq, -l1p * fp);
      E1[t] = fma(-l2q, gq, -l1p * gp);
      E2[t] = -l2p * fp;
      E3[t] = -l2p * gp;
      R0[t] = fma(-l2q, uq, fma(-l1p, up, x[m - 2]));
      R1[t] = fma(-l2p, up, x[m - 1]);
      // what eliminating this chunk adds to the block before it: kept in the
      // next level's space until that block has taken it
      Aa[T + t] = Spp;
      Ab[T + t] = Spq;
      Ad[T + t] = Sqq;
      R0[T + t] = sp;
      R1[T + t] = sq;
    }
    __syncthreads();
    if (t + 1 < T) {
      Aa[t] -= Aa[T + t + 1];
      Ab[t] -= Ab[T + t + 1];
      Ad[t] -= Ad[T + t + 1];
      R0[t] -= R0[T + t + 1];
      R1[t] -= R1[T + t + 1];
    }
    __syncthreads();
    // the levels over nb blocks. At full width nb is the constant T and the loops over
    // the levels unroll (190 systems of 256 channels 25 us, 27 us with nb = Tn alone);
    // 512 threads have no registers left for that (9000 channels 179 us rolled, 192)
    auto solve_reduced = [&](const int nb) __attribute__((always_inline)) {
      // reduction: the odd blocks of a level survive, each absorbing its two
      // even neighbours
      int o = 0;
      for (int n = nb; n > 1; n >>= 1) {
        const int on = o + n;
        if (t < n / 2) {
          const int s = o + 2 * t + 1, e = s - 1;
          double a0 = Aa[s], b0 = Ab[s], d0 = Ad[s], r0 = R0[s], r1 = R1[s];
          const double p0 = E0[s], p1 = E1[s], p2 = E2[s], p3 = E3[s];   // rows of E_s
          const Sym2 L0(Aa[e], Ab[e], Ad[e]);
          // columns of A_e^-1 E_s^T are the rows of E_s solved
          double x0 = p0, x1 = p1, y0 = p2, y1 = p3;
          L0.solve(x0, x1);
          L0.solve(y0, y1);
          a0 -= fma(p0, x0, p1 * x1);
          b0 -= fma(p2, x0, p3 * x1);
          d0 -= fma(p2, y0, p3 * y1);
          const double re0 = R0[e], re1 = R1[e];
          r0 -= fma(x0, re0, x1 * re1);
          r1 -= fma(y0, re0, y1 * re1);
          const double q0 = E0[e], q1 = E1[e], q2 = E2[e], q3 = E3[e];
          E0[on + t] = -fma(x0, q0, x1 * q2);
          E1[on + t] = -fma(x0, q1, x1 * q3);
          E2[on + t] = -fma(y0, q0, y1 * q2);
          E3[on + t] = -fma(y0, q1, y1 * q3);
          if (2 * t + 2 < n) {
            const int g = s + 1;
            const Sym2 L1(Aa[g], Ab[g], Ad[g]);
            // columns of E_g, solved
            const double c0 = E0[g], c1 = E1[g], c2 = E2[g], c3 = E3[g];
            double v0 = c0, v1 = c2, w0 = c1, w1 = c3;
            L1.solve(v0, v1);
            L1.solve(w0, w1);
            a0 -= fma(c0, v0, c2 * v1);
            b0 -= fma(c0, w0, c2 * w1);
            d0 -= fma(c1, w0, c3 * w1);
            const double rg0 = R0[g], rg1 = R1[g];
            r0 -= fma(v0, rg0, v1 * rg1);
            r1 -= fma(w0, rg0, w1 * rg1);
          }
          Aa[on + t] = a0;
          Ab[on + t] = b0;
          Ad[on + t] = d0;
          R0[on + t] = r0;
          R1[on + t] = r1;
        }
        o = on;
        __syncthreads();
      }
      if (t == 0) {
        const Sym2 L0(Aa[o], Ab[o], Ad[o]);
        double x0 = R0[o], x1 = R1[o];
        L0.solve(x0, x1);
        R0[o] = x0;
        R1[o] = x1;
      }
      __syncthreads();
      // back: the solution of each block replaces its right-hand side
      for (int n = 2; n <= nb; n <<= 1) {
        const int oc = 2 * nb - 2 * n, on = oc + n;
        if (t < n / 2) {
          const int e = oc + 2 * t, s = e + 1;
          const double xs0 = R0[on + t], xs1 = R1[on + t];
          double r0 = R0[e], r1 = R1[e];
          r0 -= fma(E0[s], xs0, E2[s] * xs1);            // E_s^T X_s
          r1 -= fma(E1[s], xs0, E3[s] * xs1);
          if (t > 0) {
            const double xb0 = R0[on + t - 1], xb1 = R1[on + t - 1];
            r0 -= fma(E0[e], xb0, E1[e] * xb1);
            r1 -= fma(E2[e], xb0, E3[e] * xb1);
          }
          const Sym2 L0(Aa[e], Ab[e], Ad[e]);
          L0.solve(r0, r1);
          R0[e] = r0;
          R1[e] = r1;
          R0[s] = xs0;
          R1[s] = xs1;
        }
        __syncthreads();
      }
    };
    if (T < 512 && Tn == T)
      solve_reduced(T);
    else
      solve_reduced(Tn);
    // inside the chunk: forward with the rows before it known, then back
    const double zp = t ? R0[t - 1] : 0.0, zq = t ? R1[t - 1] : 0.0;
    double u1 = 0.0, u2 = 0.0;
    double la = 0.0, lb = 0.0, lc = 0.0;               // l1[i-1], l2[i-2], l2[i-1]
#pragma unroll
    for (int i = 0; i < m - 2; ++i) {
      double rhs = x[i];
      if (i == 0) rhs -= fma(f0, zp, g0 * zq);
      if (i == 1) rhs -= g1 * zq;
      const double u = fma(-lb, u2, fma(-la, u1, rhs));
      x[i] = u;
      u2 = u1;
      u1 = u;
      la = l1[i];
      lb = lc;
      lc = l2[i];
    }
    double z1 = R0[t], z2 = R1[t];
    x[m - 1] = z2;
    x[m - 2] = z1;
#pragma unroll
    for (int i = m - 3; i >= 0; --i) {
      const double zi = fma(-l2[i], z2, fma(-l1[i], z1, x[i] * di[i]));
      x[i] = zi;
      z2 = z1;
      z1 = zi;
    }
    if constexpr (R) {
      if (fix) {
#pragma unroll kU
        for (int i = 0; i < m; ++i) x[i] += zo[s0 + i < F ? s0 + i : F - 1];
      }
    } else if (fix) {
      break;
    }
    if (fix || !R) {
      ++passes;
      const bool last = passes == a.itermax;
      // negative residuals: mean and sample standard deviation
      double sn = 0.0, cnt = 0.0;
#pragma unroll
      for (int i = 0; i < m; ++i) {
        const double d = y[i] - x[i];
        if (s0 + i < F && d < 0.0) {
          sn += d;
          cnt += 1.0;
        }
      }
      sn = bp_sum<T>(sn, red);
      cnt = bp_sum<T>(cnt, red);
      const double mean = sn / cnt;
      double ss = 0.0;
#pragma unroll
      for (int i = 0; i < m; ++i) {
        const double d = y[i] - x[i];
        if (s0 + i < F && d < 0.0) ss = fma(d - mean, d - mean, ss);
      }
      ss = bp_sum<T>(ss, red);
      const double sd = sqrt(ss / (cnt - 1.0));
      bool stop = cnt < 2.0 || !(sd > 0.0);
      if (!stop && !last) {
        // new weights (over l1, free until the next solve), kept until the test
        double dw = 0.0, nw = 0.0;
#pragma unroll kU
        for (int i = 0; i < m; ++i) {
          const double d = y[i] - x[i];
          const double wt = 1.0 / (1.0 + exp(2.0 * (d - (2.0 * sd - mean)) / sd));
          const double wo = w[i];
          if (s0 + i < F) {
            dw = fma(wo - wt, wo - wt, dw);
            nw = fma(wo, wo, nw);
            l1[i] = wt;
          } else {
            l1[i] = 1.0;
          }
        }
        dw = bp_sum<T>(dw, red);
        nw = bp_sum<T>(nw, red);
        stop = sqrt(dw) / sqrt(nw) < a.ratio;
      }
      if (!stop && !last) {
#pragma unroll kU
        for (int i = 0; i < m; ++i) {
          w[i] = l1[i];
          x[i] = w[i] * y[i];
        }
        fix = false;
        continue;
      }
      if constexpr (R) break;
    }
    // z goes out, and its residual W (y - z) - lam D^T (D z) is the next
    // right-hand side. The differences of neighbouring z are exact or nearly so, so
    // the residual is accurate far below the rounding of the solve and one more
    // solve takes that rounding out of z.
    __syncthreads();                      // the reduced system is read no more
#pragma unroll kU
    for (int i = 0; i < m; ++i)
      if (s0 + i < F) {
        if constexpr (M > 0) lds[pos(s0 + i)] = x[i];
        else zo[s0 + i] = x[i];
      }
    __syncthreads();
    auto z_at = [&](int j) {
      const int c = j < 0 ? 0 : (j < F ? j : F - 1);
      if constexpr (M > 0) return lds[pos(c)];
      else return zo[c];
    };
    // row r of D z (0 outside 0 .. F - 3)
    auto d_at = [&](int r) {
      const double e = (z_at(r) - z_at(r + 1)) - (z_at(r + 1) - z_at(r + 2));
      return r >= 0 && r <= F - 3 ? e : 0.0;
    };
    double e2 = d_at(s0 - 2), e1 = d_at(s0 - 1);
#pragma unroll
    for (int i = 0; i < m; ++i) {
      const double e0 = d_at(s0 + i);
      const double res = fma(-a.lam, (e0 - e1) - (e1 - e2), w[i] * (y[i] - x[i]));
      x[i] = s0 + i < F ? res : 0.0;
      e2 = e1;
      e1 = e0;
    }
    if constexpr (M > 0) {
      for (int j = t; j < F; j += T) zo[j] = lds[pos(j)];
    }
    fix = true;
  }
  __syncthreads();
  if constexpr (M > 0) {
#pragma unroll
    for (int i = 0; i < M; ++i)
      if (s0 + i < F) lds[pos(s0 + i)] = x[i];
    __syncthreads();
    for (int j = t; j < F; j += T) zo[j] = R ? lds[pos(j)] : zo[j] + lds[pos(j)];
  } else {
    for (int i = 0; i < m; ++i)
      if (s0 + i < F) zo[s0 + i] = R ? x[i] : zo[s0 + i] + x[i];
  }
  if (a.passes && t == 0) a.passes[k * a.nbeam + b] = passes;
}

template <int T, int M, bool R>
hipError_t launch_bp(BpArgs a, int nsys, hipStream_t s) {
  a.m = M ? M : (a.nchan + T - 1) / T;
  if (a.m < kMinRows) a.m = kMinRows;
  size_t shm = (size_t)kLdsVecs * 2 * T * sizeof(double);
  const size_t stage = (size_t)(T * M + T * M / 16 + 1) * sizeof(double);
  if (M && stage > shm) shm = stage;
  const auto kern = arpls_kernel<T, M, R>;
  hipError_t e = hipFuncSetAttribute((const void*)kern,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)nsys), dim3(T), shm, s, a);
  return hipGetLastError();
}

}  // namespace

size_t bandpass_workspace_size(int nbeam, int nchan, int nsub) {
  return (size_t)kVecs * nchan * nbeam * nsub * sizeof(double);
}

// Chunks by channel count: up to 16 rows of a chunk (six vectors of FP64) in
// registers, so T = 64, 256 or 512 threads cover 8192 channels; one wavefront
// suffices (and needs no barrier) up to 1024. At 512 threads (4097 channels and more)
// a thread has 256 registers and 488 bytes a lane go to scratch inside the solve: 190
// systems of 4096 / 4097 / 8192 channels, two passes, 44 / 96 / 105 us (one thread per
// system and a sequential Cholesky 6811 / 6786 / 13643). Beyond 8192 channels the
// vectors live in the workspace (6 vectors of at most nchan + 511 <= 7/6 nchan rows):
// 8193 channels 178 us (13573).
template <bool R>
hipError_t launch_sized(const BpArgs& a, int nsys, hipStream_t s) {
  if (a.nchan <= 64 * 4) return launch_bp<64, 4, R>(a, nsys, s);
  if (a.nchan <= 64 * 16) return launch_bp<64, 16, R>(a, nsys, s);
  if (a.nchan <= 256 * 8) return launch_bp<256, 8, R>(a, nsys, s);
  if (a.nchan <= 256 * 16) return launch_bp<256, 16, R>(a, nsys, s);
  if (a.nchan <= 512 * 16) return launch_bp<512, 16, R>(a, nsys, s);
  return launch_bp<512, 0, R>(a, nsys, s);
}

// The rounding of a solve grows with lam (condition number about 16 lam / the smallest
// weight), enters the next pass through the weights and is not taken out by a last
// solve alone: with only the last pass refined, 38 systems of 1024 channels at lam =
// 1e9 were 2.5e-5 off (median 1.4e-5) against 7.8e-6 (3.5e-6) of one sequential FP64
// Cholesky per pass; at 1e7, 256 channels 8.4e-8 (median) against 5.8e-8; at the default
// 1e5 it is the more accurate one (median 3.9e-10 against 1.1e-9), and at 1e6 still
// (2.6e-9 against 8.2e-9). With every pass refined 4.3e-9 (1.3e-9) at 1e9, for up to
// twice the solves: 13 passes of 1024 channels 222 us instead of 135 (the Cholesky
// 10433).
hipError_t launch_arpls(int nbeam, int nsub, int nchan, const int32_t* sum_x,
                        const int32_t* count, double lam, double ratio, int itermax, double* z,
                        int32_t* passes, void* ws, hipStream_t s) {
  const int nsys = nbeam * nsub;
  if (nsys == 0) return hipSuccess;
  BpArgs a{nbeam, nsub, nchan, itermax, 0, lam, ratio, sum_x, count, z, passes, (double*)ws};
  return lam >= kRefineLam ? launch_sized<true>(a, nsys, s) : launch_sized<false>(a, nsys, s);
}

}  // namespace rfi
