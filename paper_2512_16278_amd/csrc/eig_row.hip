// Per-cell eigen stage up to 40 beams, one cell per 16-LANE ROW of a wavefront
// (four cells per wave), in FP64 (Sec. 3.2-3.3, Eq. 1-2): Householder reduction
// of the correlation matrix to tridiagonal form, then the dominant eigenvalue
// from sign sequences of the tridiagonal's leading minors (Golub & Van Loan,
// Matrix Computations, Sec. 8.3 and 8.4).
//
// Layout: lane l of a row holds rows E + l + 16 a (a < S) of the matrix, every
// column in registers, plus (l < E) the first E columns of row l: n <= 16 S + E.
// A vector lives in the same places (x[a], and xe for the first E entries), so
// its entry j is lane (j - E) mod 16 of one register, and the products of the
// reduction take it from there: v_fmac_f64_dpp with row_newbcast multiplies by
// one lane's value in all 16 lanes. A step therefore needs no LDS, no barrier
// and no index arithmetic, and what remains beside its multiply-adds (norm,
// square root, reciprocal, two 16-lane sums) is shared by four cells. Step k:
//  - x = column k below the diagonal; sigma = |x|^2, mu = sqrt(sigma), v = x +
//    sign(x_{k+1}) mu e_{k+1} (no cancellation), gamma = 1 / (sigma + mu
//    |x_{k+1}|), so that H = I - gamma v v^T;
//  - p = A v: complete within each lane for its rows; the few rows of the first
//    E indices, held as columns by symmetry, are 16-lane sums in steps k < E;
//  - w = gamma p - (gamma^2 p.v / 2) v and A -= v w^T + w v^T on the columns
//    beyond k (rows already reduced gather values that nothing reads).
// The steps are unrolled completely (every register index a constant). Column
// k keeps x after its step: the reflectors of v1's back transformation.
//
// The dominant eigenvalue: the 16 lanes of a row test 16 points of the bracket;
// x is above every eigenvalue when all leading minors of x I - T are positive,
// P_i = (x - alpha_i) P_{i-1} - off_{i-1}^2 P_{i-2} (two multiply-adds per step
// instead of a reciprocal and three, rescaled every eight steps).
//
// Bound: FP64 instruction issue, at two to three wavefronts per SIMD. 36 beams,
// 39000 cells with eigenvalues and vectors: 5290 -> 1140 us; 19 beams, raw
// moments, 40960 cells: 407 -> 117 us (before: one wavefront per cell with the
// matrix on an 8 x 8 lane grid and the vectors in LDS). Launches of a few hundred
// cells are a wavefront's latency, and four cells to it are longer than one was: 256
// cells of 37..40 beams (80 bytes of scratch) 43 -> 49 us, 33..36 41 -> 43, fewer as
// before or faster.
#include <math.h>

#include "internal.h"
#include "tridiag.h"

namespace rfi {
namespace {

constexpr int kRowCells = kTriCellPad;   // cells per workgroup
// Launches of at most this many cells take one wavefront (four cells) per workgroup
// instead, to reach more CUs' LDS and load paths: 20 beams, 1024 cells 26 -> 21 us, 40
// beams 57 -> 49, 2048 cells 57 -> 52, 4096 57 -> 58.
constexpr int64_t kRowFew = 2048;
constexpr int kRowThreads = 256;
constexpr int kVecs = 8;           // doubles of LDS per row index and cell

__device__ __forceinline__ int64_t xcd_order_row(int64_t b, int64_t total) {
  const int64_t q = total >> 3, rem = total & 7, x = b & 7;
  return x * q + (x < rem ? x : rem) + (b >> 3);
}

// S, E: rows per lane and leading rows as above; N: columns held (<= 16 S + E).
// W: int64 cell records; NC: the non-centred matrix (see eig_tri.hip). cell0:
// first cell of each item, every item's range padded to kRowCells. A workgroup has
// 16 lanes to a cell.
template <int S, int E, int N, bool W, bool NC>
__global__ __launch_bounds__(kRowThreads, (S == 1 ? 3 : 2)) void eig_row_kernel(
    EigArgs g, const EigArgs* items, const int64_t* cell0, int nitem, const double* zb) {
  static_assert(E % 4 == 0 && N <= 16 * S + E && N > 16 * (S - 1) + E, "row layout");
  using ST = std::conditional_t<W, int64_t, int32_t>;
  typedef const __attribute__((address_space(1))) ST gst;
  extern __shared__ __attribute__((aligned(16))) double lds[];
  const int nthr = blockDim.x, ncl = nthr >> 4;        // threads, cells of a workgroup
  int64_t c0 = xcd_order_row(blockIdx.x, gridDim.x) * ncl;
  if (items) {
    int lo = 0, hi = nitem - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (cell0[mid] <= c0) lo = mid; else hi = mid - 1;
    }
    g = items[lo];
    c0 -= cell0[lo];
  }
  const int n = g.nbeam, np = n * (n + 1) / 2, nrow = n + np;
  const int64_t ncell = (int64_t)g.nsub * g.nchan;
  if (c0 >= ncell) return;                             // padding of an item's range
  const int valid = ncell - c0 < ncl ? (int)(ncell - c0) : ncl;
  // stage the sums of the workgroup's cells, [cell][row]
  ST* const st = (ST*)lds;
  if (W || g.layout) {
    // contiguous records of consecutive cells, 16 bytes per load where the
    // records start on 16 bytes (the library's own always do); a thread's
    // loads are in flight before the first is stored
    typedef int v4 __attribute__((ext_vector_type(4)));
    typedef const __attribute__((address_space(1))) v4 gv4;
    const int64_t base = c0 * nrow;
    const int words = valid * nrow * (int)(sizeof(ST) / 4);
    const int quads = ((uintptr_t)g.sum_x & 15) ? 0 : words / 4;
    gv4* src = (gv4*)((gst*)g.sum_x + base);
    constexpr int kQuads = kRowCells * (N + N * (N + 1) / 2) * (int)(sizeof(ST) / 4) / 4;
    constexpr int kQ = (kQuads + kRowThreads - 1) / kRowThreads;
    constexpr int kB = kQ < 12 ? kQ : 12;
    for (int q0 = threadIdx.x; q0 < quads; q0 += nthr * kB) {
      v4 v[kB];
#pragma unroll
      for (int u = 0; u < kB; ++u) {
        const int q = q0 + u * nthr;
        v[u] = src[q < quads ? q : quads - 1];
      }
#pragma unroll
      for (int u = 0; u < kB; ++u)
        if (q0 + u * nthr < quads) ((v4*)st)[q0 + u * nthr] = v[u];
    }
    // the rest: a last workgroup may end inside 16 bytes
    for (int q = 4 * quads + threadIdx.x; q < words; q += nthr)
      ((int*)st)[q] = ((const __attribute__((address_space(1))) int*)src)[q];
  } else {
    // rows layout: 16 consecutive cells of a row per 16 threads
    constexpr int kLd = 16;
    const int c = threadIdx.x & (ncl - 1);
    const int64_t cell = c0 + (c < valid ? c : valid - 1);
    for (int q0 = threadIdx.x / ncl; q0 < nrow; q0 += 16 * kLd) {
      ST v[kLd];
#pragma unroll
      for (int u = 0; u < kLd; ++u) {
        int q = q0 + u * 16;
        q = q < nrow ? q : nrow - 1;
        v[u] = *((gst*)(q < n ? g.sum_x + (int64_t)q * ncell
                              : g.sum_xy + (int64_t)(q - n) * ncell) + cell);
      }
#pragma unroll
      for (int u = 0; u < kLd; ++u) {
        const int q = q0 + u * 16;
        if (q < nrow) st[c * nrow + q] = v[u];
      }
    }
  }
  __syncthreads();

  const int l = threadIdx.x & 15;
  const int grp = threadIdx.x >> 4;                    // this row's cell
  const int lc = grp < valid ? grp : valid - 1;        // a row past the end repeats the last cell
  const int64_t cell = c0 + lc;
  const bool mine = grp < valid;
  const int64_t cnt = g.count[cell / g.nchan];
  const bool bad = cnt < 2 || cnt > (W ? RFI_MAX_COUNT_LONG : RFI_MAX_COUNT);
  const double cd = (double)cnt;
  const ST* SX = st + lc * nrow;
  const ST* SP = SX + n;

  // the row values of S and 1 / sqrt(N_aa) (NC: of S and the baseline z), 0 at
  // padding indices
  double A[S][N], B[E ? E : 1];
  double Sr[S], dr[S], Se = 0.0, de = 0.0;
  int rb[S], re = 0;                                   // SP index of (i, j >= i) is rb + j
  bool dead = false;
  auto row_values = [&](int i, double& Sv, double& dv, int& base) {
    const int ic = i < n ? i : 0;
    base = ic * n - ic * (ic - 1) / 2 - ic;
    Sv = (double)SX[ic];
    if constexpr (NC) {
      dv = zb ? zb[(int64_t)ic * ncell + cell] : 0.0;
    } else {
      const int64_t Naa = cnt * (int64_t)SP[base + ic] - (int64_t)SX[ic] * SX[ic];
      dv = Naa > 0 ? 1.0 / sqrt((double)Naa) : 0.0;
      dead |= i < n && Naa <= 0;
    }
    if (i >= n) dv = 0.0;
  };
  static_for<0, S>([&](auto A_) {
    constexpr int a = RFI_CI(A_);
    row_values(E + l + 16 * a, Sr[a], dr[a], rb[a]);
  });
  if constexpr (E > 0) row_values(l, Se, de, re);
  auto entry = [&](int i, int j, int base, double Si, double di, double Sj, double dj) -> double {
    // j is a constant, uniform; base the row's offset
    const int jc = j < n ? j : 0;
    const int ic = i < n ? i : 0;
    const int cb = jc * n - jc * (jc - 1) / 2 - jc;
    const double sab = (double)SP[ic <= jc ? base + jc : cb + ic];
    if constexpr (NC) {
#pragma clang fp contract(off)
      if (i >= n || j >= n) return 0.0;
      const double za = i < j ? di : dj, zc = i < j ? dj : di;
      const double Sa = i < j ? Si : Sj, Sc = i < j ? Sj : Si;
      return (((sab - zc * Sa) - za * Sc) + (cd * za) * zc) / cd;
    } else {
      // N_ab = cnt S_ab - S_a S_b is exact in FP64 (integers below 2^53); the
      // product d_a d_b keeps both triangles bit-identical
      const double Nab = fma(cd, sab, -Si * Sj);
      return i == j ? (i < n ? 1.0 : 0.0) : Nab * (di * dj);
    }
  };
  double offsq = 0.0, dgsq = 0.0;
  static_for<0, N>([&](auto J_) {
    constexpr int j = RFI_CI(J_);
    if constexpr (NC && j >= 2)
      if (j >= n) {                                    // no divisions for padding columns
        static_for<0, S>([&](auto A_) { A[RFI_CI(A_)][j] = 0.0; });
        if constexpr (j < E) B[j] = 0.0;
        return;
      }
    double Sj, dj;
    if constexpr (j < E) {
      Sj = bcast<j & 15>(Se);
      dj = bcast<j & 15>(de);
    } else {
      Sj = bcast<(j - E) & 15>(Sr[(j - E) / 16]);
      dj = bcast<(j - E) & 15>(dr[(j - E) / 16]);
    }
    static_for<0, S>([&](auto A_) {
      constexpr int a = RFI_CI(A_);
      const int i = E + l + 16 * a;
      const double v = bad ? 0.0 : entry(i, j, rb[a], Sr[a], dr[a], Sj, dj);
      A[a][j] = v;
      // each pair once: (j, i) with j < E as a column, else j > i
      if (j < E || j > i) offsq += v * v;
      if (NC && j == i) dgsq += v * v;
    });
    if constexpr (j < E) {
      const double v = bad || l >= E ? 0.0 : entry(l, j, re, Se, de, Sj, dj);
      B[j] = v;
      if (j > l) offsq += v * v;
      if (NC && j == l) dgsq += v * v;
    }
  });
  // a dead beam may belong to any lane of the row
  bool degenerate = (__ballot(dead) >> (threadIdx.x & 48) & 0xffff) != 0;
  double frob2 = NC ? group_sum<16>(dgsq) + 2.0 * group_sum<16>(offsq)
                    : (double)n + 2.0 * group_sum<16>(offsq);
  int scale = 0;                                       // the matrix held is M 2^-scale
  if constexpr (NC) {
    degenerate = !(frob2 > 0.0);
    scale = unit_scale(frob2);
    const double sc = ldexp(1.0, -scale);
    static_for<0, N>([&](auto J_) {
      constexpr int j = RFI_CI(J_);
      static_for<0, S>([&](auto A_) { A[RFI_CI(A_)][j] *= sc; });
      if constexpr (j < E) B[j] *= sc;
    });
  }
  __syncthreads();                                     // the staged sums have been read

  // the cell's tridiagonal in LDS, over the staged sums
  double* const T = lds + grp * (kVecs * N + 2);
  double2* const ae = (double2*)T;                     // (alpha_i, off_{i-1}^2)
  double* const off = T + 2 * N;                       // off_i (signed)
  double* const gam = T + 3 * N;                       // gamma of step i
  double* const del = T + 4 * N;                       // sign mu of step i
  if (l == 0) ae[0].y = 0.0;

  static_for<0, N>([&](auto K_) {
    constexpr int k = RFI_CI(K_);
    if (k < n) {
      // diagonal entry k is final
      if constexpr (k < E) {
        if (l == k) ae[k].x = B[k < E ? k : 0];
      } else {
        if (l == ((k - E) & 15)) ae[k].x = A[(k - E) / 16][k];
      }
    }
    if constexpr (k + 1 < N) {
      if (k + 1 < n) {
        constexpr bool ext = k + 1 < E;                // first rows still active
        constexpr int a0 = k + 1 < E ? 0 : (k + 1 - E) / 16;   // first active slot
        double x[S], xe = 0.0;
        static_for<0, S>([&](auto A_) {
          constexpr int a = RFI_CI(A_);
          x[a] = a < a0 ? 0.0 : (E + 16 * a > k || l > k - E - 16 * a) ? A[a][k] : 0.0;
        });
        if constexpr (ext) xe = l > k ? B[k] : 0.0;
        double s = xe * xe;
        static_for<a0, S>([&](auto A_) { s = fma(x[RFI_CI(A_)], x[RFI_CI(A_)], s); });
        const double sigma = group_sum<16>(s);
        constexpr int j1 = k + 1;                      // where v differs from x
        constexpr int p1 = j1 < E ? j1 : (j1 - E) & 15;
        const double x0 = j1 < E ? bcast<p1>(xe) : bcast<p1>(x[a0]);
        // nothing below the diagonal: gamma = 0, the step changes nothing
        const bool some = sigma > 1e-290;
        const double mu = some ? sigma * rsqrt2(sigma) : 0.0;
        const double d = copysign(mu, x0);
        const double gm = some ? rcp2(fma(mu, fabs(x0), sigma)) : 0.0;
        if constexpr (j1 < E) xe = l == p1 ? x0 + d : xe;
        else x[a0] = l == p1 ? x0 + d : x[a0];
        if (l == 0) {
          off[k] = -d;
          gam[k] = gm;
          del[k] = d;
          ae[k + 1].y = d * d;
        }
        // p = A v over columns k + 1 ..
        double p[S], pb = 0.0, pe = 0.0;
        static_for<0, S>([&](auto A_) { p[RFI_CI(A_)] = 0.0; });
        static_for<(k + 1) / 4, (N + 3) / 4>([&](auto G_) {
          constexpr int j = RFI_CI(G_) * 4 < k + 1 ? k + 1 : RFI_CI(G_) * 4;
          constexpr int C = (RFI_CI(G_) * 4 + 4 < N ? RFI_CI(G_) * 4 + 4 : N) - j;
          constexpr int J = j < E ? j : (j - E) & 15;
          const double src = j < E ? xe : x[j < E ? 0 : (j - E) / 16];
          constexpr int z1 = C > 1 ? j + 1 : j, z2 = C > 2 ? j + 2 : j, z3 = C > 3 ? j + 3 : j;
          if constexpr (S - a0 == 2) {
            mv2<J, C>(p[0], p[S - 1], src, &A[0][j], &A[S - 1][j]);
          } else {
            mv1<J, C>(p[S - 1], pb, src, A[S - 1][j], A[S - 1][z1], A[S - 1][z2], A[S - 1][z3]);
          }
        });
        if constexpr (S - a0 == 1) p[S - 1] += pb;
        if constexpr (ext) {
          // rows k + 1 .. E - 1: from their own columns, and from the lanes'
          // columns by symmetry
          pe = 0.0;
          static_for<k + 1, E>([&](auto R_) {
            constexpr int r = RFI_CI(R_);
            pe = fma(B[r], bcast<r & 15>(xe), pe);
            double t = 0.0;
            static_for<0, S>([&](auto A_) {
              t = fma(A[RFI_CI(A_)][r], x[RFI_CI(A_)], t);
            });
            t = group_sum<16>(t);
            pe += l == r ? t : 0.0;
          });
        }
        double pv = pe * xe;
        static_for<a0, S>([&](auto A_) { pv = fma(p[RFI_CI(A_)], x[RFI_CI(A_)], pv); });
        pv = group_sum<16>(pv);
        const double kk = 0.5 * gm * (gm * pv);   // (gm^2 may overflow)
        double w[S], we = 0.0;
        static_for<0, S>([&](auto A_) {
          constexpr int a = RFI_CI(A_);
          w[a] = a < a0 ? 0.0 : fma(-kk, x[a], gm * p[a]);
        });
        if constexpr (ext) we = fma(-kk, xe, gm * pe);
        static_for<(k + 1) / 4, (N + 3) / 4>([&](auto G_) {
          constexpr int j = RFI_CI(G_) * 4 < k + 1 ? k + 1 : RFI_CI(G_) * 4;
          constexpr int C = (RFI_CI(G_) * 4 + 4 < N ? RFI_CI(G_) * 4 + 4 : N) - j;
          constexpr int J = j < E ? j : (j - E) & 15;
          const double sv = j < E ? xe : x[j < E ? 0 : (j - E) / 16];
          const double sw = j < E ? we : w[j < E ? 0 : (j - E) / 16];
          static_for<a0, S>([&](auto A_) {
            constexpr int a = RFI_CI(A_);
            up1<J, C>(&A[a][j], sv, sw, x[a], w[a]);
          });
          if constexpr (ext && j < E) up1<J, C>(&B[j], sv, sw, xe, we);
        });
      }
    }
  });
  wave_sync();

  // the non-centred matrix has no eigenvalue of order 1 that its stops could lean on
  constexpr double kFloor = NC ? 1e-300 : 1.0;
  const Spectrum sp = spectrum_bounds<16>(ae, off, n, l);
  const double lam1 = largest_eigenvalue<16>(ae, n, l, sp, kFloor);
  if (l == 0 && mine) {
    g.stat[cell] = bad || (NC && degenerate) ? 0.0 : lam1 * lam1 / frob2;
    g.status[cell] = bad ? RFI_CELL_BAD_COUNT | RFI_CELL_DEGENERATE
                         : (degenerate ? RFI_CELL_DEGENERATE : 0);
  }

  if (g.eigvals) {
    // the matrix is positive semidefinite up to rounding, so |lambda|
    // descending is about index n - 1 - i
    constexpr int Q = (N + 15) / 16;
    double* const z = T + 5 * N;
    double ev[Q];
    all_eigenvalues<16, Q>(ae, n, l, sp, kFloor, z, ev);
#pragma unroll
    for (int s = 0; s < Q; ++s)
      if (l + 16 * s < n) z[l + 16 * s] = ev[s];
    wave_sync();
    if (mine) {
#pragma unroll
      for (int s = 0; s < Q; ++s) {
        const int i = l + 16 * s;
        if (i >= n) continue;
        const double li = fabs(ev[s]);
        int rank = 0;
        for (int j = 0; j < n; ++j) {
          const double lj = fabs(z[j]);
          rank += (lj > li) || (lj == li && j > i);
        }
        g.eigvals[rank * g.out_stride + cell] = bad ? 0.f : (float)(NC ? ldexp(ev[s], scale) : ev[s]);
      }
    }
    wave_sync();
  }

  if (g.v1) {
    double* const z = T + 7 * N;
    top_eigenvector<16>(ae, off, n, l, lam1 + 1e-13 * fmax(fabs(lam1), kFloor), T + 5 * N,
                        T + 6 * N, z);
    // back transformation H_0 H_1 ... H_{n-2} z, applied from the last; the
    // reflectors are the columns of A, entry k + 1 of step k shifted by del
    double zr[S], ze = 0.0;
    static_for<0, S>([&](auto A_) {
      const int i = E + l + 16 * RFI_CI(A_);
      zr[RFI_CI(A_)] = i < n ? z[i < n ? i : 0] : 0.0;
    });
    if constexpr (E > 0) ze = l < E && l < n ? z[l] : 0.0;
    static_for<0, N - 1>([&](auto R_) {
      constexpr int k = N - 2 - RFI_CI(R_);
      if (k + 1 < n) {
        constexpr bool ext = k + 1 < E;
        constexpr int a0 = k + 1 < E ? 0 : (k + 1 - E) / 16;
        constexpr int p1 = k + 1 < E ? k + 1 : (k + 1 - E) & 15;
        const double d = del[k];
        double v[S], ve = 0.0, s = 0.0;
        if constexpr (ext) {
          ve = l > k ? B[k] : 0.0;
          ve = l == p1 ? ve + d : ve;
          s = ve * ze;
        }
        static_for<a0, S>([&](auto A_) {
          constexpr int a = RFI_CI(A_);
          v[a] = (E + 16 * a > k || l > k - E - 16 * a) ? A[a][k] : 0.0;
          if constexpr (!ext && a == a0) v[a] = l == p1 ? v[a] + d : v[a];
          s = fma(v[a], zr[a], s);
        });
        const double t = gam[k] * group_sum<16>(s);
        static_for<a0, S>([&](auto A_) {
          zr[RFI_CI(A_)] = fma(-t, v[RFI_CI(A_)], zr[RFI_CI(A_)]);
        });
        if constexpr (ext) ze = fma(-t, ve, ze);
      }
    });
    // sign: sum_b v_b >= 0, else first non-zero component positive
    double s = ze;
    static_for<0, S>([&](auto A_) { s += zr[RFI_CI(A_)]; });
    s = group_sum<16>(s);
    if (__any(s == 0.0)) {
      static_for<0, S>([&](auto A_) {
        const int i = E + l + 16 * RFI_CI(A_);
        if (i < n) z[i] = zr[RFI_CI(A_)];
      });
      if (l < E && l < n) z[l] = ze;
      wave_sync();
      if (s == 0.0)
        for (int i = 0; i < n; ++i)
          if (z[i] != 0.0) {
            s = z[i];
            break;
          }
    }
    const double sgn = s < 0.0 ? -1.0 : 1.0;
    if (mine) {
      static_for<0, S>([&](auto A_) {
        const int i = E + l + 16 * RFI_CI(A_);
        if (i < n) g.v1[i * g.out_stride + cell] = bad ? 0.f : (float)(sgn * zr[RFI_CI(A_)]);
      });
      if (l < E && l < n) g.v1[l * g.out_stride + cell] = bad ? 0.f : (float)(sgn * ze);
    }
  }
}

template <int S, int E, int N, bool W, bool NC>
hipError_t launch_row(const EigArgs& a, const EigArgs* items, const int64_t* cell0, int nitem,
                      int64_t total, const double* zb, hipStream_t s) {
  const int ncl = total <= kRowFew ? 4 : kRowCells;
  const size_t stage = (size_t)ncl * (N + N * (N + 1) / 2) * (W ? 8 : 4);
  const size_t tri = (size_t)ncl * (kVecs * N + 2) * 8;
  const size_t shm = stage > tri ? stage : tri;
  const auto kern = eig_row_kernel<S, E, N, W, NC>;
  hipError_t e = hipFuncSetAttribute((const void*)kern,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
  if (e != hipSuccess) return e;
  const int64_t wg = (total + ncl - 1) / ncl;
  hipLaunchKernelGGL(kern, dim3((unsigned)wg), dim3(ncl * 16), shm, s, a, items, cell0, nitem,
                     zb);
  return hipGetLastError();
}

template <bool W, bool NC>
hipError_t launch_n(int cls, const EigArgs& a, const EigArgs* items, const int64_t* cell0,
                    int nitem, int64_t total, const double* zb, hipStream_t s) {
  switch (cls) {
    case 16: return launch_row<1, 0, 16, W, NC>(a, items, cell0, nitem, total, zb, s);
    case 20: return launch_row<1, 4, 20, W, NC>(a, items, cell0, nitem, total, zb, s);
    case 24: return launch_row<1, 8, 24, W, NC>(a, items, cell0, nitem, total, zb, s);
    case 32: return launch_row<2, 0, 32, W, NC>(a, items, cell0, nitem, total, zb, s);
    case 36: return launch_row<2, 4, 36, W, NC>(a, items, cell0, nitem, total, zb, s);
    case 40: return launch_row<2, 8, 40, W, NC>(a, items, cell0, nitem, total, zb, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

int eig_row_class(int n) {
  return n < 2 ? 0 : n <= 16 ? 16 : n <= 20 ? 20 : n <= 24 ? 24 : n <= 32 ? 32 : n <= 36 ? 36
         : n <= 40 ? 40 : 0;
}

hipError_t launch_eig_row(int cls, const EigArgs& a, const EigArgs* items, const int64_t* cell0,
                          int nitem, int64_t total, bool wide, const double* zb, bool nc,
                          hipStream_t s) {
  if (nc) return launch_n<false, true>(cls, a, items, cell0, nitem, total, zb, s);
  return wide ? launch_n<true, false>(cls, a, items, cell0, nitem, total, zb, s)
              : launch_n<false, false>(cls, a, items, cell0, nitem, total, zb, s);
}

}  // namespace rfi
