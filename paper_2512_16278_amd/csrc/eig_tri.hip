// Per-cell eigen stage for more than 40 beams, one cell per WAVEFRONT, in
// FP64 (Sec. 3.2-3.3, Eq. 1-2): Householder reduction of the correlation
// matrix to tridiagonal form, then the dominant eigenvalue from sign sequences
// of the tridiagonal's leading minors (Golub & Van Loan, Matrix Computations,
// Sec. 8.3 and 8.4). Up to 40 beams eig_row.hip packs four cells into a
// wavefront; the two share their steps and tridiag.h.
//
// Layout: lane l holds row E + l of the matrix, every column in registers;
// beyond 64 beams the first E rows are held as columns (by symmetry), their
// own first E columns once per 16-lane row of the wave. Step k, in blocks of
// four columns (k = 4 IB + rk, IB a constant, so that every register index is
// one and the code stays within the instruction cache):
//  - x = column k below the diagonal goes to LDS and comes back with entries
//    16 g .. 16 g + 15 in register V[g], the same in each 16-lane row: from
//    there v_fmac_f64_dpp broadcasts one entry to all lanes of the row, and a
//    16-lane sum over the registers is a sum over all entries;
//  - sigma = |x|^2, mu = sqrt(sigma), v = x + sign(x_{k+1}) mu e_{k+1},
//    gamma = 1 / (sigma + mu |x_{k+1}|), H = I - gamma v v^T;
//  - p = A v is complete within each lane for its own row; p makes the same
//    way through LDS, so p.v and w = gamma p - (gamma^2 p.v / 2) v need no
//    further exchange;
//  - A -= v w^T + w v^T on the block's and all later columns; v and w vanish
//    at rows <= k, so finished columns keep x: the reflectors of v1's back
//    transformation.
//
// Bound: FP64 instruction issue at two wavefronts per SIMD. 72 beams, 40960
// cells: 2536 -> 2070 us (before: the matrix on an 8 x 8 lane grid and every
// vector read from LDS in both of its forms, about 70 LDS reads per step instead
// of 10). 49..72 beams need at most 24 bytes of scratch; from 73 on 220 bytes a lane
// (int64 sums 332) are spilled, some inside the steps: 79 beams, 8192 cells 1034 ->
// 641 us, 3000 cells of long sub-intervals 371 -> 327.
#include <math.h>

#include "internal.h"
#include "tridiag.h"

namespace rfi {
namespace {

constexpr int kVecs = 8;           // doubles of LDS per row index

// Workgroup b runs on XCD b mod 8; give each XCD a contiguous run of cells
// (a bijection of [0, total)), so the cells that share the cache lines of the
// structure-of-arrays sums are read through one L2 at about the same time.
__device__ __forceinline__ int64_t xcd_order(int64_t b, int64_t total) {
  const int64_t q = total >> 3, rem = total & 7, x = b & 7;
  return x * q + (x < rem ? x : rem) + (b >> 3);
}

// the value of entry rk (uniform, 0 .. 3) of four registers
__device__ __forceinline__ double pick(const double* a, int rk) {
  const double lo = rk & 1 ? a[1] : a[0], hi = rk & 1 ? a[3] : a[2];
  return rk & 2 ? hi : lo;
}

// E: leading rows held as columns; N: columns held (<= 64 + E).
// W: the sums are int64 cell records (sub-intervals longer than the int32
// bound, summed in time chunks and widened).
// NC: the non-centred matrix of the bandpass-subtracted power instead of the
// correlation matrix: M_ab = (S_ab - z_b S_a - z_a S_b + L z_a z_b) / L from
// the exact sums and the baseline zb [nbeam][ncell] (NULL: 0), every entry
// formed in that operation order (no fused multiply-add), ||M||_F^2 over all
// entries.
// cell0: first cell of each item (ranges padded to kTriCellPad).
template <int E, int N, bool W, bool NC>
__global__ __launch_bounds__(64, N <= 48 ? 3 : 2) void eig_tri_kernel(
    EigArgs g, const EigArgs* items, const int64_t* cell0, int nitem, const double* zb) {
  static_assert(E % 4 == 0 && N % 4 == 0 && N <= 64 + E && (E == 0 || N == 64 + E), "layout");
  constexpr int NV = (N - E + 15) / 16;
  using ST = std::conditional_t<W, int64_t, int32_t>;
  // the sums are global memory (batched launches read their pointers from the
  // item table, where the compiler cannot tell the address space)
  typedef const __attribute__((address_space(1))) int gint;
  typedef const __attribute__((address_space(1))) ST gst;
  typedef int v4 __attribute__((ext_vector_type(4)));
  typedef const __attribute__((address_space(1))) v4 gv4;
  extern __shared__ __attribute__((aligned(16))) double lds[];
  int64_t cell = xcd_order(blockIdx.x, gridDim.x);
  if (items) {
    int lo = 0, hi = nitem - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (cell0[mid] <= cell) lo = mid; else hi = mid - 1;
    }
    g = items[lo];
    cell -= cell0[lo];
  }
  const int n = g.nbeam, nrow = n + n * (n + 1) / 2;
  const int l = threadIdx.x, l16 = l & 15;
  const int64_t ncell = (int64_t)g.nsub * g.nchan;
  if (cell >= ncell) return;               // padding of the item's range of cells
  const int64_t cnt = g.count[cell / g.nchan];
  if (cnt < 2 || cnt > (W ? RFI_MAX_COUNT_LONG : RFI_MAX_COUNT)) {
    for (int i = l; i < n; i += 64) {
      if (g.eigvals) g.eigvals[i * g.out_stride + cell] = 0.f;
      if (g.v1) g.v1[i * g.out_stride + cell] = 0.f;
    }
    if (l == 0) {
      g.stat[cell] = 0.0;
      g.status[cell] = RFI_CELL_BAD_COUNT | RFI_CELL_DEGENERATE;
    }
    return;
  }
  // stage the cell's sums in LDS, many loads in flight before the first store
  const ST* SX;
  if (W || g.layout) {
    // one contiguous record: 16-byte loads between its aligned ends, LDS
    // offset like the record
    constexpr int kB = 12;
    gint* src = (gint*)((gst*)g.sum_x + cell * nrow);
    const int words = nrow * (int)(sizeof(ST) / 4);
    const int mis = (int)((uintptr_t)src / 4 & 3), lead = -mis & 3;
    const int quads = (words - lead) / 4, tail = lead + 4 * quads;
    int* const dst = (int*)lds + mis;
    for (int q0 = l; q0 < quads; q0 += 64 * kB) {
      v4 v[kB];
#pragma unroll
      for (int u = 0; u < kB; ++u) {
        const int q = q0 + 64 * u;
        v[u] = ((gv4*)(src + lead))[q < quads ? q : quads - 1];
      }
#pragma unroll
      for (int u = 0; u < kB; ++u)
        if (q0 + 64 * u < quads) ((v4*)(dst + lead))[q0 + 64 * u] = v[u];
    }
    if (l < lead) dst[l] = src[l];
    if (tail + l < words) dst[tail + l] = src[tail + l];
    SX = (const ST*)dst;
  } else {
    // rows layout: row q of the record is sum_x[q] (q < n) or sum_xy[q - n]
    constexpr int kB = 16;
    ST* const dst = (ST*)lds;
    for (int q0 = l; q0 < nrow; q0 += 64 * kB) {
      ST v[kB];
#pragma unroll
      for (int u = 0; u < kB; ++u) {
        int q = q0 + 64 * u;
        q = q < nrow ? q : nrow - 1;
        v[u] = *((gst*)(q < n ? g.sum_x + (int64_t)q * ncell
                              : g.sum_xy + (int64_t)(q - n) * ncell) + cell);
      }
#pragma unroll
      for (int u = 0; u < kB; ++u)
        if (q0 + 64 * u < nrow) dst[q0 + 64 * u] = v[u];
    }
    SX = dst;
  }
  wave_sync();
  const ST* const SP = SX + n;

  // S and 1 / sqrt(N_aa) (NC: S and the baseline z) of this lane's row and of
  // the leading row l16, and of all rows in the broadcast registers; 0 at
  // padding indices
  const double cd = (double)cnt;
  bool dead = false;
  auto row_values = [&](int i, double& Sv, double& dv) {
    const int ic = i < n ? i : 0;
    Sv = (double)SX[ic];
    if constexpr (NC) {
      dv = zb ? zb[(int64_t)ic * ncell + cell] : 0.0;
    } else {
      const int64_t Naa = cnt * (int64_t)SP[ic * n - ic * (ic - 1) / 2] - (int64_t)SX[ic] * SX[ic];
      dv = Naa > 0 ? 1.0 / sqrt((double)Naa) : 0.0;
      dead |= i < n && Naa <= 0;
    }
    if (i >= n) dv = 0.0;
  };
  auto row_base = [&](int i) {             // SP index of (i, j >= i) is row_base(i) + j
    const int ic = i < n ? i : 0;
    return ic * n - ic * (ic - 1) / 2 - ic;
  };
  double A[N], B[E ? E : 1];
  double Sr, dr, Se = 0.0, de = 0.0, SV[NV], dV[NV];
  row_values(E + l, Sr, dr);
  if constexpr (E > 0) row_values(l16, Se, de);
  if constexpr (E > 0)
    if (l16 >= E) de = 0.0;
  static_for<0, NV>([&](auto G_) {
    row_values(E + 16 * RFI_CI(G_) + l16, SV[RFI_CI(G_)], dV[RFI_CI(G_)]);
  });
  const int rb = row_base(E + l), re = row_base(l16);
  auto entry = [&](int i, int j, int base, double Si, double di, double Sj, double dj) -> double {
#pragma clang fp contract(off)
    const int jc = j < n ? j : 0, ic = i < n ? i : 0;
    const int cb = jc * n - jc * (jc - 1) / 2 - jc;
    const double sab = (double)SP[ic <= jc ? base + jc : cb + ic];
    if constexpr (NC) {
      if (i >= n || j >= n) return 0.0;
      const double za = i < j ? di : dj, zc = i < j ? dj : di;
      const double Sa = i < j ? Si : Sj, Sc = i < j ? Sj : Si;
      return (((sab - zc * Sa) - za * Sc) + (cd * za) * zc) / cd;
    } else {
      // N_ab = cnt S_ab - S_a S_b is exact in FP64 (integers below 2^53); the
      // product d_a d_b keeps both triangles bit-identical
      const double Nab = fma(cd, sab, -(Si * Sj));
      return i == j ? (i < n ? 1.0 : 0.0) : Nab * (di * dj);
    }
  };
  double offsq = 0.0, dgsq = 0.0, offe = 0.0, dge = 0.0;
  static_for<0, N>([&](auto J_) {
    constexpr int j = RFI_CI(J_);
    // at most eight columns' sums in flight (each group's inputs follow the last
    // group's outputs): more would spill
    if constexpr (j % 8 == 0) {
      asm volatile("" : "+v"(Sr), "+v"(dr), "+v"(offsq)::"memory");
    }
    constexpr int gj = j < E ? 0 : (j - E) / 16, pj = j < E ? j : (j - E) & 15;
    const double Sj = bcast<pj>(j < E ? Se : SV[gj]), dj = bcast<pj>(j < E ? de : dV[gj]);
    const int i = E + l;
    A[j] = entry(i, j, rb, Sr, dr, Sj, dj);
    if (j < E || j > i) offsq = fma(A[j], A[j], offsq);   // each pair once
    if (NC && j == i) dgsq = A[j] * A[j];
    if constexpr (j < E) {
      const double v = l16 < E ? entry(l16, j, re, Se, de, Sj, dj) : 0.0;
      B[j] = v;
      if (j > l16) offe = fma(v, v, offe);
      if (NC && j == l16) dge = v * v;
    }
  });
  int degenerate = __any(dead);
  const double off2 = group_sum<64>(offsq) + group_sum<16>(offe);
  double frob2 = NC ? group_sum<64>(dgsq) + group_sum<16>(dge) + 2.0 * off2
                    : (double)n + 2.0 * off2;
  int scale = 0;                           // the matrix held is M 2^-scale
  if constexpr (NC) {
    degenerate = !(frob2 > 0.0);
    scale = unit_scale(frob2);
    const double sc = ldexp(1.0, -scale);
    static_for<0, N>([&](auto J_) {
      A[RFI_CI(J_)] *= sc;
      if constexpr (RFI_CI(J_) < E) B[RFI_CI(J_)] *= sc;
    });
  }
  wave_sync();                             // the staged sums have been read

  double2* const ae = (double2*)lds;       // (alpha_i, off_{i-1}^2)
  double* const off = lds + 2 * N;         // off_i (signed)
  double* const gam = lds + 3 * N;         // gamma of step i
  double* const del = lds + 4 * N;         // sign mu of step i
  double* const X = lds + 5 * N;           // exchange of x and p [64]
  if (l == 0) ae[0].y = 0.0;

  static_for<0, N / 4>([&](auto IB_) {
    constexpr int j0 = 4 * RFI_CI(IB_);
    constexpr bool ext = j0 < E;           // leading rows still active
    constexpr int g0 = j0 < E ? 0 : (j0 - E) / 16;   // first register with active entries
    const int nk = n - j0 < 4 ? n - j0 : 4;
#pragma unroll 1
    for (int rk = 0; rk < nk; ++rk) {
      const int k = j0 + rk;
      // this lane's and the leading row's entry of column k; the diagonal one
      // is final
      double x = pick(&A[j0], rk), xe = 0.0;
      if constexpr (ext) {
        xe = pick(&B[j0 < E ? j0 : 0], rk);
        if (l == k) ae[k].x = xe;
        xe = l16 > k ? xe : 0.0;           // (0 beyond the leading rows)
      } else {
        if (E + l == k) ae[k].x = x;
        x = E + l > k ? x : 0.0;
      }
      if (k + 1 == n) break;
      X[l] = x;
      wave_sync();
      double V[NV];
      static_for<g0, NV>([&](auto G_) { V[RFI_CI(G_)] = X[16 * RFI_CI(G_) + l16]; });
      double s = xe * xe;
      static_for<g0, NV>([&](auto G_) { s = fma(V[RFI_CI(G_)], V[RFI_CI(G_)], s); });
      const double sigma = group_sum<16>(s);
      // entry k + 1: one of the leading rows (in the lanes' xe) or a lane's row
      const int i1 = k + 1 - E;
      const double x0 = ext && i1 < 0 ? lane_f64(xe, k + 1 < 16 ? k + 1 : 0)
                                      : lane_f64(x, i1 < 0 ? 0 : i1);
      // nothing below the diagonal: gamma = 0, the step changes nothing
      const bool some = sigma > 1e-290;
      const double mu = some ? sigma * rsqrt2(sigma) : 0.0;
      const double d = copysign(mu, x0);
      const double gm = some ? rcp2(fma(mu, fabs(x0), sigma)) : 0.0;
      if constexpr (ext) xe = l16 == k + 1 && k + 1 < E ? x0 + d : xe;
      x = l == i1 ? x0 + d : x;
      // (entry k + 1 may be the first of the next register)
      static_for<g0, (g0 + 2 < NV ? g0 + 2 : NV)>([&](auto G_) {
        constexpr int q = RFI_CI(G_);
        V[q] = 16 * q + l16 == i1 ? x0 + d : V[q];
      });
      if (l == 0) {
        off[k] = -d;
        gam[k] = gm;
        del[k] = d;
        ae[k + 1].y = d * d;
      }
      // p = A v for this lane's row
      double pa = 0.0, pb = 0.0;
      static_for<j0 / 4, N / 4>([&](auto G_) {
        constexpr int j = RFI_CI(G_) * 4;
        constexpr int gj = j < E ? 0 : (j - E) / 16, pj = j < E ? j : (j - E) & 15;
        mv1<pj, 4>(pa, pb, j < E ? xe : V[gj], A[j], A[j + 1], A[j + 2], A[j + 3]);
      });
      const double p = pa + pb;
      wave_sync();                         // V has been read
      X[l] = p;
      wave_sync();
      double P[NV], pe = 0.0;
      static_for<g0, NV>([&](auto G_) { P[RFI_CI(G_)] = X[16 * RFI_CI(G_) + l16]; });
      if constexpr (ext) {
        // the leading rows: their own first E columns, and the lanes' columns
        // by symmetry
        double qa = 0.0, qb = 0.0;
        static_for<j0 / 4, E / 4>([&](auto G_) {
          constexpr int j = RFI_CI(G_) * 4;
          mv1<j, 4>(qa, qb, xe, B[j], B[j + 1], B[j + 2], B[j + 3]);
        });
        pe = qa + qb;
        static_for<j0, E>([&](auto R_) {
          constexpr int r = RFI_CI(R_);
          const double t = group_sum<64>(A[r] * x);
          pe += l16 == r ? t : 0.0;
        });
        pe = l16 > k && l16 < E ? pe : 0.0;
      }
      double pv = pe * xe;
      static_for<g0, NV>([&](auto G_) { pv = fma(P[RFI_CI(G_)], V[RFI_CI(G_)], pv); });
      pv = group_sum<16>(pv);
      const double kk = 0.5 * gm * (gm * pv);   // (gm^2 may overflow)
      // w vanishes at the rows already reduced, so their columns stay
      const double w = E + l > k ? fma(-kk, x, gm * p) : 0.0;
      const double we = fma(-kk, xe, gm * pe);
      static_for<g0, NV>([&](auto G_) {
        constexpr int q = RFI_CI(G_);
        P[q] = fma(-kk, V[q], gm * P[q]);
        if constexpr (!ext && q == g0) P[q] = E + 16 * q + l16 > k ? P[q] : 0.0;
      });
      static_for<j0 / 4, N / 4>([&](auto G_) {
        constexpr int j = RFI_CI(G_) * 4;
        constexpr int gj = j < E ? 0 : (j - E) / 16, pj = j < E ? j : (j - E) & 15;
        up1<pj, 4>(&A[j], j < E ? xe : V[gj], j < E ? we : P[gj], x, w);
        if constexpr (ext && j < E) up1<pj, 4>(&B[j < E ? j : 0], xe, we, xe, we);
      });
      wave_sync();                         // P has been read
    }
  });
  wave_sync();

  constexpr double kFloor = NC ? 1e-300 : 1.0;
  const Spectrum sp = spectrum_bounds<64>(ae, off, n, l);
  const double lam1 = largest_eigenvalue<64>(ae, n, l, sp, kFloor);
  if (l == 0) {
    g.stat[cell] = (NC && degenerate) ? 0.0 : lam1 * lam1 / frob2;
    g.status[cell] = degenerate ? RFI_CELL_DEGENERATE : 0;
  }

  if (g.eigvals) {
    constexpr int Q = (N + 63) / 64;
    double* const z = lds + 5 * N;
    double ev[Q];
    all_eigenvalues<64, Q>(ae, n, l, sp, kFloor, z, ev);
#pragma unroll
    for (int s = 0; s < Q; ++s)
      if (l + 64 * s < n) z[l + 64 * s] = ev[s];
    wave_sync();
#pragma unroll
    for (int s = 0; s < Q; ++s) {
      const int i = l + 64 * s;
      if (i >= n) continue;
      // |lambda| descending (positive semidefinite up to rounding)
      const double li = fabs(ev[s]);
      int rank = 0;
      for (int j = 0; j < n; ++j) {
        const double lj = fabs(z[j]);
        rank += (lj > li) || (lj == li && j > i);
      }
      g.eigvals[rank * g.out_stride + cell] = (float)(NC ? ldexp(ev[s], scale) : ev[s]);
    }
    wave_sync();
  }

  if (g.v1) {
    double* const z = lds + 7 * N;
    top_eigenvector<64>(ae, off, n, l, lam1 + 1e-13 * fmax(fabs(lam1), kFloor), lds + 5 * N,
                        lds + 6 * N, z);
    // back transformation H_0 H_1 ... H_{n-2} z, applied from the last; the
    // reflectors are the columns of A, entry k + 1 of step k shifted by del
    double zr = E + l < n ? z[E + l < n ? E + l : 0] : 0.0, ze = 0.0;
    if constexpr (E > 0) ze = l16 < E ? z[l16] : 0.0;
    static_for<0, N / 4>([&](auto R_) {
      constexpr int j0 = N - 4 - 4 * RFI_CI(R_);
      constexpr bool ext = j0 < E;
#pragma unroll 1
      for (int rk = 3; rk >= 0; --rk) {
        const int k = j0 + rk;
        if (k + 1 >= n) continue;
        const double d = del[k];
        double v = pick(&A[j0], rk), ve = 0.0;
        v = E + l > k ? v : 0.0;
        v = E + l == k + 1 ? v + d : v;
        double s = group_sum<64>(v * zr);
        if constexpr (ext) {
          ve = pick(&B[j0 < E ? j0 : 0], rk);
          ve = l16 > k ? ve : 0.0;
          ve = l16 == k + 1 && k + 1 < E ? ve + d : ve;
          s += group_sum<16>(ve * ze);
        }
        const double t = gam[k] * s;
        zr = fma(-t, v, zr);
        if constexpr (ext) ze = fma(-t, ve, ze);
      }
    });
    // sign: sum_b v_b >= 0, else first non-zero component positive
    double s = group_sum<64>(zr) + (E > 0 ? group_sum<16>(ze) : 0.0);
    if (s == 0.0) {
      wave_sync();
      if (E + l < n) z[E + l] = zr;
      if (l < E) z[l] = ze;
      wave_sync();
      for (int i = 0; i < n; ++i)
        if (z[i] != 0.0) {
          s = z[i];
          break;
        }
    }
    const double sgn = s < 0.0 ? -1.0 : 1.0;
    if (E + l < n) g.v1[(E + l) * g.out_stride + cell] = (float)(sgn * zr);
    if (l < E) g.v1[l * g.out_stride + cell] = (float)(sgn * ze);
  }
}

template <int E, int N, bool W, bool NC>
hipError_t launch_one(const EigArgs& a, const EigArgs* items, const int64_t* cell0, int nitem,
                      int64_t total, const double* zb, hipStream_t s) {
  const size_t stage = (size_t)(N + N * (N + 1) / 2) * (W ? 8 : 4) + 16;
  const size_t tri = (size_t)kVecs * N * 8 > (size_t)(5 * N + 128) * 8 ? (size_t)kVecs * N * 8
                                                                      : (size_t)(5 * N + 128) * 8;
  hipLaunchKernelGGL((eig_tri_kernel<E, N, W, NC>), dim3((unsigned)total), dim3(64),
                     stage > tri ? stage : tri, s, a, items, cell0, nitem, zb);
  return hipGetLastError();
}

template <bool W, bool NC = false>
hipError_t launch_cls(int cls, const EigArgs& a, const EigArgs* items, const int64_t* cell0,
                      int nitem, int64_t total, hipStream_t s, const double* zb = nullptr) {
  switch (cls) {
    case 48: return launch_one<0, 48, W, NC>(a, items, cell0, nitem, total, zb, s);
    case 64: return launch_one<0, 64, W, NC>(a, items, cell0, nitem, total, zb, s);
    case 72: return launch_one<8, 72, W, NC>(a, items, cell0, nitem, total, zb, s);
    case 80: return launch_one<16, 80, W, NC>(a, items, cell0, nitem, total, zb, s);
    default: return launch_eig_row(cls, a, items, cell0, nitem, total, W, zb, NC, s);
  }
}

}  // namespace

int eig_tri_class(int n) {
  if (n <= 40) return eig_row_class(n);
  return n <= 48 ? 48 : n <= 64 ? 64 : n <= 72 ? 72 : n <= 80 ? 80 : 0;
}

hipError_t launch_eig_tri(const EigArgs& a, hipStream_t s) {
  const int64_t ncell = (int64_t)a.nsub * a.nchan;
  if (ncell == 0) return hipSuccess;
  const int cls = eig_tri_class(a.nbeam);
  return a.layout == 2 ? launch_cls<true>(cls, a, nullptr, nullptr, 0, ncell, s)
                       : launch_cls<false>(cls, a, nullptr, nullptr, 0, ncell, s);
}

hipError_t launch_eig_tri_nc(const EigArgs& a, const double* zb, hipStream_t s) {
  const int64_t ncell = (int64_t)a.nsub * a.nchan;
  if (ncell == 0) return hipSuccess;
  return launch_cls<false, true>(eig_tri_class(a.nbeam), a, nullptr, nullptr, 0, ncell, s, zb);
}

hipError_t launch_eig_tri_batch(int cls, const EigArgs* items, const int64_t* cell0, int nitem,
                                int64_t total, hipStream_t s) {
  if (total == 0) return hipSuccess;
  return launch_cls<false>(cls, EigArgs{}, items, cell0, nitem, total, s);
}

}  // namespace rfi
