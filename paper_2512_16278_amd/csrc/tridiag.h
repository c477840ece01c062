// Eigenvalues of a symmetric tridiagonal held in LDS, by a group of W lanes of
// one wavefront (W = 16 or 64), and the FP64 helpers of the Householder
// kernels. The matrix is ae[i] = (alpha_i, off_{i-1}^2), ae[0].y = 0.
//
// Everything rests on the leading minors of x I - T,
//     P_i = (x - alpha_i) P_{i-1} - off_{i-1}^2 P_{i-2},
// whose sign changes count the eigenvalues above x (Golub & Van Loan, Matrix
// Computations, Sec. 8.4); two multiply-adds per row, no division, rescaled by
// a common power of two every eight rows. P_n itself, the characteristic
// polynomial, places the next points (secant); the brackets move by the signs
// alone, so the result does not depend on how well it does.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace rfi {

template <int CTRL>
__device__ __forceinline__ double dpp_mov(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// lane J's value in every lane of its 16-lane row
template <int J>
__device__ __forceinline__ double bcast(double x) {
  return __builtin_amdgcn_mov_dpp(x, 0x150 + J, 0xF, 0xF, true);
}
__device__ __forceinline__ double lane_f64(double x, int l) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)b, l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// Sum / minimum / maximum over the W lanes of a group, the same bits in every
// lane (each stage pairs the same two operands): mirrors within 16 lanes, then
// (W = 64) the four rows' results read as scalars.
template <int W, class Op>
__device__ __forceinline__ double group_reduce(double x, Op op) {
  x = op(x, dpp_mov<0xB1>(x));    // lane ^ 1
  x = op(x, dpp_mov<0x4E>(x));    // lane ^ 2
  x = op(x, dpp_mov<0x141>(x));   // mirror in 8 lanes
  x = op(x, dpp_mov<0x140>(x));   // mirror in 16 lanes
  if constexpr (W == 64)
    x = op(op(lane_f64(x, 0), lane_f64(x, 16)), op(lane_f64(x, 32), lane_f64(x, 48)));
  return x;
}
template <int W>
__device__ __forceinline__ double group_sum(double x) {
  return group_reduce<W>(x, [](double a, double b) { return a + b; });
}
template <int W>
__device__ __forceinline__ double group_min(double x) {
  return group_reduce<W>(x, [](double a, double b) { return fmin(a, b); });
}
template <int W>
__device__ __forceinline__ double group_max(double x) {
  return group_reduce<W>(x, [](double a, double b) { return fmax(a, b); });
}

// Compile-time loop: every index into a register-resident matrix must be a
// constant.
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}
#define RFI_CI(v) decltype(v)::value

// Multiply-adds with one lane's value of a source register in all 16 lanes of
// its row (v_fmac_f64_dpp, row_newbcast), four columns to a block: the compiler
// does not fold a 64-bit row broadcast into the multiply-add. A block starts
// with the two wait states that a DPP read needs after a write of its source.
// acc += bcast(src, J + i) * m[i], i < C, alternating two accumulators
#define RFI_FB "row_mask:0xf bank_mask:0xf\n\t"
template <int J, int C>
__device__ __forceinline__ void mv1(double& p0, double& p1, double src, double a0, double a1,
                                    double a2, double a3) {
  if constexpr (C == 4)
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %2, %3 row_newbcast:%7 " RFI_FB
        "v_fmac_f64_dpp %1, %2, %4 row_newbcast:%8 " RFI_FB
        "v_fmac_f64_dpp %0, %2, %5 row_newbcast:%9 " RFI_FB
        "v_fmac_f64_dpp %1, %2, %6 row_newbcast:%10 row_mask:0xf bank_mask:0xf"
        : "+&v"(p0), "+&v"(p1)
        : "v"(src), "v"(a0), "v"(a1), "v"(a2), "v"(a3), "n"(J), "n"(J + 1), "n"(J + 2),
          "n"(J + 3));
  else if constexpr (C == 3)
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %2, %3 row_newbcast:%6 " RFI_FB
        "v_fmac_f64_dpp %1, %2, %4 row_newbcast:%7 " RFI_FB
        "v_fmac_f64_dpp %0, %2, %5 row_newbcast:%8 row_mask:0xf bank_mask:0xf"
        : "+&v"(p0), "+&v"(p1)
        : "v"(src), "v"(a0), "v"(a1), "v"(a2), "n"(J), "n"(J + 1), "n"(J + 2));
  else if constexpr (C == 2)
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %2, %3 row_newbcast:%5 " RFI_FB
        "v_fmac_f64_dpp %1, %2, %4 row_newbcast:%6 row_mask:0xf bank_mask:0xf"
        : "+&v"(p0), "+&v"(p1)
        : "v"(src), "v"(a0), "v"(a1), "n"(J), "n"(J + 1));
  else
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
        : "+&v"(p0)
        : "v"(src), "v"(a0), "n"(J));
}
// two rows' accumulators at once
template <int J, int C>
__device__ __forceinline__ void mv2(double& p, double& q, double src, const double* a,
                                    const double* b) {
  if constexpr (C == 4)
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %2, %3 row_newbcast:%11 " RFI_FB
        "v_fmac_f64_dpp %1, %2, %7 row_newbcast:%11 " RFI_FB
        "v_fmac_f64_dpp %0, %2, %4 row_newbcast:%12 " RFI_FB
        "v_fmac_f64_dpp %1, %2, %8 row_newbcast:%12 " RFI_FB
        "v_fmac_f64_dpp %0, %2, %5 row_newbcast:%13 " RFI_FB
        "v_fmac_f64_dpp %1, %2, %9 row_newbcast:%13 " RFI_FB
        "v_fmac_f64_dpp %0, %2, %6 row_newbcast:%14 " RFI_FB
        "v_fmac_f64_dpp %1, %2, %10 row_newbcast:%14 row_mask:0xf bank_mask:0xf"
        : "+&v"(p), "+&v"(q)
        : "v"(src), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(b[0]), "v"(b[1]), "v"(b[2]),
          "v"(b[3]), "n"(J), "n"(J + 1), "n"(J + 2), "n"(J + 3));
  else if constexpr (C == 3)
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %2, %3 row_newbcast:%9 " RFI_FB
        "v_fmac_f64_dpp %1, %2, %6 row_newbcast:%9 " RFI_FB
        "v_fmac_f64_dpp %0, %2, %4 row_newbcast:%10 " RFI_FB
        "v_fmac_f64_dpp %1, %2, %7 row_newbcast:%10 " RFI_FB
        "v_fmac_f64_dpp %0, %2, %5 row_newbcast:%11 " RFI_FB
        "v_fmac_f64_dpp %1, %2, %8 row_newbcast:%11 row_mask:0xf bank_mask:0xf"
        : "+&v"(p), "+&v"(q)
        : "v"(src), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(b[0]), "v"(b[1]), "v"(b[2]), "n"(J),
          "n"(J + 1), "n"(J + 2));
  else if constexpr (C == 2)
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %2, %3 row_newbcast:%7 " RFI_FB
        "v_fmac_f64_dpp %1, %2, %5 row_newbcast:%7 " RFI_FB
        "v_fmac_f64_dpp %0, %2, %4 row_newbcast:%8 " RFI_FB
        "v_fmac_f64_dpp %1, %2, %6 row_newbcast:%8 row_mask:0xf bank_mask:0xf"
        : "+&v"(p), "+&v"(q)
        : "v"(src), "v"(a[0]), "v"(a[1]), "v"(b[0]), "v"(b[1]), "n"(J), "n"(J + 1));
  else
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %2, %3 row_newbcast:%5 " RFI_FB
        "v_fmac_f64_dpp %1, %2, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf"
        : "+&v"(p), "+&v"(q)
        : "v"(src), "v"(a[0]), "v"(b[0]), "n"(J));
}
// a[i] -= bcast(sv, J + i) w + bcast(sw, J + i) v, i < C
template <int J, int C>
__device__ __forceinline__ void up1(double* a, double sv, double sw, double v, double w) {
  if constexpr (C == 4)
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%4, %7 row_newbcast:%8 " RFI_FB
        "v_fmac_f64_dpp %1, -%4, %7 row_newbcast:%9 " RFI_FB
        "v_fmac_f64_dpp %2, -%4, %7 row_newbcast:%10 " RFI_FB
        "v_fmac_f64_dpp %3, -%4, %7 row_newbcast:%11 " RFI_FB
        "v_fmac_f64_dpp %0, -%5, %6 row_newbcast:%8 " RFI_FB
        "v_fmac_f64_dpp %1, -%5, %6 row_newbcast:%9 " RFI_FB
        "v_fmac_f64_dpp %2, -%5, %6 row_newbcast:%10 " RFI_FB
        "v_fmac_f64_dpp %3, -%5, %6 row_newbcast:%11 row_mask:0xf bank_mask:0xf"
        : "+&v"(a[0]), "+&v"(a[1]), "+&v"(a[2]), "+&v"(a[3])
        : "v"(sv), "v"(sw), "v"(v), "v"(w), "n"(J), "n"(J + 1), "n"(J + 2), "n"(J + 3));
  else if constexpr (C == 3)
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%3, %6 row_newbcast:%7 " RFI_FB
        "v_fmac_f64_dpp %1, -%3, %6 row_newbcast:%8 " RFI_FB
        "v_fmac_f64_dpp %2, -%3, %6 row_newbcast:%9 " RFI_FB
        "v_fmac_f64_dpp %0, -%4, %5 row_newbcast:%7 " RFI_FB
        "v_fmac_f64_dpp %1, -%4, %5 row_newbcast:%8 " RFI_FB
        "v_fmac_f64_dpp %2, -%4, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf"
        : "+&v"(a[0]), "+&v"(a[1]), "+&v"(a[2])
        : "v"(sv), "v"(sw), "v"(v), "v"(w), "n"(J), "n"(J + 1), "n"(J + 2));
  else if constexpr (C == 2)
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%2, %5 row_newbcast:%6 " RFI_FB
        "v_fmac_f64_dpp %1, -%2, %5 row_newbcast:%7 " RFI_FB
        "v_fmac_f64_dpp %0, -%3, %4 row_newbcast:%6 " RFI_FB
        "v_fmac_f64_dpp %1, -%3, %4 row_newbcast:%7 row_mask:0xf bank_mask:0xf"
        : "+&v"(a[0]), "+&v"(a[1])
        : "v"(sv), "v"(sw), "v"(v), "v"(w), "n"(J), "n"(J + 1));
  else
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%1, %4 row_newbcast:%5 " RFI_FB
        "v_fmac_f64_dpp %0, -%2, %3 row_newbcast:%5 row_mask:0xf bank_mask:0xf"
        : "+&v"(a[0])
        : "v"(sv), "v"(sw), "v"(v), "v"(w), "n"(J));
}

// 1 / sqrt(x) and 1 / x to full FP64 precision (hardware estimate, two Newton
// steps), x positive and normal
__device__ __forceinline__ double rsqrt2(double x) {
  double r = __builtin_amdgcn_rsq(x);
  r = fma(r, fma(-0.5 * x * r, r, 0.5), r);
  return fma(r, fma(-0.5 * x * r, r, 0.5), r);
}
__device__ __forceinline__ double rcp2(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  return fma(r, fma(-x, r, 1.0), r);
}

// The power of two that brings a matrix of squared norm frob2 to a norm of about
// 1 when divided out, and frob2 with it (an exact step). The minors below multiply
// up to eight of a matrix's entries before they are rescaled, which leaves FP64's
// range outside 1e-36 .. 1e36: a correlation matrix is always inside, the
// non-centred matrix of a blanked band (its baseline decays to 1e-20 and less) not.
__device__ __forceinline__ int unit_scale(double& frob2) {
  const int e = __builtin_amdgcn_frexp_exp(frob2) >> 1;
  frob2 = ldexp(frob2, -2 * e);
  return e;
}

// orders this wavefront's LDS accesses among its lanes
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// The characteristic polynomial at a point: p 2^e.
struct CharPoly {
  double p;
  int e;
};
// |b| / |a|, saturating
__device__ __forceinline__ double poly_ratio(const CharPoly& a, const CharPoly& b) {
  return ldexp(fabs(b.p) * __builtin_amdgcn_rcp(fabs(a.p)), b.e - a.e);
}

// Brings the last two minors back to the order of 1; returns the power of two.
__device__ __forceinline__ int rescale(double& p1, double& p2) {
  const int e = __builtin_amdgcn_frexp_exp(fmax(fabs(p1), fabs(p2)));
  p1 = ldexp(p1, -e);
  p2 = ldexp(p2, -e);
  return e;
}

// Whether x lies above every eigenvalue: all minors positive. A minor that is
// exactly zero makes the next one negative, or (T decoupled there) the last
// one zero.
__device__ __forceinline__ bool above_all(const double2* ae, int n, double x, CharPoly& f) {
  double p1 = 1.0, p2 = 0.0;
  int sg = 0, e = 0;
  for (int i0 = 0; i0 < n; i0 += 8) {
    double2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = ae[i0 + u < n ? i0 + u : n - 1];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (i0 + u < n) {
        const double p = fma(x - v[u].x, p1, -(v[u].y * p2));
        p2 = p1;
        p1 = p;
        sg |= __double2hiint(p);
      }
    }
    e += rescale(p1, p2);
  }
  f = {p1, e};
  return sg >= 0 && p1 > 0.0;
}

// Number of eigenvalues below x[s] (n minus the sign changes) and P_n there,
// Q points at once. The signs are gathered 32 rows to a word. A zero minor is
// rare (x on an eigenvalue of a leading block) and would lose the rows after
// it where T decouples: those points are counted again with the zero replaced
// by a tiny value of its predecessor's sign.
template <int Q>
__device__ __forceinline__ void count_below(const double2* ae, int n, const double (&x)[Q],
                                            int (&cnt)[Q], CharPoly (&f)[Q]) {
  double p1[Q], p2[Q], least[Q];
  unsigned h[Q];
#pragma unroll
  for (int s = 0; s < Q; ++s) {
    p1[s] = 1.0;
    p2[s] = 0.0;
    least[s] = 1.0;
    h[s] = 0;
    cnt[s] = n;
    f[s].e = 0;
  }
  for (int i0 = 0; i0 < n; i0 += 8) {
    double2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = ae[i0 + u < n ? i0 + u : n - 1];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (i0 + u < n) {
#pragma unroll
        for (int s = 0; s < Q; ++s) {
          const double p = fma(x[s] - v[u].x, p1[s], -(v[u].y * p2[s]));
          p2[s] = p1[s];
          p1[s] = p;
          least[s] = fmin(least[s], fabs(p));
          h[s] = __builtin_amdgcn_alignbit(h[s], (unsigned)__double2hiint(p), 31);
        }
      }
    }
    // signs of rows i0 - 1 .. i0 + 7 (the newest in bit 0): changes between
    // neighbours, the rows of this block only
    const int m = n - i0 < 8 ? n - i0 : 8;
#pragma unroll
    for (int s = 0; s < Q; ++s) {
      cnt[s] -= __popc((h[s] ^ (h[s] >> 1)) & ((1u << m) - 1u));
      f[s].e += rescale(p1[s], p2[s]);
    }
  }
#pragma unroll
  for (int s = 0; s < Q; ++s) {
    f[s].p = p1[s];
    if (__any(least[s] == 0.0)) {
      double a = 1.0, b = 0.0;
      int c = n;
      for (int i = 0; i < n; ++i) {
        const double2 v = ae[i];
        double p = fma(x[s] - v.x, a, -(v.y * b));
        p = p == 0.0 ? copysign(1e-290, a) : p;
        c -= (unsigned)(__double2hiint(p) ^ __double2hiint(a)) >> 31;
        b = a;
        a = p;
        if ((i & 7) == 7) (void)rescale(a, b);
      }
      cnt[s] = c;
    }
  }
}

// Bracket of the spectrum: Gershgorin, and from below the largest eigenvalue
// of every 2 x 2 principal block (Cauchy interlacing). off: |off_i| or signed.
struct Spectrum {
  double lo, hi, top;      // all eigenvalues in [lo, hi], lambda_1 >= top
};
template <int W>
__device__ __forceinline__ Spectrum spectrum_bounds(const double2* ae, const double* off, int n,
                                                    int l) {
  double glo = 1e300, ghi = -1e300, lb = -1e300;
  for (int i = l; i < n; i += W) {
    const double al = ae[i].x, ol = i > 0 ? fabs(off[i - 1]) : 0.0;
    const double on = i + 1 < n ? fabs(off[i]) : 0.0;
    glo = fmin(glo, al - (ol + on));
    ghi = fmax(ghi, al + (ol + on));
    double m = al;
    if (i + 1 < n) {
      const double an = ae[i + 1].x, h = 0.5 * (al - an);
      m = 0.5 * (al + an) + sqrt(h * h + on * on);
    }
    lb = fmax(lb, m);
  }
  glo = group_min<W>(glo);
  ghi = group_max<W>(ghi);
  lb = group_max<W>(lb);
  const double span = fmax(ghi - glo, 1e-300);
  // (two rows: the block is the matrix)
  return {glo - 1e-12 * span, (n == 2 ? lb : ghi) + 1e-12 * span, lb - 1e-12 * span};
}

// The largest eigenvalue, to 2e-14 of max(|lambda_1|, floor) (the order of the
// backward error of an FP64 reduction). The W lanes of the group test W points
// of the bracket per pass: W + 1 equal parts at first; once P_n is negative at
// its lower end (only lambda_1 lies above), points crowded around the secant's
// root, 4^-j of the bracket on either side, until a pass gains less than equal
// parts would. 36 beams: 6 to 7 passes of 16 points instead of 12.
template <int W>
__device__ __forceinline__ double largest_eigenvalue(const double2* ae, int n, int l,
                                                     const Spectrum& sp, double floor_) {
  const int base = threadIdx.x & 63 & ~(W - 1);
  double lo = fmax(sp.lo, sp.top), hi = sp.hi;
  CharPoly flo{1.0, 0}, fhi{1.0, 0};
  bool have_lo = false, have_hi = false, guided = true;
  for (int it = 0; it < 40; ++it) {
    const double w = hi - lo;
    const bool open = w > 2e-14 * fmax(fabs(hi), floor_);
    if (!__any(open)) break;
    const bool secant = guided && have_lo && have_hi && flo.p < 0.0;
    double x;
    if (secant) {
      const double t = __builtin_amdgcn_rcp(1.0 + poly_ratio(flo, fhi));
      const int j = l < W / 2 ? l : W - 1 - l;           // 0: farthest from the root
      const double d = ldexp(w, -3 - (W == 16 ? 2 * j : j));
      x = fma(t, w, lo) + (l < W / 2 ? -d : d);
      x = fmin(fmax(x, lo), hi);
    } else {
      x = fma((l + 1) * (1.0 / (W + 1)), w, lo);
    }
    CharPoly f;
    const bool up = above_all(ae, n, x, f);
    const unsigned long long bal = __ballot(up) >> base;
    const unsigned long long b = W == 64 ? bal : bal & ((1ull << (W & 63)) - 1);
    const int first = b ? __builtin_ctzll(b) : W;        // first point above all
    // the new ends and P_n there
    const int ihi = base + (first < W ? first : W - 1), ilo = base + (first > 0 ? first - 1 : 0);
    const double xh = __shfl(x, ihi), xl = __shfl(x, ilo);
    const CharPoly fh{__shfl(f.p, ihi), __shfl(f.e, ihi)};
    const CharPoly fl{__shfl(f.p, ilo), __shfl(f.e, ilo)};
    if (open) {
      if (first < W) {
        hi = xh;
        fhi = fh;
        have_hi = true;
      }
      if (first > 0) {
        lo = xl;
        flo = fl;
        have_lo = true;
      }
      guided = !secant || (hi - lo) * (W + 1) <= w;
    }
  }
  return 0.5 * (lo + hi);
}

// Every eigenvalue, index i = l + W s ascending, to 2e-16 of max(|lambda|,
// floor). The counts and P_n at W Q equally spaced points, shared through LDS
// (scratch: 12 W Q bytes), bracket them; each is then bisected until it is
// alone in its bracket and closed in on with the ITP steps of Oliveira and
// Takahashi (2020): the secant's root (the older end's P_n halved when the
// same end moves twice), moved towards the middle by 0.2 w^2 / h but by the
// tolerance at least, and never further from the middle than bisection's own
// schedule with six evaluations' slack. 13 evaluations on average and rarely
// over 20, instead of 53.
template <int W, int Q>
__device__ __forceinline__ void all_eigenvalues(const double2* ae, int n, int l,
                                                const Spectrum& sp, double floor_, double* scratch,
                                                double (&ev)[Q]) {
  constexpr int M = W * Q;
  double* const gp = scratch;
  int* const gc = (int*)(scratch + M);     // count + 128 exponent
  const double h = (sp.hi - sp.lo) * (1.0 / (M + 1));
  double a[Q], b[Q], x[Q], R[Q];
  int c[Q];
  CharPoly f[Q], fa[Q], fb[Q];
  // bits: 1 P_n known at a, 2 at b, 4 count(a) == i, 8 count(b) == i + 1, 16
  // the last move was b's, 32 a's
  int state[Q];
#pragma unroll
  for (int s = 0; s < Q; ++s) x[s] = fma((double)(l + W * s + 1), h, sp.lo);
  count_below<Q>(ae, n, x, c, f);
#pragma unroll
  for (int s = 0; s < Q; ++s) {
    gp[l + W * s] = f[s].p;
    gc[l + W * s] = c[s] + f[s].e * 128;
  }
  wave_sync();
#pragma unroll
  for (int s = 0; s < Q; ++s) c[s] = 0;
  for (int m = 0; m < M; ++m) {
    const int g = gc[m] & 127;
#pragma unroll
    for (int s = 0; s < Q; ++s) c[s] += g <= l + W * s;
  }
#pragma unroll
  for (int s = 0; s < Q; ++s) {
    const int i = l + W * s, k = c[s];
    a[s] = sp.lo;
    b[s] = sp.hi;
    fa[s] = fb[s] = CharPoly{1.0, 0};
    state[s] = (i == 0 ? 4 : 0) | (i == n - 1 ? 8 : 0);
    if (k > 0) {
      const int g = gc[k - 1];
      a[s] = fma((double)k, h, sp.lo);
      fa[s] = {gp[k - 1], g >> 7};
      state[s] = (state[s] & 8) | 1 | ((g & 127) == i ? 4 : 0);
    }
    if (k < M) {
      const int g = gc[k];
      b[s] = fma((double)(k + 1), h, sp.lo);
      fb[s] = {gp[k], g >> 7};
      state[s] = (state[s] & 5) | 2 | ((g & 127) == i + 1 ? 8 : 0);
    }
    R[s] = 0.0;
  }
  const double k1 = 0.2 / fmax(h, 1e-300);
  for (int it = 0; it < 160; ++it) {
    bool any = false;
    bool open[Q];
#pragma unroll
    for (int s = 0; s < Q; ++s) {
      const double wd = b[s] - a[s], mid = 0.5 * (a[s] + b[s]);
      const double tol = 2e-16 * fmax(fabs(b[s]), floor_);
      open[s] = l + W * s < n && wd > tol && mid > a[s] && mid < b[s];
      any |= open[s];
      x[s] = mid;
      if ((state[s] & 15) == 15) {
        R[s] = R[s] > 0.0 ? 0.5 * R[s] : 64.0 * wd;
        const double xf = fma(wd, __builtin_amdgcn_rcp(1.0 + poly_ratio(fa[s], fb[s])), a[s]);
        const double to = mid - xf, sg = copysign(1.0, to), dl = fmax(k1 * wd * wd, 2.0 * tol);
        const double xt = fabs(to) > dl ? fma(sg, dl, xf) : mid;
        const double r = fma(-0.5, wd, R[s]);
        const double xi = fabs(xt - mid) <= r ? xt : fma(-sg, r, mid);
        if (xi > a[s] && xi < b[s]) x[s] = xi;
      }
    }
    if (!__any(any)) break;
    count_below<Q>(ae, n, x, c, f);
#pragma unroll
    for (int s = 0; s < Q; ++s) {
      if (!open[s]) continue;
      const int i = l + W * s;
      if (c[s] > i) {
        fa[s].e -= state[s] >> 4 & 1;
        b[s] = x[s];
        fb[s] = f[s];
        state[s] = (state[s] & 5) | 18 | (c[s] == i + 1 ? 8 : 0);
      } else {
        fb[s].e -= state[s] >> 5 & 1;
        a[s] = x[s];
        fa[s] = f[s];
        state[s] = (state[s] & 10) | 33 | (c[s] == i ? 4 : 0);
      }
    }
  }
#pragma unroll
  for (int s = 0; s < Q; ++s) ev[s] = 0.5 * (a[s] + b[s]);
  wave_sync();                             // scratch is free again
}

// Eigenvector z (unit norm, in LDS) of T for the eigenvalue just below sg:
// three steps of inverse iteration on sg I - T from the all-ones vector. sg
// lies above every eigenvalue, so LDL^T needs no pivoting. Every lane of the
// group runs the same recurrences (16 lanes or 64 cost the same); iq, lm: LDS
// scratch [n]. Blocks of eight rows are read before they are worked on, so
// that a step waits on arithmetic alone.
template <int W>
__device__ __forceinline__ void top_eigenvector(const double2* ae, const double* off, int n, int l,
                                                double sg, double* iq, double* lm, double* z) {
  double q = sg - ae[0].x;
  for (int i0 = 0; i0 < n; i0 += 8) {
    double o[8], an[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + u + 1 < n ? i0 + u : n - 2;
      o[u] = i0 + u + 1 < n ? off[i] : 0.0;
      an[u] = ae[i + 1].x;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (i0 + u < n) {
        const double r = rcp2(q > 1e-290 ? q : 1e-290), m = -o[u] * r;
        iq[i0 + u] = r;
        lm[i0 + u] = m;
        q = fma(m, o[u], sg - an[u]);     // sg - alpha_{i+1} - off_i^2 / q
      }
    }
  }
  wave_sync();
  double sc = 1.0;
  for (int iter = 0; iter < 3; ++iter) {
    double y = 0.0, m = 0.0;
    for (int i0 = 0; i0 < n; i0 += 8) {
      double zb[8], mb[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int i = i0 + u < n ? i0 + u : n - 1;
        zb[u] = iter ? z[i] : 1.0;
        mb[u] = lm[i];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (i0 + u < n) {
          y = fma(-m, y, zb[u] * sc);
          m = mb[u];
          z[i0 + u] = y;
        }
      }
    }
    wave_sync();
    double t = 0.0, nrm = 0.0;
    for (int i1 = n - 1; i1 >= 0; i1 -= 8) {
      double zb[8], mb[8], qb[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int i = i1 - u >= 0 ? i1 - u : 0;
        zb[u] = z[i];
        mb[u] = lm[i];
        qb[u] = iq[i];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (i1 - u >= 0) {
          t = fma(-mb[u], t, zb[u] * qb[u]);
          z[i1 - u] = t;
          nrm = fma(t, t, nrm);
        }
      }
    }
    wave_sync();
    sc = 1.0 / sqrt(nrm);
  }
  for (int i = l; i < n; i += W) z[i] *= sc;
  wave_sync();
}

#undef RFI_FB

}  // namespace rfi
