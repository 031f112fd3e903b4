// lbm_vn.hip -- batched Von Neumann analysis of the linearised scheme with
// the absorbing term (Xu & Sagaut, arXiv:1203.6350, Section 3.2, eqs.
// eq:linearized, perturb-w-f, sec:matrix), FP64 on gfx950.
//
// For each parameter set the block first forms the real 9x9 Jacobian of the
// collision at f^eq(q_ref) in moment space,
//   A_m = I + S (J D P - I) - chi X,
// (P: picks rho, jx, jy; D = diag(1/(1+n chi), 1/(1+m chi), 1/(1+m chi)) is
// the derivative of the shifted rho*, j*; J = d m^eq/d(rho, j) at q_ref;
// X = I for Type I, J D P for Type II, L D P for Type III with
// L = d m^L/d(rho, j); X = 0 and D = I without damping), then
// A = M^-1 A_m M. Each thread takes one wavenumber k and
//   G(k) = diag(exp(-i k.c_j)) A
// (the streaming phase, pull form), reduces G to upper Hessenberg form with
// complex Householder reflections and finds its eigenvalues with single-shift
// complex QR (Wilkinson shifts, deflation on negligible subdiagonals,
// exceptional shifts after 10 and 20 stalled sweeps). Eigenvalues are
// returned sorted by (-|lambda|, arg lambda).
//
// Each lane holds its wavenumber's matrix in registers (every index fixed at
// compile time: the loops are fully unrolled). The QR sweeps are wave-wide and
// run level by level: at level h (8 down to 2) a sweep works on rows and columns
// 0..h only, and a lane takes part while the bottom of its active window is h or
// h - 1, so that the entries at the bottom are one of two fixed positions; a lane
// further ahead waits, masked off. With that slack of one a wave needs no more
// sweeps than lanes running freely would (29 a wave, 26 a lane on MRT sets
// with flow), and the sweep has neither gathers nor predicates. A lane's own
// sequence of checks, shifts and rotations does not depend on the others: where
// eigenvalues tie in modulus (waves along an axis), their order hangs on the last
// bit, so the arithmetic is kept as it is, without fused products. (Fused, and
// with a real subdiagonal, the same sweep takes 6.5 ms, in another order there.)
//
// Bound by VALU issue at one wave per SIMD: two thirds of a sweep's instructions
// are FP64, at level 8 a fifth move the window between the two halves of the
// register file. Registers that do not fit go to scratch memory; so four rows of
// the matrix lie in LDS while it is reduced, and the window's last column at levels
// 8 and 7 (38 KB, a quarter of the CU's; level 6 too: no gain).
//
// 64 sets x 256^2 wavenumbers: 15.7 ms (268 M eigenproblems/s) with one window 0..8
// in every sweep and the entries at a lane's own bottom selected over all
// positions, now 12 to 13 ms (traced launches 11.9 to 13.3, 334 M/s on average).
#include "lbm_device.h"
#include "lbm_internal.h"

namespace lbm {

namespace {

struct cplx {
  double re, im;
};
__device__ __forceinline__ cplx mk(double r, double i) { return cplx{r, i}; }
__device__ __forceinline__ cplx add(cplx a, cplx b) { return mk(a.re + b.re, a.im + b.im); }
__device__ __forceinline__ cplx sub(cplx a, cplx b) { return mk(a.re - b.re, a.im - b.im); }
__device__ __forceinline__ cplx mul(cplx a, cplx b) {
  return mk(a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re);
}
__device__ __forceinline__ cplx conjc(cplx a) { return mk(a.re, -a.im); }
__device__ __forceinline__ cplx scal(double s, cplx a) { return mk(s * a.re, s * a.im); }
__device__ __forceinline__ double abs1(cplx a) { return fabs(a.re) + fabs(a.im); }
__device__ __forceinline__ double absc(cplx a) { return hypot(a.re, a.im); }
__device__ __forceinline__ cplx divc(cplx a, cplx b) {
  // Smith's algorithm
  if (fabs(b.re) >= fabs(b.im)) {
    const double r = b.im / b.re, d = b.re + b.im * r;
    return mk((a.re + a.im * r) / d, (a.im - a.re * r) / d);
  }
  const double r = b.re / b.im, d = b.re * r + b.im;
  return mk((a.re * r + a.im) / d, (a.im * r - a.re) / d);
}
__device__ __forceinline__ cplx sqrtc(cplx z) {
  const double r = absc(z);
  if (r == 0.0) return mk(0.0, 0.0);
  if (z.re >= 0.0) {
    const double t = sqrt(0.5 * (r + z.re));
    return mk(t, z.im / (2.0 * t));
  }
  const double t = sqrt(0.5 * (r - z.re));
  return mk(fabs(z.im) / (2.0 * t), copysign(t, z.im));
}

constexpr int N = 9;

// The D2Q9 transform of Appendix A.1, row-major; rows (rho, jx, jy, e, eps,
// qx, qy, pxx, pxy).
__constant__ double kM[81] = {
     1,  1,  1,  1,  1, 1,  1,  1,  1,
     0,  1,  0, -1,  0, 1, -1, -1,  1,
     0,  0,  1,  0, -1, 1,  1, -1, -1,
    -4, -1, -1, -1, -1, 2,  2,  2,  2,
     4, -2, -2, -2, -2, 1,  1,  1,  1,
     0, -2,  0,  2,  0, 1, -1, -1,  1,
     0,  0, -2,  0,  2, 1,  1, -1, -1,
     0,  1, -1,  1, -1, 0,  0,  0,  0,
     0,  0,  0,  0,  0, 1, -1,  1, -1};
// Squared row norms (M M^T)_kk; the rows are orthogonal, so
// (M^-1)_{ik} = M_{ki} / (M M^T)_kk.
__constant__ double kMnorm[9] = {9, 6, 6, 36, 36, 12, 12, 4, 4};

// Moment-space Jacobian A_m (row-major 81) for one parameter set.
__device__ void build_Am(const VnParamsDev &p, double *Am) {
  const double chi = p.variant == V_NONE ? 0.0 : p.chi;
  const double ux = p.ux_f, uy = p.uy_f, u2 = ux * ux + uy * uy;
  const double J[9][3] = {{1, 0, 0}, {0, 1, 0}, {0, 0, 1},
                          {-2.0 - 3.0 * u2, 6.0 * ux, 6.0 * uy},
                          {1.0 + 3.0 * u2, -6.0 * ux, -6.0 * uy},
                          {0, -1, 0}, {0, 0, -1},
                          {-(ux * ux - uy * uy), 2.0 * ux, -2.0 * uy},
                          {-ux * uy, uy, ux}};
  const double L[9][3] = {{1, 0, 0}, {0, 1, 0}, {0, 0, 1}, {-2, 0, 0}, {1, 0, 0},
                          {0, -1, 0}, {0, 0, -1}, {0, 0, 0}, {0, 0, 0}};
  const double D[3] = {1.0 / (1.0 + p.n * chi), 1.0 / (1.0 + p.m * chi),
                       1.0 / (1.0 + p.m * chi)};
  for (int k = 0; k < 9; ++k) {
    for (int l = 0; l < 9; ++l) {
      const double JDP = l < 3 ? J[k][l] * D[l] : 0.0;
      const double LDP = l < 3 ? L[k][l] * D[l] : 0.0;
      const double id = k == l ? 1.0 : 0.0;
      double X = 0.0;
      if (p.variant == V_I) X = id;
      else if (p.variant == V_II) X = JDP;
      else if (p.variant == V_III) X = LDP;
      Am[k * 9 + l] = id + p.s[k] * (JDP - id) - chi * X;
    }
  }
}

// Eigenvalues of the 2x2 block [a b; c d].
__device__ void eig2(cplx a, cplx b, cplx c, cplx d, cplx &l1, cplx &l2) {
  const cplx p = scal(0.5, sub(a, d));
  const cplx bc = mul(b, c);
  cplx y = sqrtc(add(mul(p, p), bc));
  if (p.re * y.re + p.im * y.im < 0.0) y = scal(-1.0, y);
  const cplx z1 = add(p, y);
  if (abs1(z1) == 0.0) {
    l1 = d;
    l2 = d;
    return;
  }
  l1 = add(d, z1);
  l2 = sub(d, divc(bc, z1));
}

}  // namespace

// 1/sqrt(x) for x > 0 to about one ulp: the hardware estimate refined by
// two Newton steps (each doubles the correct bits).
__device__ __forceinline__ double rsqrt_f64(double x) {
  double y = __builtin_amdgcn_rsq(x);
  const double hx = 0.5 * x;
  y = y * __builtin_fma(-hx * y, y, 1.5);
  y = y * __builtin_fma(-hx * y, y, 1.5);
  return y;
}

// One lane's matrix: H = R + i I, row-major, static indices only.
struct RegMat {
  double r[N][N], m[N][N];
  __device__ __forceinline__ cplx at(int i, int j) const { return mk(r[i][j], m[i][j]); }
  __device__ __forceinline__ void put(int i, int j, cplx v) {
    r[i][j] = v.re;
    m[i][j] = v.im;
  }
};

// The matrix while it is reduced: its first VN_LDS_ROWS rows lie in LDS (a lane's
// entries [(row * N + column) * 64]), which leaves the registers room for the
// rest. The clobbers keep the compiler from carrying those rows in registers
// after all.
constexpr int VN_LDS_ROWS = 4;
struct SplitMat {
  RegMat H;
  double2 *rows;
  __device__ __forceinline__ cplx at(int i, int j) const {
    if (i >= VN_LDS_ROWS) return H.at(i, j);
    const double2 v = rows[(i * N + j) * 64];
    return mk(v.x, v.y);
  }
  __device__ __forceinline__ void put(int i, int j, cplx v) {
    if (i >= VN_LDS_ROWS)
      H.put(i, j, v);
    else
      rows[(i * N + j) * 64] = make_double2(v.re, v.im);
  }
  __device__ __forceinline__ void settle() const { asm volatile("" ::: "memory"); }
};

__device__ __forceinline__ cplx pick2(bool first, cplx a, cplx b) {
  return mk(first ? a.re : b.re, first ? a.im : b.im);
}

// Householder reduction to upper Hessenberg form, H <- Q^H H Q: the reflection of
// column k.
template <int k>
__device__ __forceinline__ void reflect(SplitMat &H) {
  double xn2 = 0.0;
  cplx v[N];
#pragma unroll
  for (int i = k + 1; i < N; ++i) {
    v[i] = H.at(i, k);
    xn2 += v[i].re * v[i].re + v[i].im * v[i].im;
  }
  const double xn = sqrt(xn2);
  const cplx x0 = v[k + 1];
  const double ax0 = absc(x0);
  const cplx ph = ax0 > 0.0 ? scal(1.0 / ax0, x0) : mk(1.0, 0.0);
  const cplx alpha = scal(-xn, ph);  // -e^{i arg x0} ||x||
  // v = x - alpha e1, normalised (v = 0, the identity, for a zero column)
  double vn2 = 0.0;
  v[k + 1] = sub(x0, alpha);
#pragma unroll
  for (int i = k + 1; i < N; ++i) vn2 += v[i].re * v[i].re + v[i].im * v[i].im;
  const double inv = vn2 > 0.0 ? rsqrt_f64(vn2) : 0.0;
#pragma unroll
  for (int i = k + 1; i < N; ++i) v[i] = scal(inv, v[i]);
  // left: rows k+1.., columns k+1..
#pragma unroll
  for (int j = k + 1; j < N; ++j) {
    cplx w = mk(0.0, 0.0), x[N];
#pragma unroll
    for (int i = k + 1; i < N; ++i) {
      x[i] = H.at(i, j);
      w = add(w, mul(conjc(v[i]), x[i]));
    }
    w = scal(2.0, w);
#pragma unroll
    for (int i = k + 1; i < N; ++i) H.put(i, j, sub(x[i], mul(v[i], w)));
    H.settle();
  }
  // column k below the subdiagonal: the reflection maps x to alpha e1
  // (with v = 0 the column was zero below x0 already); the entries below
  // the subdiagonal become compile-time zeros, which frees their registers
  // for the QR sweeps (they never read them)
  H.put(k + 1, k, vn2 > 0.0 ? alpha : x0);
#pragma unroll
  for (int i = k + 2; i < N; ++i)
    if (i >= VN_LDS_ROWS) H.put(i, k, mk(0.0, 0.0));
  // right: all rows, columns k+1..
#pragma unroll
  for (int i = 0; i < N; ++i) {
    cplx w = mk(0.0, 0.0), x[N];
#pragma unroll
    for (int j = k + 1; j < N; ++j) {
      x[j] = H.at(i, j);
      w = add(w, mul(x[j], v[j]));
    }
    w = scal(2.0, w);
#pragma unroll
    for (int j = k + 1; j < N; ++j) H.put(i, j, sub(x[j], mul(w, conjc(v[j]))));
    H.settle();
  }
}

template <int k>
__device__ __forceinline__ void reflect_from(SplitMat &H) {
  reflect<k>(H);
  if constexpr (k + 1 < N - 2) reflect_from<k + 1>(H);
}

__device__ __forceinline__ void hessenberg_reg(SplitMat &H) {
  reflect_from<0>(H);
  // all in registers from here on
#pragma unroll
  for (int i = 0; i < VN_LDS_ROWS; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) H.H.put(i, j, j >= i - 1 ? H.at(i, j) : mk(0.0, 0.0));
  H.settle();
}

// Rotation [c s; -conj(s) conj(c)] with c = conj(x)/r, s = conj(y)/r,
// r = sqrt(|x|^2 + |y|^2), which maps (x, y) to (r, 0); the identity when
// inactive or when x = y = 0.
__device__ __forceinline__ void givens(cplx x, cplx y, bool act, cplx &c, cplx &s) {
  const double n2 = x.re * x.re + x.im * x.im + y.re * y.re + y.im * y.im;
  const bool on = act && n2 > 0.0;
  const double ir = on ? rsqrt_f64(n2) : 0.0;
  c = on ? mk(x.re * ir, -x.im * ir) : mk(1.0, 0.0);
  s = on ? mk(y.re * ir, -y.im * ir) : mk(0.0, 0.0);
}

// A left rotation of the pair (a, b) of one column, and a right one of one row.
__device__ __forceinline__ void left_rot(cplx c, cplx s, cplx &a, cplx &b) {
  const cplx t1 = a, t2 = b;
  a = add(mul(c, t1), mul(s, t2));
  b = sub(mul(conjc(c), t2), mul(conjc(s), t1));
}
__device__ __forceinline__ void right_rot(cplx c, cplx s, cplx &a, cplx &b) {
  const cplx t1 = a, t2 = b;
  a = add(mul(t1, conjc(c)), mul(t2, conjc(s)));
  b = sub(mul(t2, c), mul(t1, s));
}

// H <- H G^H on columns q, q + 1 for rows 0..q + 1, G = [c s; -conj(s) conj(c)].
__device__ __forceinline__ void right_rots(RegMat &H, int q, cplx c, cplx s) {
#pragma unroll
  for (int i = 0; i <= q + 1; ++i) {
    cplx a = H.at(i, q), b = H.at(i, q + 1);
    right_rot(c, s, a, b);
    H.put(i, q, a);
    H.put(i, q + 1, b);
  }
}

// From this level on the last column above its diagonal lies in LDS (a lane's
// entries [row * 64]).
constexpr int VN_LDS_LEVEL = 7;
constexpr int VN_MAX_SWEEPS = 40 * N;  // a lane's own, over all its eigenvalues

// The entries of the level's window as new values. Without it an entry is one
// value from the reduction to the last sweep, and what the reduction (324
// registers) spills stays spilled in sweeps that would fit.
__device__ __forceinline__ double detach(double x) {
  double y;
  asm("v_mov_b64 %0, %1" : "=v"(y) : "v"(x));
  return y;
}
template <int h>
__device__ __forceinline__ void detach_window(RegMat &H) {
#pragma unroll
  for (int i = 0; i <= h; ++i)
#pragma unroll
    for (int j = i > 0 ? i - 1 : 0; j <= h; ++j) {
      if (j == h && i < h && h >= VN_LDS_LEVEL) continue;
      H.r[i][j] = detach(H.r[i][j]);
      H.m[i][j] = detach(H.m[i][j]);
    }
}

// QR sweeps of level h: until no lane's active window 0..hi ends at h (each
// sweep: Wilkinson shift from the window's trailing 2 x 2, exceptional
// shifts after 10 and 20 stalled sweeps; a bottom eigenvalue deflates when its
// subdiagonal is negligible, two checks per sweep). A lane that has used up its
// sweeps (one with a NaN does) leaves with hi = -1 and the wave goes on without
// it; every sweep is one of some lane at h, so the loop ends.
template <int h>
__device__ __forceinline__ void qr_level(RegMat &H, int &hi, int &it, int &sweeps, int &deflated, double2 *ev,
                                         int stride, double2 *col) {
  constexpr bool LDS = h >= VN_LDS_LEVEL;
  constexpr int l = h > 2 ? h - 1 : h;  // the lowest window end that takes part
  const double eps = 2.220446049250313e-16;
  auto last = [&](int i) {  // H(i, h), i < h
    if (!LDS) return H.at(i, h);
    const double2 v = col[i * 64];
    return mk(v.x, v.y);
  };
  auto set_last = [&](int i, cplx v) {
    if (LDS)
      col[i * 64] = make_double2(v.re, v.im);
    else
      H.put(i, h, v);
  };
  if (LDS) {
#pragma unroll
    for (int i = 0; i < h; ++i) col[i * 64] = make_double2(H.r[i][h], H.m[i][h]);
  }
  detach_window<h>(H);
  for (;;) {
    if (hi >= l && sweeps >= VN_MAX_SWEEPS) hi = -1;
#pragma unroll
    for (int rep = 0; rep < 2; ++rep) {
      const bool top = hi == h;
      const cplx d = pick2(top, H.at(h, h - 1), H.at(l, l - 1));
      const cplx a = pick2(top, H.at(h - 1, h - 1), H.at(l - 1, l - 1));
      const cplx b = pick2(top, H.at(h, h), H.at(l, l));
      if (hi >= l && deflated < 2 && abs1(d) <= eps * (abs1(a) + abs1(b))) {
        ev[hi * stride] = make_double2(b.re, b.im);
        --hi;
        ++deflated;
        it = 0;
      }
    }
    if (!__any(hi == h)) return;
    if (hi < l) continue;
    const bool top = hi == h;
    const cplx c0 = pick2(top, H.at(h, h - 1), H.at(l, l - 1));
    const cplx d0 = pick2(top, H.at(h, h), H.at(l, l));
    cplx mu;
    if (it == 10 || it == 20) {
      const double e2 = fabs(top || l < 2 ? H.r[h - 1][h - 2] : H.r[l - 1][l - 2]);
      mu = add(d0, mk(0.75 * fabs(c0.re) + e2, 0.0));
    } else {
      cplx l1, l2;
      eig2(pick2(top, H.at(h - 1, h - 1), H.at(l - 1, l - 1)),
           pick2(top, last(h - 1), H.at(l - 1, l)), c0, d0, l1, l2);
      mu = abs1(sub(l1, d0)) <= abs1(sub(l2, d0)) ? l1 : l2;
    }
    ++it;
    ++sweeps;
    deflated = 0;
    // H - mu I on the window; what lies below it (row and column h of a window
    // that ends at h - 1) is no longer read, and takes part in any way
#pragma unroll
    for (int i = 0; i <= h; ++i) H.put(i, i, sub(H.at(i, i), mu));
    // R = G_{h-1} ... G_0 (H - mu I), then R G_0^H ... G_{h-1}^H, with each
    // right rotation applied once the next left one is: the left rotation k
    // reads H(k, k) before the right rotation k - 1 changes it. The rotation
    // h - 1 is the identity for a window that ends there.
    cplx cp = mk(1.0, 0.0), sp = mk(0.0, 0.0), run = last(0);  // run: H(k, h)
#pragma unroll
    for (int k = 0; k < h; ++k) {
      cplx c, s;
      givens(H.at(k, k), H.at(k + 1, k), k < h - 1 || top, c, s);
#pragma unroll
      for (int j = k; j < h; ++j) {
        cplx a = H.at(k, j), b = H.at(k + 1, j);
        left_rot(c, s, a, b);
        H.put(k, j, a);
        H.put(k + 1, j, b);
      }
      cplx b = k + 1 < h ? last(k + 1) : H.at(h, h);
      left_rot(c, s, run, b);
      set_last(k, run);
      run = b;
      if (k > 0) right_rots(H, k - 1, cp, sp);
      cp = c;
      sp = s;
    }
#pragma unroll
    for (int i = 0; i <= h; ++i) {
      cplx a = H.at(i, h - 1), b = i < h ? last(i) : run;
      right_rot(cp, sp, a, b);
      H.put(i, h - 1, a);
      if (i < h)
        set_last(i, b);
      else
        H.put(h, h, b);
    }
#pragma unroll
    for (int i = 0; i <= h; ++i) H.put(i, i, add(H.at(i, i), mu));
  }
}

template <int h>
__device__ __forceinline__ void qr_levels(RegMat &H, int &hi, int &it, int &sweeps, int &deflated, double2 *ev,
                                          int stride, double2 *col) {
  qr_level<h>(H, hi, it, sweeps, deflated, ev, stride, col);
  if constexpr (h > 2) qr_levels<h - 1>(H, hi, it, sweeps, deflated, ev, stride, col);
}

// Eigenvalues of the upper Hessenberg H. Returns false if the lane did not
// converge within VN_MAX_SWEEPS sweeps.
__device__ __forceinline__ bool qr_reg(RegMat &H, double2 *ev, int stride, double2 *col) {
  const double eps = 2.220446049250313e-16;
  int hi = N - 1, it = 0, sweeps = 0, deflated = 0;
  qr_levels<N - 1>(H, hi, it, sweeps, deflated, ev, stride, col);
  if (hi < 0) return false;
  cplx a = H.at(0, 0), b = H.at(0, 1), c = H.at(1, 0), d = H.at(1, 1);
  if (hi == 1 && deflated == 2) {  // a sweep on the 2 x 2
    cplx l1, l2, g, s;
    eig2(a, b, c, d, l1, l2);
    const cplx mu = abs1(sub(l1, d)) <= abs1(sub(l2, d)) ? l1 : l2;
    a = sub(a, mu);
    d = sub(d, mu);
    givens(a, c, true, g, s);
    left_rot(g, s, a, c);
    left_rot(g, s, b, d);
    right_rot(g, s, a, b);
    right_rot(g, s, c, d);
    a = add(a, mu);
    d = add(d, mu);
    deflated = 0;
  }
  if (hi == 1) {
    if (abs1(c) <= eps * (abs1(a) + abs1(d))) {
      ev[stride] = make_double2(d.re, d.im);
      hi = 0;
      ++deflated;
    } else {
      cplx l0, l1;
      eig2(a, b, c, d, l0, l1);
      a = l0;
      ev[stride] = make_double2(l1.re, l1.im);
      deflated = 0;
    }
  }
  if (deflated == 2) {  // a sweep on the last entry alone: its shift out and in again
    cplx l1, l2;
    const cplx z0 = mk(0.0, 0.0);
    eig2(z0, z0, z0, a, l1, l2);
    const cplx mu = abs1(sub(l1, a)) <= abs1(sub(l2, a)) ? l1 : l2;
    a = add(sub(a, mu), mu);
  }
  ev[0] = make_double2(a.re, a.im);
  return true;
}

// One wavenumber per lane, 64 lanes per workgroup (one wave); blockIdx.y
// is the parameter set.
__global__ __launch_bounds__(64) void vn_kernel(const VnParamsDev *__restrict__ params,
                                                int64_t nk,
                                                const double *__restrict__ kx,
                                                const double *__restrict__ ky,
                                                double *__restrict__ eig,
                                                double *__restrict__ G) {
  __shared__ double Are[81];  // A = M^-1 A_m M
  __shared__ double Am[81];
  // the reduction's rows; then the eigenvalues as they deflate, [index][lane],
  // and the window's last column, [row][lane]. 38 KB with A: a block per SIMD.
  __shared__ double2 work[VN_LDS_ROWS * N * 64];
  static_assert(VN_LDS_ROWS * N >= 2 * N - 1, "eigenvalues and column");
  const int pset = blockIdx.y;
  const int t = threadIdx.x;
  if (t == 0) build_Am(params[pset], Am);
  __syncthreads();
  for (int e = t; e < 81; e += 64) {
    const int i = e / 9, j = e % 9;
    double acc = 0.0;
    for (int k = 0; k < 9; ++k) {
      double inner = 0.0;
      for (int l = 0; l < 9; ++l) inner += Am[k * 9 + l] * kM[l * 9 + j];
      acc += kM[k * 9 + i] / kMnorm[k] * inner;
    }
    Are[e] = acc;
  }
  __syncthreads();
  const int64_t kidx = (int64_t)blockIdx.x * 64 + t;
  // lanes past the end solve a copy of the last wavenumber and store nothing,
  // so that every lane of the wave runs the same sweeps
  const int64_t kk = kidx < nk ? kidx : nk - 1;
  const double k1 = kx[kk], k2 = ky[kk];
  double2 *const evs = work, *const col = work + N * 64;
  const int64_t out = (int64_t)pset * nk + kidx;
  SplitMat S;
  S.rows = work + t;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const double ph = -(k1 * cx_of(i) + k2 * cy_of(i));
    double sp, cp;
    sincos(ph, &sp, &cp);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const double a = Are[i * 9 + j];
      S.put(i, j, mk(cp * a, sp * a));
      if (G && kidx < nk) {
        G[(out * 81 + i * N + j) * 2] = cp * a;
        G[(out * 81 + i * N + j) * 2 + 1] = sp * a;
      }
    }
  }
  S.settle();
  hessenberg_reg(S);
  const bool ok = qr_reg(S.H, evs + t, 64, col + t);
  if (kidx >= nk) return;
  cplx ev[N];
  double mag[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const double2 v = evs[i * 64 + t];
    ev[i] = ok ? mk(v.x, v.y) : mk(__builtin_nan(""), __builtin_nan(""));
    mag[i] = absc(ev[i]);
  }
  // insertion sort by (-|lambda|, arg lambda), as a network of neighbours
#pragma unroll
  for (int i = 1; i < N; ++i)
#pragma unroll
    for (int j = i; j > 0; --j) {
      bool swap = mag[j] > mag[j - 1];
      if (mag[j] == mag[j - 1])
        swap = atan2(ev[j].im, ev[j].re) < atan2(ev[j - 1].im, ev[j - 1].re);
      const cplx u = ev[j - 1], v = ev[j];
      ev[j - 1] = swap ? v : u;
      ev[j] = swap ? u : v;
      const double mu = mag[j - 1], mv = mag[j];
      mag[j - 1] = swap ? mv : mu;
      mag[j] = swap ? mu : mv;
    }
#pragma unroll
  for (int i = 0; i < N; ++i)
    ((double2 *)eig)[out * 9 + i] = make_double2(ev[i].re, ev[i].im);
}

hipError_t launch_vn(const VnParamsDev *params_dev, int nparams, int64_t nk,
                     const double *kx, const double *ky, double *eig, double *G,
                     hipStream_t stream) {
  if (nk < 1) return hipSuccess;
  const int64_t bx = (nk + 63) / 64;
  if (bx > 0x7fffffff) return hipErrorInvalidValue;
  vn_kernel<<<dim3((unsigned)bx, (unsigned)nparams), dim3(64), 0, stream>>>(
      params_dev, nk, kx, ky, eig, G);
  return hipGetLastError();
}

}  // namespace lbm
