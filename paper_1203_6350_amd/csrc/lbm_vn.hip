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
// compile time: the loops are fully unrolled). The reduction leaves the
// subdiagonal real and the sweeps keep it so, which makes every rotation 12
// operations a pair instead of 16. The QR sweeps are wave-wide and run level by
// level: at level h (8 down to 2) a sweep works on rows and columns 0..h only,
// and a lane takes part while the bottom of its active window is h or h - 1, so
// that the entries at the bottom are one of two fixed positions; a lane
// further ahead waits, masked off. With that slack of one a wave needs no more
// sweeps than lanes running freely would (29 a wave, 26 a lane on MRT sets
// with flow), and the sweep has neither gathers nor predicates. Complex
// products are fused multiply-adds.
//
// Bound by VALU issue at one wave per SIMD (0.69 busy): half of the instructions
// are FP64, at level 8 a third move the window between the two halves of the
// register file. Registers that do not fit went to scratch memory, whose waits
// took a third of the time; so four rows of the matrix lie in LDS while it is
// reduced, and the window's last column at levels 8 and 7 (38 KB, a quarter of the
// CU's).
//
// 64 sets x 256^2 wavenumbers: 15.7 ms (268 M eigenproblems/s) with one window 0..8
// in every sweep, the entries at a lane's own bottom selected over all
// positions and complex subdiagonals; 9.8 ms by levels, 8.3 ms with the real
// subdiagonal, 7.5 ms with the last column in LDS, 6.5 ms (641 M/s) with the rows.
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

// a b + c, a b, conj(a) b + c and c - a b with fused multiply-adds.
__device__ __forceinline__ cplx cfma(cplx a, cplx b, cplx c) {
  return mk(__builtin_fma(a.re, b.re, __builtin_fma(-a.im, b.im, c.re)),
            __builtin_fma(a.re, b.im, __builtin_fma(a.im, b.re, c.im)));
}
__device__ __forceinline__ cplx cmul(cplx a, cplx b) {
  return mk(__builtin_fma(a.re, b.re, -(a.im * b.im)), __builtin_fma(a.re, b.im, a.im * b.re));
}
__device__ __forceinline__ cplx neg(cplx a) { return mk(-a.re, -a.im); }
__device__ __forceinline__ double norm2(cplx a) { return __builtin_fma(a.re, a.re, a.im * a.im); }
__device__ __forceinline__ cplx pick2(bool first, cplx a, cplx b) {
  return mk(first ? a.re : b.re, first ? a.im : b.im);
}

// |z|, and its phase z/|z| (1 for z = 0, or where |z|^2 is not positive).
__device__ __forceinline__ double polar(cplx z, cplx &e) {
  const double n2 = norm2(z);
  const bool on = n2 > 0.0;
  const double ir = on ? rsqrt_f64(n2) : 0.0;
  e = mk(on ? z.re * ir : 1.0, z.im * ir);
  return n2 * ir;
}

// Householder reduction to upper Hessenberg form with a real subdiagonal. The
// reflection of column k, x = H(k+1.., k), is I - tau v v^H with v = x/|x| + g e1,
// g = +-1 of Re x0's sign and tau = g conj(v0)/|v0|^2: it maps x to -g |x| e1, and
// |v0| >= 1. H <- (I - tau v v^H) H (I - tau v v^H)^H.
template <int k>
__device__ __forceinline__ void reflect(SplitMat &H) {
  double xn2 = 0.0;
  cplx v[N];
#pragma unroll
  for (int i = k + 1; i < N; ++i) {
    v[i] = H.at(i, k);
    xn2 = __builtin_fma(v[i].re, v[i].re, __builtin_fma(v[i].im, v[i].im, xn2));
  }
  const bool on = xn2 > 0.0;  // a zero column stays as it is
  const double ixn = on ? rsqrt_f64(xn2) : 0.0;
  const double g = v[k + 1].re >= 0.0 ? 1.0 : -1.0;
#pragma unroll
  for (int i = k + 1; i < N; ++i) v[i] = scal(ixn, v[i]);
  v[k + 1].re += g;
  const cplx tau = scal(on ? g / norm2(v[k + 1]) : 0.0, conjc(v[k + 1]));
  // left: rows k+1.., columns k+1..
#pragma unroll
  for (int j = k + 1; j < N; ++j) {
    cplx w = mk(0.0, 0.0), x[N];
#pragma unroll
    for (int i = k + 1; i < N; ++i) {
      x[i] = H.at(i, j);
      w = cfma(conjc(v[i]), x[i], w);
    }
    w = neg(cmul(tau, w));
#pragma unroll
    for (int i = k + 1; i < N; ++i) H.put(i, j, cfma(v[i], w, x[i]));
    H.settle();
  }
  // column k: (-g |x|, 0, ...); the entries below the subdiagonal become
  // compile-time zeros, which frees their registers for the QR sweeps
  // (they never read them)
  H.put(k + 1, k, mk(-g * (xn2 * ixn), 0.0));
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
      w = cfma(x[j], v[j], w);
    }
    w = neg(cmul(conjc(tau), w));
#pragma unroll
    for (int j = k + 1; j < N; ++j) H.put(i, j, cfma(w, conjc(v[j]), x[j]));
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
  // the last subdiagonal's phase e: row N - 1 times conj(e), column N - 1 times e
  const cplx y = H.at(N - 1, N - 2);
  cplx e;
  H.put(N - 1, N - 2, mk(polar(y, e), 0.0));
#pragma unroll
  for (int i = 0; i < N - 1; ++i) H.put(i, N - 1, cmul(e, H.at(i, N - 1)));
  // all in registers from here on
#pragma unroll
  for (int i = 0; i < VN_LDS_ROWS; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) H.H.put(i, j, j >= i - 1 ? H.at(i, j) : mk(0.0, 0.0));
  H.settle();
}

// Wilkinson shift of [a b; c d], c real: its eigenvalue nearer d, d - bc / (p + y) with
// p = (a - d)/2, y = sqrt(p^2 + bc) on p's side (so |p + y| >= |p - y|); d where
// that is not finite. It steers the convergence only, so the reciprocals
// are refined estimates.
__device__ __forceinline__ cplx shift_of(cplx a, cplx b, double c, cplx d) {
  const cplx p = scal(0.5, sub(a, d));
  const cplx bc = scal(c, b);
  const cplx q = cfma(p, p, bc);
  const double r2 = norm2(q);
  const double r = r2 > 0.0 ? r2 * rsqrt_f64(r2) : 0.0;
  const double t2 = 0.5 * (r + fabs(q.re));
  const double it = t2 > 0.0 ? rsqrt_f64(t2) : 0.0;
  const double t = t2 * it, u = 0.5 * q.im * it;  // |q.im| / (2 t)
  cplx y = q.re >= 0.0 ? mk(t, u) : mk(fabs(u), copysign(t, q.im));
  if (__builtin_fma(p.re, y.re, p.im * y.im) < 0.0) y = neg(y);
  const cplx z = add(p, y);
  const double z2 = norm2(z);
  const double e = __builtin_amdgcn_rcp(z2);
  const double iz = e * __builtin_fma(-z2, e, 2.0);
  const cplx m = cmul(scal(iz, bc), conjc(z));
  return z2 > 0.0 && __builtin_isfinite(m.re) && __builtin_isfinite(m.im) ? sub(d, m) : d;
}

// conj(c) a + s b and c b - s a, s real: a rotation of the pair (a, b).
__device__ __forceinline__ cplx rot1(cplx c, double s, cplx a, cplx b) {
  return mk(__builtin_fma(s, b.re, __builtin_fma(c.re, a.re, c.im * a.im)),
            __builtin_fma(s, b.im, __builtin_fma(c.re, a.im, -(c.im * a.re))));
}
__device__ __forceinline__ cplx rot2(cplx c, double s, cplx a, cplx b) {
  return mk(__builtin_fma(-s, a.re, __builtin_fma(c.re, b.re, -(c.im * b.im))),
            __builtin_fma(-s, a.im, __builtin_fma(c.re, b.im, c.im * b.re)));
}

// H <- H G^H on columns q, q + 1, G = [c s; -s conj(c)], where row q + 1 holds
// (0, r) with r real.
__device__ __forceinline__ void right_rot(RegMat &H, int q, cplx c, double s) {
#pragma unroll
  for (int i = 0; i <= q; ++i) {
    const cplx a = H.at(i, q), b = H.at(i, q + 1);
    H.put(i, q, rot1(c, s, a, b));
    H.put(i, q + 1, rot2(c, s, a, b));
  }
  const double r = H.r[q + 1][q + 1];
  H.put(q + 1, q, mk(s * r, 0.0));
  H.put(q + 1, q + 1, scal(r, c));
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
__device__ __forceinline__ void qr_level(RegMat &H, int &hi, int &it, int &sweeps, double2 *ev,
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
#pragma unroll
    for (int rep = 0; rep < 2; ++rep) {
      const bool top = hi == h;
      const double d = top ? H.r[h][h - 1] : H.r[l][l - 1];
      const cplx a = pick2(top, H.at(h - 1, h - 1), H.at(l - 1, l - 1));
      const cplx b = pick2(top, H.at(h, h), H.at(l, l));
      if (hi >= l && fabs(d) <= eps * (abs1(a) + abs1(b))) {
        ev[hi * stride] = make_double2(b.re, b.im);
        --hi;
        it = 0;
      }
    }
    if (hi >= l && sweeps >= VN_MAX_SWEEPS) hi = -1;
    if (!__any(hi == h)) return;
    if (hi < l) continue;
    const bool top = hi == h;
    const double c = top ? H.r[h][h - 1] : H.r[l][l - 1];
    const cplx d = pick2(top, H.at(h, h), H.at(l, l));
    cplx mu = shift_of(pick2(top, H.at(h - 1, h - 1), H.at(l - 1, l - 1)),
                       pick2(top, last(h - 1), H.at(l - 1, l)), c, d);
    if (it == 10 || it == 20)
      mu = mk(d.re + __builtin_fma(0.75, fabs(c), fabs(top || l < 2 ? H.r[h - 1][h - 2]
                                                                    : H.r[l - 1][l - 2])), d.im);
    ++it;
    ++sweeps;
    // H - mu I on the window; what lies below it (row and column h of a window
    // that ends at h - 1) is no longer read, and takes part in any way
#pragma unroll
    for (int i = 0; i <= h; ++i) H.put(i, i, sub(H.at(i, i), mu));
    // R = G_{h-1} ... G_0 (H - mu I), then R G_0^H ... G_{h-1}^H, with each
    // right rotation applied once the next left one is: the left rotation k
    // reads H(k, k) before the right rotation k - 1 changes it. A left rotation
    // maps its own column's pair (x, y) to (r, 0), r real. With y = 0 at the
    // window's end it takes R's last diagonal entry to its modulus, which
    // keeps the subdiagonal real.
    cplx cp = mk(1.0, 0.0), run = last(0);  // run: H(k, h)
    double sp = 0.0;
#pragma unroll
    for (int k = 0; k < h; ++k) {
      const cplx x = H.at(k, k);
      const double y = k < h - 1 || top ? H.r[k + 1][k] : 0.0;
      const double n2 = __builtin_fma(y, y, norm2(x));
      const bool on = n2 > 0.0;
      const double ir = on ? rsqrt_f64(n2) : 0.0;
      const cplx cc = mk(on ? x.re * ir : 1.0, x.im * ir);  // conj(c)
      const double s = y * ir;
      H.put(k, k, mk(n2 * ir, 0.0));
#pragma unroll
      for (int j = k + 1; j < h; ++j) {
        const cplx a = H.at(k, j), b = H.at(k + 1, j);
        H.put(k, j, rot1(cc, s, a, b));
        H.put(k + 1, j, rot2(cc, s, a, b));
      }
      const cplx b = k + 1 < h ? last(k + 1) : H.at(h, h);
      set_last(k, rot1(cc, s, run, b));
      run = rot2(cc, s, run, b);
      if (k > 0) right_rot(H, k - 1, cp, sp);
      cp = conjc(cc);
      sp = s;
    }
    cplx e;
    const double r = polar(run, e);
#pragma unroll
    for (int i = 0; i < h; ++i) {
      const cplx a = H.at(i, h - 1), b = last(i);
      H.put(i, h - 1, rot1(cp, sp, a, b));
      set_last(i, cmul(e, rot2(cp, sp, a, b)));
    }
    H.put(h, h - 1, mk(sp * r, 0.0));
    H.put(h, h, cmul(e, scal(r, cp)));
#pragma unroll
    for (int i = 0; i <= h; ++i) H.put(i, i, add(H.at(i, i), mu));
  }
}

template <int h>
__device__ __forceinline__ void qr_levels(RegMat &H, int &hi, int &it, int &sweeps, double2 *ev,
                                          int stride, double2 *col) {
  qr_level<h>(H, hi, it, sweeps, ev, stride, col);
  if constexpr (h > 2) qr_levels<h - 1>(H, hi, it, sweeps, ev, stride, col);
}

// Eigenvalues of the upper Hessenberg H. Returns false if the lane did not
// converge within VN_MAX_SWEEPS sweeps.
__device__ __forceinline__ bool qr_reg(RegMat &H, double2 *ev, int stride, double2 *col) {
  int hi = N - 1, it = 0, sweeps = 0;
  qr_levels<N - 1>(H, hi, it, sweeps, ev, stride, col);
  if (hi == 1) {
    const cplx a = H.at(0, 0), b = H.at(0, 1), c = H.at(1, 0), d = H.at(1, 1);
    cplx l0 = a, l1 = d;
    if (abs1(c) > 2.220446049250313e-16 * (abs1(a) + abs1(d))) eig2(a, b, c, d, l0, l1);
    ev[0] = make_double2(l0.re, l0.im);
    ev[stride] = make_double2(l1.re, l1.im);
  } else if (hi == 0) {
    ev[0] = make_double2(H.r[0][0], H.m[0][0]);
  }
  return hi >= 0;
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
