// lbm_tile.h -- the tile kernel of liblbm (Xu & Sagaut, arXiv:1203.6350: up to
// 14 applications of the step of Section 2 per launch on a two-dimensional
// tile held in LDS) and its launcher. Instantiated once per storage type, in
// lbm_tile_f64.hip, lbm_tile_f32.hip and lbm_tile_f16.hip.
//
// For lattices that the strip kernel (lbm_strip.h) cannot fill the device
// with: a strip marches its rows one after the other, and a one-step launch
// of a small lattice is all launch and memory latency (128^2 FP64: 3.6 us a
// step, 512^2 FP32: 9.1 us, both far above their arithmetic). Here a
// workgroup takes R x R cells. Step 1 pulls from the lattice for all of them,
// each further step from the neighbours' results in LDS, on a region that
// shrinks by one cell per side and step, so that after `steps` steps the
// inner T x T cells are left, T = R - 2 (steps - 1), which the last step
// stores. Nothing but the launch order joins the workgroups.
//
// Per step, one step per launch -> tiles (Type II): 128^2 FP64 3.6 -> 1.2 us, 128^2
// FP32 4.5 -> 0.9, 256^2 FP32 4.8 -> 1.1, 512^2 FP32 9.8 -> 2.4 (107 G updates/s),
// 512^2 FP16 7.3 -> 2.7, the 800 x 200 FP64 channel 7.9 -> 3.2. Traced launches of eight
// steps take some 10 us (24^2 FP64 and 32^2 FP32) and 19 (48^2 FP32) where their tiles run
// at once: 5 to 10 us for the first loads, the last stores and a wave's start, and
// 0.4 to 1.1 a step. VALU issue is busy 0.27, 0.63 and 0.82 of the time that waves are on
// the chip: the small regions are bound by latency (first loads, one barrier
// and one LDS round trip a step), the 48^2 one by VALU issue, half of it on the
// shrinking halo. LDS has no bank conflicts.
//
// The same tiles of many small lattices make one launch of a batch (us a step,
// FP32): 2 of 64^2 3.3 -> 1.05, 8 of 256^2 12.7 -> 4.3, 50 of 128^2 14.0 -> 7.7, 36 of
// 200^2 15.1 -> 10.4.
//
// The eight moving populations live in LDS in two copies (step j writes copy
// j mod 2 and reads it after one barrier); the resting one stays in its
// thread's register. Every intermediate result is rounded through the storage
// format, so the result is bit-identical to that many one-step launches, up to the
// sign of zeros (waves clear of the layer run the collision's FREE form).
#pragma once

#include "lbm_device.h"
#include "lbm_internal.h"
#include "lbm_launch.h"

namespace lbm {

// One lattice as a tile launch sees it, in the compute precision.
template <typename S>
struct TileLat {
  typedef typename Store<S>::C C;
  const S *src;
  S *dst;
  int nx, ny;
  int64_t pitch, ps;
  C scale[9], inv_scale[9];
  CollideParams<C> p;
  int variant, chi_mode;
  const C *chi_field, *chix, *chiy;
  const C *qf;   // TILE_QF: [3][qps] reference-state deviations, rows of `pitch`
  C *qf_out;     // with alpha != 0: the running mean after the launch's steps
  int64_t qps;
  C alpha;
};

// TILE_CH: a channel in x. Post-collision deviations of the source column for
// each step of the launch, and whether column nx - 1 copies nx - 2.
template <typename C, bool CH>
struct TileChannel {
  C src[TILE_MAX_STEPS][9];
  int outflow;
};
template <typename C>
struct TileChannel<C, false> {};

// Forms of the kernel: TILE_DEF the collision's default form (conserved rates
// 0, n = m), TILE_QF per-cell reference states, TILE_CH a channel in x.
constexpr int TILE_DEF = 1;
constexpr int TILE_QF = 2;
constexpr int TILE_CH = 4;

// a mod n in [0, n) for -R <= a < n + R; a lattice at least as wide as the region
// (the same answer in all lanes) needs no division.
template <int R>
__device__ __forceinline__ int wrap_mod(int a, int n) {
  if (n < R) a %= n;
  return a < 0 ? a + n : (a >= n ? a - n : a);
}

// A workgroup's region of R x R cells on NT threads of N cells each.
template <int R_, int NT_>
struct TileGeom {
  static constexpr int R = R_, NT = NT_;
  static constexpr int PLANE = R * R, N = (PLANE + NT - 1) / NT;
  static constexpr int PAD = 8;  // a channel's last column reads up to two cells before row 0
};

template <typename S, typename G, int FORM, int VAR>
__device__ __forceinline__ void tile_run(const TileLat<S> &L, int X0, int Y0, int steps, int inset,
                                         typename Store<S>::C *lds,
                                         const TileChannel<typename Store<S>::C, (FORM & TILE_CH) != 0> *ch) {
  typedef typename Store<S>::C C;
  constexpr bool DEF = (FORM & TILE_DEF) != 0, QF = (FORM & TILE_QF) != 0,
                 CH = (FORM & TILE_CH) != 0;
  constexpr int R = G::R, N = G::N;
  // halo: the outputs are the cells H .. R-H-1; a launch of fewer steps than its
  // tiles were cut for leaves a frame of `inset` cells out
  const int in0 = inset + (CH ? 1 : 0), H = steps - 1 + in0;
  constexpr int BUF = 8 * G::PLANE;
  int lx[N], ly[N];
  C g0[N], chi[N], q[N][QF ? 3 : 1];
  bool over[N];  // CH: the source column
  int back[N];   // CH: 1 where column nx - 1 takes the update of nx - 2
  bool give[N];  // CH: column nx - 2, whose resting population column nx - 1 reads too
  bool any_chi = false;
  C mref[9];
  if (!QF && (VAR == V_I || VAR == V_II)) ref_moments(L.p, mref);
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const int id = threadIdx.x + k * G::NT;
    ly[k] = id / R;
    lx[k] = id - ly[k] * R;
    if (G::PLANE % G::NT != 0 && id >= G::PLANE) ly[k] = 4 * R;  // no cell: never needed
    chi[k] = C(0);
    over[k] = false;
    back[k] = 0;
    give[k] = false;
  }
  // Step j runs on the cells within steps - j of the outputs.
#define LBM_TILE_NEED(k, j)                                                        \
  ((unsigned)(lx[k] - ((j) - 1 + in0)) < (unsigned)(R - 2 * ((j) - 1 + in0)) &&    \
   (unsigned)(ly[k] - ((j) - 1 + in0)) < (unsigned)(R - 2 * ((j) - 1 + in0)))
  auto finish = [&](C g[9], int k, int j) {  // collide, then store or hand on
    C c0, c1, c2;
    if constexpr (QF) {
      CollideParams<C> pc = L.p;
      pc.dcf0 = q[k][0];
      pc.dcf1 = q[k][1];
      pc.dcf2 = q[k][2];
      // pre-collision conserved moments, summed as the collision sums them
      c0 = g[0] + ((g[1] + g[3]) + (g[2] + g[4])) + ((g[5] + g[7]) + (g[6] + g[8]));
      c1 = (g[1] - g[3]) + ((g[5] - g[7]) + (g[8] - g[6]));
      c2 = (g[2] - g[4]) + ((g[5] - g[7]) + (g[6] - g[8]));
      C mr[9];
      if (VAR == V_I || VAR == V_II) ref_moments(pc, mr);
      collide<C, VAR, DEF>(g, chi[k], pc, mr);
      if (L.alpha != C(0)) {
        q[k][0] = fmaC(L.alpha, c0 - q[k][0], q[k][0]);
        q[k][1] = fmaC(L.alpha, c1 - q[k][1], q[k][1]);
        q[k][2] = fmaC(L.alpha, c2 - q[k][2], q[k][2]);
      }
    } else if (VAR != V_NONE && !any_chi) {
      collide<C, VAR, DEF, true>(g, C(0), L.p, mref);
    } else {
      collide<C, VAR, DEF>(g, chi[k], L.p, mref);
    }
    if constexpr (CH) {
      if (over[k]) {
#pragma unroll
        for (int i = 0; i < 9; ++i) g[i] = ch->src[j - 1][i];
      }
    }
    if (j < steps) {
#pragma unroll
      for (int i = 0; i < 9; ++i) g[i] = roundtrip<S>(g[i], L.scale[i], L.inv_scale[i]);
      g0[k] = g[0];
      C *w = lds + (j & 1) * BUF + ly[k] * R + lx[k];
#pragma unroll
      for (int i = 1; i < 9; ++i) w[(i - 1) * G::PLANE] = g[i];
      if (CH && give[k]) lds[2 * BUF + (j & 1) * R + ly[k]] = g[0];
    } else {
      const int x = X0 + lx[k] - H, y = Y0 + ly[k] - H;
      if (x < L.nx && y < L.ny) {
        const int64_t cell = (int64_t)y * L.pitch + x;
#pragma unroll
        for (int i = 0; i < 9; ++i) Store<S>::store(L.dst + i * L.ps + cell, g[i], L.inv_scale[i]);
        if constexpr (QF) {
          if (L.alpha != C(0)) {
            L.qf_out[cell] = q[k][0];
            L.qf_out[L.qps + cell] = q[k][1];
            L.qf_out[2 * L.qps + cell] = q[k][2];
          }
        }
      }
    }
  };
  // ---- step 1, pulled from the lattice
  {
    C g[N][9];
#pragma unroll
    for (int k = 0; k < N; ++k) {
      if (LBM_TILE_NEED(k, 1)) {
        const int xo = wrap_mod<R>(X0 + lx[k] - H, L.nx), y = wrap_mod<R>(Y0 + ly[k] - H, L.ny);
        if constexpr (CH) {
          // The source column cuts the lattice in x, so of the periodic images in a
          // region only columns 0 .. nx - 1 and the next source column matter.
          const int gx = X0 + lx[k] - H;
          over[k] = xo == 0;
          back[k] = ch->outflow && gx == L.nx - 1 ? 1 : 0;
          give[k] = ch->outflow && gx == L.nx - 2;
        }
        const int x = xo - back[k];
        const int xm = x == 0 ? L.nx - 1 : x - 1, xp = x == L.nx - 1 ? 0 : x + 1;
        const int ym = y == 0 ? L.ny - 1 : y - 1, yp = y == L.ny - 1 ? 0 : y + 1;
        const int64_t r0 = (int64_t)y * L.pitch, rm = (int64_t)ym * L.pitch,
                      rp = (int64_t)yp * L.pitch;
        const S *s = L.src;
        const int64_t ps = L.ps;
        g[k][0] = Store<S>::load(s + r0 + x, L.scale[0]);
        g[k][1] = Store<S>::load(s + 1 * ps + r0 + xm, L.scale[1]);
        g[k][2] = Store<S>::load(s + 2 * ps + rm + x, L.scale[2]);
        g[k][3] = Store<S>::load(s + 3 * ps + r0 + xp, L.scale[3]);
        g[k][4] = Store<S>::load(s + 4 * ps + rp + x, L.scale[4]);
        g[k][5] = Store<S>::load(s + 5 * ps + rm + xm, L.scale[5]);
        g[k][6] = Store<S>::load(s + 6 * ps + rm + xp, L.scale[6]);
        g[k][7] = Store<S>::load(s + 7 * ps + rp + xp, L.scale[7]);
        g[k][8] = Store<S>::load(s + 8 * ps + rp + xm, L.scale[8]);
        switch (L.chi_mode) {
          case CHI_FIELD: chi[k] = L.chi_field[r0 + x]; break;
          case CHI_SEP_MAX: chi[k] = chi_at<C, CHI_SEP_MAX>(nullptr, L.chix, L.chiy, 0, x, y); break;
          case CHI_SEP_SUM: chi[k] = chi_at<C, CHI_SEP_SUM>(nullptr, L.chix, L.chiy, 0, x, y); break;
          default: break;
        }
        if constexpr (QF) {
          q[k][0] = L.qf[r0 + x];
          q[k][1] = L.qf[L.qps + r0 + x];
          q[k][2] = L.qf[2 * L.qps + r0 + x];
        }
        any_chi |= chi[k] != C(0);
      }
    }
    // one form per wave: a wave clear of the layer skips the damping's products with 0
    any_chi = __builtin_amdgcn_ballot_w64(any_chi) != 0;
#pragma unroll
    for (int k = 0; k < N; ++k)
      if (LBM_TILE_NEED(k, 1)) finish(g[k], k, 1);
  }
  // ---- further steps, pulled from LDS
#pragma unroll 1
  for (int j = 2; j <= steps; ++j) {
    __syncthreads();
    const C *buf = lds + ((j - 1) & 1) * BUF;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      if (LBM_TILE_NEED(k, j)) {
        const C *r = buf + ly[k] * R + lx[k] - back[k];
        C g[9];
        g[0] = g0[k];
        if (CH && back[k]) g[0] = lds[2 * BUF + ((j - 1) & 1) * R + ly[k]];
        g[1] = r[0 * G::PLANE - 1];
        g[2] = r[1 * G::PLANE - R];
        g[3] = r[2 * G::PLANE + 1];
        g[4] = r[3 * G::PLANE + R];
        g[5] = r[4 * G::PLANE - R - 1];
        g[6] = r[5 * G::PLANE - R + 1];
        g[7] = r[6 * G::PLANE + R + 1];
        g[8] = r[7 * G::PLANE + R - 1];
        finish(g, k, j);
      }
    }
  }
#undef LBM_TILE_NEED
}

template <typename S, typename G, int FORM>
__device__ __forceinline__ void tile_variant(const TileLat<S> &L, int X0, int Y0, int steps, int inset,
                                             typename Store<S>::C *lds,
                                             const TileChannel<typename Store<S>::C, (FORM & TILE_CH) != 0> *ch) {
  switch (L.variant) {
    case V_I: tile_run<S, G, FORM, V_I>(L, X0, Y0, steps, inset, lds, ch); break;
    case V_II: tile_run<S, G, FORM, V_II>(L, X0, Y0, steps, inset, lds, ch); break;
    case V_III: tile_run<S, G, FORM, V_III>(L, X0, Y0, steps, inset, lds, ch); break;
    case V_VISC: tile_run<S, G, FORM, V_VISC>(L, X0, Y0, steps, inset, lds, ch); break;
    default: tile_run<S, G, FORM, V_NONE>(L, X0, Y0, steps, inset, lds, ch); break;
  }
}

template <typename G, int FORM>
constexpr int tile_lds_elems() {
  return G::PAD + 2 * 8 * G::PLANE + ((FORM & TILE_CH) ? 2 * G::R : 0);
}

template <typename S, typename G, int FORM>
__global__ __launch_bounds__(G::NT) void tile_kernel(
    TileLat<S> L, TileChannel<typename Store<S>::C, (FORM & TILE_CH) != 0> ch, int steps, int ntx, int per_xcd,
    int nwg) {
  typedef typename Store<S>::C C;
  __shared__ C lds[tile_lds_elems<G, FORM>()];
  // workgroup i runs on XCD i % 8: each XCD gets a contiguous band of tiles
  const int v = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (v >= nwg) return;
  const int ty = v / ntx, tx = v - ty * ntx;
  const int T = G::R - 2 * (steps - 1 + ((FORM & TILE_CH) ? 1 : 0));
  int X0 = tx * T;
  // a channel's last column takes the update of the one before it, two cells
  // from its inputs: a last tile of that column alone starts one cell earlier
  // (column nx - 2 is then stored twice, with the same values)
  if ((FORM & TILE_CH) && X0 > L.nx - 2) X0 = L.nx - 2;
  tile_variant<S, G, FORM>(L, X0, ty * T, steps, 0, lds + G::PAD, &ch);
}

template <typename S>
static TileLat<S> make_tile_lat(const StepConfig &c, const void *src, void *dst) {
  typedef typename Store<S>::C C;
  const Lat<S> B = make_lat<S>(c);
  TileLat<S> L;
  L.src = (const S *)src;
  L.dst = (S *)dst;
  L.nx = B.nx;
  L.ny = B.ny;
  L.pitch = B.pitch;
  L.ps = B.ps;
  for (int i = 0; i < 9; ++i) {
    L.scale[i] = B.scale[i];
    L.inv_scale[i] = B.inv_scale[i];
  }
  L.p = make_params<C>(c);
  L.variant = c.variant;
  L.chi_mode = c.chi_mode;
  L.chi_field = (const C *)c.chi_field;
  L.chix = (const C *)c.chi_x;
  L.chiy = (const C *)c.chi_y;
  L.qf = (const C *)c.qfield;
  L.qf_out = (C *)c.qfield_out;
  L.qps = c.qps;
  L.alpha = C(c.qalpha);
  return L;
}

template <typename S, typename G, int FORM>
static hipError_t launch_tile_g(const StepConfig &c, int steps, const double *source,
                                const void *src, void *dst, hipStream_t stream) {
  typedef typename Store<S>::C C;
  // (a channel's last column depends on two cells to its left per step)
  const int T = G::R - 2 * (steps - 1 + ((FORM & TILE_CH) ? 1 : 0));
  if (steps < 1 || steps > TILE_MAX_STEPS || T < 1) return hipErrorInvalidValue;
  TileChannel<C, (FORM & TILE_CH) != 0> ch;
  if constexpr ((FORM & TILE_CH) != 0) {
    ch.outflow = c.outflow;
    for (int j = 0; j < TILE_MAX_STEPS; ++j)
      for (int i = 0; i < 9; ++i) ch.src[j][i] = j < steps ? C(source[9 * j + i]) : C(0);
  }
  const int ntx = (c.nx + T - 1) / T, nty = (c.ny + T - 1) / T;
  const int64_t nwg = (int64_t)ntx * nty, per = (nwg + 7) / 8;
  if (8 * per > 0x7fffffff) return hipErrorInvalidValue;
  tile_kernel<S, G, FORM><<<dim3((unsigned)(8 * per)), dim3(G::NT), 0, stream>>>(
      make_tile_lat<S>(c, src, dst), ch, steps, ntx, (int)per, (int)nwg);
  return hipGetLastError();
}

template <typename S, typename G>
static hipError_t launch_tile_form(const StepConfig &c, int steps, const double *source,
                                   const void *src, void *dst, hipStream_t stream) {
  typedef typename Store<S>::C C;
  const bool def = C(c.s[0]) == C(0) && C(c.s[1]) == C(0) && C(c.s[2]) == C(0) &&
                   C(c.n) == C(c.m);
  // a fixed reference field is read by the damped variants only
  const bool qf = c.qfield && (c.qalpha != 0.0 || (c.variant >= V_I && c.variant <= V_III));
  if (c.channel)
    return def ? launch_tile_g<S, G, TILE_CH | TILE_DEF>(c, steps, source, src, dst, stream)
               : launch_tile_g<S, G, TILE_CH>(c, steps, source, src, dst, stream);
  if (qf)
    return def ? launch_tile_g<S, G, TILE_QF | TILE_DEF>(c, steps, nullptr, src, dst, stream)
               : launch_tile_g<S, G, TILE_QF>(c, steps, nullptr, src, dst, stream);
  return def ? launch_tile_g<S, G, TILE_DEF>(c, steps, nullptr, src, dst, stream)
             : launch_tile_g<S, G, 0>(c, steps, nullptr, src, dst, stream);
}

template <typename S>
static hipError_t launch_tile_storage(const StepConfig &c, int region, int steps,
                                      const double *source, const void *src, void *dst,
                                      hipStream_t stream) {
  if (c.qfield && c.qalpha != 0.0 && !c.qfield_out) return hipErrorInvalidValue;
  switch (region) {
    case 24: return launch_tile_form<S, TileGeom<24, 576>>(c, steps, source, src, dst, stream);
    case 32: return launch_tile_form<S, TileGeom<32, 1024>>(c, steps, source, src, dst, stream);
    // (two copies of these regions' populations fit the 160 KB of LDS in FP32 only)
    case 40:
      if constexpr (sizeof(typename Store<S>::C) == 4)
        return launch_tile_form<S, TileGeom<40, 832>>(c, steps, source, src, dst, stream);
      break;
    case 48:
      if constexpr (sizeof(typename Store<S>::C) == 4)
        return launch_tile_form<S, TileGeom<48, 768>>(c, steps, source, src, dst, stream);
      break;
  }
  return hipErrorInvalidValue;
}

// Tiles of many lattices in one launch (launch j of a tick): the table lists
// (member, first column, first row) of the outputs, cut for `most` steps. Each
// member takes its steps of the tick evenly over batch_tile_launches of them.
// The descriptors' numbers become the same scalar operands as kernel arguments.
template <typename C>
__device__ __forceinline__ C uniform(double v) {
  if constexpr (sizeof(C) == 4)
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, (float)v)));
  else
    return v;
}

template <typename S, typename G>
__global__ __launch_bounds__(G::NT) void batch_tile_kernel(
    const BatchDomain *__restrict__ doms, const int4 *__restrict__ tiles,
    const int *__restrict__ ntiles, int j, int most) {
  typedef typename Store<S>::C C;
  __shared__ C lds[tile_lds_elems<G, TILE_DEF>()];
  const int nt = *ntiles, per_xcd = (nt + 7) / 8;
  const int v = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per_xcd || v >= nt) return;
  const int4 t = tiles[v];
  const BatchDomain &d = doms[t.x];
  const int stop = d.stop_at, launches = batch_tile_launches(stop, most);
  if (j >= launches) return;
  const int steps = stop * (j + 1) / launches - stop * j / launches;
  const int par = (d.parity + j) & 1;
  TileLat<S> L;
  L.src = (const S *)d.lat[par];
  L.dst = (S *)d.lat[par ^ 1];
  L.nx = d.nx;
  L.ny = d.ny;
  L.pitch = d.pitch;
  L.ps = d.ps;
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    L.scale[i] = uniform<C>(d.scale[i]);
    L.inv_scale[i] = uniform<C>(d.inv_scale[i]);
    L.p.s[i] = uniform<C>(d.s[i]);
  }
  L.p.n = uniform<C>(d.n);
  L.p.m = uniform<C>(d.m);
  L.p.rho_b = uniform<C>(d.rho_b);
  L.p.ubx = uniform<C>(d.ubx);
  L.p.uby = uniform<C>(d.uby);
  L.p.dcf0 = uniform<C>(d.dcf[0]);
  L.p.dcf1 = uniform<C>(d.dcf[1]);
  L.p.dcf2 = uniform<C>(d.dcf[2]);
  set_relax_coeffs(L.p);
  if constexpr (sizeof(C) == 4)
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      L.p.sig[i] = uniform<C>(L.p.sig[i]);
      L.p.tau[i] = uniform<C>(L.p.tau[i]);
    }
  L.variant = d.variant;
  L.chi_mode = d.chi_mode;
  L.chi_field = (const C *)d.chi_field;
  L.chix = (const C *)d.chi_x;
  L.chiy = (const C *)d.chi_y;
  L.qf = nullptr;
  L.qf_out = nullptr;
  L.qps = 0;
  L.alpha = C(0);
  tile_variant<S, G, TILE_DEF>(L, t.y, t.z, steps, most - steps, lds + G::PAD, nullptr);
}

template <typename S>
static hipError_t launch_batch_tile_storage(int region, int most, const BatchDomain *doms,
                                            const int4 *tiles, const int *ntiles, int grid, int j,
                                            hipStream_t stream) {
  if (most < 1 || most > TILE_MAX_STEPS || region - 2 * (most - 1) < 1 || grid < 1)
    return hipErrorInvalidValue;
#define LBM_BTILE(R, NT)                                                                        \
  batch_tile_kernel<S, TileGeom<R, NT>><<<dim3((unsigned)grid), dim3(NT), 0, stream>>>(          \
      doms, tiles, ntiles, j, most);                                                             \
  return hipGetLastError();
  switch (region) {
    case 24: LBM_BTILE(24, 576)
    case 32: LBM_BTILE(32, 1024)
    case 40:
      if constexpr (sizeof(typename Store<S>::C) == 4) { LBM_BTILE(40, 832) }
      break;
    case 48:
      if constexpr (sizeof(typename Store<S>::C) == 4) { LBM_BTILE(48, 768) }
      break;
  }
#undef LBM_BTILE
  return hipErrorInvalidValue;
}

}  // namespace lbm
