// Semi-Lagrangian transports of the state, adjoint, incremental state and incremental
// adjoint, the departure-point setup and the body-force accumulation.
//
// Discretisation (paper Section 2.2 equations StateEquation and FirstOrder1-4, the
// commented incremental system of Section 2.2, Section 3.2 with iota(v~)):
//   u = dt * N_ref * v                      velocity in voxels per step
//   X = -(u + Interp(u, i - u)) / 2         forward characteristic (Heun)
//   Y = +(u + Interp(u, i + u)) / 2         backward characteristic (Heun)
//   a = 1 + dt/2 [R + (1 + dt R) r],  R = Interp(r, i + Y),  r = div v
//   m^{n+1} = Interp(m^n, i + X)
//   lambda^n = a Interp(lambda^{n+1}, i + Y),  b = sum_n w_n lambda^n grad m^n
//   t^0 = dt/2 f^0, t^{n+1} = Interp(t^n, i + X) + dt f^{n+1},
//   dm^Nt = Interp(t^{Nt-1}, i + X) + dt/2 f^Nt,  f^n = -grad m^n . dv
// with periodic d-linear interpolation, central differences grad f = (f(i+e) - f(i-e)) N_ref/2
// and trapezoid weights w_n in time.
//
// Layout: grid fields are float32 planes with x fastest; vector fields are dim consecutive
// planes.  The backward offsets and the reaction factor are packed into one 16-byte voxel,
// YA = (Y, a), which costs no extra bytes and saves three loads.  The kernels stream at the
// HBM rate, so they read every field once per voxel (12 + 4 + ... bytes) and nothing more;
// the two x-neighbours of every interpolation row come in one 8-byte load.
#include "bl_field.h"

namespace bl {
namespace {

// ---------------------------------------------------------------------------------- setup
template <int DIM, int ZV>
__global__ __launch_bounds__(kTB) void k_setup(Geo g, const float* __restrict__ v,
                                               float* __restrict__ X,
                                               float4* __restrict__ YA) {
  BL_BATCH_Z1(g.bat)
  BL_AT_NN(v, g.bat);
  BL_AT_NN(X, g.bat);
  BL_AT_NN(YA, g.bat);
  COLUMN
  setup_voxels<DIM, ZV>(g, t, v, X, YA);
}

// every step n of a non-stationary velocity's time grid in one launch: n = blockIdx.y, the
// velocities V[n] and V[n + 1] (dim + 1 planes per node), X[n], YA[n]
template <int DIM>
__global__ __launch_bounds__(kTB) void k_setup_ns(Geo g, const float* __restrict__ V,
                                                  float* __restrict__ Xall,
                                                  float4* __restrict__ YAall) {
  BL_BATCH_Z1(g.bat)
  BL_AT_NN(V, g.bat);
  BL_AT_NN(Xall, g.bat);
  BL_AT_NN(YAall, g.bat);
  constexpr int ZV = 1;
  COLUMN
  const size_t M = (size_t)g.M, n = blockIdx.y;
  setup_voxel_ns<DIM>(g, t, V + n * (DIM + 1) * M, Xall + n * DIM * M, YAall + n * M);
}

// ----------------------------------------------------------------------------- transports
template <int DIM, int ZV>
__global__ __launch_bounds__(kTB) void k_state_step(Geo g, const float* __restrict__ m_in,
                                                    const float* __restrict__ X,
                                                    float* __restrict__ m_out) {
  BL_BATCH_Z1(g.bat)
  BL_AT_NN(m_in, g.bat);
  BL_AT_NN(X, g.bat);
  BL_AT_NN(m_out, g.bat);
  COLUMN
  Tap tp[ZV];
  taps_x<DIM, ZV>(g, t, X, tp);
  float val[ZV];
  gather_zv<DIM, ZV>(g, field_rsrc(m_in, g), tp, val);
  store_zv<ZV>(g, t, m_out, val);
}

template <int DIM, int ZV>
__global__ __launch_bounds__(kTB) void k_adj_step(Geo g, const float* __restrict__ lam_in,
                                                  const float4* __restrict__ YA,
                                                  float* __restrict__ lam_out) {
  BL_BATCH_Z1(g.bat)
  BL_AT_NN(lam_in, g.bat);
  BL_AT_NN(YA, g.bat);
  BL_AT_NN(lam_out, g.bat);
  COLUMN
  Tap tp[ZV];
  float aw[ZV], val[ZV];
  taps_ya<DIM, ZV>(g, t, YA, tp, aw);
  gather_zv<DIM, ZV>(g, field_rsrc(lam_in, g), tp, val);
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) val[zz] = aw[zz] * val[zz];
  store_zv<ZV>(g, t, lam_out, val);
}

template <int DIM>
__global__ __launch_bounds__(kTB) void k_terminal(Geo g, const float* __restrict__ mT,
                                                  const float* __restrict__ I1,
                                                  float* __restrict__ lam) {
  BL_BATCH_Z1(g.bat)
  BL_AT_NN(mT, g.bat);
  BL_AT_NN(I1, g.bat);
  BL_AT_NN(lam, g.bat);
  constexpr int ZV = 1;
  COLUMN
  VOXEL(0)
  st(field_rsrc(lam, g), t.c, zo,
     g.lam_scale * (ld(field_rsrc(mT, g), t.c, zo) - ld(field_rsrc(I1, g), t.c, zo)));
}

// ---------------------------------------------------------------- stencil + gather kernels
template <int DIM, int ZV>
__global__ __launch_bounds__(kTB) void k_inc_init(Geo g, const float* __restrict__ m0,
                                                  const float* __restrict__ dv,
                                                  float* __restrict__ t0) {
  BL_BATCH_Z1(g.bat)
  BL_AT_NN(m0, g.bat);
  BL_AT_NN(dv, g.bat);
  BL_AT_NN(t0, g.bat);
  COLUMN
  float val[ZV];
  source_f<DIM, ZV>(g, t, m0, dv, val);
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) val[zz] = 0.5f * g.dt * val[zz];
  store_zv<ZV>(g, t, t0, val);
}

template <int DIM, int ZV>
__global__ __launch_bounds__(kTB) void k_inc_step(Geo g, const float* __restrict__ t_in,
                                                  const float* __restrict__ X,
                                                  const float* __restrict__ m_next,
                                                  const float* __restrict__ dv,
                                                  float* __restrict__ t_out) {
  BL_BATCH_Z1(g.bat)
  BL_AT_NN(t_in, g.bat);
  BL_AT_NN(X, g.bat);
  BL_AT_NN(m_next, g.bat);
  BL_AT_NN(dv, g.bat);
  BL_AT_NN(t_out, g.bat);
  COLUMN
  Tap tp[ZV];
  float src[ZV], val[ZV];
  taps_x<DIM, ZV>(g, t, X, tp);
  source_f<DIM, ZV>(g, t, m_next, dv, src);
  gather_zv<DIM, ZV>(g, field_rsrc(t_in, g), tp, val);
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) val[zz] = fmaf(g.dt, src[zz], val[zz]);
  store_zv<ZV>(g, t, t_out, val);
}

template <int DIM, int ZV>
__global__ __launch_bounds__(kTB) void k_inc_last(Geo g, const float* __restrict__ t_in,
                                                  const float* __restrict__ X,
                                                  const float* __restrict__ mT,
                                                  const float* __restrict__ dv,
                                                  float* __restrict__ dlam) {
  BL_BATCH_Z1(g.bat)
  BL_AT_NN(t_in, g.bat);
  BL_AT_NN(X, g.bat);
  BL_AT_NN(mT, g.bat);
  BL_AT_NN(dv, g.bat);
  BL_AT_NN(dlam, g.bat);
  COLUMN
  Tap tp[ZV];
  float src[ZV], val[ZV];
  taps_x<DIM, ZV>(g, t, X, tp);
  source_f<DIM, ZV>(g, t, mT, dv, src);
  gather_zv<DIM, ZV>(g, field_rsrc(t_in, g), tp, val);
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) val[zz] = g.lam_scale * fmaf(0.5f * g.dt, src[zz], val[zz]);
  store_zv<ZV>(g, t, dlam, val);
}

// b = sum_n w_n lambda^n grad m^n (body_sum)
template <int DIM, int ZV>
__global__ __launch_bounds__(kTB) void k_body_force(Geo g, const float* __restrict__ lam,
                                                    const float* __restrict__ m,
                                                    float* __restrict__ b,
                                                    const float4* __restrict__ YA) {
  BL_BATCH_Z1(g.bat)
  BL_AT_NN(lam, g.bat);
  BL_AT_NN(m, g.bat);
  BL_AT_NN(b, g.bat);
  BL_AT(YA, g.bat);
  COLUMN
  const size_t M = (size_t)g.M;
  float acc[ZV][3];
  body_sum<DIM, ZV>(g, t, lam, m, YA, acc);
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    VOXEL(zz)
    if (live)
      for (int c = 0; c < DIM; ++c) st(field_rsrc(b + c * M, g), t.c, zo, acc[zz][c]);
  }
}

// ------------------------------------------------------------ full Newton Hessian product
// The Newton product keeps the adjoint terms the Gauss-Newton one drops: the source
// s^n = div(lambda^n dv) of the incremental adjoint and lambda^n grad dm^n in the body force.
// The incremental state steps also store dm^n; the incremental adjoint runs on
//   q^Nt = -(2/sigma^2) dm^Nt,  dlambda^Nt = u^Nt = q^Nt + dt/2 s^Nt,
//   q^n = a Interp(u^{n+1}, i + Y) + dt/2 s^n,  dlambda^n = q^n,  u^n = q^n + dt/2 s^n  (0 < n < Nt),
//   dlambda^0 = a Interp(u^1, i + Y).

// central-difference divergence of lambda dv: sum_j (lam dv_j)(i + e_j) - (i - e_j)
template <int DIM, int ZV>
__device__ __forceinline__ void div_lam_dv(const Geo& g, const Col& t, const float* lam,
                                           const float* dv, float (&out)[ZV]) {
  const Rsrc rl = field_rsrc(lam, g);
  const Vec<DIM> rd = vec_rsrc<DIM>(dv, g);
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    VOXEL(zz)
    float s = ld(rl, t.xp, zo) * ld(rd.c[0], t.xp, zo) - ld(rl, t.xm, zo) * ld(rd.c[0], t.xm, zo);
    s += ld(rl, t.yp, zo) * ld(rd.c[1], t.yp, zo) - ld(rl, t.ym, zo) * ld(rd.c[1], t.ym, zo);
    if constexpr (DIM == 3)
      s += ld(rl, t.c, zp) * ld(rd.c[2], t.c, zp) - ld(rl, t.c, zm) * ld(rd.c[2], t.c, zm);
    out[zz] = s * g.half_nref;
  }
}

// incremental state step that also stores dm^{n+1} = Interp(t^n, i + X) + dt/2 f^{n+1}
template <int DIM, int ZV>
__global__ __launch_bounds__(kTB) void k_inc_step_n(Geo g, const float* __restrict__ t_in,
                                                    const float* __restrict__ X,
                                                    const float* __restrict__ m_next,
                                                    const float* __restrict__ dv,
                                                    float* __restrict__ t_out,
                                                    float* __restrict__ dm_out) {
  BL_BATCH_Z1(g.bat)
  BL_AT_NN(t_in, g.bat);
  BL_AT_NN(X, g.bat);
  BL_AT_NN(m_next, g.bat);
  BL_AT_NN(dv, g.bat);
  BL_AT_NN(t_out, g.bat);
  BL_AT_NN(dm_out, g.bat);
  COLUMN
  Tap tp[ZV];
  float src[ZV], val[ZV], dmv[ZV];
  taps_x<DIM, ZV>(g, t, X, tp);
  source_f<DIM, ZV>(g, t, m_next, dv, src);
  gather_zv<DIM, ZV>(g, field_rsrc(t_in, g), tp, val);
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    dmv[zz] = fmaf(0.5f * g.dt, src[zz], val[zz]);
    val[zz] = fmaf(g.dt, src[zz], val[zz]);
  }
  store_zv<ZV>(g, t, t_out, val);
  store_zv<ZV>(g, t, dm_out, dmv);
}

// last incremental state step: dm^Nt, and dlambda^Nt = u^Nt = -(2/sigma^2) dm^Nt + dt/2 s^Nt
template <int DIM, int ZV>
__global__ __launch_bounds__(kTB) void k_inc_last_n(Geo g, const float* __restrict__ t_in,
                                                    const float* __restrict__ X,
                                                    const float* __restrict__ mT,
                                                    const float* __restrict__ dv,
                                                    const float* __restrict__ lamT,
                                                    float* __restrict__ dm_out,
                                                    float* __restrict__ dlam) {
  BL_BATCH_Z1(g.bat)
  BL_AT_NN(t_in, g.bat);
  BL_AT_NN(X, g.bat);
  BL_AT_NN(mT, g.bat);
  BL_AT_NN(dv, g.bat);
  BL_AT_NN(lamT, g.bat);
  BL_AT_NN(dm_out, g.bat);
  BL_AT_NN(dlam, g.bat);
  COLUMN
  Tap tp[ZV];
  float src[ZV], dmv[ZV], val[ZV];
  taps_x<DIM, ZV>(g, t, X, tp);
  source_f<DIM, ZV>(g, t, mT, dv, src);
  div_lam_dv<DIM, ZV>(g, t, lamT, dv, val);
  gather_zv<DIM, ZV>(g, field_rsrc(t_in, g), tp, dmv);
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    dmv[zz] = fmaf(0.5f * g.dt, src[zz], dmv[zz]);
    val[zz] = fmaf(0.5f * g.dt, val[zz], g.lam_scale * dmv[zz]);
  }
  store_zv<ZV>(g, t, dm_out, dmv);
  store_zv<ZV>(g, t, dlam, val);
}

// one incremental adjoint step of the Newton product: q = a Interp(u^{n+1}, i + Y) (+ dt/2 s^n
// when own); dlambda^n = q; with u_out, u^n = q + dt/2 s^n
template <int DIM, int ZV>
__global__ __launch_bounds__(kTB) void k_adj_step_n(Geo g, const float* __restrict__ u_in,
                                                    const float4* __restrict__ YA,
                                                    const float* __restrict__ lam_n,
                                                    const float* __restrict__ dv, int own,
                                                    float* __restrict__ dlam,
                                                    float* __restrict__ u_out) {
  BL_BATCH_Z1(g.bat)
  BL_AT_NN(u_in, g.bat);
  BL_AT_NN(YA, g.bat);
  BL_AT_NN(lam_n, g.bat);
  BL_AT_NN(dv, g.bat);
  BL_AT_NN(dlam, g.bat);
  BL_AT(u_out, g.bat);
  COLUMN
  Tap tp[ZV];
  float aw[ZV], hs[ZV], qv[ZV], uv[ZV];
  taps_ya<DIM, ZV>(g, t, YA, tp, aw);
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) hs[zz] = 0.f;
  if (own) {
    div_lam_dv<DIM, ZV>(g, t, lam_n, dv, hs);
#pragma unroll
    for (int zz = 0; zz < ZV; ++zz) hs[zz] = 0.5f * g.dt * hs[zz];
  }
  gather_zv<DIM, ZV>(g, field_rsrc(u_in, g), tp, qv);
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    qv[zz] = aw[zz] * qv[zz] + hs[zz];
    uv[zz] = qv[zz] + hs[zz];
  }
  store_zv<ZV>(g, t, dlam, qv);
  if (u_out) store_zv<ZV>(g, t, u_out, uv);
}

// Newton body force: sum_n w_n (dlambda^n grad m^n + lambda^n grad dm^n); the node loop is
// outside the thread's z run and the z differences of m^n and dm^n come from sliding windows,
// as in k_body_force
template <int DIM, int ZV>
__global__ __launch_bounds__(kTB) void k_body_force_n(Geo g, const float* __restrict__ dlam,
                                                      const float* __restrict__ m,
                                                      const float* __restrict__ lam,
                                                      const float* __restrict__ dm,
                                                      float* __restrict__ b) {
  BL_BATCH_Z1(g.bat)
  BL_AT_NN(dlam, g.bat);
  BL_AT_NN(m, g.bat);
  BL_AT_NN(lam, g.bat);
  BL_AT_NN(dm, g.bat);
  BL_AT_NN(b, g.bat);
  COLUMN
  const size_t M = (size_t)g.M;
  float acc[ZV][3];
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) acc[zz][0] = acc[zz][1] = acc[zz][2] = 0.f;
  for (int n = 0; n <= g.nt; ++n) {
    const float w = (n == 0 || n == g.nt) ? 0.5f * g.dt : g.dt;
    const Rsrc rm = field_rsrc(m + n * M, g), rd = field_rsrc(dm + n * M, g);
    const Rsrc rq = field_rsrc(dlam + n * M, g), rl = field_rsrc(lam + n * M, g);
    float mprev = 0.f, mcur = 0.f, dprev = 0.f, dcur = 0.f;
    if (DIM == 3) {
      VOXEL(0)
      mprev = ld(rm, t.c, zm);
      mcur = ld(rm, t.c, zo);
      dprev = ld(rd, t.c, zm);
      dcur = ld(rd, t.c, zo);
    }
#pragma unroll
    for (int zz = 0; zz < ZV; ++zz) {
      VOXEL(zz)
      float gr[3], gd[3];
      gr[0] = (ld(rm, t.xp, zo) - ld(rm, t.xm, zo)) * g.half_nref;
      gr[1] = (ld(rm, t.yp, zo) - ld(rm, t.ym, zo)) * g.half_nref;
      gd[0] = (ld(rd, t.xp, zo) - ld(rd, t.xm, zo)) * g.half_nref;
      gd[1] = (ld(rd, t.yp, zo) - ld(rd, t.ym, zo)) * g.half_nref;
      gr[2] = gd[2] = 0.f;
      if (DIM == 3) {
        const float mnext = ld(rm, t.c, zp), dnext = ld(rd, t.c, zp);
        gr[2] = (mnext - mprev) * g.half_nref;
        gd[2] = (dnext - dprev) * g.half_nref;
        mprev = mcur;
        mcur = mnext;
        dprev = dcur;
        dcur = dnext;
      }
      const float wl = w * ld(rq, t.c, zo);
      const float wa = w * ld(rl, t.c, zo);
#pragma unroll
      for (int c = 0; c < DIM; ++c) acc[zz][c] = fmaf(wa, gd[c], fmaf(wl, gr[c], acc[zz][c]));
    }
  }
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    VOXEL(zz)
    if (live)
      for (int c = 0; c < DIM; ++c) st(field_rsrc(b + c * M, g), t.c, zo, acc[zz][c]);
  }
}

// b^n = lambda^n grad m^n at the time node n = blockIdx.y (a non-stationary gradient or
// product has one body force per node, not a time integral); all nodes in one launch
template <int DIM, int ZV>
__global__ __launch_bounds__(kTB) void k_body_node(Geo g, const float* __restrict__ lam,
                                                   const float* __restrict__ m,
                                                   float* __restrict__ b,
                                                   const float4* __restrict__ YA0) {
  BL_BATCH_Z1(g.bat)
  BL_AT_NN(lam, g.bat);
  BL_AT_NN(m, g.bat);
  BL_AT_NN(b, g.bat);
  BL_AT(YA0, g.bat);
  COLUMN
  const size_t M = (size_t)g.M;
  // with YA0 (the first step's (Y, a)), the blocks of node 0 form lambda^0 = a Interp(lambda^1,
  // i + Y) as the adjoint step would, with the same arithmetic, instead of reading it
  float l[ZV];
  if (YA0 != nullptr && blockIdx.y == 0) {
    Tap tp[ZV];
    float aw[ZV];
    taps_ya<DIM, ZV>(g, t, YA0, tp, aw);
    gather_zv<DIM, ZV>(g, field_rsrc(lam + M, g), tp, l);
#pragma unroll
    for (int zz = 0; zz < ZV; ++zz) l[zz] = aw[zz] * l[zz];
  } else {
    const Rsrc rl = field_rsrc(lam + blockIdx.y * M, g);
#pragma unroll
    for (int zz = 0; zz < ZV; ++zz) {
      VOXEL(zz)
      l[zz] = ld(rl, t.c, zo);
    }
  }
  const Rsrc rm = field_rsrc(m + blockIdx.y * M, g);
  b += blockIdx.y * (size_t)DIM * M;
  float acc[ZV][3];
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    VOXEL(zz)
    float gr[3];
    grad_c<DIM>(g, rm, t, zo, zm, zp, gr);
    for (int c = 0; c < DIM; ++c) acc[zz][c] = l[zz] * gr[c];
  }
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    VOXEL(zz)
    if (live)
      for (int c = 0; c < DIM; ++c) st(field_rsrc(b + c * M, g), t.c, zo, acc[zz][c]);
  }
}

// Deterministic partial sums of (mT - I1)^2: a fixed grid of kRedBlocks blocks, each thread
// a fixed strided subset, then the fixed-order block reduction (wavefront shuffles).
__global__ __launch_bounds__(256) void k_energy_partial(int64_t n, const float* __restrict__ a,
                                                        const float* __restrict__ b,
                                                        double* __restrict__ partial,
                                                        float* __restrict__ lam, float lam_scale,
                                                        Batch bt) {
  BL_BATCH_Z1(bt)
  BL_AT_NN(a, bt);
  BL_AT_NN(b, bt);
  BL_AT_NN(partial, bt);
  BL_AT(lam, bt);
  // the thread's elements i, i + stride, ... in that order; kEU of them per round with all of
  // the round's loads issued before its stores (a loop that loads and stores one element per
  // iteration waits for each iteration's loads)
  constexpr int kEU = 8;
  const int64_t stride = (int64_t)gridDim.x * 256;
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  double acc = 0.0;
  for (; i + (kEU - 1) * stride < n; i += kEU * stride) {
    float av[kEU], bv[kEU];
#pragma unroll
    for (int u = 0; u < kEU; ++u) {
      av[u] = a[i + u * stride];
      bv[u] = b[i + u * stride];
    }
#pragma unroll
    for (int u = 0; u < kEU; ++u) {
      const double d = (double)av[u] - (double)bv[u];
      acc = fma(d, d, acc);
      if (lam) lam[i + u * stride] = lam_scale * (av[u] - bv[u]);   // as k_terminal forms it
    }
  }
  for (; i < n; i += stride) {
    const float ai = a[i], bi = b[i];
    const double d = (double)ai - (double)bi;
    acc = fma(d, d, acc);
    if (lam) lam[i] = lam_scale * (ai - bi);
  }
  const double r = block_reduce_256<false>(acc);
  if (threadIdx.x == 0) partial[blockIdx.x] = r;
}

// One component of packed float4 data into a plane.
__global__ __launch_bounds__(256) void k_unpack4(int64_t n, int comp,
                                                 const float4* __restrict__ src,
                                                 float* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float4 v = src[i];
  dst[i] = comp == 0 ? v.x : comp == 1 ? v.y : comp == 2 ? v.z : v.w;
}

inline dim3 gather_grid(const Geo& g, int zv) {
  const long long nb = (long long)g.nqb * ((g.nz + zv - 1) / zv);
  return dim3((unsigned)((nb + kXCD - 1) / kXCD * kXCD));
}
}  // namespace

// 3D launches take the class's voxels per thread along z (1, 2, 4 or 8); 2D runs one per thread.
// NY > 1 repeats the grid over blockIdx.y (one copy per time node).
#define GRID_N(ZV_, NY) batch_grid(dim3(gather_grid(g, ZV_).x, (NY)), g.bat)
#define DISPATCH_GATHER_N(KERNEL, CLS, NY, ...)                                                 \
  do {                                                                                          \
    if (g.dim == 3) {                                                                           \
      const int zv_ = g.zv[CLS];                                                                \
      if (zv_ == 8)                                                                             \
        BL_LAUNCH((KERNEL<3, 8>), GRID_N(8, NY), dim3(kTB), 0, s, __VA_ARGS__);    \
      else if (zv_ == 4)                                                                        \
        BL_LAUNCH((KERNEL<3, 4>), GRID_N(4, NY), dim3(kTB), 0, s, __VA_ARGS__);    \
      else if (zv_ == 2)                                                                        \
        BL_LAUNCH((KERNEL<3, 2>), GRID_N(2, NY), dim3(kTB), 0, s, __VA_ARGS__);    \
      else                                                                                      \
        BL_LAUNCH((KERNEL<3, 1>), GRID_N(1, NY), dim3(kTB), 0, s, __VA_ARGS__);    \
    } else {                                                                                    \
      BL_LAUNCH((KERNEL<2, 1>), GRID_N(1, NY), dim3(kTB), 0, s, __VA_ARGS__);     \
    }                                                                                           \
  } while (0)
#define DISPATCH_GATHER(KERNEL, CLS, ...) DISPATCH_GATHER_N(KERNEL, CLS, 1, __VA_ARGS__)
#define DISPATCH_ONE(KERNEL, ...)                                                          \
  do {                                                                                     \
    if (g.dim == 3)                                                                        \
      hipLaunchKernelGGL(KERNEL<3>, batch_grid(gather_grid(g, 1), g.bat), dim3(kTB), 0, s, \
                         __VA_ARGS__);                                                     \
    else                                                                                   \
      hipLaunchKernelGGL(KERNEL<2>, batch_grid(gather_grid(g, 1), g.bat), dim3(kTB), 0, s, \
                         __VA_ARGS__);                                                     \
  } while (0)
void setup(const Geo& g, const float* v, float* X, float4* YA, hipStream_t s) {
  if (g.dim == 3 && g.zv[TR_SETUP] >= 4) return setup_box(g, v, X, YA, s);
  if (g.dim == 3 && g.zv[TR_SETUP] == 2)
    BL_LAUNCH((k_setup<3, 2>), GRID_N(2, 1), dim3(kTB), 0, s, g, v, X, YA);
  else if (g.dim == 3)
    BL_LAUNCH((k_setup<3, 1>), GRID_N(1, 1), dim3(kTB), 0, s, g, v, X, YA);
  else
    BL_LAUNCH((k_setup<2, 1>), GRID_N(1, 1), dim3(kTB), 0, s, g, v, X, YA);
}
void setup_ns(const Geo& g, const float* V, float* X, float4* YA, int steps, hipStream_t s) {
  const dim3 grid = batch_grid(dim3(gather_grid(g, 1).x, (unsigned)steps), g.bat);
  if (g.dim == 3 && g.zv[TR_SETUP] >= 4)
    setup_box_ns(g, V, X, YA, steps, s);
  else if (g.dim == 3)
    hipLaunchKernelGGL(k_setup_ns<3>, grid, dim3(kTB), 0, s, g, V, X, YA);
  else
    hipLaunchKernelGGL(k_setup_ns<2>, grid, dim3(kTB), 0, s, g, V, X, YA);
}
void body_nodes(const Geo& g, const float* lam, const float* m, float* b, int nodes,
                hipStream_t s, const float4* YA0) {
  DISPATCH_GATHER_N(k_body_node, TR_FORCE, nodes, g, lam, m, b, YA0);
}
void state_step(const Geo& g, const float* m_in, const float* X, float* m_out, hipStream_t s) {
  DISPATCH_GATHER(k_state_step, TR_STATE, g, m_in, X, m_out);
}
void terminal(const Geo& g, const float* mT, const float* I1, float* lam, hipStream_t s) {
  DISPATCH_ONE(k_terminal, g, mT, I1, lam);
}
void adj_step(const Geo& g, const float* lam_in, const float4* YA, float* lam_out,
              hipStream_t s) {
  DISPATCH_GATHER(k_adj_step, TR_ADJ, g, lam_in, YA, lam_out);
}
void body_force(const Geo& g, const float* lam, const float* m, float* b, hipStream_t s,
                const float4* YA) {
  DISPATCH_GATHER(k_body_force, TR_FORCE, g, lam, m, b, YA);
}
void inc_init(const Geo& g, const float* m0, const float* dv, float* t0, hipStream_t s) {
  DISPATCH_GATHER(k_inc_init, TR_INC, g, m0, dv, t0);
}
void inc_step(const Geo& g, const float* t_in, const float* X, const float* m_next,
              const float* dv, float* t_out, hipStream_t s) {
  DISPATCH_GATHER(k_inc_step, TR_INC, g, t_in, X, m_next, dv, t_out);
}
void inc_last(const Geo& g, const float* t_in, const float* X, const float* mT,
              const float* dv, float* dlam, hipStream_t s) {
  DISPATCH_GATHER(k_inc_last, TR_INC, g, t_in, X, mT, dv, dlam);
}
void inc_step_n(const Geo& g, const float* t_in, const float* X, const float* m_next,
                const float* dv, float* t_out, float* dm_out, hipStream_t s) {
  DISPATCH_GATHER(k_inc_step_n, TR_INC, g, t_in, X, m_next, dv, t_out, dm_out);
}
void inc_last_n(const Geo& g, const float* t_in, const float* X, const float* mT,
                const float* dv, const float* lamT, float* dm_out, float* dlam, hipStream_t s) {
  DISPATCH_GATHER(k_inc_last_n, TR_INC, g, t_in, X, mT, dv, lamT, dm_out, dlam);
}
void adj_step_n(const Geo& g, const float* u_in, const float4* YA, const float* lam_n,
                const float* dv, int own, float* dlam, float* u_out, hipStream_t s) {
  DISPATCH_GATHER(k_adj_step_n, TR_ADJ, g, u_in, YA, lam_n, dv, own, dlam, u_out);
}
void body_force_n(const Geo& g, const float* dlam, const float* m, const float* lam,
                  const float* dm, float* b, hipStream_t s) {
  DISPATCH_GATHER(k_body_force_n, TR_FORCE, g, dlam, m, lam, dm, b);
}
void energy_partial(const Geo& g, const float* mT, const float* I1, double* partial,
                    hipStream_t s, float* lam) {
  hipLaunchKernelGGL(k_energy_partial, batch_grid(dim3(kRedBlocks), g.bat), dim3(256), 0, s, g.M,
                     mT, I1, partial, lam, g.lam_scale, g.bat);
}
void unpack4(const Geo& g, int comp, const float4* in, float* plane, hipStream_t s) {
  hipLaunchKernelGGL(k_unpack4, dim3((unsigned)((g.M + 255) / 256)), dim3(256), 0, s, g.M, comp,
                     in, plane);
}

}  // namespace bl
