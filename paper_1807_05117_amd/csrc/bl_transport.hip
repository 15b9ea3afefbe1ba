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
                                                    const float4* __restrict__ YA, BodyStart b0) {
  BL_BATCH_Z1(g.bat)
  BL_AT_NN(lam, g.bat);
  BL_AT_NN(m, g.bat);
  BL_AT_NN(b, g.bat);
  BL_AT(YA, g.bat);
  COLUMN
  const size_t M = (size_t)g.M;
  float acc[ZV][3];
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    VOXEL(zz)
    for (int c = 0; c < 3; ++c)
      acc[zz][c] = c < DIM && b0.c[c] ? ld(field_rsrc(batch_ptr_nn(b0.c[c], g.bat, bpair_), g), t.c, zo) : 0.f;
  }
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
// One pass over all time nodes (k_newton_terms) forms what does not depend on the adjoint: dt/2 s^n
// and the body force's second term.  The adjoint steps then read one field more than the
// Gauss-Newton ones, and both they and the incremental state run as sweeps where those do
// (bl_sweep.hip).  At 128^3 with ten steps (us): incremental state 86 (184 as steps), terms 95,
// adjoint with the body force 97.  Steps that formed s^n themselves took 182 and a body force of
// both terms 100; as steps it is 148 + 54 now.

// incremental state step that also stores dm^{n+1} = Interp(t^n, i + X) + dt/2 f^{n+1} (t_out
// null: the last step)
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
  BL_AT(t_out, g.bat);
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
  if (t_out) store_zv<ZV>(g, t, t_out, val);
  store_zv<ZV>(g, t, dm_out, dmv);
}

// hs^n = dt/2 s^n for 0 < n < Nt, u^Nt in plane Nt of hs, and b2 = sum_n w_n lambda^n grad dm^n
// (dm^0 = 0); the nodes in turn, dv around the voxels in registers, z neighbours from sliding
// windows as in body_sum
template <int DIM, int ZV>
__global__ __launch_bounds__(kTB) void k_newton_terms(Geo g, const float* __restrict__ lam,
                                                      const float* __restrict__ dm,
                                                      const float* __restrict__ dv,
                                                      float* __restrict__ hs, float* __restrict__ bx,
                                                      float* __restrict__ by, float* __restrict__ bz) {
  BL_BATCH_Z1(g.bat)
  BL_AT_NN(lam, g.bat);
  BL_AT_NN(dm, g.bat);
  BL_AT_NN(dv, g.bat);
  BL_AT_NN(hs, g.bat);
  BL_AT_NN(bx, g.bat);
  BL_AT_NN(by, g.bat);
  BL_AT_NN(bz, g.bat);
  COLUMN
  const size_t M = (size_t)g.M;
  const Vec<DIM> rd = vec_rsrc<DIM>(dv, g);
  float d[ZV][6], acc[ZV][3];
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    VOXEL(zz)
    d[zz][0] = ld(rd.c[0], t.xm, zo);
    d[zz][1] = ld(rd.c[0], t.xp, zo);
    d[zz][2] = ld(rd.c[1], t.ym, zo);
    d[zz][3] = ld(rd.c[1], t.yp, zo);
    d[zz][4] = d[zz][5] = 0.f;
    if constexpr (DIM == 3) {
      d[zz][4] = ld(rd.c[2], t.c, zm);
      d[zz][5] = ld(rd.c[2], t.c, zp);
    }
    acc[zz][0] = acc[zz][1] = acc[zz][2] = 0.f;
  }
  for (int n = g.nt; n >= 1; --n) {
    const float w = n == g.nt ? 0.5f * g.dt : g.dt;
    const Rsrc rl = field_rsrc(lam + n * M, g), rm = field_rsrc(dm + n * M, g);
    const Rsrc out = field_rsrc(hs + n * M, g);
    float lprev = 0.f, lcur = 0.f, prev = 0.f, cur = 0.f;
    {
      VOXEL(0)
      lcur = ld(rl, t.c, zo);
      cur = ld(rm, t.c, zo);
      if (DIM == 3) {
        lprev = ld(rl, t.c, zm);
        prev = ld(rm, t.c, zm);
      }
    }
#pragma unroll
    for (int zz = 0; zz < ZV; ++zz) {
      VOXEL(zz)
      float lnext = 0.f, next = 0.f;
      if (DIM == 3) {
        lnext = ld(rl, t.c, zp);
        next = ld(rm, t.c, zp);
      }
      const float gx = (ld(rm, t.xp, zo) - ld(rm, t.xm, zo)) * g.half_nref;
      const float gy = (ld(rm, t.yp, zo) - ld(rm, t.ym, zo)) * g.half_nref;
      const float wl = w * lcur;
      acc[zz][0] = fmaf(wl, gx, acc[zz][0]);
      acc[zz][1] = fmaf(wl, gy, acc[zz][1]);
      if (DIM == 3) acc[zz][2] = fmaf(wl, (next - prev) * g.half_nref, acc[zz][2]);
      const float s = div_lam_dv<DIM>(ld(rl, t.xm, zo), ld(rl, t.xp, zo), ld(rl, t.ym, zo),
                                      ld(rl, t.yp, zo), lprev, lnext, d[zz]) * g.half_nref;
      const float h = 0.5f * g.dt * s;
      // (2D: one voxel per thread, so cur is its own)
      if (live) st(out, t.c, zo, n == g.nt ? g.lam_scale * cur + h : h);
      lprev = lcur;
      lcur = lnext;
      prev = cur;
      cur = next;
    }
  }
  const Rsrc r0 = field_rsrc(bx, g), r1 = field_rsrc(by, g), r2 = field_rsrc(bz, g);
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    VOXEL(zz)
    if (!live) continue;
    st(r0, t.c, zo, acc[zz][0]);
    st(r1, t.c, zo, acc[zz][1]);
    if (DIM == 3) st(r2, t.c, zo, acc[zz][2]);
  }
}

// one incremental adjoint step of the Newton product: q^n = a Interp(u^{n+1}, i + Y) + hs^n in
// place of hs^n, u^n = q^n + hs^n (u_out null: the last step, without hs)
template <int DIM, int ZV>
__global__ __launch_bounds__(kTB) void k_adj_step_n(Geo g, const float* __restrict__ u_in,
                                                    const float4* __restrict__ YA,
                                                    float* __restrict__ hs, float* __restrict__ u_out) {
  BL_BATCH_Z1(g.bat)
  BL_AT_NN(u_in, g.bat);
  BL_AT_NN(YA, g.bat);
  BL_AT_NN(hs, g.bat);
  BL_AT(u_out, g.bat);
  COLUMN
  Tap tp[ZV];
  float aw[ZV], h[ZV], q[ZV], u[ZV];
  taps_ya<DIM, ZV>(g, t, YA, tp, aw);
  const Rsrc rh = field_rsrc(hs, g);
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    VOXEL(zz)
    h[zz] = u_out ? ld(rh, t.c, zo) : 0.f;
  }
  gather_zv<DIM, ZV>(g, field_rsrc(u_in, g), tp, q);
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    q[zz] = fmaf(aw[zz], q[zz], h[zz]);
    u[zz] = q[zz] + h[zz];
  }
  store_zv<ZV>(g, t, hs, q);
  if (u_out) store_zv<ZV>(g, t, u_out, u);
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
                const float4* YA, BodyStart b0) {
  DISPATCH_GATHER(k_body_force, TR_FORCE, g, lam, m, b, YA, b0);
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
void newton_terms(const Geo& g, const float* lam, const float* dm, const float* dv, float* hs,
                  const BodyStart& b2, hipStream_t s) {
  DISPATCH_GATHER(k_newton_terms, TR_FORCE, g, lam, dm, dv, hs, b2.c[0], b2.c[1], b2.c[2]);
}
void adj_step_n(const Geo& g, const float* u_in, const float4* YA, float* hs, float* u_out,
                hipStream_t s) {
  DISPATCH_GATHER(k_adj_step_n, TR_ADJ, g, u_in, YA, hs, u_out);
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
