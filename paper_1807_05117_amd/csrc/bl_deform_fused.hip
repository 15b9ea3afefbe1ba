// Fused stage kernels of the deformation state equation on the product grid (3D).
//
// One Runge-Kutta stage (or one stage of the transposed sweep) is three launches instead of a
// chain of separate transform, product and band kernels:
//   1. xy:  band (kz >= 0 half) -> F2[c][h][y][x]: the x and y contractions of iota
//           (bl_dft_mfma.hip).  In the derivative form the components are the spectral derivatives
//           d~_j U_i (c = i dim + j) formed on the fly from the state U.
//   2. col: per (y, x) column of the product grid: the z contraction of iota, the pointwise
//           products (and their side outputs), and the z contraction of pi, the column's z
//           values exchanged through LDS; two lanes per column split the kz spectrum.
//   3. yx:  G[c][h][y][x] -> the band: the x and y contractions of pi for 16 ky by 32 kx of one
//           (component, h) plane (the transposed sweep takes its three derivative planes
//           together), followed by the band-side update of the
//           stage (forward) or of the transposed sweep (backward) at kz = h and at the
//           conjugate-mirror index -k.  On the kz = 0 plane the entry k is owned by the half
//           ky > 0 or (ky = 0, kx >= 0); its owner writes k and -k, so the result is exactly
//           Hermitian, and k = 0 takes the real part.
// Twiddle tables are those of the product grid's transform plan (bl_dft.hip layout).
// These kernels are bound by memory latency at ~1.5 waves per SIMD, so every global load a
// phase needs is issued before its first wait: no load sits behind a condition (a guarded load
// compiles to a branch and a wait) and no runtime loop alternates loads and LDS stores.
#include <algorithm>

#include "bl_mfma.h"

namespace bl {
namespace {

constexpr int kColW = 32;     // columns per column-kernel block (two lanes each)
constexpr int kColWaves = 8;  // waves per column-kernel block

__device__ __forceinline__ int wave_uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// q = 2 pi k / l of band index j on axis a (l from the image grid)
__device__ __forceinline__ float qaxis(const Geo& g, int a, int j) {
  const float two_pi = 6.283185307179586f;
  const int kv = a == 0 ? j - g.kx / 2 : (a == 1 ? j - g.ky / 2 : j - g.kz0);
  const int n = a == 0 ? g.nx : (a == 1 ? g.ny : g.nz);
  return two_pi * (float)kv * ((float)g.nref / (float)n);
}

// Staging of tables into LDS with a thread's loads in flight together.  A runtime loop of
// load-then-store waits for one memory round trip per iteration; here a thread first loads R
// entries of a table into registers (entries past the end read the clamped last entry), and
// only then stores them.  Loads of several tables are issued before any of their stores.
template <int NT, int R>
struct Stager {
  float2 v[R];
  template <class Ld>
  __device__ __forceinline__ void load(int n, int base, Ld ld) {
#pragma unroll
    for (int u = 0; u < R; ++u) v[u] = ld(min(base + (int)threadIdx.x + NT * u, n - 1));
  }
  template <class St>
  __device__ __forceinline__ void store(int n, int base, St st) const {
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const int o = base + (int)threadIdx.x + NT * u;
      if (o < n) st(o, v[u]);
    }
  }
};

// ---------------------------------------------------------------------------- 2. columns
// Block (32 columns, component), eight waves: lane l of a wave serves column l mod 32 and the
// half l / 32 of the kz spectrum (h in [half KZH / 2, (half + 1) KZH / 2)), so each lane holds
// half of a column's coefficients and the two halves' partial sums meet in one lane swap.  Wave
// w handles the z planes w, w + 8, ... of the block's columns.  The block's z twiddles
// exp(+2 pi i h z / pz) are staged in LDS (tz[z][h], KZH per row) and read as broadcasts, each
// shared by the three fields a block contracts.

// this lane's half of the column of one field (h < kzh; zero past kzh).  Every load is made,
// at the clamped plane past kzh, and zeroed afterwards: a guarded load compiles to a branch and
// a wait per load, an unguarded one lets all of them be in flight together.
template <int KZH>
__device__ __forceinline__ void load_half(const float2* __restrict__ Fc, size_t hstride, int kzh,
                                          int half, float2* F) {
  constexpr int NHH = KZH / 2;
  float2 v[NHH];
#pragma unroll
  for (int u = 0; u < NHH; ++u) v[u] = Fc[(size_t)min(half * NHH + u, kzh - 1) * hstride];
#pragma unroll
  for (int u = 0; u < NHH; ++u) F[u] = half * NHH + u < kzh ? v[u] : make_float2(0.f, 0.f);
}

// the block's z twiddles tz[z][h] (zero past kzh): pz * KZH <= 48 * 16 entries, two per thread;
// the loads are issued here and the LDS stores made later by tz_store, so that the caller's
// other loads are in flight at the same time
template <int KZH>
struct TzStage {
  Stager<64 * kColWaves, 2> st;
  __device__ __forceinline__ void load(const float2* __restrict__ tw_zT, int pz, int kzh) {
    st.load(pz * KZH, 0, [&](int o) {
      const int z = o / KZH, h = o - z * KZH;
      return tw_zT[(size_t)z * kZP + min(h, kzh - 1)];
    });
  }
  __device__ __forceinline__ void store(int pz, int kzh, float2* tz) const {
    st.store(pz * KZH, 0, [&](int o, float2 v) {
      const int h = o % KZH;
      tz[o] = h < kzh ? v : make_float2(0.f, 0.f);
    });
  }
};

// f_j(z) = Re F_j[0] + 2 sum_{h >= 1} Re(F_j[h] tz[z][h]) for three fields at one plane z: each
// half sums its h range, then the halves exchange partial sums (lane l <-> l ^ 32)
template <int KZH>
__device__ __forceinline__ void iota_z3(const float2 (*F)[KZH / 2], const float2* tz, int z,
                                        int half, float* f) {
  constexpr int NHH = KZH / 2;
#pragma unroll
  for (int j = 0; j < 3; ++j) f[j] = 0.f;
#pragma unroll
  for (int u = 0; u < NHH; ++u) {
    const int h = half * NHH + u;
    const float2 t = tz[z * KZH + h];
    const float sc = h == 0 ? 1.f : 2.f;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      f[j] = fmaf(sc * F[j][u].x, t.x, f[j]);
      f[j] = fmaf(-sc * F[j][u].y, t.y, f[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < 3; ++j) f[j] += __shfl_xor(f[j], 32);
}

// Forward stage, block (column chunk, component i): f_(i,j)(z) = iota_z(F2[i dim + j]);
// out(z) = sum_j f_(i,j)(z) V_j(z) (+ sum_j DUGr_(i,j)(z) DVP_j(z) for products); the state
// pass stores DUGw_(i,j)(z) = f_(i,j)(z); G[i][h] = sum_z out(z) conj tz[z][h], wave w taking
// h = half KZH / 2 + w.
template <int NZS, int KZH, bool INC>
__global__ __launch_bounds__(64 * kColWaves) void k_fx_col_fwd(Geo gp, const float2* __restrict__ F2,
                                                    const float* __restrict__ VP,
                                                    float* __restrict__ DUGw,
                                                    const float* __restrict__ DUGr,
                                                    const float* __restrict__ DVP,
                                                    const float2* __restrict__ tw_zT,
                                                    float2* __restrict__ G) {
  __shared__ float2 tz[kColWaves * NZS * KZH];
  __shared__ float buf[kColWaves * NZS][kColW];
  const int lane = threadIdx.x & 63;
  const int col = lane & (kColW - 1), half = lane >> 5;
  const int w = wave_uniform(threadIdx.x >> 6);
  const int i = blockIdx.y;
  const int nq = gp.nx * gp.ny;
  const int q = blockIdx.x * kColW + col;
  const int qc = q < nq ? q : nq - 1;
  const bool live = q < nq;
  const int pz = gp.nz, kzh = gp.kzh;
  const int64_t MP = gp.M;
  float2 F[3][KZH / 2];
#pragma unroll
  for (int j = 0; j < 3; ++j)
    load_half<KZH>(F2 + (size_t)(3 * i + j) * kzh * nq + qc, (size_t)nq, kzh, half, F[j]);
  TzStage<KZH> tzs;
  tzs.load(tw_zT, pz, kzh);
  // planes past pz are computed at the clamped plane pz - 1 and not stored: no branch keeps the
  // loads of later planes from being issued early.  Every load of the block's inputs is issued
  // before the first LDS store and barrier.
  float vp[3][NZS], dg[3][NZS], dw[3][NZS];
#pragma unroll
  for (int s = 0; s < NZS; ++s) {
    const int64_t at = (int64_t)min(w + kColWaves * s, pz - 1) * nq + qc;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      vp[j][s] = VP[j * MP + at];
      if (INC) {
        dg[j][s] = DUGr[(int64_t)(3 * i + j) * MP + at];
        dw[j][s] = DVP[j * MP + at];
      }
    }
  }
  tzs.store(pz, kzh, tz);
  __syncthreads();
#pragma unroll
  for (int s = 0; s < NZS; ++s) {
    const int z = w + kColWaves * s;
    const int zc = min(z, pz - 1);
    const int64_t at = (int64_t)zc * nq + qc;
    float f[3];
    iota_z3<KZH>(F, tz, zc, half, f);
    float o = 0.f;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      o = fmaf(f[j], vp[j][s], o);
      const int64_t ac = (int64_t)(3 * i + j) * MP + at;
      if (INC) o = fmaf(dg[j][s], dw[j][s], o);
      else if (live && half == 0 && z < pz) DUGw[ac] = f[j];
    }
    if (half == 0) buf[z][col] = o;
  }
  __syncthreads();
  if (!live) return;
  const int h = half * (KZH / 2) + w;
  if (w >= KZH / 2 || h >= kzh) return;
  float2 a = make_float2(0.f, 0.f), b = a;
  int z = 0;
#pragma unroll 4
  for (; z + 1 < pz; z += 2) {
    const float v0 = buf[z][col], v1 = buf[z + 1][col];
    const float2 t0 = tz[z * KZH + h], t1 = tz[(z + 1) * KZH + h];
    a.x = fmaf(v0, t0.x, a.x);
    a.y = fmaf(-v0, t0.y, a.y);
    b.x = fmaf(v1, t1.x, b.x);
    b.y = fmaf(-v1, t1.y, b.y);
  }
  if (z < pz) {
    const float v0 = buf[z][col];
    const float2 t0 = tz[z * KZH + h];
    a.x = fmaf(v0, t0.x, a.x);
    a.y = fmaf(-v0, t0.y, a.y);
  }
  G[((size_t)i * kzh + h) * nq + q] = make_float2(a.x + b.x, a.y + b.y);
}

// Backward stage, block (column chunk, component j): kg_i(z) = iota_z(F2[i]) of the cotangent;
// GACC_j (+)= sum_i DUG_(i,j)(z) kg_i(z); G[i dim + j][h] = sum_z kg_i(z) V_j(z) conj tz[z][h]
// for i < 3, wave w taking h = half KZH / 2 + w.
template <int NZS, int KZH>
__global__ __launch_bounds__(64 * kColWaves) void k_fx_col_bwd(Geo gp, const float2* __restrict__ F2,
                                                    const float* __restrict__ VP,
                                                    const float* __restrict__ DUG,
                                                    float* __restrict__ GACC, int first,
                                                    const float2* __restrict__ tw_zT,
                                                    float2* __restrict__ G) {
  __shared__ float2 tz[kColWaves * NZS * KZH];
  __shared__ float bk[3][kColWaves * NZS][kColW];   // kg_i(z) V_j(z)
  const int lane = threadIdx.x & 63;
  const int col = lane & (kColW - 1), half = lane >> 5;
  const int w = wave_uniform(threadIdx.x >> 6);
  const int j = blockIdx.y;
  const int nq = gp.nx * gp.ny;
  const int q = blockIdx.x * kColW + col;
  const int qc = q < nq ? q : nq - 1;
  const bool live = q < nq;
  const int pz = gp.nz, kzh = gp.kzh;
  const int64_t MP = gp.M;
  float2 F[3][KZH / 2];
#pragma unroll
  for (int c = 0; c < 3; ++c)
    load_half<KZH>(F2 + (size_t)c * kzh * nq + qc, (size_t)nq, kzh, half, F[c]);
  TzStage<KZH> tzs;
  tzs.load(tw_zT, pz, kzh);
  // the planes' accumulator, state derivatives and velocity, loaded before the barrier
  float ga[NZS], du[3][NZS], vv[NZS];
#pragma unroll
  for (int s = 0; s < NZS; ++s) {
    const int64_t at = (int64_t)min(w + kColWaves * s, pz - 1) * nq + qc;
    ga[s] = GACC[j * MP + at];
    vv[s] = VP[j * MP + at];
#pragma unroll
    for (int c = 0; c < 3; ++c) du[c][s] = DUG[(int64_t)(3 * c + j) * MP + at];
  }
  tzs.store(pz, kzh, tz);
  __syncthreads();
#pragma unroll
  for (int s = 0; s < NZS; ++s) {
    const int z = w + kColWaves * s;
    const int64_t at = (int64_t)min(z, pz - 1) * nq + qc;
    float kg[3];
    iota_z3<KZH>(F, tz, min(z, pz - 1), half, kg);
    float a = first ? 0.f : ga[s];
#pragma unroll
    for (int c = 0; c < 3; ++c) a = fmaf(du[c][s], kg[c], a);
    if (live && half == 0 && z < pz) GACC[j * MP + at] = a;
    const float vj = vv[s];
    if (half == 0) {
#pragma unroll
      for (int c = 0; c < 3; ++c) bk[c][z][col] = kg[c] * vj;
    }
  }
  __syncthreads();
  if (!live) return;
  const int h = half * (KZH / 2) + w;
  if (w >= KZH / 2 || h >= kzh) return;
  float2 a[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) a[c] = make_float2(0.f, 0.f);
#pragma unroll 4
  for (int z = 0; z < pz; ++z) {
    const float2 t = tz[z * KZH + h];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float v = bk[c][z][col];
      a[c].x = fmaf(v, t.x, a[c].x);
      a[c].y = fmaf(-v, t.y, a[c].y);
    }
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) G[((size_t)(3 * c + j) * kzh + h) * nq + q] = a[c];
}

// ------------------------------------------------------------------------------ 3. pi yx
// the band entries a thread of a yx block writes: entry k = (jx, jy, kz0 + h) with value R and,
// where its mirror is written by the same thread, the mirror -k with conj(R).  Unpaired entries
// (jx = 0 or jy = 0) are written as zero by their own k; the unpaired plane jz = 0 by h = 0.
struct Target {
  int b;        // band index of k
  int bm;       // band index of -k, or -1
  int bz;       // unpaired k with h > 0: the unpaired entry (jx, jy) of the plane kz = -h, else -1
  bool zero;    // k is unpaired
  bool real;    // k = 0
};

__device__ __forceinline__ Target target(const Geo& g, int h, int jx, int jy) {
  Target t;
  const int jz = g.kz0 + h;
  t.b = (jz * g.ky + jy) * g.kx + jx;
  t.zero = jx == 0 || jy == 0;
  t.real = false;
  t.bm = -1;
  t.bz = -1;
  if (t.zero) {
    if (h > 0) t.bz = ((g.kz0 - h) * g.ky + jy) * g.kx + jx;
    return t;
  }
  const int mx = g.kx - jx, my = g.ky - jy;
  if (h > 0) {
    t.bm = ((g.kz0 - h) * g.ky + my) * g.kx + mx;
  } else {
    const int ky = jy - g.ky / 2, kx = jx - g.kx / 2;
    const bool own = ky > 0 || (ky == 0 && kx >= 0);
    if (!own) {
      t.b = -1;   // written by the owner of -k
      return t;
    }
    if (ky == 0 && kx == 0) t.real = true;
    else t.bm = (g.kz0 * g.ky + my) * g.kx + mx;
  }
  return t;
}

// the band values a forward stage update of component i at band index b reads (b < 0: a
// harmless in-bounds load of entry 0, not used)
struct StageIn {
  float2 s, u, p;
};
__device__ __forceinline__ StageIn stage_load(const Geo& g, int i, int b,
                                              const float2* __restrict__ src,
                                              const float2* __restrict__ un,
                                              const float2* __restrict__ acc) {
  const size_t o = (size_t)i * g.B + max(b, 0);
  return StageIn{src[o], un[o], acc[o]};
}

// Forward stage update of component i at band index b with conv (unscaled)
__device__ __forceinline__ void stage_entry(const Geo& g, int i, int b, float2 cv, float scaleP,
                                            const StageIn& in, float2* __restrict__ acc, int st,
                                            float2* __restrict__ wout) {
  const size_t o = (size_t)i * g.B + b;
  const float h = g.dt;
  const float2 sv = in.s;
  const float2 k = make_float2(-sv.x - scaleP * cv.x, -sv.y - scaleP * cv.y);
  const float2 u = in.u;
  float2 a;
  if (st == 1) {
    a = k;
  } else {
    const float2 p = in.p;
    const float f = st == 4 ? 1.f : 2.f;
    a = make_float2(fmaf(f, k.x, p.x), fmaf(f, k.y, p.y));
  }
  if (st < 4) {
    acc[o] = a;
    const float c = st == 3 ? h : 0.5f * h;
    wout[o] = make_float2(fmaf(c, k.x, u.x), fmaf(c, k.y, u.y));
  } else {
    const float s6 = h / 6.f;
    wout[o] = make_float2(fmaf(s6, a.x, u.x), fmaf(s6, a.y, u.y));
  }
}

__device__ __forceinline__ void stage_zero(const Geo& g, int i, int b, float2* __restrict__ acc,
                                           int st, float2* __restrict__ wout) {
  const size_t o = (size_t)i * g.B + b;
  if (st < 4) acc[o] = make_float2(0.f, 0.f);
  wout[o] = make_float2(0.f, 0.f);
}

// the band values a transposed-sweep update of component i at band index b reads (b < 0: a
// harmless in-bounds load of entry 0, not used)
struct AdjIn {
  float2 r, p, ks;
};
__device__ __forceinline__ AdjIn adj_load(const Geo& g, int i, int b,
                                          const float2* __restrict__ rho,
                                          const float2* __restrict__ Asum,
                                          const float2* __restrict__ Ksum) {
  const size_t o = (size_t)i * g.B + max(b, 0);
  return AdjIn{rho[o], Asum[o], Ksum[o]};
}

// Transposed-sweep update of component i at band index b with A = sum_j i q_j R_j / MP
__device__ __forceinline__ void adj_entry(const Geo& g, int i, int b, float2 A, int st, int more,
                                          const AdjIn& in, float2* __restrict__ rho,
                                          float2* __restrict__ Asum, float2* __restrict__ Ksum,
                                          float2* __restrict__ kap) {
  const size_t o = (size_t)i * g.B + b;
  const float h = g.dt;
  const float cr = st == 2 ? h / 6.f : h / 3.f;
  const float ca = st == 4 ? h : 0.5f * h;
  const float2 r = in.r;
  float2 as = A;
  if (st != 4) {
    const float2 p = in.p;
    as = make_float2(p.x + A.x, p.y + A.y);
  }
  float2 kp;
  if (st > 1) {
    Asum[o] = as;
    kp = make_float2(fmaf(ca, A.x, cr * r.x), fmaf(ca, A.y, cr * r.y));
  } else {
    const float2 rn = make_float2(r.x + as.x, r.y + as.y);
    rho[o] = rn;
    if (!more) return;
    kp = make_float2(h / 6.f * rn.x, h / 6.f * rn.y);
  }
  kap[o] = kp;
  const float2 ks = in.ks;
  Ksum[o] = make_float2(ks.x + kp.x, ks.y + kp.y);
}

// A block takes 16 ky by 32 kx of one (component i, kz = h) plane: R = sum_y sum_x G conj Tx conj
// Ty on the matrix cores (as k_pi_yx, bl_dft_mfma.hip), then the update of its band entries, one per
// thread, whose operands are loaded first.  Wavefront (x tile, part):
//   forward sweep: part of 3 of the terms y, R is the sum of all;
//   transposed sweep: derivative plane j, and R = q_x R_0 + q_y R_1 + q_z R_2, A = i scaleP R.
// At a 48^3 product grid (96 blocks) a launch takes 7.8 and 10.1 us; with the planes and
// twiddles staged in LDS for the vector units it took 8.1 and 13.0.
constexpr int kKY = 16, kKX = 32;      // entries of a block
constexpr int kYxTiles = 3;            // x tiles at a time
constexpr int kYxWaves = 3 * kYxTiles;
struct YxArgs {
  float scaleP;
  int st, more;
  const float2 *src, *un;              // forward
  float2 *acc, *wout;
  float2 *rho, *Asum, *Ksum, *kap;     // transposed
};
template <bool ADJ>
__global__ __launch_bounds__(64 * kYxWaves) void k_fx_pi_yx(Geo g, Geo gp, const float2* __restrict__ G,
                                                            const float2* __restrict__ tw_x,
                                                            const float2* __restrict__ tw_yT, int kyp,
                                                            int nyp, int ntx, YxArgs a) {
  __shared__ float part[kYxWaves][2][8][65];
  const int lane = threadIdx.x & 63, m = lane & 15, q = lane >> 4, w = wave_of(threadIdx.x);
  const int KX = g.kx, KY = g.ky, PX = gp.nx, PY = gp.ny;
  const int ih = blockIdx.x, i = ih / g.kzh, h = ih - i * g.kzh;
  const int kyt = (int)blockIdx.y / ((KX + kKX - 1) / kKX), ky0 = kyt * kKY;
  const int kx0 = ((int)blockIdx.y - kyt * ((KX + kKX - 1) / kKX)) * kKX;
  // this thread's entry and what its update reads
  const int e = (int)threadIdx.x, el = e & (kKX - 1), ey = e / kKX;
  const int jx = kx0 + el, jy = ky0 + ey;
  const bool entry = ey < kKY && jx < KX && jy < KY;
  Target t = target(g, h, min(jx, KX - 1), min(jy, KY - 1));
  if (!entry) t.b = -1;
  StageIn sin[2];
  AdjIn ain[3];
  if constexpr (ADJ) {
    ain[0] = adj_load(g, i, t.b, a.rho, a.Asum, a.Ksum);
    ain[1] = adj_load(g, i, t.bm, a.rho, a.Asum, a.Ksum);
    ain[2] = adj_load(g, i, t.bz, a.rho, a.Asum, a.Ksum);
  } else {
    sin[0] = stage_load(g, i, t.zero ? -1 : t.b, a.src, a.un, a.acc);
    sin[1] = stage_load(g, i, t.bm, a.src, a.un, a.acc);
  }
  const int p = w / ntx, xt = w - p * ntx;   // part, x tile
  if (p < 3) {
    const size_t plane = ADJ ? (size_t)(3 * i + p) * g.kzh + h : (size_t)ih;
    const Rsrc rg = rsrc(G + plane * PY * PX, (uint32_t)PY * (uint32_t)PX * 8u);
    const Rsrc ry = rsrc(tw_yT, (uint32_t)nyp * (uint32_t)kyp * 8u);
    const Rsrc rx = rsrc(tw_x, (uint32_t)KX * (uint32_t)PX * 8u);
    f4 pre[2], pim[2];
#pragma unroll
    for (int v = 0; v < 2; ++v) pre[v] = pim[v] = f4{0.f, 0.f, 0.f, 0.f};
    for (int x0 = xt * 16; x0 < PX; x0 += 16 * ntx) {
      f4 tx[2][2];   // twiddles of the terms x = x0 + 4 q + n
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const int kx = kx0 + 16 * v + m;
        const uint32_t off = kx < KX ? ((uint32_t)kx * (uint32_t)PX + (uint32_t)(x0 + 4 * q)) * 8u : kPast;
        tx[v][0] = ld4(rx, off);
        tx[v][1] = ld4(rx, off == kPast ? kPast : off + 16u);
      }
      f4 cr[2], ci[2], sr[2], si[2];
#pragma unroll
      for (int v = 0; v < 2; ++v) cr[v] = ci[v] = sr[v] = si[v] = f4{0.f, 0.f, 0.f, 0.f};
      const uint32_t xoff = (uint32_t)(x0 + m) * 8u;
      const bool on = x0 + m < PX;
      constexpr int U = ADJ ? 4 : 3;
      const int first = ADJ ? 0 : 4 * p, step = ADJ ? 4 : 12;
      for (int y0 = first; y0 <= PY / 2; y0 += step * U) {
        f2 s[U], d[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const uint32_t y = (uint32_t)(y0 + step * u + q), ym = (uint32_t)PY - y;
          const bool one = on && (int)y <= PY / 2, two = one && y > 0 && y != ym;
          const f2 v0 = ld2(rg, one ? y * (uint32_t)PX * 8u + xoff : kPast);
          const f2 v1 = ld2(rg, two ? ym * (uint32_t)PX * 8u + xoff : kPast);
          b[u] = ld2(ry, (y * (uint32_t)kyp + (uint32_t)(ky0 + m)) * 8u);
          s[u] = v0 + v1;
          d[u] = v0 - v1;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          cr[u & 1] = mfma(s[u].x, b[u].x, cr[u & 1]);
          ci[u & 1] = mfma(s[u].y, b[u].x, ci[u & 1]);
          sr[u & 1] = mfma(d[u].y, b[u].y, sr[u & 1]);
          si[u & 1] = mfma(d[u].x, b[u].y, si[u & 1]);
        }
      }
      const f4 hr = (cr[0] + cr[1]) + (sr[0] + sr[1]), hi = (ci[0] + ci[1]) - (si[0] + si[1]);
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const f4 t0 = tx[v][0], t1 = tx[v][1];
        f4 pa[2], pb[2], pc[2], pd[2];
#pragma unroll
        for (int n = 0; n < 2; ++n) pa[n] = pb[n] = pc[n] = pd[n] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int n = 0; n < 4; ++n) {
          const float tr = n < 2 ? t0[2 * n] : t1[2 * n - 4], ti = n < 2 ? t0[2 * n + 1] : t1[2 * n - 3];
          pa[n & 1] = mfma(tr, hr[n], pa[n & 1]);
          pb[n & 1] = mfma(tr, hi[n], pb[n & 1]);
          pc[n & 1] = mfma(ti, hi[n], pc[n & 1]);
          pd[n & 1] = mfma(ti, hr[n], pd[n & 1]);
        }
        pre[v] += (pa[0] + pa[1]) + (pc[0] + pc[1]);
        pim[v] += (pb[0] + pb[1]) - (pd[0] + pd[1]);
      }
    }
    // row 4 q + n of tile v is kx = kx0 + 16 v + 4 q + n, column m is ky = ky0 + m (65: the
    // entries of a wavefront's readers lie in different banks)
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        part[w][v][2 * n][lane] = pre[v][n];
        part[w][v][2 * n + 1][lane] = pim[v][n];
      }
  }
  __syncthreads();
  if (entry) {
    const int v = el >> 4, n = el & 3, l = (el >> 2 & 3) * 16 + ey;
    float2 r = make_float2(0.f, 0.f);
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      float2 s = make_float2(0.f, 0.f);
#pragma unroll
      for (int o = 0; o < kYxTiles; ++o)
        if (o < ntx) {
          s.x += part[j * ntx + o][v][2 * n][l];
          s.y += part[j * ntx + o][v][2 * n + 1][l];
        }
      const float qj = !ADJ ? 1.f : j == 0 ? qaxis(g, 0, jx) : j == 1 ? qaxis(g, 1, jy) : qaxis(g, 2, g.kz0 + h);
      r.x = fmaf(qj, s.x, r.x);
      r.y = fmaf(qj, s.y, r.y);
    }
    if constexpr (ADJ) {
      float2 A = t.zero ? make_float2(0.f, 0.f) : make_float2(-a.scaleP * r.y, a.scaleP * r.x);
      if (t.real) A.y = 0.f;
      if (t.b >= 0) {
        adj_entry(g, i, t.b, A, a.st, a.more, ain[0], a.rho, a.Asum, a.Ksum, a.kap);
        if (t.bm >= 0)
          adj_entry(g, i, t.bm, make_float2(A.x, -A.y), a.st, a.more, ain[1], a.rho, a.Asum, a.Ksum, a.kap);
        if (t.bz >= 0)
          adj_entry(g, i, t.bz, make_float2(0.f, 0.f), a.st, a.more, ain[2], a.rho, a.Asum, a.Ksum, a.kap);
      }
    } else if (t.b >= 0) {
      if (t.zero) {
        stage_zero(g, i, t.b, a.acc, a.st, a.wout);
        if (t.bz >= 0) stage_zero(g, i, t.bz, a.acc, a.st, a.wout);
      } else {
        if (t.real) r.y = 0.f;
        stage_entry(g, i, t.b, r, a.scaleP, sin[0], a.acc, a.st, a.wout);
        if (t.bm >= 0)
          stage_entry(g, i, t.bm, make_float2(r.x, -r.y), a.scaleP, sin[1], a.acc, a.st, a.wout);
      }
    }
  }
  if (h == 0 && blockIdx.y == 0) {   // the unpaired plane kz = -K/2 (A = 0 there)
    for (int o = threadIdx.x; o < KY * KX; o += (int)blockDim.x) {
      if constexpr (ADJ)
        adj_entry(g, i, o, make_float2(0.f, 0.f), a.st, a.more, adj_load(g, i, o, a.rho, a.Asum, a.Ksum),
                  a.rho, a.Asum, a.Ksum, a.kap);
      else
        stage_zero(g, i, o, a.acc, a.st, a.wout);
    }
  }
}

template <bool ADJ>
void launch_yx(const Geo& g, const Geo& gp, const DftPlan& pl, const float2* G, const YxArgs& a,
               hipStream_t s) {
  const int ntx = std::min((gp.nx + 15) / 16, kYxTiles);
  const int waves = std::max(3 * ntx, kKY * kKX / 64);   // at least a thread per entry
  const dim3 grid(g.dim * g.kzh, ((g.ky + kKY - 1) / kKY) * ((g.kx + kKX - 1) / kKX));
  hipLaunchKernelGGL(k_fx_pi_yx<ADJ>, grid, dim3(64 * waves), 0, s, g, gp, G, pl.tw_x, pl.tw_yT, pl.kyp,
                     pl.nyp, ntx, a);
}

int nzs_of(int pz) { return pz <= 16 ? 2 : pz <= 32 ? 4 : 6; }
int kzh_of(int kzh) { return kzh <= 8 ? 8 : 16; }

}  // namespace

bool fused_ok(const Geo& g, const Geo& gp) {
  return g.dim == 3 && gp.nz <= 48 && g.kzh <= 16 && g.kzh >= 2 && g.ky <= 128 && gp.nx * gp.ny <= 6144;
}

void fx_iota_xy(const Geo& g, const Geo& gp, const DftPlan& pl, const float2* in, int deriv,
                float2* F2, hipStream_t s) {
  // (fused_ok: ky is below the bound of these)
  if (deriv) iota_xy_deriv_mfma(g, gp, pl, in, F2, s);
  else iota_xy_mfma(gp, pl, in, g.dim, F2, s);
}

namespace {
// f(planes of a wavefront, kz of a block) with the compile-time sizes that hold gp's
template <class F>
void with_sizes(const Geo& gp, F&& f) {
  using std::integral_constant;
  const auto kz = [&](auto nzs) {
    if (kzh_of(gp.kzh) == 8) f(nzs, integral_constant<int, 8>{});
    else f(nzs, integral_constant<int, 16>{});
  };
  switch (nzs_of(gp.nz)) {
    case 2: kz(integral_constant<int, 2>{}); break;
    case 4: kz(integral_constant<int, 4>{}); break;
    default: kz(integral_constant<int, 6>{}); break;
  }
}
dim3 col_grid(const Geo& gp) { return dim3((unsigned)((gp.nx * gp.ny + kColW - 1) / kColW), 3); }
}  // namespace

void fx_col_fwd(const Geo& gp, const DftPlan& pl, const float2* F2, const float* VP,
                float* DUGw, const float* DUGr, const float* DVP, float2* G, hipStream_t s) {
  with_sizes(gp, [&](auto nzs, auto kzh) {
    constexpr int N = decltype(nzs)::value, K = decltype(kzh)::value;
    if (DUGr != nullptr)   // products: read the stored stage derivatives
      hipLaunchKernelGGL((k_fx_col_fwd<N, K, true>), col_grid(gp), dim3(64 * kColWaves), 0, s, gp, F2, VP,
                         DUGw, DUGr, DVP, pl.tw_zT, G);
    else
      hipLaunchKernelGGL((k_fx_col_fwd<N, K, false>), col_grid(gp), dim3(64 * kColWaves), 0, s, gp, F2, VP,
                         DUGw, DUGr, DVP, pl.tw_zT, G);
  });
}

void fx_col_bwd(const Geo& gp, const DftPlan& pl, const float2* F2, const float* VP,
                const float* DUG, float* GACC, int first, float2* G, hipStream_t s) {
  with_sizes(gp, [&](auto nzs, auto kzh) {
    constexpr int N = decltype(nzs)::value, K = decltype(kzh)::value;
    hipLaunchKernelGGL((k_fx_col_bwd<N, K>), col_grid(gp), dim3(64 * kColWaves), 0, s, gp, F2, VP, DUG, GACC,
                       first, pl.tw_zT, G);
  });
}

void fx_pi_yx_stage(const Geo& g, const Geo& gp, const DftPlan& pl, const float2* G, float scaleP,
                    const float2* src, const float2* un, float2* acc, int st, float2* wout,
                    hipStream_t s) {
  YxArgs a{};
  a.scaleP = scaleP;
  a.st = st;
  a.src = src;
  a.un = un;
  a.acc = acc;
  a.wout = wout;
  launch_yx<false>(g, gp, pl, G, a, s);
}

void fx_pi_yx_adj(const Geo& g, const Geo& gp, const DftPlan& pl, const float2* G, float scaleP,
                  float2* rho, float2* Asum, float2* Ksum, float2* kap, int st, int more,
                  hipStream_t s) {
  YxArgs a{};
  a.scaleP = scaleP;
  a.st = st;
  a.more = more;
  a.rho = rho;
  a.Asum = Asum;
  a.Ksum = Ksum;
  a.kap = kap;
  launch_yx<true>(g, gp, pl, G, a, s);
}

}  // namespace bl
