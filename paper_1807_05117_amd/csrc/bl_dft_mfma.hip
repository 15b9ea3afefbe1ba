// Band <-> grid transforms on the FP32 matrix cores (v_mfma_f32_16x16x4_f32: products and sums
// in FP32, K = 4 terms per instruction).
//
// The stages of bl_dft.hip's comment are products of small dense twiddle matrices with fields.
// With one thread per output the vector units waited for twiddles (scalar loads of whole rows,
// or a table row again per wavefront from the L2) rather than for their arithmetic.  Here a
// wavefront keeps tiles of 16 x 16 outputs, one register of a twiddle matrix feeds 16 x 4
// multiply-adds, and the x and y stages are one launch each way, their intermediate in
// registers and LDS.  Axes are folded (index i with n - i: sums meet the cosines, differences
// the sines), which halves the products.  Per launch (us), before and now:
//                      128^3          181x211x179     256^3
//   iota x and y       7.3 + 8.6, 7.6   25 + 37, 24     50 + 62, 38
//   iota z             11.8, 10.3       38, 27          72, 58
//   pi z               14.5, 8.3        61, 27          127, 54
//   pi y and x         10.1 + 8.6, 11.9 35 + 29, 33     60 + 89, 55
// Chains of sums are split where registers allow, since the rounding of a sum grows with the
// terms of its chain: against FP64, iota is off by 1.0 to 1.6e-7 (1.1 to 2.1e-7 before) and pi of
// white noise by 1.2 to 1.8e-7 (1.2 to 2.0e-7) over ten shapes up to 256 points and 64 terms an axis.
// The z stages are bound by their fields (256^3: 201 MB at 3.4 to 3.7 TB/s).  pi y and x has one
// workgroup per (component, kz, 16 ky) and does not fill the device at 128^3 (96 of them).
#include "bl_mfma.h"

namespace bl {
namespace {

// Consecutive workgroups go to the 8 XCDs in turn, each with an L2 of its own; so that neighbours,
// which share cache lines where rows are not aligned, meet in one L2, workgroup b takes unit
// (b % 8) (n / 8) + b / 8 of n (a multiple of 8; the last ones may have no unit).
constexpr unsigned kXcd = 8;
__device__ __forceinline__ unsigned unit_of() {
  return (blockIdx.x % kXcd) * (gridDim.x / kXcd) + blockIdx.x / kXcd;
}
inline unsigned units(int64_t n) { return (unsigned)((n + kXcd - 1) / kXcd * kXcd); }

// ---------------------------------------------------------------------- iota, x and y stages
// A block takes 16 columns x of one (component, kz) plane and a run of y tiles: its wavefronts
// share the x stage (F1[ky][x] for all ky, through LDS), then each forms y tiles of 16 rows.
// KYM: tiles of 16 ky.  DERIV: component c = i dim + j is the derivative of band field i along
// axis j, i q_j band_i with q_j = 2 pi k_j ratio_j.
constexpr int kIW = 4;   // wavefronts of a block
struct Ratios {
  float r[3];
};
template <int KYM, bool DERIV>
__global__ __launch_bounds__(64 * kIW) void k_iota_xy(Geo g, Ratios ratio, const float2* __restrict__ band,
                                                      const float2* __restrict__ tw_x,
                                                      const float2* __restrict__ tw_yT, int kyp, int nyp,
                                                      int nxt, int nyr, int yrun, int nch,
                                                      float2* __restrict__ F2) {
  BL_BATCH_Z1(g.bat)
  BL_AT(band, g.bat);
  BL_AT(F2, g.bat);
  __shared__ f2 F1[KYM * 16][16];
  const int lane = threadIdx.x & 63, m = lane & 15, q = lane >> 4, w = wave_of(threadIdx.x);
  const int unit = (int)unit_of(), run = unit / nxt, ch = run / nyr;
  if (ch >= nch) return;
  const int xt = unit - run * nxt, yb = run - ch * nyr;
  const int c = ch / g.kzh, h = ch - c * g.kzh;
  const int x = xt * 16 + m, xc = min(x, g.nx - 1);
  const size_t plane = (size_t)g.ky * g.kx;
  const int ci = DERIV ? c / g.dim : c, axis = c - ci * g.dim;
  const Rsrc rb = rsrc(band + (size_t)(ci * g.kz + g.kz0 + h) * plane, (uint32_t)plane * 8u);
  const Rsrc rx = rsrc(tw_x, (uint32_t)g.kx * (uint32_t)g.nx * 8u);
  for (int t = w; t < KYM; t += kIW) {
    const int row = t * 16 + m;
    f4 re[4], im[4];   // four chains: the rounding of a sum grows with the terms of its chain
#pragma unroll
    for (int j = 0; j < 4; ++j) re[j] = im[j] = f4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < g.kx; k0 += 32) {   // four loads of terms kx = k + 2 q, k + 2 q + 1 ahead
      f4 a[4];
      f2 b[4][2];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t k = (uint32_t)(k0 + 8 * u + 2 * q);
        a[u] = ld4(rb, row < g.ky && (int)k < g.kx ? ((uint32_t)row * (uint32_t)g.kx + k) * 8u : kPast);
        if constexpr (DERIV) {
          const float two_pi = 6.283185307179586f;
          const int k0i = axis == 0 ? (int)k - g.kx / 2 : axis == 1 ? row - g.ky / 2 : h;
          const int k1i = axis == 0 ? k0i + 1 : k0i;
          const float q0 = two_pi * (float)k0i * ratio.r[axis], q1 = two_pi * (float)k1i * ratio.r[axis];
          a[u] = f4{-q0 * a[u].y, q0 * a[u].x, -q1 * a[u].w, q1 * a[u].z};
        }
        b[u][0] = ld2(rx, (k * (uint32_t)g.nx + (uint32_t)xc) * 8u);
        b[u][1] = ld2(rx, ((k + 1u) * (uint32_t)g.nx + (uint32_t)xc) * 8u);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        re[0] = mfma(a[u].x, b[u][0].x, re[0]);
        im[0] = mfma(a[u].y, b[u][0].x, im[0]);
        re[1] = mfma(a[u].y, b[u][0].y, re[1]);
        im[1] = mfma(a[u].x, b[u][0].y, im[1]);
        re[2] = mfma(a[u].z, b[u][1].x, re[2]);
        im[2] = mfma(a[u].w, b[u][1].x, im[2]);
        re[3] = mfma(a[u].w, b[u][1].y, re[3]);
        im[3] = mfma(a[u].z, b[u][1].y, im[3]);
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      F1[t * 16 + 4 * q + i][m] = f2{(re[0][i] + re[2][i]) - (re[1][i] + re[3][i]),
                                     (im[0][i] + im[2][i]) + (im[1][i] + im[3][i])};
  }
  __syncthreads();
  f2 f[KYM][4];
#pragma unroll
  for (int t = 0; t < KYM; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) f[t][i] = F1[t * 16 + 4 * q + i][m];
  const Rsrc ry = rsrc(tw_yT, (uint32_t)nyp * (uint32_t)kyp * 8u);
  const Rsrc out = rsrc(F2 + (size_t)ch * g.ny * g.nx, (uint32_t)g.ny * (uint32_t)g.nx * 8u);
  // rows y <= ny / 2: with A = sum Tr Fr, B = sum Ti Fi, C = sum Tr Fi and D = sum Ti Fr, row y is
  // (A - B, C + D) and row ny - y is (A + B, C - D)
  const int y1 = min(g.ny / 2 + 1, (yb + 1) * yrun);
  for (int y0 = yb * yrun + w * 16; y0 < y1; y0 += 16 * kIW) {
    f4 ra = {0.f, 0.f, 0.f, 0.f}, rb2 = ra, rc = ra, rd = ra;
    f4 a[KYM][2];   // twiddles of the terms ky = 16 t + 4 q + i, i = 0..3
    const uint32_t row = (uint32_t)(y0 + m) * (uint32_t)kyp * 8u;
#pragma unroll
    for (int t = 0; t < KYM; ++t) {
      a[t][0] = ld4(ry, row + (uint32_t)(t * 16 + 4 * q) * 8u);
      a[t][1] = ld4(ry, row + (uint32_t)(t * 16 + 4 * q + 2) * 8u);
    }
#pragma unroll
    for (int t = 0; t < KYM; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float tr = a[t][i / 2][2 * (i & 1)], ti = a[t][i / 2][2 * (i & 1) + 1];
        ra = mfma(tr, f[t][i].x, ra);
        rb2 = mfma(ti, f[t][i].y, rb2);
        rc = mfma(tr, f[t][i].y, rc);
        rd = mfma(ti, f[t][i].x, rd);
      }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int y = y0 + 4 * q + i, ym = g.ny - y;
      if (y >= y1 || x >= g.nx) continue;
      st2(out, ((uint32_t)y * (uint32_t)g.nx + (uint32_t)x) * 8u, f2{ra[i] - rb2[i], rc[i] + rd[i]});
      if (y > 0 && ym != y)
        st2(out, ((uint32_t)ym * (uint32_t)g.nx + (uint32_t)x) * 8u, f2{ra[i] + rb2[i], rc[i] - rd[i]});
    }
  }
}

// ------------------------------------------------------------------------------ iota, z stage
// Planes z and nz - z share their twiddles up to conjugation: over z <= nz / 2, A = sum_h
// f.x t.x and B = sum_h f.y t.y give A - B for plane z and A + B for plane nz - z.  A wavefront
// holds the half spectrum of 16 NT columns in registers and forms tiles of 16 z; a lane's NT
// columns are consecutive, so it stores 4 NT bytes at a time.  T: groups of 4 kz.
template <int T, int NT>
__global__ __launch_bounds__(256) void k_iota_z(Geo g, const float2* __restrict__ F2,
                                                const float2* __restrict__ tw_zT, int nzp,
                                                float* __restrict__ out, int zchunk) {
  BL_BATCH(g.bat)
  BL_AT(F2, g.bat);
  BL_AT(out, g.bat);
  const int lane = threadIdx.x & 63, m = lane & 15, q = lane >> 4, w = wave_of(threadIdx.x);
  const uint32_t nq = (uint32_t)g.nx * (uint32_t)g.ny;
  const int c = batch_bz(g.bat, bpair_);
  const uint32_t col0 = (unit_of() * 4u + (uint32_t)w) * (16u * NT), col = col0 + NT * (uint32_t)m;
  if (col0 >= nq) return;
  const Rsrc rf = rsrc(F2 + (size_t)c * g.kzh * nq, (uint32_t)g.kzh * nq * 8u);
  const Rsrc rt = rsrc(tw_zT, (uint32_t)nzp * kZP * 8u);
  const Rsrc ro = rsrc(out + (size_t)c * g.M, (uint32_t)g.M * 4u);
  float bx[T][NT], by[T][NT];   // kz = 4 t + q
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int h = 4 * t + q;
    const float sc = h > 0 ? 2.f : 1.f;
    const uint32_t off = h < g.kzh ? ((uint32_t)h * nq + col) * 8u : kPast;
#pragma unroll
    for (int j = 0; j < NT; j += 2) {
      const f4 v = ld4(rf, off == kPast ? kPast : off + 8u * j);
      bx[t][j] = sc * v.x;
      by[t][j] = sc * v.y;
      bx[t][j + 1] = sc * v.z;
      by[t][j + 1] = sc * v.w;
    }
  }
  const int zmax = g.nz / 2;
  const int z1 = min(zmax + 1, (int)(blockIdx.y + 1) * zchunk);
  f2 next[T];   // twiddles of the next tile
  auto load = [&](int z) {
    const uint32_t row = ((uint32_t)(z + m) * kZP + (uint32_t)q) * 8u;
#pragma unroll
    for (int t = 0; t < T; ++t) next[t] = ld2(rt, row + (uint32_t)t * 32u);
  };
  int z0 = blockIdx.y * zchunk;
  if (z0 < z1) load(z0);
  for (; z0 < z1; z0 += 16) {
    f4 a[NT], b[NT];
    f2 tw[T];
#pragma unroll
    for (int j = 0; j < NT; ++j) a[j] = b[j] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < T; ++t) tw[t] = next[t];
    if (z0 + 16 < z1) load(z0 + 16);
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        a[j] = mfma(tw[t].x, bx[t][j], a[j]);
        b[j] = mfma(tw[t].y, by[t][j], b[j]);
      }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int z = z0 + 4 * q + i, zm = g.nz - z;
      if (z >= z1) continue;
      const bool two = z > 0 && zm != z;
      const uint32_t o0 = ((uint32_t)z * nq + col) * 4u, o1 = ((uint32_t)zm * nq + col) * 4u;
      if (col + NT <= nq) {
        if constexpr (NT == 4) {
          st4(ro, o0, f4{a[0][i] - b[0][i], a[1][i] - b[1][i], a[2][i] - b[2][i], a[3][i] - b[3][i]});
          if (two) st4(ro, o1, f4{a[0][i] + b[0][i], a[1][i] + b[1][i], a[2][i] + b[2][i], a[3][i] + b[3][i]});
        } else {
          st2(ro, o0, f2{a[0][i] - b[0][i], a[1][i] - b[1][i]});
          if (two) st2(ro, o1, f2{a[0][i] + b[0][i], a[1][i] + b[1][i]});
        }
      } else {
#pragma unroll
        for (int j = 0; j < NT; ++j)
          if (col + j < nq) {
            st1(ro, o0 + 4u * j, a[j][i] - b[j][i]);
            if (two) st1(ro, o1 + 4u * j, a[j][i] + b[j][i]);
          }
      }
    }
  }
}

// -------------------------------------------------------------------------------- pi, z stage
// With s = f(z) + f(nz - z) and d = f(z) - f(nz - z) over z <= nz / 2 (the planes that are their
// own mirror alone), G.x = sum_z s t.x and G.y = -sum_z d t.y: half the products.  The
// wavefronts of a block share 32 columns and take every kPW-th group of four z; their sums
// are added in LDS in a fixed order.  HM: tiles of 16 kz.
constexpr int kPW = 4;
template <int HM>
__global__ __launch_bounds__(64 * kPW) void k_pi_z(Geo g, const float* __restrict__ f,
                                                   const float2* __restrict__ tw_zT, int nzp,
                                                   float2* __restrict__ G) {
  BL_BATCH(g.bat)
  BL_AT(f, g.bat);
  BL_AT(G, g.bat);
  __shared__ float part[kPW][16][64];
  const int lane = threadIdx.x & 63, m = lane & 15, q = lane >> 4, w = wave_of(threadIdx.x);
  const uint32_t nq = (uint32_t)g.nx * (uint32_t)g.ny;
  const int c = blockIdx.y;
  const uint32_t col0 = unit_of() * (32u), col = col0 + 2u * (uint32_t)m;
  if (col0 >= nq) return;
  const Rsrc rf = rsrc(f + (size_t)c * g.M, (uint32_t)g.M * 4u);
  const Rsrc rt = rsrc(tw_zT, (uint32_t)nzp * kZP * 8u);
  const Rsrc ro = rsrc(G + (size_t)c * g.kzh * nq, (uint32_t)g.kzh * nq * 8u);
  f4 re[HM][2], im[HM][2];
#pragma unroll
  for (int t = 0; t < HM; ++t)
#pragma unroll
    for (int j = 0; j < 2; ++j) re[t][j] = im[t][j] = f4{0.f, 0.f, 0.f, 0.f};
  const int zmax = g.nz / 2;
  constexpr int U = 4;   // groups of a wavefront whose loads are in flight together
  for (int z0 = 4 * w; z0 <= zmax; z0 += 4 * kPW * U) {
    float s[U][2], d[U][2];
    f2 tw[U][HM];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int zu = z0 + 4 * kPW * u + q, z = min(zu, zmax), zm = z > 0 ? g.nz - z : 0;
      const uint32_t o0 = ((uint32_t)z * nq + col) * 4u, o1 = ((uint32_t)zm * nq + col) * 4u;
      const bool one = zu <= zmax, two = one && zm != z;
#pragma unroll
      for (int t = 0; t < HM; ++t) tw[u][t] = ld2(rt, ((uint32_t)z * kZP + (uint32_t)(16 * t + m)) * 8u);
      const f2 a = ld2(rf, o0), b = ld2(rf, o1);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const float x = one ? a[j] : 0.f, y = two ? b[j] : 0.f;
        s[u][j] = x + y;
        d[u][j] = y - x;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (z0 + 4 * kPW * u > zmax) break;   // the same for the wavefront
#pragma unroll
      for (int t = 0; t < HM; ++t)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          re[t][j] = mfma(tw[u][t].x, s[u][j], re[t][j]);
          im[t][j] = mfma(tw[u][t].y, d[u][j], im[t][j]);
        }
    }
  }
#pragma unroll
  for (int t = 0; t < HM; ++t) {
    if (t > 0) __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        part[w][(i * 2 + j) * 2][lane] = re[t][j][i];
        part[w][(i * 2 + j) * 2 + 1][lane] = im[t][j][i];
      }
    __syncthreads();
    // wavefront w adds the rows kz = 16 t + 4 q + w
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[j] = part[0][w * 4 + j][lane];
#pragma unroll
      for (int o = 1; o < kPW; ++o) v[j] += part[o][w * 4 + j][lane];
    }
    const int h = 16 * t + 4 * q + w;
    if (h < g.kzh) {
      const uint32_t o = ((uint32_t)h * nq + col) * 8u;
      if (col + 2 <= nq) st4(ro, o, f4{v[0], v[1], v[2], v[3]});
      else if (col < nq) st2(ro, o, f2{v[0], v[1]});
    }
  }
}
static_assert(kPW == 4, "a wavefront adds one of the four rows of a lane");

// ------------------------------------------------------------------------ pi, y and x stages
// A block takes 16 ky of one (component, kz) plane.  A wavefront forms H[ky][x] for 16 columns x
// (terms y) as the tile D[x][ky], whose registers then are the terms x of P[ky][kx]; the
// wavefronts' sums are added in LDS in a fixed order.  KXM: tiles of 16 kx.
constexpr int kMaxW = 16;
template <int KXM>
__global__ __launch_bounds__(64 * kMaxW) void k_pi_yx(Geo g, const float2* __restrict__ G,
                                                      const float2* __restrict__ tw_yT, int kyp, int nyp,
                                                      const float2* __restrict__ tw_x,
                                                      float2* __restrict__ P) {
  BL_BATCH(g.bat)
  BL_AT(G, g.bat);
  BL_AT(P, g.bat);
  __shared__ float part[kMaxW][8][64];
  const int lane = threadIdx.x & 63, m = lane & 15, q = lane >> 4, w = wave_of(threadIdx.x);
  const int waves = (int)blockDim.x >> 6;
  const int ch = batch_bz(g.bat, bpair_), ky0 = blockIdx.x * 16;
  const Rsrc rg = rsrc(G + (size_t)ch * g.ny * g.nx, (uint32_t)g.ny * (uint32_t)g.nx * 8u);
  const Rsrc ry = rsrc(tw_yT, (uint32_t)nyp * (uint32_t)kyp * 8u);
  const Rsrc rx = rsrc(tw_x, (uint32_t)g.kx * (uint32_t)g.nx * 8u);
  f4 pre[KXM], pim[KXM];
#pragma unroll
  for (int t = 0; t < KXM; ++t) pre[t] = pim[t] = f4{0.f, 0.f, 0.f, 0.f};
  for (int x0 = w * 16; x0 < g.nx; x0 += 16 * waves) {
    // the sums of the cosines and of the sines apart, even and odd groups apart: the rounding of a
    // sum grows with the terms of its chain
    f4 cr[2], ci[2], sr[2], si[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) cr[j] = ci[j] = sr[j] = si[j] = f4{0.f, 0.f, 0.f, 0.f};
    const uint32_t xoff = (uint32_t)(x0 + m) * 8u;
    const bool on = x0 + m < g.nx;
    // terms y = y0 + 4 u + q and ny - y together: sums meet the cosines, differences the sines
    constexpr int U = 4;   // groups whose loads are in flight together
    for (int y0 = 0; y0 <= g.ny / 2; y0 += 4 * U) {
      f2 s[U], d[U], b[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t y = (uint32_t)(y0 + 4 * u + q), ym = (uint32_t)g.ny - y;
        const bool one = on && (int)y <= g.ny / 2, two = one && y > 0 && y != ym;
        const f2 v0 = ld2(rg, one ? y * (uint32_t)g.nx * 8u + xoff : kPast);
        const f2 v1 = ld2(rg, two ? ym * (uint32_t)g.nx * 8u + xoff : kPast);
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
    for (int t = 0; t < KXM; ++t) {   // terms x = x0 + 4 q + i
      const int kx = 16 * t + m;
      const uint32_t off = kx < g.kx ? ((uint32_t)kx * (uint32_t)g.nx + (uint32_t)(x0 + 4 * q)) * 8u : kPast;
      const f4 t0 = ld4(rx, off), t1 = ld4(rx, off == kPast ? kPast : off + 16u);
      f4 pa[2], pb[2], pc[2], pd[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) pa[j] = pb[j] = pc[j] = pd[j] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float tr = i < 2 ? t0[2 * i] : t1[2 * i - 4], ti = i < 2 ? t0[2 * i + 1] : t1[2 * i - 3];
        pa[i & 1] = mfma(tr, hr[i], pa[i & 1]);
        pb[i & 1] = mfma(tr, hi[i], pb[i & 1]);
        pc[i & 1] = mfma(ti, hi[i], pc[i & 1]);
        pd[i & 1] = mfma(ti, hr[i], pd[i & 1]);
      }
      pre[t] += (pa[0] + pa[1]) + (pc[0] + pc[1]);
      pim[t] += (pb[0] + pb[1]) - (pd[0] + pd[1]);
    }
  }
  float2* const dst = P + (size_t)ch * g.ky * g.kx;
#pragma unroll
  for (int t = 0; t < KXM; ++t) {
    if (t > 0) __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      part[w][2 * i][lane] = pre[t][i];
      part[w][2 * i + 1][lane] = pim[t][i];
    }
    __syncthreads();
    for (int e = (int)threadIdx.x; e < 256; e += (int)blockDim.x) {
      const int i = e >> 6, l = e & 63, ky = ky0 + (l & 15), kx = 16 * t + 4 * (l >> 4) + i;
      float2 s = make_float2(part[0][2 * i][l], part[0][2 * i + 1][l]);
      for (int o = 1; o < waves; ++o) {
        s.x += part[o][2 * i][l];
        s.y += part[o][2 * i + 1][l];
      }
      if (ky < g.ky && kx < g.kx) dst[(size_t)ky * g.kx + kx] = s;
    }
  }
}

template <int T, int NT>
void launch_iota_z(const Geo& g, const DftPlan& p, const float2* F2, float* out, int C, hipStream_t s) {
  const int64_t nq = (int64_t)g.nx * g.ny;
  const unsigned qb = units((nq + 64 * NT - 1) / (64 * NT));
  // z tiles of 16 planes (z, nz - z), split over blocks until the launch fills the device; the
  // launch shape asks for further splits
  const int tiles = (g.nz / 2 + 16) / 16;
  int n = 1;
  while ((int64_t)qb * C * n < 1024 && 2 * n <= tiles) n *= 2;
  for (int k = g.zv[TR_IOTA_Z]; k > 1 && 2 * n <= tiles; k /= 2) n *= 2;
  const int zchunk = (tiles + n - 1) / n * 16;
  BL_LAUNCH((k_iota_z<T, NT>), batch_grid(dim3(qb, (unsigned)((g.nz / 2 + zchunk) / zchunk), C), g.bat),
            dim3(256), 0, s, g, F2, p.tw_zT, p.nzp, out, zchunk);
}
template <int HM>
void launch_pi_z(const Geo& g, const DftPlan& p, const float* f, int C, float2* G, hipStream_t s) {
  const int64_t nq = (int64_t)g.nx * g.ny;
  BL_LAUNCH((k_pi_z<HM>), batch_grid(dim3(units((nq + 31) / 32), C), g.bat),
            dim3(64 * kPW), 0, s, g, f, p.tw_zT, p.nzp, G);
}

}  // namespace

void iota_z_mfma(const Geo& g, const DftPlan& p, const float2* F2, float* out, int C, hipStream_t s) {
  switch ((g.kzh + 3) / 4) {
    case 1: launch_iota_z<1, 4>(g, p, F2, out, C, s); break;
    case 2: launch_iota_z<2, 4>(g, p, F2, out, C, s); break;
    case 3: launch_iota_z<3, 4>(g, p, F2, out, C, s); break;
    case 4: launch_iota_z<4, 4>(g, p, F2, out, C, s); break;
    case 5: launch_iota_z<5, 4>(g, p, F2, out, C, s); break;
    case 6: launch_iota_z<6, 4>(g, p, F2, out, C, s); break;
    case 7:
    case 8: launch_iota_z<8, 4>(g, p, F2, out, C, s); break;
    case 9:
    case 10:
    case 11:
    case 12: launch_iota_z<12, 2>(g, p, F2, out, C, s); break;
    default: launch_iota_z<16, 2>(g, p, F2, out, C, s); break;
  }
}

void pi_z_mfma(const Geo& g, const DftPlan& p, const float* f, int C, float2* G, hipStream_t s) {
  switch ((g.kzh + 15) / 16) {
    case 1: launch_pi_z<1>(g, p, f, C, G, s); break;
    case 2: launch_pi_z<2>(g, p, f, C, G, s); break;
    case 3: launch_pi_z<3>(g, p, f, C, G, s); break;
    default: launch_pi_z<4>(g, p, f, C, G, s); break;
  }
}

namespace {
bool launch_iota_xy(const Geo& g, const DftPlan& p, const float2* band, int C, float2* F2, bool deriv,
                    const Ratios& r, hipStream_t s) {
  if (g.ky > 128) return false;
  const unsigned xt = (unsigned)((g.nx + 15) / 16);
  // y tiles over blocks until the launch fills the device (each repeats the x stage)
  const int rows = g.ny / 2 + 1, tiles = (rows + 16 * kIW - 1) / (16 * kIW);
  int n = 1;
  while ((int64_t)xt * C * g.kzh * n < 512 && 2 * n <= tiles) n *= 2;
  const int yrun = (tiles + n - 1) / n * 16 * kIW;
  const int nyr = (rows + yrun - 1) / yrun, nch = C * g.kzh;
  const dim3 grid = batch_grid(dim3(units((int64_t)xt * nyr * nch)), g.bat);
#define XY_D(K, D)                                                                               \
  hipLaunchKernelGGL((k_iota_xy<K, D>), grid, dim3(64 * kIW), 0, s, g, r, band, p.tw_x, p.tw_yT, p.kyp, \
                     p.nyp, (int)xt, nyr, yrun, nch, F2)
#define XY(K)              \
  do {                     \
    if (deriv) XY_D(K, true); \
    else XY_D(K, false);   \
  } while (0)
  switch ((g.ky + 15) / 16) {
    case 1: XY(1); break;
    case 2: XY(2); break;
    case 3: XY(3); break;
    case 4: XY(4); break;
    case 5:
    case 6: XY(6); break;
    default: XY(8); break;
  }
#undef XY
#undef XY_D
  return true;
}
}  // namespace

bool iota_xy_mfma(const Geo& g, const DftPlan& p, const float2* band, int C, float2* F2, hipStream_t s) {
  return launch_iota_xy(g, p, band, C, F2, false, Ratios{}, s);
}
bool iota_xy_deriv_mfma(const Geo& g, const Geo& gp, const DftPlan& p, const float2* band, float2* F2,
                        hipStream_t s) {
  const Ratios r{{(float)g.nref / (float)g.nx, (float)g.nref / (float)g.ny, (float)g.nref / (float)g.nz}};
  return launch_iota_xy(gp, p, band, g.dim * g.dim, F2, true, r, s);
}

bool pi_yx_mfma(const Geo& g, const DftPlan& p, const float2* G, int C, float2* P, hipStream_t s) {
  if (g.kx > 128) return false;
  const int tiles = (g.nx + 15) / 16, rounds = (tiles + kMaxW - 1) / kMaxW;
  const int waves = (tiles + rounds - 1) / rounds;
  const dim3 grid = batch_grid(dim3((unsigned)((g.ky + 15) / 16), 1, (unsigned)(C * g.kzh)), g.bat);
#define YX(K)                                                                                           \
  hipLaunchKernelGGL(k_pi_yx<K>, grid, dim3(64 * (unsigned)waves), 0, s, g, G, p.tw_yT, p.kyp, p.nyp,   \
                     p.tw_x, P)
  switch ((g.kx + 15) / 16) {
    case 1: YX(1); break;
    case 2: YX(2); break;
    case 3: YX(3); break;
    case 4: YX(4); break;
    case 5:
    case 6: YX(6); break;
    default: YX(8); break;
  }
#undef YX
  return true;
}

}  // namespace bl
