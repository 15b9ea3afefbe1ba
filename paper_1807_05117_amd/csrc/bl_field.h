// Device helpers shared by the kernels that transport grid fields: the threads' place in the
// grid, field access through raw buffer resources, interpolation and central differences.
#pragma once

#include "bl_internal.h"

namespace bl {
namespace {

// quotient by a host constant (FastDiv), exact for n < 2^31
__device__ __forceinline__ uint32_t fast_div(uint32_t n, const FastDiv& d) {
  return (__umulhi(n, d.m) + n * d.one) >> d.s;
}

// Fields are read through raw buffer resources: the plane's z offset is a scalar operand of the
// load, an 8-byte load of two consecutive floats needs only 4-byte alignment, and the hardware
// range check returns 0 for any dword past the buffer instead of faulting.
typedef float f2v __attribute__((ext_vector_type(2)));
typedef __amdgpu_buffer_rsrc_t Rsrc;

__device__ __forceinline__ Rsrc field_rsrc(const float* f, const Geo& g) {
  const uint64_t bytes = (uint64_t)g.M * 4u;   // < 2^32: the host limits prod(n) to < 2^30
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(f), (short)0, (int)(uint32_t)bytes,
                                           0x00020000);
}
// POLICY: the access's cache policy (kSC1: device scope, not served from a line that another XCD's
// stores have left stale)
constexpr int kSC1 = 16;
template <int POLICY = 0>
__device__ __forceinline__ float ld(Rsrc rs, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)voff, (int)soff, POLICY));
}
__device__ __forceinline__ void st(Rsrc rs, uint32_t voff, uint32_t soff, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), rs, (int)voff, (int)soff, 0);
}
// Periodic index of any |i| < 2^21 (i is exact in float): the quotient from i * (1/n) may be
// off by one near multiples of n, which the two selects correct.
__device__ __forceinline__ int wrap(int i, int n, float inv_n) {
  const int q = (int)floorf((float)i * inv_n);
  int r = i - q * n;
  r += r < 0 ? n : 0;
  r -= r >= n ? n : 0;
  return r;
}
// Lower cell index (periodic) and fractional weight of an offset.  General form: offsets are
// clamped to +-2^20 voxels and non-finite offsets are mapped to 0, so every index that
// reaches memory lies in [0, n).
__device__ __forceinline__ uint32_t split_any(float o, int base, int n, float inv_n, float& w) {
  if (!(fabsf(o) <= 1048576.0f)) o = 0.0f;
  const float f = floorf(o);
  w = o - f;
  return (uint32_t)wrap(base + (int)f, n, inv_n);
}

// ------------------------------------------------------------------ threads and addresses
// One thread per (x, y) column entry and ZV voxels of it along z.  A block takes kTB
// consecutive entries of the flattened (y, x) plane, whatever nx is: every wavefront reads and
// writes 64 consecutive floats of each plane and only a plane's last block has idle lanes
// (tiles of whole 64-voxel x runs leave a quarter of the lanes idle at nx = 96).
//
// While their fields come from the caches these kernels are bound by the issue of vector
// instructions and by the address path of the gathers, not by bandwidth: a wavefront
// instruction takes four cycles of its SIMD, 128^3 voxels are 32 wavefront-voxels per SIMD, so
// every instruction per voxel costs about 53 ns of a launch, and a 32-bit integer multiply
// four times that.  So
//   - the place of a voxel within its plane is one 32-bit byte offset per thread, shared by
//     every field (raw buffer loads: the plane's resource and the z offset are scalars), its
//     stencil neighbours four more; all divisions are scalar multiplications by host constants;
//   - an interpolation tap wraps each axis with two unsigned minima and forms its four row
//     addresses with two 24-bit multiply-adds; offsets of a whole period or more (and
//     non-finite ones) take a general path that a wavefront enters only if a lane needs it.
// A tap with its interpolation takes about 55 instructions per voxel; with 64 x 4 tiles, 64-bit
// addresses and multiplied wraps it took about 190 instruction times.  Per launch, before and
// after: state step 13.1 -> 12.1 us at 128^3, 8.2 -> 6.4 at 96^3, 26.2 -> 22.3 at 160x192x160,
// 73 -> 61 at 256^3 (5.5 TB/s); incremental step 15.9 -> 15.4, 9.9 -> 8.3, 32.7 -> 28.8, 136 -> 135.
constexpr int kTB = kTransportBlock;

// XCD-aware tile order: the hardware deals consecutive workgroups round-robin to the 8
// XCDs, each with its own L2.  The launch is 1D with a multiple of 8 workgroups and workgroup
// b works on tile (b % 8) * (nb / 8) + b / 8 of the plane-fastest tile order, so every XCD
// sweeps one contiguous slab of the volume and the y / z neighbours that gathers and central
// differences touch are mostly in its own L2.
constexpr int kXCD = 8;

// the thread's column entry and the byte offsets of its stencil within a plane (periodic)
struct Col {
  int x, y;
  uint32_t q;                 // y nx + x
  uint32_t c, xm, xp, ym, yp; // byte offsets of the entry and its x and y neighbours
  int zb;                     // the block's first plane / ZV
  uint32_t plane4;            // bytes of a plane
};

// for the block of entries from q0 on and the planes from zb ZV on; false: no entry of the plane
__device__ __forceinline__ bool place(const Geo& g, uint32_t q0, uint32_t zb, Col& t) {
  const uint32_t y0 = fast_div(q0, g.div_nx);
  const uint32_t xx = q0 - y0 * (uint32_t)g.nx + threadIdx.x;
  const uint32_t dy = fast_div(xx, g.div_nx);
  t.zb = (int)zb;
  t.x = (int)(xx - __umul24(dy, (uint32_t)g.nx));
  t.y = (int)(y0 + dy);
  t.q = q0 + threadIdx.x;
  t.c = t.q * 4u;
  t.plane4 = (uint32_t)g.nx * (uint32_t)g.ny * 4u;
  const uint32_t row = (uint32_t)g.nx * 4u, wx = row - 4u, wy = ((uint32_t)g.ny - 1u) * row;
  t.xm = t.x == 0 ? t.c + wx : t.c - 4u;
  t.xp = t.x + 1 == g.nx ? t.c - wx : t.c + 4u;
  t.ym = t.y == 0 ? t.c + wy : t.c - row;
  t.yp = t.y + 1 == g.ny ? t.c - wy : t.c + row;
  return t.q < (uint32_t)g.nx * (uint32_t)g.ny;
}
__device__ __forceinline__ bool locate(const Geo& g, int zv, Col& t) {
  const uint32_t nb = gridDim.x;            // multiple of kXCD
  const uint32_t b = blockIdx.x;
  const uint32_t tile = (b % kXCD) * (nb / kXCD) + b / kXCD;
  const uint32_t zb = fast_div(tile, g.div_nqb);
  if ((int)zb * zv >= g.nz) return false;
  return place(g, (tile - zb * (uint32_t)g.nqb) * kTB, zb, t);
}

#define COLUMN                         \
  Col t;                               \
  if (!locate(g, ZV, t)) return;
// plane z of the thread's voxel zz, clamped to the grid so that every load stays in bounds and
// the ZV voxels' loads can be issued together (only the stores are guarded), and the byte
// offsets of the plane and its periodic z neighbours; all scalar
#define VOXEL(zz)                                                               \
  const int zr = t.zb * ZV + (zz);                                              \
  const int z = zr < g.nz ? zr : g.nz - 1;                                      \
  const bool live = zr < g.nz;                                                  \
  const uint32_t zo = (uint32_t)z * t.plane4;                                   \
  const uint32_t zm = z == 0 ? (uint32_t)(g.nz - 1) * t.plane4 : zo - t.plane4; \
  const uint32_t zp = z + 1 == g.nz ? 0u : zo + t.plane4;                       \
  (void)live; (void)zo; (void)zm; (void)zp;

// (Y, a) of the thread's voxel: plane z as a scalar base, 16 bytes per column entry (< 2^26)
__device__ __forceinline__ float4 ld_ya(const Geo& g, const float4* YA, int z, const Col& t) {
  const char* base = reinterpret_cast<const char*>(YA + (size_t)z * ((size_t)g.nx * g.ny));
  return *reinterpret_cast<const float4*>(base + (uint32_t)(t.q << 4));
}

__device__ __forceinline__ void st_ya(const Geo& g, float4* YA, int z, const Col& t, float4 v) {
  char* base = reinterpret_cast<char*>(YA + (size_t)z * ((size_t)g.nx * g.ny));
  *reinterpret_cast<float4*>(base + (uint32_t)(t.q << 4)) = v;
}

// -------------------------------------------------------------------------- interpolation
// Byte addresses of the four (2D: two) rows' x0 entries, the weights, and whether the x1
// neighbour wraps to the row's start.
struct Tap {
  uint32_t a00, a01, a10, a11;   // (z0,y0) (z0,y1) (z1,y0) (z1,y1)
  float wx, wy, wz;
  bool wrapped;
};

// The same for |o| < n: base + floor(o) lies in [-n, 2n - 2], which two unsigned minima fold
// into [0, n) (a negative value is a huge unsigned one, so the first minimum takes i + n, and
// for i < n the second keeps i).
__device__ __forceinline__ uint32_t split_near(float o, int base, int n, float& w) {
  const float f = floorf(o);
  w = o - f;
  uint32_t i = (uint32_t)(base + (int)f);
  i = min(i, i + (uint32_t)n);
  return min(i, i - (uint32_t)n);
}

__device__ __forceinline__ uint64_t lanes_far(float o, int n) {
  return __builtin_amdgcn_ballot_w64(!(fabsf(o) < (float)n));   // NaN: far
}

template <int DIM>
__device__ __forceinline__ void tap_rows(const Geo& g, uint32_t x0, uint32_t y0, uint32_t z0,
                                         Tap& t) {
  // nx ny < 2^23 and every index < 2^11: 24-bit multiplies are exact
  const uint32_t nx = (uint32_t)g.nx, ny = (uint32_t)g.ny, row = nx * 4u;
  uint32_t e = __umul24(y0, nx) + x0;
  if (DIM == 3) e += __umul24(z0, nx * ny);
  t.a00 = e * 4u;
  const uint32_t dy = y0 == ny - 1u ? 0u - (ny - 1u) * row : row;
  t.a01 = t.a00 + dy;
  if (DIM == 3) {
    const uint32_t pl = ny * row;
    const uint32_t dz = z0 == (uint32_t)g.nz - 1u ? 0u - ((uint32_t)g.nz - 1u) * pl : pl;
    t.a10 = t.a00 + dz;
    t.a11 = t.a01 + dz;
  } else {
    t.a10 = t.a00;
    t.a11 = t.a01;
  }
  t.wrapped = x0 == nx - 1u;
}

// the taps of a thread's ZV voxels at (x, y, z[zz]) + o[zz]
template <int DIM, int ZV>
__device__ __forceinline__ void make_taps(const Geo& g, const Col& t, const float (&ox)[ZV],
                                          const float (&oy)[ZV], const float (&oz)[ZV],
                                          Tap (&tp)[ZV]) {
  uint64_t far = 0;   // lanes with an offset of a period or more, or a non-finite one
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    far |= lanes_far(ox[zz], g.nx) | lanes_far(oy[zz], g.ny);
    if (DIM == 3) far |= lanes_far(oz[zz], g.nz);
  }
  uint32_t x0[ZV], y0[ZV], z0[ZV];
  if (far == 0) {
#pragma unroll
    for (int zz = 0; zz < ZV; ++zz) {
      VOXEL(zz)
      x0[zz] = split_near(ox[zz], t.x, g.nx, tp[zz].wx);
      y0[zz] = split_near(oy[zz], t.y, g.ny, tp[zz].wy);
      tp[zz].wz = 0.0f;
      z0[zz] = 0;
      if (DIM == 3) z0[zz] = split_near(oz[zz], z, g.nz, tp[zz].wz);
    }
  } else {
#pragma unroll
    for (int zz = 0; zz < ZV; ++zz) {
      VOXEL(zz)
      x0[zz] = split_any(ox[zz], t.x, g.nx, g.inv_nx, tp[zz].wx);
      y0[zz] = split_any(oy[zz], t.y, g.ny, g.inv_ny, tp[zz].wy);
      tp[zz].wz = 0.0f;
      z0[zz] = 0;
      if (DIM == 3) z0[zz] = split_any(oz[zz], z, g.nz, g.inv_nz, tp[zz].wz);
    }
  }
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) tap_rows<DIM>(g, x0[zz], y0[zz], z0[zz], tp[zz]);
}

// Interpolated values of f at the ZV taps of a thread.  f[x0] and f[x0 + 1] of a row come in
// one 8-byte load: with the addresses of a real gather (runs of consecutive floats broken
// where the offset crosses a voxel) a wavefront's load occupies its compute unit's address path
// for about 16 cycles whatever its width, so two 4-byte loads per row cost more (state step
// 13.4 against 12.1 us, setup 60 against 47 us at 128^3).  Where x1 wraps to the row's start
// its value comes from a second load, issued only by waves in which some lane wraps (one
// wave-uniform branch after every row load of the thread is in flight) and, by lanes that do
// not wrap, past the end of the buffer, where the range check returns 0 without touching memory.
constexpr uint32_t kPastEnd = 0xFFFFFFFCu;   // >= the byte size of any field (< 2^32)

template <int DIM, int ZV, int POLICY = 0>
__device__ __forceinline__ void gather_zv(const Geo& g, Rsrc f, const Tap (&t)[ZV],
                                          float (&out)[ZV]) {
  constexpr int R = DIM == 3 ? 4 : 2;
  f2v v[ZV][R];
  uint64_t any = 0;
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    const uint32_t a[4] = {t[zz].a00, t[zz].a01, t[zz].a10, t[zz].a11};
#pragma unroll
    for (int r = 0; r < R; ++r)
      v[zz][r] = __builtin_bit_cast(f2v, __builtin_amdgcn_raw_buffer_load_b64(f, (int)a[r], 0, POLICY));
    any |= __builtin_amdgcn_ballot_w64(t[zz].wrapped);
  }
  if (any != 0) {
    const uint32_t back = ((uint32_t)g.nx - 1u) * 4u;
    float w[ZV][R];
#pragma unroll
    for (int zz = 0; zz < ZV; ++zz) {
      const uint32_t a[4] = {t[zz].a00, t[zz].a01, t[zz].a10, t[zz].a11};
#pragma unroll
      for (int r = 0; r < R; ++r) w[zz][r] = ld<POLICY>(f, t[zz].wrapped ? a[r] - back : kPastEnd, 0);
    }
#pragma unroll
    for (int zz = 0; zz < ZV; ++zz)
#pragma unroll
      for (int r = 0; r < R; ++r) v[zz][r].y = t[zz].wrapped ? w[zz][r] : v[zz][r].y;
  }
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    float rr[R];
#pragma unroll
    for (int r = 0; r < R; ++r) rr[r] = fmaf(t[zz].wx, v[zz][r].y - v[zz][r].x, v[zz][r].x);
    const float pa = fmaf(t[zz].wy, rr[1] - rr[0], rr[0]);
    if (DIM == 2) {
      out[zz] = pa;
    } else {
      const float pb = fmaf(t[zz].wy, rr[3] - rr[2], rr[2]);
      out[zz] = fmaf(t[zz].wz, pb - pa, pa);
    }
  }
}

// d-linear interpolation from the eight (four) corner values, as the step launches form it
template <int DIM>
__device__ __forceinline__ float blend(const float (&v)[8], float wx, float wy, float wz) {
  const float ra = fmaf(wx, v[1] - v[0], v[0]);
  const float rb = fmaf(wx, v[3] - v[2], v[2]);
  if constexpr (DIM == 2) return fmaf(wz, rb - ra, ra);
  const float pa = fmaf(wy, rb - ra, ra);
  const float rc = fmaf(wx, v[5] - v[4], v[4]);
  const float rd = fmaf(wx, v[7] - v[6], v[6]);
  const float pb = fmaf(wy, rd - rc, rc);
  return fmaf(wz, pb - pa, pa);
}

// X offsets of the thread's voxels (dim planes at X) as taps
template <int DIM, int ZV>
__device__ __forceinline__ void taps_x(const Geo& g, const Col& t, const float* X, Tap (&tp)[ZV]) {
  const size_t M = (size_t)g.M;
  const Rsrc r0 = field_rsrc(X, g), r1 = field_rsrc(X + M, g);
  const Rsrc r2 = field_rsrc(DIM == 3 ? X + 2 * M : X, g);
  float ox[ZV], oy[ZV], oz[ZV];
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    VOXEL(zz)
    ox[zz] = ld(r0, t.c, zo);
    oy[zz] = ld(r1, t.c, zo);
    oz[zz] = DIM == 3 ? ld(r2, t.c, zo) : 0.f;
  }
  make_taps<DIM, ZV>(g, t, ox, oy, oz, tp);
}

// (Y, a) of the thread's voxels as taps and factors
template <int DIM, int ZV>
__device__ __forceinline__ void taps_ya(const Geo& g, const Col& t, const float4* YA,
                                        Tap (&tp)[ZV], float (&aw)[ZV]) {
  float ox[ZV], oy[ZV], oz[ZV];
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    VOXEL(zz)
    const float4 o = ld_ya(g, YA, z, t);
    ox[zz] = o.x;
    oy[zz] = o.y;
    oz[zz] = o.z;
    aw[zz] = o.w;
  }
  make_taps<DIM, ZV>(g, t, ox, oy, oz, tp);
}

// The values of a thread's ZV voxels are computed first and stored afterwards, so no store
// sits between the voxels' loads.  Large grids store with the streaming hint (Geo::stream_out).
// Both forms are raw buffer stores that differ in their cache-policy immediate (bit 1: nt), so
// the compiler cannot merge the two branches into one plain store.
template <int ZV>
__device__ __forceinline__ void store_zv(const Geo& g, const Col& t, float* out,
                                         const float (&val)[ZV]) {
  const Rsrc rs = field_rsrc(out, g);
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    VOXEL(zz)
    if (!live) continue;
    const uint32_t v = __builtin_bit_cast(uint32_t, val[zz]);
    if (g.stream_out)
      __builtin_amdgcn_raw_buffer_store_b32(v, rs, (int)t.c, (int)zo, 2);
    else
      __builtin_amdgcn_raw_buffer_store_b32(v, rs, (int)t.c, (int)zo, 0);
  }
}

// ---------------------------------------------------------------------------------- setup
// Departure offsets X, Y and the reaction factor a at the thread's ZV voxels, with the gathers
// from global memory; v: dim planes of the velocity, then r.
template <int DIM, int ZV>
__device__ __forceinline__ void setup_voxels(const Geo& g, const Col& t, const float* __restrict__ v,
                                             float* __restrict__ X, float4* __restrict__ YA) {
  const size_t M = (size_t)g.M;
  const float s = g.dt * (float)g.nref;
  // the ZV voxels of the thread are computed first and stored afterwards (their gathers can
  // all be in flight)
  float u[3][ZV], nu[3][ZV];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const Rsrc vc = field_rsrc(v + (c < DIM ? c : 0) * M, g);
#pragma unroll
    for (int zz = 0; zz < ZV; ++zz) {
      VOXEL(zz)
      u[c][zz] = c < DIM ? s * ld(vc, t.c, zo) : 0.f;
      nu[c][zz] = -u[c][zz];
    }
  }
  Tap tf[ZV], tb[ZV];
  make_taps<DIM, ZV>(g, t, nu[0], nu[1], nu[2], tf);   // X = -(u + Interp(u, i - u)) / 2
  make_taps<DIM, ZV>(g, t, u[0], u[1], u[2], tb);      // Y = +(u + Interp(u, i + u)) / 2
  float xo[3][ZV], yo[3][ZV], av[ZV];
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) xo[2][zz] = yo[2][zz] = 0.f;
#pragma unroll
  for (int c = 0; c < DIM; ++c) {
    const Rsrc vc = field_rsrc(v + c * M, g);
    float gf[ZV], gb[ZV];
    gather_zv<DIM, ZV>(g, vc, tf, gf);
    gather_zv<DIM, ZV>(g, vc, tb, gb);
#pragma unroll
    for (int zz = 0; zz < ZV; ++zz) {
      xo[c][zz] = -0.5f * (u[c][zz] + s * gf[zz]);
      yo[c][zz] = 0.5f * (u[c][zz] + s * gb[zz]);
    }
  }
  // reaction factor of the adjoint along the backward characteristic (Heun)
  const Rsrc rr = field_rsrc(v + DIM * M, g);
  Tap ty[ZV];
  make_taps<DIM, ZV>(g, t, yo[0], yo[1], yo[2], ty);
  float R[ZV];
  gather_zv<DIM, ZV>(g, rr, ty, R);
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    VOXEL(zz)
    const float ri = ld(rr, t.c, zo);
    av[zz] = 1.0f + 0.5f * g.dt * (R[zz] + (1.0f + g.dt * R[zz]) * ri);
  }
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    VOXEL(zz)
    if (!live) continue;
    for (int c = 0; c < DIM; ++c) st(field_rsrc(X + c * M, g), t.c, zo, xo[c][zz]);
    st_ya(g, YA, z, t, make_float4(yo[0][zz], yo[1][zz], yo[2][zz], av[zz]));
  }
}

// Non-stationary step t_n -> t_{n+1}: the Heun characteristics take the velocity at both
// ends of the step: X = -(u1 + Interp(u0, i - u1)) / 2 (end point i at t_{n+1}),
// Y = +(u0 + Interp(u1, i + u0)) / 2 (start point i at t_n), R = Interp(r1, i + Y),
// a = 1 + dt/2 [R + (1 + dt R) r0].  With v0 = v1 these are the stationary formulas.
// (v1 follows v0, dim + 1 planes per node)
template <int DIM>
__device__ __forceinline__ void setup_voxel_ns(const Geo& g, const Col& t, const float* __restrict__ v0,
                                               float* __restrict__ X, float4* __restrict__ YA) {
  constexpr int ZV = 1;
  VOXEL(0)
  const size_t M = (size_t)g.M;
  const float* __restrict__ v1 = v0 + (DIM + 1) * M;
  const float s = g.dt * (float)g.nref;
  float u0[3][1] = {{0.f}, {0.f}, {0.f}}, u1[3] = {0.f, 0.f, 0.f}, nu1[3][1];
#pragma unroll
  for (int c = 0; c < DIM; ++c) {
    u0[c][0] = s * ld(field_rsrc(v0 + c * M, g), t.c, zo);
    u1[c] = s * ld(field_rsrc(v1 + c * M, g), t.c, zo);
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) nu1[c][0] = -u1[c];
  Tap tf[1], tb[1];
  make_taps<DIM, 1>(g, t, nu1[0], nu1[1], nu1[2], tf);
  make_taps<DIM, 1>(g, t, u0[0], u0[1], u0[2], tb);
  float xo[3] = {0.f, 0.f, 0.f}, yo[3][1] = {{0.f}, {0.f}, {0.f}};
#pragma unroll
  for (int c = 0; c < DIM; ++c) {
    float gf[1], gb[1];
    gather_zv<DIM, 1>(g, field_rsrc(v0 + c * M, g), tf, gf);
    gather_zv<DIM, 1>(g, field_rsrc(v1 + c * M, g), tb, gb);
    xo[c] = -0.5f * (u1[c] + s * gf[0]);
    yo[c][0] = 0.5f * (u0[c][0] + s * gb[0]);
  }
  Tap ty[1];
  make_taps<DIM, 1>(g, t, yo[0], yo[1], yo[2], ty);
  const float ri = ld(field_rsrc(v0 + DIM * M, g), t.c, zo);
  float Rv[1];
  gather_zv<DIM, 1>(g, field_rsrc(v1 + DIM * M, g), ty, Rv);
  const float R = Rv[0];
  const float a = 1.0f + 0.5f * g.dt * (R + (1.0f + g.dt * R) * ri);
  for (int c = 0; c < DIM; ++c) st(field_rsrc(X + c * M, g), t.c, zo, xo[c]);
  st_ya(g, YA, z, t, make_float4(yo[0][0], yo[1][0], yo[2][0], a));
}

// ------------------------------------------------------------------------------- stencils
// Central differences of the field at the thread's entry of plane zo (z neighbours zm, zp),
// scaled by N_ref / 2.
template <int DIM>
__device__ __forceinline__ void grad_c(const Geo& g, Rsrc f, const Col& t, uint32_t zo,
                                       uint32_t zm, uint32_t zp, float* gr) {
  gr[0] = (ld(f, t.xp, zo) - ld(f, t.xm, zo)) * g.half_nref;
  gr[1] = (ld(f, t.yp, zo) - ld(f, t.ym, zo)) * g.half_nref;
  if (DIM == 3) gr[2] = (ld(f, t.c, zp) - ld(f, t.c, zm)) * g.half_nref;
}

// dim planes of a vector field
template <int DIM>
struct Vec {
  Rsrc c[DIM];
};
template <int DIM>
__device__ __forceinline__ Vec<DIM> vec_rsrc(const float* f, const Geo& g) {
  Vec<DIM> v;
#pragma unroll
  for (int c = 0; c < DIM; ++c) v.c[c] = field_rsrc(f + c * (size_t)g.M, g);
  return v;
}

// central-difference divergence of lambda dv, unscaled: sum_j (lam dv_j)(i + e_j) - (i - e_j);
// lz: lambda at z - 1 and z + 1, dz: dv_z there
template <int DIM>
__device__ __forceinline__ float div_lam_dv(float lxm, float lxp, float lym, float lyp, float lzm, float lzp,
                                            const float (&d)[6]) {
  float s = lxp * d[1] - lxm * d[0];
  s += lyp * d[3] - lym * d[2];
  if constexpr (DIM == 3) s += lzp * d[5] - lzm * d[4];
  return s;
}

// f = -grad m . dv at the thread's ZV voxels
template <int DIM, int ZV>
__device__ __forceinline__ void source_f(const Geo& g, const Col& t, const float* m,
                                         const float* dv, float (&src)[ZV]) {
  const Rsrc rm = field_rsrc(m, g);
  const Vec<DIM> rd = vec_rsrc<DIM>(dv, g);
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) {
    VOXEL(zz)
    float gr[3];
    grad_c<DIM>(g, rm, t, zo, zm, zp, gr);
    float s = gr[0] * ld(rd.c[0], t.c, zo);
    s = fmaf(gr[1], ld(rd.c[1], t.c, zo), s);
    if constexpr (DIM == 3) s = fmaf(gr[2], ld(rd.c[2], t.c, zo), s);
    src[zz] = -s;
  }
}


// b = sum_n w_n lambda^n grad m^n over the stored adjoint and state planes (trapezoid in
// time), one pass after the backward transport.  A thread takes its ZV voxels of a z run for
// every time node in turn (node loop outside, voxel loop inside), so its z differences come
// from a sliding window of three planes held in registers: each m^n plane of the run is read
// once, plus one plane above and below, and the ZV voxels' loads of a node are in flight
// together.  With YA given, lambda^0 is not read: it is formed here as the last adjoint step
// would, a Interp(lambda^1, i + Y), with the same arithmetic (the caller then stops the
// backward transport at lambda^1; lambda^0 is needed by nothing but this sum).  The sum starts at
// what acc holds.  POLICY: of the loads of lambda.
template <int DIM, int ZV, int POLICY = 0>
__device__ __forceinline__ void body_sum(const Geo& g, const Col& t, const float* lam, const float* m,
                                         const float4* YA, float (&acc)[ZV][3]) {
  const size_t M = (size_t)g.M;
  for (int n = g.nt; n >= 0; --n) {   // in the order of the backward sweep (bl_sweep.hip)
    const float w = (n == 0 || n == g.nt) ? 0.5f * g.dt : g.dt;
    const Rsrc rm = field_rsrc(m + n * M, g);
    float l[ZV];
    if (n == 0 && YA != nullptr) {   // lambda^0 from lambda^1, as k_adj_step
      Tap tp[ZV];
      float aw[ZV];
      taps_ya<DIM, ZV>(g, t, YA, tp, aw);
      gather_zv<DIM, ZV>(g, field_rsrc(lam + M, g), tp, l);
#pragma unroll
      for (int zz = 0; zz < ZV; ++zz) l[zz] = aw[zz] * l[zz];
    } else {
      const Rsrc rl = field_rsrc(lam + n * M, g);
#pragma unroll
      for (int zz = 0; zz < ZV; ++zz) {
        VOXEL(zz)
        l[zz] = ld<POLICY>(rl, t.c, zo);
      }
    }
    float prev = 0.f, cur = 0.f;   // m at z - 1 and z
    if (DIM == 3) {                // the run starts below nz
      VOXEL(0)
      prev = ld(rm, t.c, zm);
      cur = ld(rm, t.c, zo);
    }
#pragma unroll
    for (int zz = 0; zz < ZV; ++zz) {
      VOXEL(zz)
      const float gx = (ld(rm, t.xp, zo) - ld(rm, t.xm, zo)) * g.half_nref;
      const float gy = (ld(rm, t.yp, zo) - ld(rm, t.ym, zo)) * g.half_nref;
      float gz = 0.f;
      if (DIM == 3) {
        // voxels past nz repeat the clamped last plane and are not stored
        const float next = ld(rm, t.c, zp);
        gz = (next - prev) * g.half_nref;
        prev = cur;
        cur = next;
      }
      const float wl = w * l[zz];
      acc[zz][0] = fmaf(wl, gx, acc[zz][0]);
      acc[zz][1] = fmaf(wl, gy, acc[zz][1]);
      if (DIM == 3) acc[zz][2] = fmaf(wl, gz, acc[zz][2]);
    }
  }
}
}  // namespace
}  // namespace bl
