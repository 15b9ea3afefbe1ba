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
#include "bl_internal.h"

namespace bl {
namespace {

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

// quotient by a host constant (FastDiv), exact for n < 2^31
__device__ __forceinline__ uint32_t fast_div(uint32_t n, const FastDiv& d) {
  return (__umulhi(n, d.m) + n * d.one) >> d.s;
}

// the thread's column entry and the byte offsets of its stencil within a plane (periodic)
struct Col {
  int x, y;
  uint32_t q;                 // y nx + x
  uint32_t c, xm, xp, ym, yp; // byte offsets of the entry and its x and y neighbours
  int zb;                     // the block's first plane / ZV
  uint32_t plane4;            // bytes of a plane
};

__device__ __forceinline__ bool locate(const Geo& g, int zv, Col& t) {
  const uint32_t nb = gridDim.x;            // multiple of kXCD
  const uint32_t b = blockIdx.x;
  const uint32_t tile = (b % kXCD) * (nb / kXCD) + b / kXCD;
  const uint32_t zb = fast_div(tile, g.div_nqb);
  const uint32_t q0 = (tile - zb * (uint32_t)g.nqb) * kTB;
  if ((int)zb * zv >= g.nz) return false;
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
__device__ __forceinline__ float ld(Rsrc rs, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)voff, (int)soff, 0));
}
__device__ __forceinline__ void st(Rsrc rs, uint32_t voff, uint32_t soff, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), rs, (int)voff, (int)soff, 0);
}
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

template <int DIM, int ZV>
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
      v[zz][r] = __builtin_bit_cast(f2v, __builtin_amdgcn_raw_buffer_load_b64(f, (int)a[r], 0, 0));
    any |= __builtin_amdgcn_ballot_w64(t[zz].wrapped);
  }
  if (any != 0) {
    const uint32_t back = ((uint32_t)g.nx - 1u) * 4u;
    float w[ZV][R];
#pragma unroll
    for (int zz = 0; zz < ZV; ++zz) {
      const uint32_t a[4] = {t[zz].a00, t[zz].a01, t[zz].a10, t[zz].a11};
#pragma unroll
      for (int r = 0; r < R; ++r) w[zz][r] = ld(f, t[zz].wrapped ? a[r] - back : kPastEnd, 0);
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
template <int DIM, int ZV>
__global__ __launch_bounds__(kTB) void k_setup(Geo g, const float* __restrict__ v,
                                               float* __restrict__ X,
                                               float4* __restrict__ YA) {
  BL_BATCH_Z1(g.bat)
  BL_AT_NN(v, g.bat);
  BL_AT_NN(X, g.bat);
  BL_AT_NN(YA, g.bat);
  COLUMN
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
// (every step n of the time grid in one launch: n = blockIdx.y, v0 = V[n], v1 = V[n + 1] with
// dim + 1 planes per node, X[n], YA[n])
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
  VOXEL(0)
  const size_t M = (size_t)g.M;
  const size_t n = blockIdx.y;
  const float* __restrict__ v0 = V + n * (DIM + 1) * M;
  const float* __restrict__ v1 = v0 + (DIM + 1) * M;
  float* __restrict__ X = Xall + n * DIM * M;
  float4* __restrict__ YA = YAall + n * M;
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

// b = sum_n w_n lambda^n grad m^n over the stored adjoint and state planes (trapezoid in
// time), one pass after the backward transport.  A thread takes its ZV voxels of a z run for
// every time node in turn (node loop outside, voxel loop inside), so its z differences come
// from a sliding window of three planes held in registers: each m^n plane of the run is read
// once, plus one plane above and below, and the ZV voxels' loads of a node are in flight
// together.  With YA given, lambda^0 is not read: it is formed here as the last adjoint step
// would, a Interp(lambda^1, i + Y), with the same arithmetic (the caller then stops the
// backward transport at lambda^1; lambda^0 is needed by nothing but this sum).
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
#pragma unroll
  for (int zz = 0; zz < ZV; ++zz) acc[zz][0] = acc[zz][1] = acc[zz][2] = 0.f;
  // lambda^0 of the thread's voxels: from lambda^1 (as k_adj_step), or its stored plane
  float l[ZV];
  if (YA != nullptr) {
    Tap tp[ZV];
    float aw[ZV];
    taps_ya<DIM, ZV>(g, t, YA, tp, aw);
    gather_zv<DIM, ZV>(g, field_rsrc(lam + M, g), tp, l);
#pragma unroll
    for (int zz = 0; zz < ZV; ++zz) l[zz] = aw[zz] * l[zz];
  } else {
    const Rsrc rl = field_rsrc(lam, g);
#pragma unroll
    for (int zz = 0; zz < ZV; ++zz) {
      VOXEL(zz)
      l[zz] = ld(rl, t.c, zo);
    }
  }
  for (int n = 0; n <= g.nt; ++n) {
    const float w = (n == 0 || n == g.nt) ? 0.5f * g.dt : g.dt;
    const Rsrc rm = field_rsrc(m + n * M, g);
    if (n > 0) {
      const Rsrc rl = field_rsrc(lam + n * M, g);
#pragma unroll
      for (int zz = 0; zz < ZV; ++zz) {
        VOXEL(zz)
        l[zz] = ld(rl, t.c, zo);
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
  DISPATCH_GATHER(k_setup, TR_SETUP, g, v, X, YA);
}
void setup_ns(const Geo& g, const float* V, float* X, float4* YA, int steps, hipStream_t s) {
  const dim3 grid = batch_grid(dim3(gather_grid(g, 1).x, (unsigned)steps), g.bat);
  if (g.dim == 3)
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
