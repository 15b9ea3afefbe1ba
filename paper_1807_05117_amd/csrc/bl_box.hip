// Departure points of 3D grids with the neighbourhood of a tile in LDS.
//
// The setup interpolates seven values per voxel: the three velocity components at i - u and at
// i + u, and r at i + Y.  A gather from global memory occupies its compute unit's address path
// for about 16 cycles per wavefront instruction whatever its width, 28 of them per voxel here;
// the same corners from LDS take a quarter of that, and the kernel is then bound by the issue
// of vector instructions (about 400 per voxel, 70 us at 181x211x179).  Per launch, gathers from
// global memory and from LDS (us): 44.3 and 31.7 at 128^3, 152 and 105 at 181x211x179, 403 and
// 225 at 256^3 (of which the bytes take 145), 22.9 and 19.6 at 96^3, 9.8 and 12.8 at 64^3, where
// there are too few tiles.
//
// A workgroup takes a tile of up to 64 x by 8 y by 4 z voxels, four of them per thread along z,
// and loads boxes around it (the tile and the halo its taps reach, periodic) straight to LDS,
// one field at a time.  No workgroup waits for another.
#include "bl_field.h"

namespace bl {
namespace {

typedef __attribute__((address_space(3))) void* LdsPtr;
constexpr int kTX = 64, kTY = 8;        // the tile's extents in x (at most) and y
constexpr int kBoxDepth = 4;            // and in z
constexpr int kBoxRows = 256, kBoxCols = 96;
constexpr int kBoxFloats = 9216;        // holds a halo of two voxels on every side
constexpr int kBoxKeep = 8;             // all of a thread's elements of a box with a halo of one

// tile of this workgroup and the thread's column in it
struct Tile {
  int x0, y0, z0;       // first voxel
  int xs, ys;           // the thread's column within the tile
  bool on;              // it lies in the grid
  Col t;                // its place in a plane (x, y, q, c, plane4)
};
__device__ __forceinline__ bool tile_of(const Geo& g, const BoxPlan& p, Tile& k) {
  const uint32_t nb = gridDim.x;   // a multiple of kXCD: every XCD sweeps one slab
  const uint32_t tile = (blockIdx.x % kXCD) * (nb / kXCD) + blockIdx.x / kXCD;
  if (tile >= (uint32_t)p.tiles) return false;
  const uint32_t row = fast_div(tile, p.div_ntx), tz = fast_div(row, p.div_nty);
  k.x0 = (int)(tile - row * (uint32_t)p.ntx) * p.sw;
  k.y0 = (int)(row - tz * (uint32_t)p.nty) * kTY;
  k.z0 = (int)tz * kBoxDepth;
  k.ys = (int)fast_div(threadIdx.x, p.div_sw);
  k.xs = (int)threadIdx.x - k.ys * p.sw;
  k.t.x = k.x0 + k.xs;
  k.t.y = k.y0 + k.ys;
  k.on = k.ys < kTY && k.t.x < g.nx && k.t.y < g.ny;
  if (!k.on) {   // addresses stay in the tile
    k.t.x = k.x0;
    k.t.y = k.y0;
    k.xs = k.ys = 0;
  }
  k.t.q = (uint32_t)k.t.y * (uint32_t)g.nx + (uint32_t)k.t.x;
  k.t.c = k.t.q * 4u;
  k.t.plane4 = (uint32_t)g.nx * (uint32_t)g.ny * 4u;
  return true;
}

// A box of a field around the tile: `bx` columns, `by` rows, `bz` planes from (x0 - hx, ...) on.
// Element e of it comes from row[e / bx] + col[e % bx] of the field's buffer; a thread keeps
// the addresses of its first K elements for the next field.
struct Box {
  int bx, by, bz, hx, hy, hz, n;
  float inv_bx;
};
struct BoxTables {
  uint32_t row[kBoxRows], col[kBoxCols];
};
__device__ __forceinline__ Box box_of(const BoxPlan& p, int hx, int hy, int hz) {
  Box b;
  b.hx = hx;
  b.hy = hy;
  b.hz = hz;
  b.bx = p.sw + 2 * hx;
  b.by = kTY + 2 * hy;
  b.bz = kBoxDepth + 2 * hz;
  b.n = b.bx * b.by * b.bz;
  b.inv_bx = 1.0f / (float)b.bx;
  return b;
}
__device__ __forceinline__ bool box_fits(const Box& b) {
  return b.n <= kBoxFloats && b.by * b.bz <= kBoxRows && b.bx <= kBoxCols;
}
// before the first load of a box; ends with a barrier
__device__ __forceinline__ void box_tables(const Geo& g, const Tile& k, const Box& b, BoxTables& tb) {
  const uint32_t plane4 = k.t.plane4, row4 = (uint32_t)g.nx * 4u;
  const float inv = 1.0f / (float)b.by;
  for (int i = (int)threadIdx.x; i < b.by * b.bz; i += (int)blockDim.x) {
    const int bz = (int)(((float)i + 0.5f) * inv), by = i - bz * b.by;
    tb.row[i] = (uint32_t)wrap(k.z0 - b.hz + bz, g.nz, g.inv_nz) * plane4 +
                (uint32_t)wrap(k.y0 - b.hy + by, g.ny, g.inv_ny) * row4;
  }
  for (int i = (int)threadIdx.x; i < b.bx; i += (int)blockDim.x)
    tb.col[i] = (uint32_t)wrap(k.x0 - b.hx + i, g.nx, g.inv_nx) * 4u;
  __syncthreads();
}
__device__ __forceinline__ uint32_t box_address(const Box& b, const BoxTables& tb, int e) {
  const int row = (int)(((float)e + 0.5f) * b.inv_bx);   // exact: e < 2^15, bx < 2^7
  return tb.row[row] + tb.col[e - row * b.bx];
}
__device__ __forceinline__ void box_addresses(const Box& b, const BoxTables& tb, uint32_t (&at)[kBoxKeep]) {
#pragma unroll
  for (int i = 0; i < kBoxKeep; ++i) {
    const int e = (int)threadIdx.x + i * (int)blockDim.x;
    const uint32_t a = box_address(b, tb, min(e, b.n - 1));
    at[i] = e < b.n ? a : kPastEnd;   // past the end reads 0
  }
}
// asynchronous: complete after box_wait.  S has room for the kept elements of all threads.
__device__ __forceinline__ void box_load(Rsrc f, const Box& b, const BoxTables& tb,
                                         const uint32_t (&at)[kBoxKeep], float* S) {
  const int nthr = (int)blockDim.x, first = __builtin_amdgcn_readfirstlane((int)threadIdx.x);
#pragma unroll
  for (int i = 0; i < kBoxKeep; ++i)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(f, (LdsPtr)(S + first + i * nthr), 4, (int)at[i], 0, 0, 0);
  for (int e0 = first + kBoxKeep * nthr; e0 < b.n; e0 += nthr) {
    const int e = e0 + (int)(threadIdx.x & 63u);
    if (e < b.n)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(f, (LdsPtr)(S + e0), 4, (int)box_address(b, tb, e), 0, 0, 0);
  }
}
__device__ __forceinline__ void box_wait() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}

// ---------------------------------------------------------------------------------- setup
// halo that holds the taps at offsets of magnitude up to the float with these bits (-1: none does)
__device__ __forceinline__ int halo(uint32_t bits) {
  const float m = __builtin_bit_cast(float, bits);
  return m < 64.0f ? (int)m + 1 : -1;   // NaN, infinities: -1
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o));
  return v;
}

// a copy that the compiler may not share between uses: what is formed from it (cells, weights) is
// formed again instead of being held in registers for the next field
__device__ __forceinline__ float fresh(float v) {
  asm volatile("" : "+v"(v));
  return v;
}
// interpolated value at offset (ox, oy, oz) from element `base` of the box
__device__ __forceinline__ float box_value(const float* S, const Box& b, int base, float ox, float oy,
                                           float oz) {
  ox = fresh(ox);
  oy = fresh(oy);
  oz = fresh(oz);
  const float fx = floorf(ox), fy = floorf(oy), fz = floorf(oz);
  const int ps = b.bx * b.by;
  const float* q = S + base + (int)fmaf(fz, (float)ps, fmaf(fy, (float)b.bx, fx));
  const float v[8] = {q[0], q[1], q[b.bx], q[b.bx + 1], q[ps], q[ps + 1], q[ps + b.bx], q[ps + b.bx + 1]};
  return blend<3>(v, ox - fx, oy - fy, oz - fz);
}

// NS: one time step of a non-stationary velocity per blockIdx.y, with the velocities of both its
// ends (see k_setup_ns).  The velocity components take turns in one box, so that three workgroups
// fit a compute unit; taps are formed again for each (a thread's cells and weights for all of its
// voxels would not fit the registers).  All components in LDS at once, with two workgroups, and
// two boxes by turns, with the next component's loads ahead, were slower (181x211x179: 117 and
// 113 against 105 us).  A tile whose offsets do not fit the box (more than about two voxels per
// time step) takes its gathers from global memory.
template <bool NS>
__global__ __launch_bounds__(kTX * kTY, 6) void k_setup_box(Geo g, BoxPlan p, const float* __restrict__ V,
                                                            float* __restrict__ Xall,
                                                            float4* __restrict__ YAall) {
  BL_BATCH_Z1(g.bat)
  BL_AT_NN(V, g.bat);
  BL_AT_NN(Xall, g.bat);
  BL_AT_NN(YAall, g.bat);
  __shared__ float S[kBoxFloats];
  __shared__ BoxTables tb;
  __shared__ uint32_t top[6];
  constexpr int R = kBoxDepth, ZV = R;
  const size_t M = (size_t)g.M, n = NS ? blockIdx.y : 0;
  const float* const v0 = V + n * 4 * M;
  const float* const v1 = NS ? v0 + 4 * M : v0;
  float* const X = Xall + n * 3 * M;
  float4* const YA = YAall + n * M;
  Tile k;
  if (!tile_of(g, p, k)) return;
  Col& t = k.t;
  const float s = g.dt * (float)g.nref;
  if (threadIdx.x < 6) top[threadIdx.x] = 0u;

  // u at the start (backward characteristic) and end (forward) of the step
  float u0[3][R], u1[3][NS ? R : 1], ri[R];
  uint32_t big[3] = {0u, 0u, 0u};
  t.zb = k.z0 / R;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const Rsrc a = field_rsrc(v0 + c * M, g), b = field_rsrc(v1 + c * M, g);
#pragma unroll
    for (int zz = 0; zz < R; ++zz) {
      VOXEL(zz)
      u0[c][zz] = s * ld(a, t.c, zo);
      if constexpr (NS) u1[c][zz] = s * ld(b, t.c, zo);
    }
  }
#pragma unroll
  for (int zz = 0; zz < R; ++zz) {
    VOXEL(zz)
    ri[zz] = ld(field_rsrc(v0 + 3 * M, g), t.c, zo);
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
#pragma unroll
    for (int zz = 0; zz < R; ++zz) {
      big[c] = max(big[c], __builtin_bit_cast(uint32_t, fabsf(u0[c][zz])));
      if constexpr (NS) big[c] = max(big[c], __builtin_bit_cast(uint32_t, fabsf(u1[c][zz])));
    }
    big[c] = wave_max(big[c]);
  }
  __syncthreads();
  if ((threadIdx.x & 63) == 0)
    for (int c = 0; c < 3; ++c) atomicMax(&top[c], big[c]);
  __syncthreads();
  const int hx = halo(top[0]), hy = halo(top[1]), hz = halo(top[2]);
  const Box b = box_of(p, hx, hy, hz);
  bool fits = min(hx, min(hy, hz)) >= 0 && box_fits(b);
  if (fits) {
    uint32_t at[kBoxKeep];
    box_tables(g, k, b, tb);
    box_addresses(b, tb, at);
    const int ps = b.bx * b.by, base = (b.hz * b.by + k.ys + b.hy) * b.bx + k.xs + b.hx;
    float yo[3][R];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      __syncthreads();   // the box's readers are done
      box_load(field_rsrc(v0 + c * M, g), b, tb, at, S);
      box_wait();
      const Rsrc rx = field_rsrc(X + c * M, g);
#pragma unroll
      for (int zz = 0; zz < R; ++zz) {   // X = -(u + Interp(u, i - u)) / 2
        VOXEL(zz)
        constexpr int kU = NS ? 1 : 0;
        const float ex = kU ? u1[0][zz * kU] : u0[0][zz], ey = kU ? u1[1][zz * kU] : u0[1][zz],
                    ez = kU ? u1[2][zz * kU] : u0[2][zz], ec = kU ? u1[c][zz * kU] : u0[c][zz];
        const float xo = -0.5f * (ec + s * box_value(S, b, base + zz * ps, -ex, -ey, -ez));
        if (live && k.on) st(rx, t.c, zo, xo);
        if (zz & 1) __builtin_amdgcn_sched_barrier(0);   // two voxels' corners at a time
      }
      if constexpr (NS) {
        __syncthreads();
        box_load(field_rsrc(v1 + c * M, g), b, tb, at, S);
        box_wait();
      }
      big[c] = 0u;
#pragma unroll
      for (int zz = 0; zz < R; ++zz) {   // Y = (u + Interp(u, i + u)) / 2
        yo[c][zz] = 0.5f * (u0[c][zz] + s * box_value(S, b, base + zz * ps, u0[0][zz], u0[1][zz], u0[2][zz]));
        big[c] = max(big[c], __builtin_bit_cast(uint32_t, fabsf(yo[c][zz])));
        if (zz & 1) __builtin_amdgcn_sched_barrier(0);
      }
      big[c] = wave_max(big[c]);
      if ((threadIdx.x & 63) == 0) atomicMax(&top[3 + c], big[c]);
    }
    __syncthreads();
    // r at i + Y, whose box is rarely larger than the velocity's
    const int rx = halo(top[3]), ry = halo(top[4]), rz = halo(top[5]);
    const Box br = box_of(p, max(rx, hx), max(ry, hy), max(rz, hz));
    fits = min(rx, min(ry, rz)) >= 0 && box_fits(br);
    if (fits) {
      if (br.n != b.n) {
        box_tables(g, k, br, tb);
        box_addresses(br, tb, at);
      }
      box_load(field_rsrc(v1 + 3 * M, g), br, tb, at, S);
      box_wait();
      const int pr = br.bx * br.by, base_r = (br.hz * br.by + k.ys + br.hy) * br.bx + k.xs + br.hx;
#pragma unroll
      for (int zz = 0; zz < R; ++zz) {
        VOXEL(zz)
        const float Rv = box_value(S, br, base_r + zz * pr, yo[0][zz], yo[1][zz], yo[2][zz]);
        const float a = 1.0f + 0.5f * g.dt * (Rv + (1.0f + g.dt * Rv) * ri[zz]);
        if (live && k.on) st_ya(g, YA, z, t, make_float4(yo[0][zz], yo[1][zz], yo[2][zz], a));
        if (zz & 1) __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  if (!fits && k.on) {
#pragma unroll 1
    for (int zz = 0; zz < R; ++zz) {
      t.zb = k.z0 + zz;
      if (t.zb >= g.nz) break;
      if constexpr (NS) setup_voxel_ns<3>(g, t, v0, X, YA);
      else setup_voxels<3, 1>(g, t, v0, X, YA);
    }
  }
}

BoxPlan box_plan(const Geo& g) {
  BoxPlan p;
  p.ntx = (g.nx + kTX - 1) / kTX;
  p.sw = (g.nx + p.ntx - 1) / p.ntx;
  p.nty = (g.ny + kTY - 1) / kTY;
  p.tiles = p.ntx * p.nty * ((g.nz + kBoxDepth - 1) / kBoxDepth);
  p.div_ntx = make_div((uint32_t)p.ntx);
  p.div_nty = make_div((uint32_t)p.nty);
  p.div_sw = make_div((uint32_t)p.sw);
  return p;
}

dim3 box_grid(const Geo& g, const BoxPlan& p, int ny) {
  return batch_grid(dim3((unsigned)((p.tiles + kXCD - 1) / kXCD * kXCD), (unsigned)ny), g.bat);
}
dim3 box_block(const BoxPlan& p) { return dim3((unsigned)((p.sw * kTY + 63) / 64 * 64)); }

}  // namespace

void setup_box(const Geo& g, const float* v, float* X, float4* YA, hipStream_t s) {
  const BoxPlan p = box_plan(g);
  BL_LAUNCH((k_setup_box<false>), box_grid(g, p, 1), box_block(p), 0, s, g, p, v, X, YA);
}
void setup_box_ns(const Geo& g, const float* V, float* X, float4* YA, int steps, hipStream_t s) {
  const BoxPlan p = box_plan(g);
  BL_LAUNCH((k_setup_box<true>), box_grid(g, p, steps), box_block(p), 0, s, g, p, V, X, YA);
}

}  // namespace bl
