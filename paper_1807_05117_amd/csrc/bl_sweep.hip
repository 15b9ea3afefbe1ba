// Every time step of a transport in one launch: the forward state, the incremental state and
// the adjoint with its body force, for grids whose tiles are resident on the device at once.
//
// As separate launches the steps of a 128^3 problem take 12 to 15 us each, of which the fields'
// bytes (from the last-level cache) need about 5: every launch loads the offsets again, forms
// the same interpolation taps from them, and pays its start, two dependent round trips and its
// tail.  Here a workgroup owns one tile of whole x rows for the entire sweep.
//   - The offsets are read and the taps formed once; addresses and weights (and dv, the reaction
//     factor, the body force) stay in registers for all steps.
//   - The tile's plane lies in LDS with the box of rows its taps reach; a step loads only the
//     rows of other tiles, gathers from LDS (a gather from global memory occupies the address
//     path about four times as long) and stores its voxels for the others.
//   - A tile waits only for the tiles its box touches, through one progress word per tile.
// Ten steps at 128^3 take 54 us for the state (121 as steps), 74 for the incremental state (162)
// and 78 for the adjoint with the body force (154); five steps at 96^3 20 us for the state and 27 for
// the adjoint (32 and 48).
// What is left is the gathers' and stencils' LDS reads and the exchange, about 2 us per step for
// a store, its progress word and the neighbours' loads.  The arithmetic per voxel is that of the
// step launches, and the results are bitwise the same.
//
// Memory order.  Within a sweep every plane is written once, by its tile's owner, with
// device-scope stores (sc1: written through to memory), and read by others with device-scope
// loads (sc1: not served from a stale L2 line).  The owner waits until its stores have
// completed (vmcnt 0, all waves: a barrier) before it publishes its progress; a reader issues
// its loads after it has seen the progress it needs.  Fields read by plain loads (offsets, m in
// the incremental and adjoint sweeps, dv) are complete before the launch.
//
// Progress.  Owners wait for each other, so they must all be resident.  The launch has at most
// one workgroup per compute unit, but nothing reserves the device for it: another stream's
// kernels may hold compute units, or another sweep may hold some while waiting for the rest.  So
// no wait is without end: a workgroup that has waited SweepRun::wait abandons the sweep for all its
// workgroups (the abort word).  Those of an abandoned sweep take (step, block of columns) tickets
// from one counter instead, in time order, each with a wait for all blocks of the step before.
// The holder of a ticket waits only for earlier tickets, and those are held by workgroups that are
// running, so this ends however many workgroups are resident.  It recomputes the sweep from its
// inputs; what was finished before is stored again with the same values.  Should a wait for earlier
// tickets not end all the same, it is given up and reported, and the call fails.
// A tile whose box does not fit the LDS (offsets of more than about four voxels per step at 128^3)
// abandons the sweep in the same way.  Either reason is reported to the host, which then takes the
// steps for a while (bl_lddmm.hip).
#include <algorithm>
#include <atomic>

#include "bl_field.h"

namespace bl {
namespace {

constexpr int kLdsBytes = 160 * 1024 - 512;
constexpr int kTabRows = 512;       // rows of other tiles a box may hold
constexpr int kXCDs = 8;
typedef __attribute__((address_space(3))) void* LdsPtr;
// words of a sweep's synchronisation area (kSweepWords): all zero before the launch
enum { SY_ABORT = 0, SY_TICKET = 16, SY_DONE = 48, SY_FLAGS = 320 };

__device__ __forceinline__ uint32_t ld_flag(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_flag(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The kernel's arguments, for code that is rarely run (reports, tickets): read again there, since as
// values they would be kept in scalar registers, which are short, for the whole sweep.  With those of
// the tickets kept, 61 (96^3) and 75 (128^3) of them were spilled to vector registers in the
// incremental sweep, 26 and 42 without; products took 121.2 and 199.8 us, now 117.2 and 198.4.
struct KernelArgs {
  Geo g;
  SweepPlan p;
  SweepArgs a;
};
typedef const __attribute__((address_space(4))) KernelArgs* KernelArgsPtr;
__device__ __forceinline__ KernelArgsPtr kernel_args() {
  KernelArgsPtr k = (KernelArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(k));
  return k;
}
// to memory that the host may read meanwhile
__device__ __forceinline__ void report(int word) {
  const KernelArgsPtr k = kernel_args();
  __hip_atomic_store(k->a.run.report + word, k->a.run.number, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ uint32_t add_flag(uint32_t* p) {
  return __hip_atomic_fetch_add(p, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev(Rsrc rs, uint32_t voff, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), rs, (int)voff, 0, kSC1);
}
// this wavefront's stores have reached their scope; no access moves across
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void keep_order() { asm volatile("" ::: "memory"); }

// The sweeps see a grid of x rows: row (y, z) is row z * ry + y.  In 2D the rows of the grid are
// the "planes" of one row each (ry = 1, rz = ny), so that one code runs along z.
template <int DIM>
struct Rows {
  int ry, rz;
  float inv_ry, inv_rz;
  uint32_t plane4;   // bytes of a plane
  // byte offset of plane z (nx ry < 2^23 and z < 2^11: a 24-bit multiply is exact)
  __device__ __forceinline__ uint32_t at(int z) const { return __umul24((uint32_t)z << 2, plane4 >> 2); }
  __device__ __forceinline__ explicit Rows(const Geo& g)
      : ry(DIM == 3 ? g.ny : 1), rz(DIM == 3 ? g.nz : g.ny),
        inv_ry(DIM == 3 ? g.inv_ny : 1.0f), inv_rz(DIM == 3 ? g.inv_nz : g.inv_ny),
        plane4((uint32_t)ry * (uint32_t)g.nx * 4u) {}
};

// a thread's voxels: x, row y, planes z0 .. z0 + R - 1, and the byte offset within a plane
struct Lane {
  bool on;
  int x, y, z0;
  uint32_t c;
};

template <int DIM, int R>
__device__ __forceinline__ Lane lane_of(const Geo& g, const SweepPlan& p, const Rows<DIM>& rw,
                                        int tile, uint32_t tid) {
  const uint32_t tz = fast_div((uint32_t)tile, p.div_nty), ty = (uint32_t)tile - tz * (uint32_t)p.nty;
  const uint32_t row = fast_div(tid, p.div_nx), gz = fast_div(row, p.div_ty);
  Lane t;
  t.x = (int)(tid - row * (uint32_t)g.nx);
  t.y = (int)(ty * (uint32_t)p.ty + (row - gz * (uint32_t)p.ty));
  t.z0 = (int)(tz * (uint32_t)p.tz + gz * (uint32_t)R);
  t.on = (int)gz < p.gz && t.y < rw.ry && t.z0 < rw.rz;
  if (!t.on) t.x = t.y = t.z0 = 0;   // addresses stay in bounds
  t.c = (uint32_t)t.y * (uint32_t)g.nx * 4u + (uint32_t)t.x * 4u;
  return t;
}
// a value the compiler may not carry over from another step: addresses formed from it are
// formed again (a run's addresses kept for all steps would not fit the registers)
__device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}
__device__ __forceinline__ int clampz(int z, int rz) { return z < rz ? z : rz - 1; }

constexpr bool is_inc(int kind) { return kind == SWEEP_INC || kind == SWEEP_INC_N; }
constexpr bool is_adj(int kind) { return kind == SWEEP_ADJ || kind == SWEEP_ADJ_N; }

// offsets along x, y, z of voxel (t, z)
typedef float f4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ Rsrc ya_rsrc(const SweepArgs& a, const Geo& g) {   // 16 M < 2^32 here
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float4*>(a.YA), (short)0,
                                           (int)((uint32_t)g.M * 16u), 0x00020000);
}
template <int KIND, int DIM>
__device__ __forceinline__ void load_offsets(const Geo& g, const Rows<DIM>& rw, const SweepArgs& a,
                                             const Lane& t, int z, float& ox, float& oy, float& oz) {
  const uint32_t off = t.c + rw.at(z);
  if constexpr (is_adj(KIND)) {
    const f4 o = __builtin_bit_cast(
        f4, __builtin_amdgcn_raw_buffer_load_b128(ya_rsrc(a, g), (int)(off * 4u), 0, 0));
    ox = o.x;
    oy = DIM == 3 ? o.y : 0.f;
    oz = DIM == 3 ? o.z : o.y;
  } else {
    ox = ld(field_rsrc(a.X, g), off, 0);
    const float o1 = ld(field_rsrc(a.X + (size_t)g.M, g), off, 0);
    oy = DIM == 3 ? o1 : 0.f;
    oz = DIM == 3 ? ld(field_rsrc(a.X + 2 * (size_t)g.M, g), off, 0) : o1;
  }
}
// the adjoint's reaction factor of voxel (t, z): by a load of its own, since the four values of one
// 16-byte load would be kept (and spilled) as a group
template <int DIM>
__device__ __forceinline__ float load_factor(const Geo& g, const Rows<DIM>& rw, const SweepArgs& a,
                                             const Lane& t, int z) {
  return ld(ya_rsrc(a, g), (t.c + rw.at(z)) * 4u + 12u, 0);
}

// The state's plane of the tile with one row around it in every direction, in LDS: rows of
// `pitch` floats in the order of the tile's rows, filled by direct loads to LDS.
struct Stencil {
  const float* m;       // the buffer
  int at;               // the thread's first voxel
  int xm, xp, sy, sz;   // to its neighbours along x (periodic), y and z
};

// central differences of the plane in LDS at the thread's R voxels (z neighbours from a sliding
// window), handed to f(r, gx, gy, gz); 2D: gy is the difference along the rows' axis
template <int DIM, int R, class F>
__device__ __forceinline__ void differences(const Geo& g, const Stencil& st, F&& f) {
  const float* m = st.m + fresh(st.at);
  float prev = m[-st.sz], cur = m[0];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    m = st.m + fresh(st.at + r * st.sz);
    const float next = m[st.sz];
    const float gx = (m[st.xp] - m[st.xm]) * g.half_nref;
    const float gz = (next - prev) * g.half_nref;
    if constexpr (DIM == 3) f(r, gx, (m[st.sy] - m[-st.sy]) * g.half_nref, gz);
    else f(r, gx, gz, 0.f);
    prev = cur;
    cur = next;
    if (R > 4 && (r & 1)) __builtin_amdgcn_sched_barrier(0);   // two voxels' reads at a time
  }
}

// -grad m . dv at the thread's R voxels
template <int DIM, int R>
__device__ __forceinline__ void source(const Geo& g, const Stencil& st, const float (&dv)[DIM][R],
                                       float (&src)[R]) {
  differences<DIM, R>(g, st, [&](int r, float gx, float gy, float gz) {
    float s = gx * dv[0][r];
    s = fmaf(gy, dv[1][r], s);
    if constexpr (DIM == 3) s = fmaf(gz, dv[2][r], s);
    src[r] = -s;
  });
}

template <int DIM, int R>
__device__ __forceinline__ void load_dv(const Geo& g, const Rows<DIM>& rw, const Lane& t, const float* dv,
                                        float (&out)[DIM][R]) {
#pragma unroll
  for (int c = 0; c < DIM; ++c)
#pragma unroll
    for (int r = 0; r < R; ++r)
      out[c][r] = ld(field_rsrc(dv + c * (size_t)g.M, g), t.c + rw.at(clampz(t.z0 + r, rw.rz)), 0);
}

// b += w_n lambda^n grad m^n
template <int DIM, int R>
__device__ __forceinline__ void add_node(const Geo& g, const Stencil& st, int n, const float (&lam)[R],
                                         float (&bx)[R], float (&by)[R], float (&bz)[R]) {
  const float w = (n == 0 || n == g.nt) ? 0.5f * g.dt : g.dt;
  differences<DIM, R>(g, st, [&](int r, float gx, float gy, float gz) {
    const float wl = w * lam[r];
    bx[r] = fmaf(wl, gx, bx[r]);
    by[r] = fmaf(wl, gy, by[r]);
    if constexpr (DIM == 3) bz[r] = fmaf(wl, gz, bz[r]);
  });
}
template <int DIM, int R>
__device__ __forceinline__ void store_b(const Geo& g, const Rows<DIM>& rw, const Lane& t, float* b,
                                        const float (&bx)[R], const float (&by)[R],
                                        const float (&bz)[R]) {
  const size_t M = (size_t)g.M;
  const Rsrc rx = field_rsrc(b, g), ry = field_rsrc(b + M, g), rz = field_rsrc(DIM == 3 ? b + 2 * M : b, g);
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (t.on && t.z0 + r < rw.rz) {
      const uint32_t at = t.c + rw.at(t.z0 + r);
      st(rx, at, 0, bx[r]);
      st(ry, at, 0, by[r]);
      if constexpr (DIM == 3) st(rz, at, 0, bz[r]);
    }
}

// step s of a sweep: the plane it reads and the plane it writes
template <int KIND>
__device__ __forceinline__ int plane_in(const Geo& g, int s) { return is_adj(KIND) ? g.nt - s : s; }
template <int KIND>
__device__ __forceinline__ int plane_out(const Geo& g, int s) { return is_adj(KIND) ? g.nt - s - 1 : s + 1; }

// the plane that step s reads
template <int KIND>
__device__ __forceinline__ const float* input(const Geo& g, const SweepArgs& a, int s) {
  const float* f = KIND == SWEEP_ADJ_N && s == 0 ? a.hs : a.planes;   // u^nt lies with hs
  return f + (size_t)plane_in<KIND>(g, s) * (size_t)g.M;
}
// the step's value from the interpolated one (src: of the Newton adjoint hs, and q is returned)
template <int KIND>
__device__ __forceinline__ float finish(const Geo& g, int s, float v, float src, float fac) {
  if constexpr (KIND == SWEEP_INC_N) return fmaf(g.dt, src, v);
  if constexpr (KIND == SWEEP_ADJ_N) return fmaf(fac, v, src);
  if constexpr (KIND == SWEEP_INC)
    return s + 1 < g.nt ? fmaf(g.dt, src, v) : g.lam_scale * fmaf(0.5f * g.dt, src, v);
  if constexpr (KIND == SWEEP_ADJ) return fac * v;
  return v;
}

// ------------------------------------------------------------- an abandoned sweep (tickets)
// A ticket is one step of one block of columns, done as the step launches do it.  What other
// workgroups of this launch have stored is read by device-scope loads (a fence in their place drops
// every line of the XCD's L2, workgroup after workgroup), and the finished blocks are counted in kDone
// words (256 additions to one word are made one by one).  Ten steps of six voxels at 128^3: a product
// 755 us, 1,330 with fences and one word, 390 in step launches.  (One that is late at once, of less
// than a voxel per step and with the host's copies: 885 us before arguments were read again, now 830.)
constexpr uint32_t kDone = 8, kDoneStride = 16;
template <int KIND, int DIM>
__device__ __forceinline__ void run_tickets(const Geo& g, const SweepArgs& a, int* sh) {
  constexpr int ZV = DIM == 3 ? 2 : 1;
  const size_t M = (size_t)g.M;
  const uint32_t nthr = blockDim.x, nq = ((uint32_t)(g.nx * g.ny) + nthr - 1u) / nthr;
  constexpr int kRuns = DIM == 3 ? 4 : 1;   // ZV planes at a time
  const uint32_t chunks = nq * (uint32_t)((g.nz + ZV * kRuns - 1) / (ZV * kRuns));
  const uint32_t stages = (uint32_t)g.nt + (KIND == SWEEP_STATE || KIND == SWEEP_ADJ_N ? 0u : 1u);
  __syncthreads();
  if (threadIdx.x == 0) sh[0] = (int)add_flag(a.run.sync + SY_TICKET);
  for (;;) {
    __syncthreads();
    const uint32_t k = (uint32_t)__builtin_amdgcn_readfirstlane(sh[0]);
    if (k >= stages * chunks) return;
    const uint32_t stage = k / chunks, chunk = k - stage * chunks, zb = chunk / nq;
    if (threadIdx.x < 64 && stage > 0) {   // every block of the stages before
      const uint32_t most = kernel_args()->a.run.polls;
      for (uint32_t polls = 0;; ++polls) {
        const uint32_t d = ld_flag(a.run.sync + SY_DONE + (threadIdx.x % kDone) * kDoneStride);
        uint32_t sum = 0;
#pragma unroll
        for (int i = 0; i < (int)kDone; ++i) sum += (uint32_t)__builtin_amdgcn_readlane((int)d, i);
        if (sum >= stage * chunks) break;
        if (polls >= most) {
          if (threadIdx.x == 0) report(SR_GAVE_UP);
          break;
        }
        __builtin_amdgcn_s_sleep(4);
      }
    }
    __syncthreads();
    Col t;
    const bool column = place(g, (chunk - zb * nq) * nthr, zb * kRuns, t);
    const int s = is_inc(KIND) ? (int)stage - 1 : (int)stage;   // incremental: -1 is t^0
#pragma unroll 1
    for (int k2 = 0; k2 < kRuns; ++k2, ++t.zb) {
      const bool on = column && t.zb * ZV < g.nz;
      if (on && KIND == SWEEP_ADJ && s == g.nt) {
        float acc[ZV][3] = {};
        body_sum<DIM, ZV, kSC1>(g, t, a.planes, a.m, nullptr, acc);
#pragma unroll
        for (int zz = 0; zz < ZV; ++zz) {
          VOXEL(zz)
          if (live)
            for (int c = 0; c < DIM; ++c) st(field_rsrc(a.b + c * M, g), t.c, zo, acc[zz][c]);
        }
      } else if (on) {
        float val[ZV], src[ZV] = {}, fac[ZV] = {};
        Tap tp[ZV];
        if constexpr (is_adj(KIND)) taps_ya<DIM, ZV>(g, t, a.YA, tp, fac);
        else taps_x<DIM, ZV>(g, t, a.X, tp);
        if constexpr (is_inc(KIND)) source_f<DIM, ZV>(g, t, a.m + (size_t)(s + 1) * M, a.dv, src);
        if (s < 0) {
#pragma unroll
          for (int zz = 0; zz < ZV; ++zz) val[zz] = 0.5f * g.dt * src[zz];
        } else {
          const int n = plane_out<KIND>(g, s);
          gather_zv<DIM, ZV, kSC1>(g, field_rsrc(input<KIND>(g, a, s), g), tp, val);
#pragma unroll
          for (int zz = 0; zz < ZV; ++zz) {
            VOXEL(zz)
            if constexpr (KIND == SWEEP_INC_N) {
              if (live) st(field_rsrc(a.dm + (size_t)n * M, g), t.c, zo, fmaf(0.5f * g.dt, src[zz], val[zz]));
            }
            if constexpr (KIND == SWEEP_ADJ_N) src[zz] = n > 0 ? ld(field_rsrc(a.hs + (size_t)n * M, g), t.c, zo) : 0.f;
            val[zz] = finish<KIND>(g, s, val[zz], src[zz], fac[zz]);
            if constexpr (KIND == SWEEP_ADJ_N) {   // b so far, in acc (others may still read b2)
              const float wn = n == 0 ? 0.5f * g.dt : g.dt;
              const float first = s == 0 ? 0.5f * g.dt * ld(field_rsrc(input<KIND>(g, a, 0), g), t.c, zo) : 0.f;
              float gr[3], g0[3];
              grad_c<DIM>(g, field_rsrc(a.m + (size_t)n * M, g), t, zo, zm, zp, gr);
              if (s == 0) grad_c<DIM>(g, field_rsrc(a.m + (size_t)g.nt * M, g), t, zo, zm, zp, g0);
              for (int c = 0; c < DIM; ++c) {
                float b = ld<kSC1>(field_rsrc(s == 0 ? a.b2.c[c] : a.acc + c * M, g), t.c, zo);
                if (s == 0) b = fmaf(first, g0[c], b);
                b = fmaf(wn * val[zz], gr[c], b);
                if (live) st_dev(field_rsrc((n == 0 ? a.b : a.acc) + c * M, g), t.c + zo, b);
              }
              val[zz] += src[zz];
            }
          }
        }
        const int n = s < 0 ? 0 : plane_out<KIND>(g, s);
        if (KIND == SWEEP_INC_N ? n < g.nt : KIND == SWEEP_ADJ_N ? n > 0 : true) {
          const Rsrc out = field_rsrc(a.planes + (size_t)n * M, g);
#pragma unroll
          for (int zz = 0; zz < ZV; ++zz) {
            VOXEL(zz)
            if (live) st_dev(out, t.c + zo, val[zz]);
          }
        }
      }
    }
    stores_done();
    __syncthreads();
    if (threadIdx.x == 0) {
      add_flag(a.run.sync + SY_DONE + (chunk % kDone) * kDoneStride);
      sh[0] = (int)add_flag(a.run.sync + SY_TICKET);
    }
  }
}

// --------------------------------------------------------------------------- the sweep
template <int KIND, int DIM, int R>
__global__ __launch_bounds__(1024) void k_sweep(Geo g, SweepPlan p, SweepArgs a) {
  extern __shared__ float4 lds4[];
  uint2* const tab = reinterpret_cast<uint2*>(lds4);                  // [kTabRows] rows of other tiles
  uint32_t* const mtab = reinterpret_cast<uint32_t*>(tab + kTabRows); // [kTabRows] the stencil's rows
  float* const S = reinterpret_cast<float*>(mtab + kTabRows);         // the tile's box of rows
  __shared__ int sh[8];   // 0-3 box, 4 abandoned, 5 by this tile, 6 how long it waits
  constexpr bool kStencil = KIND != SWEEP_STATE;
  const Rows<DIM> rw(g);
  const size_t M = (size_t)g.M;
  const uint32_t nb = gridDim.x;   // a multiple of kXCDs: every XCD owns a contiguous run of tiles
  const int tile = (int)((blockIdx.x % kXCDs) * (nb / kXCDs) + blockIdx.x / kXCDs);
  const uint32_t tid = threadIdx.x, nthr = blockDim.x;
  const bool shared = p.tiles > 1;   // a single tile waits for nobody
  uint32_t* const flags = a.run.sync + SY_FLAGS;

  if (tile >= p.tiles) return;
  {
    const Lane t = lane_of<DIM, R>(g, p, rw, tile, tid);
    const int tz = (int)fast_div((uint32_t)tile, p.div_nty), ty = tile - tz * p.nty;
    const int y0 = ty * p.ty, z0 = tz * p.tz;
    const int ey = min(p.ty, rw.ry - y0), ez = min(p.tz, rw.rz - z0);   // the tile's extent
    const uint32_t n4 = (uint32_t)(g.nx + 3) / 4u;   // 16-byte entries of a row
    const uint32_t row4 = (uint32_t)g.nx * 4u;

    float wx[R], wy[R], wz[R];
#pragma unroll
    for (int r = 0; r < R; ++r)
      load_offsets<KIND, DIM>(g, rw, a, t, clampz(t.z0 + r, rw.rz), wx[r], wy[r], wz[r]);
    if (tid < 4) sh[tid] = (tid & 1) ? -(1 << 28) : (1 << 28);
    if (tid == 4) sh[4] = shared && ld_flag(a.run.sync + SY_ABORT) != 0;   // abandoned already
    if (tid == 5) sh[5] = 0;
    if (tid == 6) sh[6] = (int)a.run.wait;

    // the state's plane around the tile, for the stencils: where its rows come from
    float* const mbuf = S + p.box_floats;
    const uint32_t mrow = DIM == 3 ? (uint32_t)p.ty + 2u : 1u;
    const uint32_t mrows = mrow * ((uint32_t)p.tz + 2u), mentries = mrows * n4;
    if constexpr (kStencil) {
      for (uint32_t i = tid; i < mrows; i += nthr) {
        const uint32_t zi = DIM == 3 ? fast_div(i, p.div_ty2) : i;
        const int gy = DIM == 3 ? wrap(y0 - 1 + (int)(i - zi * mrow), rw.ry, rw.inv_ry) : 0;
        const int gz = wrap(min(z0 - 1 + (int)zi, rw.rz), rw.rz, rw.inv_rz);
        mtab[i] = (uint32_t)gz * rw.plane4 + (uint32_t)gy * row4;
      }
    }
    auto load_m = [&](int n) {   // asynchronous: complete after stores_done() and a barrier
      if constexpr (kStencil) {
        const Rsrc rm = field_rsrc(a.m + (size_t)n * M, g);
        for (uint32_t e = tid; e < mentries; e += nthr) {
          const uint32_t row = fast_div(e, p.div_n4);
          __builtin_amdgcn_raw_ptr_buffer_load_lds(
              rm, (LdsPtr)(mbuf + (size_t)__builtin_amdgcn_readfirstlane(e) * 4), 16,
              (int)(mtab[row] + (e - row * n4) * 16u), 0, 0, 0);
        }
      }
    };
    Stencil st;
    {
      const int pm = (int)n4 * 4, zl = t.on ? t.z0 - z0 : 0, yl = t.on ? t.y - y0 : 0;
      st.sy = pm;
      st.sz = (int)mrow * pm;
      st.xm = t.x == 0 ? g.nx - 1 : -1;
      st.xp = t.x + 1 == g.nx ? 1 - g.nx : 1;
      st.m = mbuf;
      st.at = (zl + 1) * st.sz + (DIM == 3 ? (yl + 1) * pm : 0) + t.x;
    }

    // taps: cells and weights.  Along an axis that the tile spans whole, cells are periodic and the
    // box has one more row, a copy of row 0; else they count on from the tile's.
    const bool fully = DIM == 3 && p.nty == 1, fullz = p.ntz == 1;
    int ax[R], ay[R], az[R];
    int ylo = 1 << 28, yhi = -(1 << 28), zlo = 1 << 28, zhi = -(1 << 28);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int z = clampz(t.z0 + r, rw.rz);
      ax[r] = (int)split_any(wx[r], t.x, g.nx, g.inv_nx, wx[r]);
      ay[r] = 0;
      if constexpr (DIM == 3) {
        wy[r] = fabsf(wy[r]) <= 1048576.0f ? wy[r] : 0.f;
        const float f = floorf(wy[r]);
        wy[r] -= f;
        ay[r] = t.y + (int)f;
        if (fully) ay[r] = wrap(ay[r], rw.ry, rw.inv_ry);
      }
      wz[r] = fabsf(wz[r]) <= 1048576.0f ? wz[r] : 0.f;
      const float f = floorf(wz[r]);
      wz[r] -= f;
      az[r] = z + (int)f;
      if (fullz) az[r] = wrap(az[r], rw.rz, rw.inv_rz);
      if (t.on) {
        ylo = min(ylo, ay[r]);
        yhi = max(yhi, ay[r]);
        zlo = min(zlo, az[r]);
        zhi = max(zhi, az[r]);
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      ylo = min(ylo, __shfl_xor(ylo, o));
      yhi = max(yhi, __shfl_xor(yhi, o));
      zlo = min(zlo, __shfl_xor(zlo, o));
      zhi = max(zhi, __shfl_xor(zhi, o));
    }
    __syncthreads();
    if ((tid & 63) == 0) {
      atomicMin(&sh[0], ylo);
      atomicMax(&sh[1], yhi);
      atomicMin(&sh[2], zlo);
      atomicMax(&sh[3], zhi);
    }
    __syncthreads();
    if constexpr (is_inc(KIND)) load_m(0);
    if constexpr (is_adj(KIND)) load_m(g.nt);
    // the box: the tile's own rows and every row its taps reach
    ylo = DIM == 2 || fully ? 0 : min(sh[0], y0);
    yhi = DIM == 2 ? 0 : fully ? rw.ry : max(sh[1] + 1, y0 + ey - 1);
    zlo = fullz ? 0 : min(sh[2], z0);
    zhi = fullz ? rw.rz : max(sh[3] + 1, z0 + ez - 1);
    const int by = yhi - ylo + 1, bz = zhi - zlo + 1;
    const int pitch = p.pitch, ps = by * pitch;
    // rows of other tiles: whole slabs below and above in z, strips beside in y
    const int hz0 = z0 - zlo, hz1 = fullz ? 0 : zhi - (z0 + ez - 1);
    const int hy0 = y0 - ylo, hy1 = DIM == 2 || fully ? 0 : yhi - (y0 + ey - 1);
    const int slab = (hz0 + hz1) * by, hy = hy0 + hy1, sz = fullz ? bz : ez;
    const long long nrows = (long long)(hz0 + hz1) * by + (long long)hy * sz;
    const bool fits = (long long)by * bz * pitch <= p.box_floats && nrows <= kTabRows;
    bool bail = sh[4] != 0 || !fits;
    if (!fits && tid == 0) {
      st_flag(a.run.sync + SY_ABORT, 1u);
      report(SR_LEFT);
    }
    const int rows = bail ? 0 : (int)nrows;
    const uint32_t entries = (uint32_t)rows * n4;
    for (int i = (int)tid; i < rows; i += (int)nthr) {
      int b, c;   // box row: b planes, c rows from its corner
      if (i < slab) {
        const int q = i / by;
        c = i - q * by;
        b = q < hz0 ? q : q + ez;
      } else {
        const int q = (i - slab) / hy, k = i - slab - q * hy;
        b = (fullz ? 0 : hz0) + q;
        c = k < hy0 ? k : k + ey;
      }
      const int gy = DIM == 3 ? wrap(ylo + c, rw.ry, rw.inv_ry) : 0, gz = wrap(zlo + b, rw.rz, rw.inv_rz);
      const uint32_t owner = (uint32_t)(gz / p.tz) * (uint32_t)p.nty + (uint32_t)(gy / p.ty);
      tab[i] = make_uint2((uint32_t)gz * rw.plane4 + (uint32_t)gy * row4,
                          (uint32_t)((b * by + c) * pitch) | owner << 16);
    }
    // first corner of each tap, in floats of the box (< 2^16), two to a register
    uint32_t ad[(R + 1) / 2] = {};
#pragma unroll
    for (int r = 0; r < R; ++r)
      ad[r / 2] |= (uint32_t)(bail || !t.on ? 0 : __mul24(__mul24(az[r] - zlo, by) + (ay[r] - ylo), pitch) + ax[r])
                   << 16 * (r & 1);
    const int own = bail || !t.on ? 0 : __mul24(__mul24(t.z0 - zlo, by) + (t.y - ylo), pitch) + t.x;
    const int run = t.on && !bail ? min(R, rw.rz - t.z0) : 0;   // the thread's voxels
    // the thread's voxels into the box, with the copies of column 0 and of spanned axes' row 0
    auto put = [&](const float (&v)[R]) {
      const int base = fresh(own);
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (r < run) S[base + r * ps] = v[r];
      if (t.x == 0) {
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (r < run) S[base + r * ps + g.nx] = v[r];
      }
      if (!fullz && !fully) return;
      const bool cy = fully && t.y == 0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (r >= run) continue;
        auto row = [&](int i) {
          S[i] = v[r];
          if (t.x == 0) S[i + g.nx] = v[r];
        };
        const int i = base + r * ps;
        const bool cz = fullz && t.z0 + r == 0;
        if (cz) row(i + rw.rz * ps);
        if (cy) row(i + rw.ry * pitch);
        if (cz && cy) row(i + rw.rz * ps + rw.ry * pitch);
      }
    };
    auto publish = [&](uint32_t v) {   // after the barrier that follows stores_done()
      if (tid == 0 && shared) st_flag(flags + tile * 16, v);
    };
    auto store = [&](int plane, const float (&v)[R]) {
      const Rsrc out = field_rsrc(a.planes + (size_t)plane * M, g);
      const int z = fresh(t.z0);
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (r < run) st_dev(out, t.c + rw.at(z + r), v[r]);
    };

    float val[R], fx[R] = {}, fy[R] = {}, fz[R] = {}, dv[is_inc(KIND) ? DIM : 1][R] = {};
    float src[R] = {}, fac[R] = {};
    if constexpr (KIND == SWEEP_ADJ_N) {
      auto start = [&](int c, float (&f)[R]) {
#pragma unroll
        for (int r = 0; r < R; ++r)
          f[r] = ld(field_rsrc(a.b2.c[c], g), t.c + rw.at(clampz(t.z0 + r, rw.rz)), 0);
      };
      start(0, fx);
      start(1, fy);
      if constexpr (DIM == 3) start(2, fz);
    }
    if constexpr (is_adj(KIND)) {
#pragma unroll
      for (int r = 0; r < R; ++r) fac[r] = load_factor<DIM>(g, rw, a, t, clampz(t.z0 + r, rw.rz));
    }
    if constexpr (is_inc(KIND)) {
      load_dv<DIM, R>(g, rw, t, a.dv, dv);
      stores_done();
      __syncthreads();
      source<DIM, R>(g, st, dv, val);
#pragma unroll
      for (int r = 0; r < R; ++r) val[r] = 0.5f * g.dt * val[r];
      store(0, val);
      put(val);
      __syncthreads();   // every stencil of m^0 is done
      load_m(1);
      stores_done();
      __syncthreads();
      if (!bail) publish(1u);   // (an abandoned tile has stored nothing)
      source<DIM, R>(g, st, dv, src);
    } else {
      const Rsrc in = field_rsrc(input<KIND>(g, a, 0), g);
#pragma unroll
      for (int r = 0; r < R; ++r) val[r] = ld(in, t.c + rw.at(clampz(t.z0 + r, rw.rz)), 0);
      put(val);
      if constexpr (is_adj(KIND)) stores_done();
      __syncthreads();
      if constexpr (is_adj(KIND)) add_node<DIM, R>(g, st, g.nt, val, fx, fy, fz);
    }
    // an entry of the other tiles' rows: where it comes from, and floats of the box | tile << 16
    auto entry = [&](uint32_t e, uint32_t& from, uint32_t& to) {
      const uint32_t row = fast_div(e, p.div_n4), c4 = e - row * n4;
      const uint2 q = tab[row];
      from = q.x + c4 * 16u;
      to = q.y + c4 * 4u;
      return c4;
    };

    for (int s = 0; s < g.nt && !bail; ++s) {
      const Rsrc in = field_rsrc(input<KIND>(g, a, s), g);
      // progress the other tiles must show: this step's input plane (the first one of the state
      // and adjoint sweeps is there before the launch)
      const uint32_t need = (uint32_t)s + (is_inc(KIND) ? 1u : 0u);
      bool out_of_time = false;
      auto wait = [&](uint32_t ta, uint32_t tb) {
        if (need == 0) return;
        const uint32_t* fa = flags + (ta >> 16) * 16u;
        const uint32_t* fb = flags + (tb >> 16) * 16u;
        uint64_t start = 0;
        const uint32_t patience = (uint32_t)sh[6];   // (read while the first look is on its way)
        for (uint32_t it = 1;; ++it) {
          const uint32_t pa = ld_flag(fa), pb = ld_flag(fb);
          if (__builtin_amdgcn_ballot_w64(min(pa, pb) < need) == 0) break;
          if ((it & 15u) == 0 || patience == 0) {
            const uint64_t now = __builtin_amdgcn_s_memrealtime();
            if (start == 0) start = now;
            if (now - start >= patience) {
              st_flag(a.run.sync + SY_ABORT, 1u);
              sh[5] = 1;
            }
            if (ld_flag(a.run.sync + SY_ABORT) != 0) {
              out_of_time = true;
              break;
            }
          }
        }
        keep_order();
      };
      auto load4 = [&](uint32_t from) {
        return __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(in, (int)from, 0, kSC1));
      };
      auto put4 = [&](uint32_t to, uint32_t c4, f4 v) {
        float* d = S + (to & 0xffffu);
        const int left = g.nx - (int)c4 * 4;   // floats of the row from this entry on
        if (left >= 4) {
          *reinterpret_cast<f4*>(d) = v;
        } else {
          d[0] = v.x;
          if (left > 1) d[1] = v.y;
          if (left > 2) d[2] = v.z;
        }
        if (c4 == 0) d[g.nx] = v.x;
      };
      for (uint32_t e = tid; e < entries && !out_of_time; e += 2 * nthr) {
        uint32_t from0, from1, to0, to1;
        const uint32_t c0 = entry(e, from0, to0), c1 = entry(e + nthr < entries ? e + nthr : e, from1, to1);
        wait(to0, to1);
        if (out_of_time) break;
        const f4 v0 = load4(from0), v1 = load4(from1);
        put4(to0, c0, v0);
        put4(to1, c1, v1);
      }
      if (out_of_time) sh[4] = 1;
      __syncthreads();
      if (sh[4] != 0) {
        if (tid == 0 && sh[5] != 0) report(SR_LATE);
        bail = true;
        break;
      }
      const int n = plane_out<KIND>(g, s);
      // the plane of the next stencils: the last ones that used the buffer are done
      if constexpr (is_inc(KIND)) {
        if (s + 2 <= g.nt) load_m(s + 2);
      }
      if constexpr (is_adj(KIND)) load_m(n);
      if constexpr (KIND == SWEEP_ADJ_N) {
        const Rsrc rh = field_rsrc(a.hs + (size_t)n * M, g);
        const int z = fresh(t.z0);
#pragma unroll
        for (int r = 0; r < R; ++r) src[r] = n > 0 ? ld(rh, t.c + rw.at(clampz(z + r, rw.rz)), 0) : 0.f;
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const uint32_t pair = (uint32_t)fresh((int)ad[r / 2]);
        const float* q = S + (r & 1 ? pair >> 16 : pair & 0xffffu);
        const float* q2 = q + ps;
        float v[8];
        v[0] = q[0];
        v[1] = q[1];
        if constexpr (DIM == 3) {
          v[2] = q[pitch];
          v[3] = q[pitch + 1];
          v[4] = q2[0];
          v[5] = q2[1];
          v[6] = q2[pitch];
          v[7] = q2[pitch + 1];
        } else {
          v[2] = q2[0];
          v[3] = q2[1];
        }
        const float at = blend<DIM>(v, wx[r], wy[r], wz[r]);
        if constexpr (KIND == SWEEP_INC_N) {
          const uint32_t o = t.c + rw.at(fresh(t.z0) + r);
          if (r < run) ::bl::st(field_rsrc(a.dm + (size_t)n * M, g), o, 0, fmaf(0.5f * g.dt, src[r], at));
        }
        val[r] = finish<KIND>(g, s, at, src[r], fac[r]);
        // few voxels' corners at a time: more would not fit the registers
        if (R > 4 && (KIND == SWEEP_STATE ? (r & 1) : true)) __builtin_amdgcn_sched_barrier(0);
      }
      const bool more = s + 1 < g.nt;
      if constexpr (KIND == SWEEP_ADJ_N) {   // q^n meets grad m^n, u^n = q^n + hs^n goes on
#pragma unroll
        for (int r = 0; r < R; ++r) src[r] += val[r];
        if (n > 0) store(n, src);
      } else if (KIND == SWEEP_INC_N ? more : KIND != SWEEP_ADJ || n > 0 || a.keep0) {
        store(n, val);
      }
      if (more || is_adj(KIND)) {
        __syncthreads();   // every gather of this step is done
        if (more) put(KIND == SWEEP_ADJ_N ? src : val);
        stores_done();
        __syncthreads();
        if (more) publish((uint32_t)s + (is_inc(KIND) ? 2u : 1u));
      }
      if constexpr (is_inc(KIND)) {
        if (more) source<DIM, R>(g, st, dv, src);
      }
      if constexpr (is_adj(KIND)) add_node<DIM, R>(g, st, n, val, fx, fy, fz);
    }
    if (bail) {   // the same for every thread of the block
      const KernelArgsPtr k = kernel_args();
      run_tickets<KIND, DIM>(*(const Geo*)&k->g, *(const SweepArgs*)&k->a, sh);
    } else if constexpr (is_adj(KIND)) {
      store_b<DIM, R>(g, rw, t, a.b, fx, fy, fz);
    }
  }
}

template <int KIND, int DIM, int R>
void launch_r(const Geo& g, const SweepPlan& p, const SweepArgs& a, hipStream_t s) {
  // more than 64 KB of LDS is asked for once per kernel and device
  static std::atomic<uint64_t> asked{0};
  int dev = 0;
  (void)hipGetDevice(&dev);
  const uint64_t bit = uint64_t(1) << (dev & 63);
  if (!(asked.load(std::memory_order_relaxed) & bit)) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_sweep<KIND, DIM, R>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    asked.fetch_or(bit, std::memory_order_relaxed);
  }
  const unsigned nb = (unsigned)((p.tiles + kXCDs - 1) / kXCDs * kXCDs);
  hipLaunchKernelGGL((k_sweep<KIND, DIM, R>), dim3(nb), dim3((unsigned)p.threads), kLdsBytes, s, g, p, a);
}
template <int KIND, int DIM>
void launch_dim(const Geo& g, const SweepPlan& p, const SweepArgs& a, hipStream_t s) {
  switch (p.run) {
    case 1: launch_r<KIND, DIM, 1>(g, p, a, s); break;
    case 2: launch_r<KIND, DIM, 2>(g, p, a, s); break;
    case 4: launch_r<KIND, DIM, 4>(g, p, a, s); break;
    case 6: launch_r<KIND, DIM, 6>(g, p, a, s); break;
    default: launch_r<KIND, DIM, 8>(g, p, a, s); break;
  }
}
template <int KIND>
void launch_kind(const Geo& g, const SweepPlan& p, const SweepArgs& a, hipStream_t s) {
  if (g.dim == 3) launch_dim<KIND, 3>(g, p, a, s);
  else launch_dim<KIND, 2>(g, p, a, s);
}

}  // namespace

// Tiles of whole x rows, ty rows by tz = gz run planes, one workgroup of nx ty gz threads each,
// every thread with `run` planes.  Of the shapes with at most one tile per compute unit, at most
// 1024 threads, at most 8 planes per thread (registers) and a box that fits the LDS with two rows
// to spare on every side, the one with the least estimated time per step: a constant for the
// exchange with other tiles (2.0 us, 0.6 for a single tile), 0.021 us per wavefront-voxel of a
// tile and half that per wavefront-load of its neighbours' rows.  Measured per step (us): 4.8
// (128^3, 8 x 8 rows: 128 wavefront-voxels), 3.2 (96^3, 6 x 6: 54), 3.3 (64^3, 8 x 8: 64), 2.3
// (64^3, 4 x 4: 16).
SweepPlan sweep_plan(const Geo& g, int compute_units) {
  SweepPlan best{};
  if (g.M >= (int64_t(1) << 28)) return best;   // 32-bit byte offsets of 16-byte voxels
  const int ry = g.dim == 3 ? g.ny : 1, rz = g.dim == 3 ? g.nz : g.ny;
  const int pitch = (g.nx + 3) / 4 * 4 + 4;
  const int lds = (kLdsBytes - kTabRows * (int)(sizeof(uint2) + sizeof(uint32_t))) / 4;
  const int most = std::min(compute_units, kSweepTiles);
  double cost = 1e30;
  for (int run : {1, 2, 4, 6, 8})
    for (int ty = 1; ty <= ry && g.nx * ty <= 1024; ++ty)
      for (int gz = 1; g.nx * ty * gz <= 1024; ++gz) {
        const int tz = gz * run;
        const int threads = (g.nx * ty * gz + 63) / 64 * 64;
        const int entries = (g.dim == 3 ? ty + 2 : 1) * (tz + 2) * ((g.nx + 3) / 4);   // of the stencil's rows
        if ((g.dim == 3 ? ty + 2 : 1) * (tz + 2) > kTabRows) continue;
        const int nty = (ry + ty - 1) / ty, ntz = (rz + tz - 1) / tz;
        if ((long long)nty * ntz > most) continue;
        const int hy = nty > 1 ? 4 : 1, hz = ntz > 1 ? 4 : 1;
        // the box floats that are left beside the stencil's rows (whole wavefronts of entries)
        const int box = lds - (entries + 63) / 64 * 256;
        if ((long long)(g.dim == 3 ? ty + hy : 1) * (tz + hz) * pitch > box) continue;
        const int waves = threads / 64;
        const double halo = ((ntz > 1 ? 2.0 * (ty + 2) : 0.0) + (nty > 1 ? 2.0 * tz : 0.0)) * g.nx / 256.0;
        const double c = (nty * ntz > 1 ? 2.0 : 0.6) + 0.021 * waves * run + 0.01 * halo;
        if (c < cost) {
          cost = c;
          best.run = run;
          best.ty = ty;
          best.gz = gz;
          best.tz = tz;
          best.nty = nty;
          best.ntz = ntz;
          best.threads = threads;
          best.box_floats = box;
        }
        if (tz >= rz) break;
      }
  if (best.run == 0) return best;   // no such shape: the steps are launched one by one
  best.tiles = best.nty * best.ntz;
  best.pitch = pitch;
  best.div_nx = make_div((uint32_t)g.nx);
  best.div_ty = make_div((uint32_t)best.ty);
  best.div_ty2 = make_div((uint32_t)best.ty + 2u);
  best.div_nty = make_div((uint32_t)best.nty);
  best.div_n4 = make_div((uint32_t)((g.nx + 3) / 4));
  return best;
}

void sweep_state(const Geo& g, const SweepPlan& p, const float* X, float* m, const SweepRun& r,
                 hipStream_t s) {
  SweepArgs a{};
  a.X = X;
  a.planes = m;
  a.run = r;
  launch_kind<SWEEP_STATE>(g, p, a, s);
}
void sweep_inc(const Geo& g, const SweepPlan& p, const float* X, const float* m, const float* dv,
               float* t, const SweepRun& r, hipStream_t s) {
  SweepArgs a{};
  a.X = X;
  a.planes = t;
  a.m = m;
  a.dv = dv;
  a.run = r;
  launch_kind<SWEEP_INC>(g, p, a, s);
}
void sweep_adj(const Geo& g, const SweepPlan& p, const float4* YA, const float* m, float* lam,
               float* b, int keep0, const SweepRun& r, hipStream_t s) {
  SweepArgs a{};
  a.YA = YA;
  a.planes = lam;
  a.m = m;
  a.b = b;
  a.keep0 = keep0;
  a.run = r;
  launch_kind<SWEEP_ADJ>(g, p, a, s);
}

void sweep_inc_n(const Geo& g, const SweepPlan& p, const float* X, const float* m, const float* dv,
                 float* t, float* dm, const SweepRun& r, hipStream_t s) {
  SweepArgs a{};
  a.X = X;
  a.planes = t;
  a.m = m;
  a.dv = dv;
  a.dm = dm;
  a.run = r;
  launch_kind<SWEEP_INC_N>(g, p, a, s);
}
void sweep_adj_n(const Geo& g, const SweepPlan& p, const float4* YA, const float* m, const float* hs,
                 const BodyStart& b2, float* acc, float* u, float* b, const SweepRun& r, hipStream_t s) {
  SweepArgs a{};
  a.YA = YA;
  a.planes = u;
  a.m = m;
  a.hs = hs;
  a.b2 = b2;
  a.acc = acc;
  a.b = b;
  a.run = r;
  launch_kind<SWEEP_ADJ_N>(g, p, a, s);
}

}  // namespace bl
