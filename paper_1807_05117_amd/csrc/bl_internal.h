// Internal declarations shared by the HIP translation units of the library.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <cstddef>
#include <cstdint>
#include <type_traits>

namespace bl {

// Several problems of one shape in one launch (the batched serving engine).  Problem p's
// device buffers lie p * stride bytes after problem 0's (one arena per problem, equal
// layouts), the launch's gridDim.z is `count` times the single-problem launch's, and the
// blocks of problem p return at once when gate[p * gate_stride] reads 0.  The default (one
// problem, no gate) is the plain launch.  Twiddle tables are read from problem 0 (they depend
// on the grid and band only, which every problem of a batch shares).
struct Batch {
  int64_t stride = 0;
  const int* gate = nullptr;
  int64_t gate_stride = 0;   // ints between consecutive problems' gates
  int count = 1;
};

// problem index of this block, and blockIdx.z within the problem's own launch
__device__ __forceinline__ int batch_pair(const Batch& b) {
  const int zper = b.count > 1 ? (int)gridDim.z / b.count : 0;
  return zper > 0 ? (int)blockIdx.z / zper : 0;
}
__device__ __forceinline__ int batch_bz(const Batch& b, int pair) {
  return (int)blockIdx.z - pair * ((int)gridDim.z / b.count);
}
__device__ __forceinline__ bool batch_gated_off(const Batch& b, int pair) {
  return b.gate != nullptr && b.gate[(size_t)pair * b.gate_stride] == 0;
}
// problem pair's copy of a buffer of problem 0 (null stays null).  Byte-pointer arithmetic,
// not an integer round trip: the compiler then still knows the result points to global memory
// (global and scalar loads; through an integer it can only use flat loads).
template <class T>
__device__ __forceinline__ T* batch_ptr(T* p, const Batch& b, int pair) {
  using Byte = typename std::conditional<std::is_const<T>::value, const char, char>::type;
  return p == nullptr ? p : reinterpret_cast<T*>(reinterpret_cast<Byte*>(p) + (int64_t)pair * b.stride);
}
template <class T>
__device__ __forceinline__ T* batch_ptr_nn(T* p, const Batch& b, int pair) {
  using Byte = typename std::conditional<std::is_const<T>::value, const char, char>::type;
  return reinterpret_cast<T*>(reinterpret_cast<Byte*>(p) + (int64_t)pair * b.stride);
}
inline dim3 batch_grid(dim3 d, const Batch& b) {
  d.z *= (unsigned)b.count;
  return d;
}
// kernel prologue: the block's problem, gated-off problems return; BL_AT shifts a buffer
#define BL_BATCH(bt)                                  \
  const int bpair_ = ::bl::batch_pair(bt);            \
  if (::bl::batch_gated_off(bt, bpair_)) return;
// the same for launches of one z per problem: no division
#define BL_BATCH_Z1(bt)               \
  const int bpair_ = (int)blockIdx.z; \
  if (::bl::batch_gated_off(bt, bpair_)) return;
// (a buffer that is never null: no test)
#define BL_AT_NN(p, bt) p = ::bl::batch_ptr_nn(p, bt, bpair_)
#define BL_AT(p, bt) p = ::bl::batch_ptr(p, bt, bpair_)

// Sum (MAX: maximum) of one double per thread of a 1D block of 256 threads, in a fixed order:
// within each 64-lane wavefront by shuffles (offsets 32, 16, ..., 1; lane 0 ends with its
// wavefront's value), then the four wavefront values in order by thread 0, which alone returns
// the result.  Every thread of the block must call it (it has two barriers).
template <bool MAX>
__device__ __forceinline__ double block_reduce_256(double v) {
  __shared__ double part[4];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double w = __shfl_down(v, (unsigned)o, 64);
    v = MAX ? fmax(v, w) : v + w;
  }
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0) {
    r = part[0];
#pragma unroll
    for (int w = 1; w < 4; ++w) r = MAX ? fmax(r, part[w]) : r + part[w];
  }
  __syncthreads();   // part may be reused by a following reduction of the same kernel
  return r;
}

// Kernel timing for the benchmark: a pair of HIP events that the next launch through
// BL_LAUNCH on the calling host thread records at its kernel's own start and end (the
// dispatch's timestamps, no gap to a neighbouring launch).  set_launch_events(e) arms it;
// BL_LAUNCH takes and clears it.
struct LaunchEvents {
  hipEvent_t start = nullptr, stop = nullptr;
};
void set_launch_events(LaunchEvents* e);
LaunchEvents* take_launch_events();
#define BL_LAUNCH(KERNEL, GRID, BLOCK, SHMEM, STREAM, ...)                                   \
  do {                                                                                     \
    if (::bl::LaunchEvents* ev_ = ::bl::take_launch_events())                              \
      hipExtLaunchKernelGGL(KERNEL, GRID, BLOCK, SHMEM, STREAM, ev_->start, ev_->stop, 0,  \
                            __VA_ARGS__);                                                  \
    else                                                                                   \
      hipLaunchKernelGGL(KERNEL, GRID, BLOCK, SHMEM, STREAM, __VA_ARGS__);                  \
  } while (0)

// Quotient by a constant d as one high multiply and a shift: n / d = umulhi(n, m) >> s for
// every n < 2^31 (d = 1: m = s = 0 and the quotient is n * one).  With s = ceil(log2 d) - 1 and m = ceil(2^(32 + s) / d) the
// excess e = m d - 2^(32 + s) is below d <= 2^(s + 1), so n e < 2^(32 + s) and the floor is exact.
struct FastDiv {
  uint32_t m = 0, s = 0, one = 0;
};
inline FastDiv make_div(uint32_t d) {
  FastDiv f;
  f.one = d < 2 ? 1 : 0;
  if (d < 2) return f;
  uint32_t s = 0;
  while ((uint64_t(2) << s) < d) ++s;
  f.s = s;
  f.m = (uint32_t)(((uint64_t(1) << (32 + s)) + d - 1) / d);
  return f;
}

// Geometry and weights of one problem, passed by value to every kernel.
struct Geo {
  int dim;            // 2 or 3
  int nx, ny, nz;     // grid (nz == 1 in 2D)
  int kx, ky, kz;     // band (kz == 1 in 2D)
  int kzh;            // stored non-negative kz planes: 1 in 2D, kz/2 in 3D
  int kz0;            // band index of kz = 0: 0 in 2D, kz/2 in 3D
  int nt;             // time steps
  int nref;           // max grid size (voxel size 1/nref)
  int64_t M;          // voxels
  int64_t B;          // band entries per component (kx*ky*kz)
  float dt;           // 1/nt
  float half_nref;    // nref/2 (central difference scale)
  float lam_scale;    // -2/sigma^2
  float inv_nx, inv_ny, inv_nz;   // 1/n per axis (periodic index wrap)
  int nqb;            // blocks of kTransportBlock column entries in a plane (transports)
  FastDiv div_nqb, div_nx;
  int gamma;          // 1: incompressible flow (velocities projected divergence-free)
  int newton;         // 1: full Newton Hessian products (else Gauss-Newton)
  int nodes;          // band velocity fields: 1 (stationary) or nt + 1 (one per time node)
  int deform;         // 1: deformation state equation (band displacement of the inverse map)
  int px, py, pz;     // product grid of the truncated convolutions (deformation method)
  // 1: the transports store their outputs with the streaming (non-temporal) hint.  Set when the
  // nine grid fields an incremental step touches exceed the 256 MiB last-level cache: there
  // the hint speeds the steps up, below it the next step's reads of the output would miss.
  int stream_out;
  // launch shapes per kernel class (TR_*): voxels per thread along z of the transports, the setup's
  // form, the z-chunk multiplier of the iota z stage, and one without effect (TR_IOTA_XY).  Every
  // choice computes bitwise the same values.
  int zv[8];
  // several problems of this shape in one launch (default: one)
  Batch bat;
};

constexpr int kTransportBlock = 256;   // threads of a transport block

// kernel classes of the launch shapes (Geo::zv)
enum { TR_STATE = 0, TR_INC, TR_ADJ, TR_FORCE, TR_SETUP, TR_IOTA_Z, TR_IOTA_XY, TR_CLASSES };

// Work buffers and twiddle tables of the band<->grid transforms.
constexpr int kYG = 4;     // y outputs per thread in the iota y stage
constexpr int kJG = 8;     // ky outputs per thread in the pi y stage
constexpr int kZP = 64;    // padded row length of the z twiddle table
constexpr int kU = 8;      // loads in flight per thread in the contraction loops
constexpr int kUY = 16;    // loads in flight per thread in the pi y stage

// Twiddle tables are zero-padded so that every chunk of kU loads stays in bounds:
// padded extents: kx, nx rounded up to 8, ny to 32, ky to kJG, nz to 128.
struct DftPlan {
  float2* tw_x = nullptr;   // [kxp][nx]   exp(+2 pi i kx x / nx), kx = j - Kx/2; zero rows >= Kx
  float2* tw_xT = nullptr;  // [nxp][kx]   the same, transposed; zero rows >= nx
  float2* tw_y = nullptr;   // [kyp][nyp]  exp(+2 pi i ky y / ny); zero outside
  float2* tw_yT = nullptr;  // [nyp][kyp]  the same, transposed
  float2* tw_zT = nullptr;  // [nzp][kZP]  exp(+2 pi i h z / nz), h = 0..kzh-1; zero outside
  int kxp = 0, nxp = 0, kyp = 0, nyp = 0, nzp = 0;
  float2* bufA = nullptr;   // stage buffers, each C_max * kzh * max(ky*nx, ny*nx) complex, C_max
                            // the widest transform (4, or every node of a non-stationary field)
  float2* bufB = nullptr;
  // split hi/lo BF16 twiddle matrices of the mixed-precision z stages (FP32 mode: unused)
  unsigned short* wi_bf16 = nullptr;   // 2 nzp32 mixed_kp     iota: (hi, lo)
  unsigned short* wp_bf16 = nullptr;   // 64 mixed_jt nzp16    pi:   (hi, lo)
  int nzp32 = 0, nzp16 = 0;
  int mixed = 0;
};

constexpr int kMaxKzh = 64;       // register arrays of the z stages: kz <= 128
constexpr int kRedBlocks = 512;   // partial sums per deterministic FP64 reduction

// ---- transforms on the matrix cores (bl_dft_mfma.hip): z stages; x and y stages of bands with at
// most 128 ky (iota) or kx (pi), else false
void iota_z_mfma(const Geo& g, const DftPlan& p, const float2* F2, float* out, int C, hipStream_t s);
void pi_z_mfma(const Geo& g, const DftPlan& p, const float* f, int C, float2* G, hipStream_t s);
bool iota_xy_mfma(const Geo& g, const DftPlan& p, const float2* band, int C, float2* F2, hipStream_t s);
// the derivatives along every axis of dim band fields (i q_j band_i as component i dim + j), with
// the symbols of g on the grid gp
bool iota_xy_deriv_mfma(const Geo& g, const Geo& gp, const DftPlan& p, const float2* band, float2* F2,
                        hipStream_t s);
bool pi_yx_mfma(const Geo& g, const DftPlan& p, const float2* G, int C, float2* P, hipStream_t s);

// ---- transforms (bl_dft.hip)
// out: C planes
void iota(const Geo& g, const DftPlan& p, const float2* band, int C, float* out, hipStream_t s);
// pi without the 1/M scale: P[c][h][ky][kx] for h = 0..kzh-1 (half spectrum)
void pi_half(const Geo& g, const DftPlan& p, const float* grid, int C, float2* P, hipStream_t s);
// the stages separately: iota = iota_xy (band -> p.bufB) then iota_z (p.bufB -> out);
// pi_half = pi_z (grid -> p.bufA) then pi_yx (p.bufA -> P)
void iota_xy(const Geo& g, const DftPlan& p, const float2* band, int C, hipStream_t s);
void iota_z(const Geo& g, const DftPlan& p, int C, float* out, hipStream_t s);
void pi_z(const Geo& g, const DftPlan& p, const float* grid, int C, hipStream_t s);
void pi_yx(const Geo& g, const DftPlan& p, int C, float2* P, hipStream_t s);

// ---- mixed-precision z stages on BF16 matrix cores (bl_mixed.hip)
int mixed_kp(const Geo& g);   // padded contraction length of the iota z stage: 2 kzh -> x16
int mixed_jt(const Geo& g);   // 32-row output tiles of the pi z stage
void iota_z_mixed(const Geo& g, const DftPlan& p, const float2* F2, int C, float* out,
                  hipStream_t s);
void pi_z_mixed(const Geo& g, const DftPlan& p, const float* f, int C, float2* G, hipStream_t s);

// ---- band kernels (bl_dft.hip)
// out[c] = projection of raw[c] (c < dim): Hermitian, and divergence-free when g.gamma = 1;
// with_div: out[dim] = spectral divergence.
// reg_partial (may be null): kRedBlocks partial sums of sum_c Lhat |out_c|^2.
// zero (may be null): nzero words set to zero by the same launch (a sweep's synchronisation words)
void band_prep(const Geo& g, const float2* raw, float2* out, int with_div, const double* Lhat64,
               double* reg_partial, hipStream_t s, uint32_t* zero = nullptr, int nzero = 0);
// the same for `nodes` band vectors in one launch, istride and ostride complex entries apart; the
// regulariser is the weighted sum (w, at the first and the last node wend)
void band_prep_nodes(const Geo& g, const float2* raw, float2* out, int nodes, size_t istride,
                     size_t ostride, hipStream_t s, int with_div = 0, const double* Lhat64 = nullptr,
                     double* reg_partial = nullptr, double w = 0.0, double wend = 0.0);
// out[c][k] = Lhat(k) vproj[c][k] + scale * P (Hermitian-completed), zero on unpaired planes;
// leray (C == dim): then projected divergence-free per index k.
// With dot_part not NULL (one node), also the finalize_blocks(g) block partials of
// Re sum conj(dotp) out over all C components (each thread sums its band index's components in
// order, then its block in the fixed order of block_reduce_256); with sq_part and max_part not
// NULL likewise the partials of sum |out|^2 and of max |out|.
// Given `done`, the launch stores done.value to done.word (host memory) when it begins: everything
// before it on the stream has then ended.
struct Done {
  uint64_t* word = nullptr;
  uint64_t value = 0;
};
__device__ __forceinline__ void report_begun(const Done& d) {
  if (d.word && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0)
    __hip_atomic_store(d.word, d.value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
void band_finalize(const Geo& g, int C, const float2* vproj, const float* Lhat,
                   const float2* P, float scale, float2* out, int* nonfinite, hipStream_t s,
                   int leray = 0, const float2* dotp = nullptr, double* dot_part = nullptr,
                   double* sq_part = nullptr, double* max_part = nullptr, Done done = {});
// blocks of a band_finalize launch (at most kRedBlocks)
int finalize_blocks(const Geo& g);
// band_finalize of `nodes` vectors in one launch: node n reads vproj + n vstride and
// P + n pstride and writes out + n ostride
void band_finalize_nodes(const Geo& g, int C, const float2* vproj, size_t vstride,
                         const float* Lhat, const float2* P, size_t pstride, float scale,
                         float2* out, size_t ostride, int nodes, int* nonfinite, hipStream_t s,
                         int leray = 0, Done done = {});

// ---- transports (bl_transport.hip)
// X: dim planes of forward offsets; YA = (Y, a) backward offsets and reaction factor
void setup(const Geo& g, const float* v, float* X, float4* YA, hipStream_t s);
// non-stationary steps t_n -> t_{n+1} for n < steps, one launch: V holds (v^n, r^n) of every
// node (dim + 1 planes each); step n writes X + n dim M and YA + n M
void setup_ns(const Geo& g, const float* V, float* X, float4* YA, int steps, hipStream_t s);
// b^n = lambda^n grad m^n for the time nodes n < nodes (lam, m: one plane per node; b: dim
// planes per node), one launch; with YA0 (the first step's (Y, a)), lambda^0 is formed from
// lambda^1 as a Interp(lambda^1, i + Y) instead of read (the plane lambda^0 is not used)
void body_nodes(const Geo& g, const float* lam, const float* m, float* b, int nodes,
                hipStream_t s, const float4* YA0 = nullptr);
void state_step(const Geo& g, const float* m_in, const float* X, float* m_out, hipStream_t s);
// kRedBlocks partials of sum (mT - I1)^2 in FP64; with lam not NULL also the terminal adjoint
// lam = lam_scale (mT - I1), the values terminal() writes
void energy_partial(const Geo& g, const float* mT, const float* I1, double* partial,
                    hipStream_t s, float* lam = nullptr);
void terminal(const Geo& g, const float* mT, const float* I1, float* lam, hipStream_t s);
void adj_step(const Geo& g, const float* lam_in, const float4* YA, float* lam_out,
              hipStream_t s);
// b_c = sum_n w_n lam^n d_c m^n over nt + 1 stored planes of lam and m; with YA, lam^0 is
// formed from lam^1 as a Interp(lam^1, i + Y) instead of read (the plane lam^0 is not used); the sum starts at b0 where given (dim planes)
struct BodyStart {
  float* c[3] = {nullptr, nullptr, nullptr};
};
void body_force(const Geo& g, const float* lam, const float* m, float* b, hipStream_t s,
                const float4* YA = nullptr, BodyStart b0 = {});
void inc_init(const Geo& g, const float* m0, const float* dv, float* t0, hipStream_t s);
void inc_step(const Geo& g, const float* t_in, const float* X, const float* m_next,
              const float* dv, float* t_out, hipStream_t s);
void inc_last(const Geo& g, const float* t_in, const float* X, const float* mT,
              const float* dv, float* dlam, hipStream_t s);
// full Newton product: incremental state step that also stores dm^{n+1} (t_out null: the last)
void inc_step_n(const Geo& g, const float* t_in, const float* X, const float* m_next,
                const float* dv, float* t_out, float* dm_out, hipStream_t s);
// hs^n = dt/2 div(lam^n dv) for 0 < n < nt, hs^nt = u^nt = -(2/sigma^2) dm^nt + dt/2 div(lam^nt dv)
// and b2 = sum_n w_n lam^n grad dm^n, from nt + 1 planes of lam and dm
void newton_terms(const Geo& g, const float* lam, const float* dm, const float* dv, float* hs,
                  const BodyStart& b2, hipStream_t s);
// q = a Interp(u_in, i + Y) + hs, in place of hs; u_out = q + hs (u_out null: without hs)
void adj_step_n(const Geo& g, const float* u_in, const float4* YA, float* hs, float* u_out,
                hipStream_t s);

// one component of packed float4 voxels into a plane
void unpack4(const Geo& g, int comp, const float4* in, float* plane, hipStream_t s);

// ---- setup of 3D grids from LDS (bl_box.hip): tiles of sw x 8 x 4 voxels, one
// workgroup each
struct BoxPlan {
  int sw = 0, ntx = 0, nty = 0, tiles = 0;
  FastDiv div_ntx, div_nty, div_sw;
};
void setup_box(const Geo& g, const float* v, float* X, float4* YA, hipStream_t s);
void setup_box_ns(const Geo& g, const float* V, float* X, float4* YA, int steps, hipStream_t s);

// ---- whole sweeps in one launch (bl_sweep.hip), stationary velocity, single problem
enum { SWEEP_STATE = 0, SWEEP_INC, SWEEP_ADJ, SWEEP_INC_N, SWEEP_ADJ_N };   // _N: full Newton product
constexpr int kSweepTiles = 256;                    // most tiles of a sweep
constexpr int kSweepWords = 320 + kSweepTiles * 16; // synchronisation words of a sweep, zero before it
// tiles of a sweep: ty rows of x by tz = gz * run planes, one workgroup each
struct SweepPlan {
  int run = 0;          // planes per thread; 0: the grid has no plan
  int ty = 0, tz = 0, gz = 0, nty = 0, ntz = 0, tiles = 0, threads = 0;
  int pitch = 0;        // floats of a row in LDS
  int box_floats = 0;   // LDS floats of a tile's rows and those its taps reach
  FastDiv div_nx, div_ty, div_ty2, div_nty, div_n4;   // by nx, ty, ty + 2, nty, 16-byte entries per row
};
// what the host gives a sweep beside its fields
// 100 us of the 100 MHz realtime counter.  A tile waits two or three microseconds for a neighbour that
// runs; others may not be resident yet because another stream's kernel still holds compute units, and
// short kernels are worth waiting for: products at 128^3 beside additions of 256 MB (73 us each)
// take 687 us with a wait of 50, 429 with 100 and with 400 (696 as steps).
constexpr uint32_t kSweepWait = 10000;
// about ten seconds of running: counted in looks, since a clock also runs while a workgroup is
// suspended for another process
constexpr uint32_t kSweepPolls = 1u << 24;
struct SweepRun {
  uint32_t* sync = nullptr;      // kSweepWords words, zero
  // SR_WORDS words: a sweep that abandons itself stores `number` to one of them
  uint64_t* report = nullptr;
  uint64_t number = 0;
  uint32_t wait = kSweepWait;    // realtime ticks that a tile waits for others (0: not once)
  uint32_t polls = kSweepPolls;  // looks at an abandoned sweep's earlier blocks before it is given up
};
// a tile's offsets left its box; a tile waited too long; the sweep was given up, its planes are not
// valid
enum { SR_LEFT = 0, SR_LATE, SR_GAVE_UP, SR_WORDS };
struct SweepArgs {
  const float* X = nullptr;      // forward offsets (state, incremental)
  const float4* YA = nullptr;    // backward offsets and reaction factor (adjoint)
  float* planes = nullptr;       // nt + 1 planes of the transported field
  const float* m = nullptr;      // nt + 1 planes of the state (incremental, adjoint)
  const float* dv = nullptr;     // dim planes (incremental)
  float* b = nullptr;            // dim planes: body force (adjoint)
  int keep0 = 0;                 // adjoint: lambda^0 is stored too
  float* dm = nullptr;           // nt + 1 planes (Newton incremental)
  const float* hs = nullptr;     // nt + 1 planes: hs^n and, in plane nt, u^nt (Newton adjoint)
  BodyStart b2;                  // dim planes: where b starts (Newton adjoint)
  float* acc = nullptr;          // dim planes to work in (Newton adjoint)
  SweepRun run;
};
// run = 0 where the grid's tiles cannot all be resident (one per compute unit) or do not fit
SweepPlan sweep_plan(const Geo& g, int compute_units);
// m^{n+1} = Interp(m^n, i + X) for n = 0..nt-1 (as nt times state_step)
void sweep_state(const Geo& g, const SweepPlan& p, const float* X, float* m, const SweepRun& r,
                 hipStream_t s);
// t^0..t^{nt-1} into the planes t (as inc_init, inc_step) and inc_last's value into plane nt
void sweep_inc(const Geo& g, const SweepPlan& p, const float* X, const float* m, const float* dv,
               float* t, const SweepRun& r, hipStream_t s);
// lam[nt] transported down to lam[1] (keep0: lam[0]) and the body force b (as adj_step and
// body_force)
void sweep_adj(const Geo& g, const SweepPlan& p, const float4* YA, const float* m, float* lam,
               float* b, int keep0, const SweepRun& r, hipStream_t s);

// the Newton product's: t^0..t^{nt-1} into the planes t and dm^1..dm^nt into dm; and, with the
// terms of newton_terms, u^{nt-1}..u^1 into the planes u and the body force b
void sweep_inc_n(const Geo& g, const SweepPlan& p, const float* X, const float* m, const float* dv,
                 float* t, float* dm, const SweepRun& r, hipStream_t s);
void sweep_adj_n(const Geo& g, const SweepPlan& p, const float4* YA, const float* m, const float* hs,
                 const BodyStart& b2, float* acc, float* u, float* b, const SweepRun& r, hipStream_t s);

// ---- deformation state equation (bl_deform.hip)
// Band fields are full centred bands of g (B entries per component); product-grid planes have
// MP = px * py * pz points; Ph is a kz >= 0 half spectrum of the product grid (pi_half output,
// kzh * ky * kx entries per component) and scaleP = 1 / MP.
// one Runge-Kutta stage st = 1..4 of d_t u~ = -src - conv, conv = Herm(Ph) / MP:
// k = -src - conv; acc = k (st 1), acc + 2k (st 2, 3), acc + k (st 4); the next state
// un + c h k (st 1, 2, 3; c = 1/2, 1/2, 1) or un + h/6 acc (st 4, also stored to unext);
// DU (may be null) receives its spectral derivatives DU[i * dim + j] = d~_j (lengths of the image grid)
void def_stage(const Geo& g, float scaleP, const float2* Ph, const float2* src, const float2* un,
               float2* acc, int st, float2* unext, float2* DU, hipStream_t s);
// out_i = sum_j DG[i dim + j] V_j (+ DG2[i dim + j] V2_j when DG2 != null), product grid
void def_prod(const Geo& g, int64_t MP, const float* DG, const float* V, const float* DG2,
              const float* V2, float* out, hipStream_t s);
// kap = h/6 rho, Ksum = kap (start of the transposed sweep)
void def_adj_init(const Geo& g, const float2* rho, float2* kap, float2* Ksum, hipStream_t s);
// KV[i dim + j] = KG_i V_j; GACC_j (+)= sum_i DUG[i dim + j] KG_i (first: =)
void def_adj_prod(const Geo& g, int64_t MP, const float* KG, const float* V, const float* DUG,
                  float* KV, float* GACC, int first, hipStream_t s);
// A_i = sum_j i q_j Herm(Ph[i dim + j]) / MP; the stage st = 4..1 of the transposed sweep
// (next kap, the running sum of A, Ksum += kap; st 1: rho += sum A, then kap = h/6 rho when
// more steps follow)
void def_adj_combine(const Geo& g, float scaleP, const float2* Ph, float2* rho, float2* Asum,
                     float2* Ksum, float2* kap, int st, int more, hipStream_t s);
// out = Lhat vproj (if vproj) + Ksum + Herm(Ph) / MP, divergence-free part when gamma = 1
void def_out(const Geo& g, float scaleP, const float2* Ph, const float2* Ksum,
             const float2* vproj, const float* Lhat, float2* out, int* nonfinite, hipStream_t s,
             Done done = {});
// image level (image grid): IG = (I0, central-difference gradient of I0)
void def_ig4(const Geo& g, const float* I0, float4* IG, hipStream_t s);
// m1 = I0 and GP = grad I0 interpolated at i + N_ref UG (UG: dim planes, domain units)
void def_warp(const Geo& g, const float* UG, const float4* IG, float* m1, float4* GP,
              hipStream_t s);
// Bf_j = -(2/sigma^2)(m1 - I1) GP_j
void def_rho1(const Geo& g, const float* m1, const float* I1, const float4* GP, float* Bf,
              hipStream_t s);
// Bf_j = -(2/sigma^2) (GP . DU) GP_j with DU = dim planes of iota(du~(1))
void def_drho1(const Geo& g, const float* DU, const float4* GP, float* Bf, hipStream_t s);

// fused stage kernels of the deformation method (bl_deform_fused.hip), 3D product grids with
// pz <= 48 and px py <= 6144 (fused_ok); F2 and G are work buffers of
// dim^2 * kzh * py * px complex entries (the product plan's bufA / bufB)
bool fused_ok(const Geo& g, const Geo& gp);
// F2[c][h][y][x] from the kz >= 0 half of `in` (dim fields; deriv: the dim^2 fields i q_j in_i)
void fx_iota_xy(const Geo& g, const Geo& gp, const DftPlan& pl, const float2* in, int deriv,
                float2* F2, hipStream_t s);
// columns: iota z, products with VP (+ DUGr . DVP), DUGw <- the derivative fields (if not
// null), pi z of the dim products into G[i][h][y][x]
void fx_col_fwd(const Geo& gp, const DftPlan& pl, const float2* F2, const float* VP,
                float* DUGw, const float* DUGr, const float* DVP, float2* G, hipStream_t s);
// columns: iota z of the cotangent, GACC (+)= (D~U)^T kap, pi z of the dim^2 products kap_i V_j
void fx_col_bwd(const Geo& gp, const DftPlan& pl, const float2* F2, const float* VP,
                const float* DUG, float* GACC, int first, float2* G, hipStream_t s);
// pi xy of G and the Runge-Kutta stage update (as def_stage; wout receives the next state)
void fx_pi_yx_stage(const Geo& g, const Geo& gp, const DftPlan& pl, const float2* G, float scaleP,
                    const float2* src, const float2* un, float2* acc, int st, float2* wout,
                    hipStream_t s);
// pi xy of the dim^2 products and the transposed-sweep update (as def_adj_combine)
void fx_pi_yx_adj(const Geo& g, const Geo& gp, const DftPlan& pl, const float2* G, float scaleP,
                  float2* rho, float2* Asum, float2* Ksum, float2* kap, int st, int more,
                  hipStream_t s);

// ---- reductions and band vector algebra (bl_reduce.hip)
// out[0] = sum of n partials in a fixed order (one block); also stored to host[0] (host-mapped
// pinned memory) when host != NULL, and *flag published to host_flag[0] when flag != NULL
void reduce_final(const double* partial, int n, double* out, hipStream_t s,
                  double* host = nullptr, const int* flag = nullptr, double* host_flag = nullptr,
                  const Batch& bt = Batch{});
// kRedBlocks partials of Re sum conj(a) b over n complex entries
void dot_partial(const float2* a, const float2* b, int64_t n, double* partial, hipStream_t s,
                 const Batch& bt = Batch{});
// the same over g.nodes * dim * B entries, node k weighted by the trapezoid weight w_k
void dot_partial_w(const Geo& g, const float2* a, const float2* b, double* partial, hipStream_t s);
// kRedBlocks partials of max |a|
void maxabs_partial(const float2* a, int64_t n, double* partial, hipStream_t s,
                    const Batch& bt = Batch{});
void reduce_max_final(const double* partial, int n, double* out, hipStream_t s,
                      double* host = nullptr, const int* flag = nullptr,
                      double* host_flag = nullptr, const Batch& bt = Batch{});
// reduce_final of pa and, in the same launch, reduce_final (max_b: reduce_max_final) of pb with
// the flag published beside it; the same values as the two separate calls
void reduce_final2(const double* pa, double* outa, double* hosta, const double* pb, double* outb,
                   double* hostb, int n, hipStream_t s, bool max_b = false,
                   const int* flag = nullptr, double* host_flag = nullptr,
                   const Batch& bt = Batch{});
// y = 0; y = x (kernels, so that a captured graph holds no memset or copy node)
void zero_band(float2* y, int64_t n, hipStream_t s, const Batch& bt = Batch{});
void copy_band(float2* y, const float2* x, int64_t n, hipStream_t s, const Batch& bt = Batch{});
// y = x + eps[0] d (step length in device memory)
void add_scaled_dev(float2* y, const float2* x, const float2* d, const double* eps, int64_t n,
                    hipStream_t s, const Batch& bt = Batch{});
// one PCG step: pHp = <p, Hp> from its nphp partials php_part (the same value as reduce_final
// of them; stored to pHp[0] and, when not NULL, host-mapped pHp_host[0]),
// alpha = rz / pHp (0 unless pHp > 0), delta += alpha p, r -= alpha Hp, z = r / Lhat,
// kRedBlocks partials of <r, r> (p0) and <r, z> (p1); php_part must not alias p0 or p1
void pcg_step(const Geo& g, const float2* p, const float2* Hp, const double* rz,
              const double* php_part, int nphp, double* pHp, double* pHp_host, float2* delta,
              float2* r, const float* Lhat, float2* z, double* p0, double* p1, hipStream_t s);
// y = x + (num[0] / den[0]) y with device scalars
void xpby_dev(float2* y, const float2* x, const double* num, const double* den, int64_t n,
              hipStream_t s, const Batch& bt = Batch{});
// p = z + (rz_next / rz) p after summing kRedBlocks partials each: rr_next (also to host-mapped
// rr_host) of p0, rz_next of p1, the same values as reduce_final2; rz and rz_next differ
void pcg_direction(float2* p, const float2* z, const double* p0, const double* p1,
                   const double* rz, double* rr_next, double* rr_host, double* rz_next, int64_t n,
                   hipStream_t s);
// delta = 0, r = -grad, z = r / Lhat (per component), p = z; also kRedBlocks partials of <r, r>
// (p0) and <r, z> (p1)
void pcg_start(const Geo& g, const float2* grad, const float* Lhat, float2* delta, float2* r,
               float2* z, float2* p, double* p0, double* p1, hipStream_t s);
// y = x + eps d
void add_scaled(float2* y, const float2* x, const float2* d, double eps, int64_t n,
                hipStream_t s);
// partials of sum (a - b)^2 over n reals
void sqdiff_partial(const float* a, const float* b, int64_t n, double* partial, hipStream_t s,
                    const Batch& bt = Batch{});

}  // namespace bl
