// Mixed-precision z stages of the band <-> grid transforms (paper Section 3.1, iota and pi)
// on BF16 matrix cores with split operands and FP32 accumulation.
//
// Each z stage is a real matrix product over one axis:
//   iota:  v[z][q] = sum_j Wi[z][j] G[j][q],  G[2h] = Re F2[h], G[2h+1] = Im F2[h],
//          Wi[z][2h] = s_h cos(2 pi h z / nz), Wi[z][2h+1] = -s_h sin(2 pi h z / nz),
//          s_0 = 1, s_h = 2 (Hermitian half spectrum, real output)
//   pi:    G[j][q] = sum_z Wp[j][z] f[z][q],  Wp[2h][z] = cos(..), Wp[2h+1][z] = -sin(..)
// with q = (y, x) the column index.  Every FP32 operand x is split into two BF16 numbers,
// x ~ hi + lo with hi = bf16(x) and lo = bf16(x - hi) (round to nearest even), and each
// product is formed as hi*hi + hi*lo + lo*hi on v_mfma_f32_32x32x16_bf16 with FP32
// accumulation; the dropped lo*lo term is below 2^-16 relative.  Twiddle splits are made on
// the host from FP64 values.
//
// Matrix-core operand layout (32x32x16, wave64): lane l holds A[i = l % 32][k = 8 (l / 32) + e]
// and B[k = 8 (l / 32) + e][j = l % 32] for e = 0..7; the accumulator register r of lane l
// holds D[i = 8 (r / 4) + 4 (l / 32) + r % 4][j = l % 32].
//
// Twiddle operands lie in the tables fragment by fragment, as a wavefront loads them: 64 lanes of
// 8 consecutive values, 1 KB in one piece.  In rows of the matrices the same loads touched 32 to
// 64 cache lines each, more cache traffic than the fields.  A lane's NT columns are consecutive,
// so that it loads and stores 4 NT bytes at a time and a wavefront uses an operand NT times
// (NT = 2 while the operands and sums of two columns leave registers for a second wavefront).
// Bound by the grid's planes.  Three components, before and now: 160x192x160 (band 40x48x40)
// iota 27.9 -> 16.7 us, pi 30.7 -> 19.8; 256^3 (band 64^3) 99.6 -> 50.6 and 97.2 -> 60.8 (5.0
// and 4.1 TB/s); 128^3 11.1 -> 9.5 and 13.1 -> 10.4; 64^3 5.5 -> 4.5 and 6.2 -> 5.9; 96^3 with
// band 96^3 (NT = 1) 11.5 -> 9.0 and 14.5 -> 11.6.
#include "bl_mfma.h"

namespace bl {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// round to nearest even
__device__ __forceinline__ void split2(f2 x, bf16x2& hi, bf16x2& lo) {
  hi = __builtin_convertvector(x, bf16x2);
  lo = __builtin_convertvector(x - __builtin_convertvector(hi, f2), bf16x2);
}

__device__ __forceinline__ f32x16 mfma3(bf16x8 ahi, bf16x8 alo, bf16x8 bhi, bf16x8 blo,
                                       f32x16 acc) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ahi, bhi, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ahi, blo, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(alo, bhi, acc, 0, 0, 0);
  return acc;
}

// the fragment of a lane: hi at f, lo at f + half
__device__ __forceinline__ void frag(const bf16x8* W, size_t half, size_t f, bf16x8& hi, bf16x8& lo) {
  hi = W[f];
  lo = W[half + f];
}

// iota z stage.  A wavefront holds the half spectrum of 32 NT columns in registers (the B
// operands) and forms z tiles of 32 planes; the next tile's twiddles are loaded meanwhile.
// Wi: KS fragments for each z tile.
template <int KS, int NT>
__global__ __launch_bounds__(256) void k_iota_z_mfma(Geo g, const float2* __restrict__ F2,
                                                     const bf16x8* __restrict__ Wi, int tiles,
                                                     float* __restrict__ out, int qblocks,
                                                     int run) {
  BL_BATCH(g.bat)
  BL_AT(F2, g.bat);
  BL_AT(out, g.bat);
  const int lane = threadIdx.x & 63, m = lane & 31, kq = lane >> 5;
  const uint32_t nq = (uint32_t)g.nx * (uint32_t)g.ny;
  const int c = blockIdx.y, chunk = (int)blockIdx.x / qblocks;
  const uint32_t unit = blockIdx.x - chunk * qblocks;
  const uint32_t col0 = (unit * 4u + (uint32_t)wave_of(threadIdx.x)) * (32u * NT);
  const uint32_t col = col0 + NT * (uint32_t)m;
  if (col0 >= nq) return;
  const Rsrc rf = rsrc(F2 + (size_t)c * g.kzh * nq, (uint32_t)g.kzh * nq * 8u);
  const Rsrc ro = rsrc(out + (size_t)c * g.M, (uint32_t)g.M * 4u);
  // B operand: k = 16 s + 8 kq + e  ->  h = 8 s + 4 kq + e/2, (Re, Im) by e parity
  bf16x8 bhi[NT][KS], blo[NT][KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    bf16x2 hi[NT][4], lo[NT][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int h = 8 * s + 4 * kq + i;
      const uint32_t off = h < g.kzh ? ((uint32_t)h * nq + col) * 8u : kPast;
      if constexpr (NT == 2) {
        const f4 v = ld4(rf, off);
        split2(f2{v.x, v.y}, hi[0][i], lo[0][i]);
        split2(f2{v.z, v.w}, hi[1][i], lo[1][i]);
      } else {
        split2(ld2(rf, off), hi[0][i], lo[0][i]);
      }
    }
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        bhi[j][s][e] = hi[j][e / 2][e & 1];
        blo[j][s][e] = lo[j][e / 2][e & 1];
      }
  }
  const size_t half = (size_t)tiles * KS * 64;
  const int t1 = min(tiles, (chunk + 1) * run);
  bf16x8 nhi[KS], nlo[KS];
  auto load = [&](int zt) {
#pragma unroll
    for (int s = 0; s < KS; ++s) frag(Wi, half, ((size_t)zt * KS + s) * 64 + lane, nhi[s], nlo[s]);
  };
  int zt = chunk * run;
  if (zt < t1) load(zt);
  for (; zt < t1; ++zt) {
    bf16x8 ahi[KS], alo[KS];
    f32x16 acc[NT];
#pragma unroll
    for (int s = 0; s < KS; ++s) ahi[s] = nhi[s], alo[s] = nlo[s];
    if (zt + 1 < t1) load(zt + 1);
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[j] = mfma3(ahi[s], alo[s], bhi[j][s], blo[j][s], acc[j]);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int z = zt * 32 + 8 * (r >> 2) + 4 * kq + (r & 3);
      const uint32_t o = ((uint32_t)z * nq + col) * 4u;
      if (z >= g.nz) continue;
      if constexpr (NT == 2) {
        if (col + 2 <= nq) {
          st2(ro, o, f2{acc[0][r], acc[1][r]});
          continue;
        }
      }
      if (col < nq) st1(ro, o, acc[0][r]);
    }
  }
}

// pi z stage.  The four wavefronts of a block share 32 NT columns; wavefront w takes the
// 16-plane steps w, w + 4, ... two at a time, for JT 32-row tiles of (Re, Im) outputs; the
// four sums are added in LDS in a fixed order.  Wp: JT fragments for each step.
template <int JT, int NT>
__global__ __launch_bounds__(256) void k_pi_z_mfma(Geo g, const float* __restrict__ f,
                                                   const bf16x8* __restrict__ Wp, int steps,
                                                   float2* __restrict__ G) {
  BL_BATCH(g.bat)
  BL_AT(f, g.bat);
  BL_AT(G, g.bat);
  __shared__ float red[4][NT][16][64];
  const int lane = threadIdx.x & 63, m = lane & 31, kq = lane >> 5, w = wave_of(threadIdx.x);
  const uint32_t nq = (uint32_t)g.nx * (uint32_t)g.ny;
  const int c = blockIdx.y;
  const uint32_t col = blockIdx.x * (32u * NT) + NT * (uint32_t)m;
  const Rsrc rf = rsrc(f + (size_t)c * g.M, (uint32_t)g.M * 4u);
  const Rsrc ro = rsrc(G + (size_t)c * g.kzh * nq, (uint32_t)g.kzh * nq * 8u);
  const size_t half = (size_t)steps * JT * 64;
  f32x16 acc[NT][JT];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int t = 0; t < JT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][t][r] = 0.f;
  for (int s0 = w; s0 < steps; s0 += 8) {
    float v[2][NT][8];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int z = 16 * (s0 + 4 * u) + 8 * kq + e;
        const uint32_t o = z < g.nz ? ((uint32_t)z * nq + col) * 4u : kPast;
        if constexpr (NT == 2) {
          const f2 x = ld2(rf, o);
          v[u][0][e] = x.x;
          v[u][1][e] = x.y;
        } else {
          v[u][0][e] = ld1(rf, o);
        }
      }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (s0 + 4 * u >= steps) break;   // the same for the wavefront
      bf16x8 bhi[NT], blo[NT];
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          bf16x2 hi, lo;
          split2(f2{v[u][j][e], v[u][j][e + 1]}, hi, lo);
          bhi[j][e] = hi.x, bhi[j][e + 1] = hi.y;
          blo[j][e] = lo.x, blo[j][e + 1] = lo.y;
        }
#pragma unroll
      for (int t = 0; t < JT; ++t) {
        bf16x8 ahi, alo;
        frag(Wp, half, ((size_t)(s0 + 4 * u) * JT + t) * 64 + lane, ahi, alo);
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[j][t] = mfma3(ahi, alo, bhi[j], blo[j], acc[j][t]);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < JT; ++t) {
    if (t > 0) __syncthreads();
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) red[w][j][r][lane] = acc[j][t][r];
    __syncthreads();
    // wavefront w adds the registers 4 w .. 4 w + 3: rows 32 t + 8 w + 4 kq + 0..3, which are
    // the (Re, Im) pairs of two h
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int h = 16 * t + 4 * w + 2 * kq + i;
      f2 sum[NT];
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int r = 4 * w + 2 * i + e;
          sum[j][e] = ((red[0][j][r][lane] + red[1][j][r][lane]) + red[2][j][r][lane]) +
                      red[3][j][r][lane];
        }
      const uint32_t o = ((uint32_t)h * nq + col) * 8u;
      if (h >= g.kzh) continue;
      if constexpr (NT == 2) {
        if (col + 2 <= nq) {
          st4(ro, o, f4{sum[0].x, sum[0].y, sum[1].x, sum[1].y});
          continue;
        }
      }
      if (col < nq) st2(ro, o, sum[0]);
    }
  }
}

template <int KS, int NT>
void launch_iota(const Geo& g, const DftPlan& p, const float2* F2, int C, float* out,
                 hipStream_t s) {
  const int64_t nq = (int64_t)g.nx * g.ny;
  const int qb = (int)((nq + 128 * NT - 1) / (128 * NT)), tiles = p.nzp32 / 32;
  // z tiles over blocks until the launch fills the device
  int n = 1;
  while ((int64_t)qb * C * n < 1024 && 2 * n <= tiles) n *= 2;
  const int run = (tiles + n - 1) / n;
  BL_LAUNCH((k_iota_z_mfma<KS, NT>), batch_grid(dim3((unsigned)(qb * ((tiles + run - 1) / run)), C), g.bat),
            dim3(256), 0, s, g, F2, reinterpret_cast<const bf16x8*>(p.wi_bf16), tiles, out, qb, run);
}
template <int JT, int NT>
void launch_pi(const Geo& g, const DftPlan& p, const float* f, int C, float2* G, hipStream_t s) {
  const int64_t nq = (int64_t)g.nx * g.ny;
  BL_LAUNCH((k_pi_z_mfma<JT, NT>), batch_grid(dim3((unsigned)((nq + 32 * NT - 1) / (32 * NT)), C), g.bat),
            dim3(256), 0, s, g, f, reinterpret_cast<const bf16x8*>(p.wp_bf16), p.nzp16 / 16, G);
}

}  // namespace

int mixed_kp(const Geo& g) { return (2 * g.kzh + 15) / 16 * 16; }
int mixed_jt(const Geo& g) { return (2 * g.kzh + 31) / 32; }

void iota_z_mixed(const Geo& g, const DftPlan& p, const float2* F2, int C, float* out,
                  hipStream_t s) {
  switch (mixed_kp(g) / 16) {
    case 1: launch_iota<1, 2>(g, p, F2, C, out, s); break;
    case 2: launch_iota<2, 2>(g, p, F2, C, out, s); break;
    case 3: launch_iota<3, 2>(g, p, F2, C, out, s); break;
    case 4: launch_iota<4, 2>(g, p, F2, C, out, s); break;
    case 5: launch_iota<5, 1>(g, p, F2, C, out, s); break;
    case 6: launch_iota<6, 1>(g, p, F2, C, out, s); break;
    case 7: launch_iota<7, 1>(g, p, F2, C, out, s); break;
    default: launch_iota<8, 1>(g, p, F2, C, out, s); break;
  }
}

void pi_z_mixed(const Geo& g, const DftPlan& p, const float* f, int C, float2* G, hipStream_t s) {
  switch (mixed_jt(g)) {
    case 1: launch_pi<1, 2>(g, p, f, C, G, s); break;
    case 2: launch_pi<2, 2>(g, p, f, C, G, s); break;
    case 3: launch_pi<3, 1>(g, p, f, C, G, s); break;
    default: launch_pi<4, 1>(g, p, f, C, G, s); break;
  }
}

}  // namespace bl
