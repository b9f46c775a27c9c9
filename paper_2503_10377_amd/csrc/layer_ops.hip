// Row-wise and elementwise kernels of a full transformer layer chunk (the
// non-attention, non-GEMM steps): LayerNorm forward and backward, the GELU
// recomputation, the weight transpose, and the packing of the chunk's
// [dQ | dK | dV] rows for the QKV projection's backward.  bf16 activations,
// fp32 statistics and parameter gradients.
#include "sppo_kernels.h"
#include "tile_common.h"

namespace sppo {
namespace {

constexpr int kLnThreads = 256;
constexpr int kLnMaxPer = 4;  // 16-byte groups per thread: H <= 256 * 8 * 4 = 8192

// Sum over the wave, in every lane: DPP within the 16-lane rows (xor 1, xor 2,
// then mirrors, whose partners hold the other half's sum), permlane swaps
// between them; no LDS round trips.
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp<0xB1>(v);
  v += dpp<0x4E>(v);
  v += dpp<0x141>(v);
  v += dpp<0x140>(v);
  return sum_groups(v);
}

// Four floats of a buffer whose caller promises a float's alignment.
using f32x4_a4 = float __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ float block_sum(float v, float* red) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  __syncthreads();  // red may still be read by a previous reduction
  if (lane == 0) red[w] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

__device__ __forceinline__ void unpack8(const u32x4& x, float (&f)[8]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f[2 * e] = __uint_as_float(x[e] << 16);
    f[2 * e + 1] = __uint_as_float(x[e] & 0xffff0000u);
  }
}
__device__ __forceinline__ u32x4 pack8(const float (&f)[8]) {
  const bf16x8 b = pack_bf16x8(f[0], f[1], f[2], f[3], f[4], f[5], f[6], f[7]);
  return __builtin_bit_cast(u32x4, b);
}

// y = (x - mean) * rstd * gamma + beta per row, with biased variance; TEAM
// threads per row with PER 16-byte column groups each (H <= 8 TEAM PER).  mean
// and rstd are kept for the backward.  A team is the whole workgroup, or one
// wave of it (TEAM = 64), which needs no barrier.  HBM-bound: 8192 x 4096 in
// 25 us, 5.4 TB/s.
template <int TEAM, int PER>
__global__ __launch_bounds__(kLnThreads) void ln_fwd_kernel(LnArgs a) {
  __shared__ float red[4];
  const int H = a.H, tid = threadIdx.x % TEAM;
  const int64_t row = (int64_t)blockIdx.x * (kLnThreads / TEAM) + threadIdx.x / TEAM;
  if (TEAM < kLnThreads && row >= a.rows) return;
  auto total = [&](float v) {
    if constexpr (TEAM == 64) return wave_sum(v);
    else return block_sum(v, red);
  };
  const uint16_t* x = a.x + row * a.ldx;
  float v[PER][8];
  float s = 0.f;
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int c = 8 * (tid + TEAM * p);
    if (c < H) {
      unpack8(ld_global16(x + c), v[p]);
#pragma unroll
      for (int e = 0; e < 8; ++e) s += v[p][e];
    }
  }
  const float mean = total(s) / H;
  float q = 0.f;
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int c = 8 * (tid + TEAM * p);
    if (c < H) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float d = v[p][e] - mean;
        q += d * d;
      }
    }
  }
  const float rstd = 1.f / sqrtf(total(q) / H + a.eps);
  uint16_t* y = a.y + row * a.ldy;
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int c = 8 * (tid + TEAM * p);
    if (c < H) {
      float o[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = (v[p][e] - mean) * rstd * a.gamma[c + e] + a.beta[c + e];
      *reinterpret_cast<u32x4*>(y + c) = pack8(o);
    }
  }
  if (tid == 0 && a.mean) {
    a.mean[row] = mean;
    a.rstd[row] = rstd;
  }
}

// Backward of y = xhat * gamma + beta, xhat = (x - mean) * rstd, per row:
//   dx = dres + rstd * (g - mean_j(g) - xhat * mean_j(g * xhat)),  g = dy * gamma
// (dres: the gradient that reaches x around the LayerNorm, the residual
// branch).  Workgroup b handles rows [b R, b R + R), two rows at a time (one
// reduction for both), and writes its partial sums of dy * xhat and dy over
// those rows (the gamma and beta gradients) to part[b]; ln_reduce adds the
// partials.  The NT threads are teams of TEAM, PER 16-byte column groups per
// thread (H <= 8 TEAM PER); the teams take the pairs in turn and add their
// partial sums through LDS at the end, in team order.
// HBM-bound: while a pair is reduced, its dres and the next pair's x and dy are
// on their way, and gamma stays in registers (with ln_reduce, 8192 x 4096:
// 90 -> 53 us, 5.1 TB/s; 30000 x 256: 125 -> 23 us).
template <int NT, int TEAM, int PER>
__global__ __launch_bounds__(NT) void ln_bwd_kernel(LnArgs a) {
  constexpr int TEAMS = NT / TEAM, NW = NT / 64;  // a team is the workgroup or one wave
  static_assert(TEAM == NT || TEAM == 64, "");
  __shared__ float red[2][NW * 4];
  const int H = a.H, tid = threadIdx.x % TEAM, team = threadIdx.x / TEAM, wv = threadIdx.x >> 6;
  const int64_t r0 = (int64_t)blockIdx.x * a.rows_per_block;
  const int64_t r1 = r0 + a.rows_per_block < a.rows ? r0 + a.rows_per_block : a.rows;
  float pg[PER][8], pb[PER][8], gm[PER][8];
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int c = 8 * (tid + TEAM * p);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      pg[p][e] = pb[p][e] = 0.f;
      gm[p][e] = c < H ? a.gamma[c + e] : 0.f;
    }
  }
  u32x4 xn[2][PER], dn[2][PER];
  float mn[2], rn[2];
  auto load = [&](int64_t row) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int64_t rr = row + j < r1 ? row + j : r1 - 1;  // a lone last row is read twice, used once
      mn[j] = a.mean[rr];
      rn[j] = a.rstd[rr];
#pragma unroll
      for (int p = 0; p < PER; ++p) {
        const int c = 8 * (tid + TEAM * p);
        xn[j][p] = dn[j][p] = u32x4{0, 0, 0, 0};
        if (c < H) {
          xn[j][p] = ld_global16(a.x + rr * a.ldx + c);
          dn[j][p] = ld_global16(a.dy + rr * a.lddy + c);
        }
      }
    }
  };
  load(r0 + 2 * team);
  int ph = 0;
  for (int64_t row = r0 + 2 * team; row < r1; row += 2 * TEAMS, ph ^= 1) {
    const bool two = row + 1 < r1;
    u32x4 xc[2][PER], dc[2][PER], rs[2][PER];
    float mean[2], rstd[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      mean[j] = mn[j];
      rstd[j] = rn[j];
#pragma unroll
      for (int p = 0; p < PER; ++p) {
        const int c = 8 * (tid + TEAM * p);
        xc[j][p] = xn[j][p];
        dc[j][p] = dn[j][p];
        rs[j][p] = u32x4{0, 0, 0, 0};
        if (c < H) rs[j][p] = ld_global16(a.dres + (j == 0 || two ? row + j : row) * a.lddres + c);
      }
    }
    if (row + 2 * TEAMS < r1) load(row + 2 * TEAMS);
    float sums[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 2; ++j) {
#pragma unroll
      for (int p = 0; p < PER; ++p) {
        if (8 * (tid + TEAM * p) < H) {
          float xv[8], dv[8];
          unpack8(xc[j][p], xv);
          unpack8(dc[j][p], dv);
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float xh = (xv[e] - mean[j]) * rstd[j], gg = dv[e] * gm[p][e];
            sums[2 * j] += gg;
            sums[2 * j + 1] += gg * xh;
            if (j == 0 || two) {
              pg[p][e] += dv[e] * xh;
              pb[p][e] += dv[e];
            }
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) sums[i] = wave_sum(sums[i]);
    if constexpr (TEAM > 64) {  // one barrier per pair: the waves' sums alternate between two LDS images
      if ((tid & 63) == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) red[ph][wv * 4 + i] = sums[i];
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        sums[i] = red[ph][i];
#pragma unroll
        for (int w = 1; w < NW; ++w) sums[i] += red[ph][w * 4 + i];
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (j == 1 && !two) break;
      const float m1 = sums[2 * j] / H, m2 = sums[2 * j + 1] / H;
#pragma unroll
      for (int p = 0; p < PER; ++p) {
        const int c = 8 * (tid + TEAM * p);
        if (c < H) {
          float xv[8], dv[8], rv[8], o[8];
          unpack8(xc[j][p], xv);
          unpack8(dc[j][p], dv);
          unpack8(rs[j][p], rv);
#pragma unroll
          for (int e = 0; e < 8; ++e)
            o[e] = rv[e] + rstd[j] * (dv[e] * gm[p][e] - m1 - (xv[e] - mean[j]) * rstd[j] * m2);
          *reinterpret_cast<u32x4*>(a.y + (row + j) * a.ldy + c) = pack8(o);
        }
      }
    }
  }
  float* part = a.part + (int64_t)blockIdx.x * 2 * H;
  if constexpr (TEAMS > 1) {
    __shared__ __attribute__((aligned(16))) float comb[TEAMS][2][8 * TEAM * PER];
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int c = 8 * (tid + TEAM * p);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        comb[team][0][c + e] = pg[p][e];
        comb[team][1][c + e] = pb[p][e];
      }
    }
    __syncthreads();
    for (int c = threadIdx.x; c < H; c += NT) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        float t = comb[0][i][c];
#pragma unroll
        for (int u = 1; u < TEAMS; ++u) t += comb[u][i][c];
        part[i * H + c] = t;
      }
    }
    return;
  }
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int c = 8 * (tid + TEAM * p);
    if (c < H) {
#pragma unroll
      for (int e = 0; e < 8; e += 4) {
        *reinterpret_cast<f32x4_a4*>(part + c + e) = f32x4_a4{pg[p][e], pg[p][e + 1], pg[p][e + 2], pg[p][e + 3]};
        *reinterpret_cast<f32x4_a4*>(part + H + c + e) = f32x4_a4{pb[p][e], pb[p][e + 1], pb[p][e + 2], pb[p][e + 3]};
      }
    }
  }
}

// dgamma[c] (+)= sum_b part[b][c], dbeta[c] (+)= sum_b part[b][H + c].  A
// workgroup covers 32 columns of the 2H partial row (eight 16-byte pieces) with
// 32 row groups: group t sums the blocks b = t, t + 32, ... in order, then the
// group sums are added pairwise (a fixed order: the result is deterministic).
constexpr int kRedCols = 32, kRedGroups = 32;
__global__ __launch_bounds__(kRedCols / 4 * kRedGroups) void ln_reduce_kernel(LnArgs a) {
  __shared__ __attribute__((aligned(16))) float red[kRedGroups][kRedCols + 4];
  const int lc = threadIdx.x % (kRedCols / 4) * 4, t = threadIdx.x / (kRedCols / 4);
  const int c = blockIdx.x * kRedCols + lc;  // column of the [2H] partial row (2H is a multiple of 16)
  const int W = 2 * a.H;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  if (c < W) {
#pragma unroll 8
    for (int b = t; b < a.nblocks; b += kRedGroups) s += *reinterpret_cast<const f32x4_a4*>(a.part + (int64_t)b * W + c);
  }
  *reinterpret_cast<f32x4*>(&red[t][lc]) = s;
  __syncthreads();
  const int oc = blockIdx.x * kRedCols + threadIdx.x;
  if (threadIdx.x < kRedCols && oc < W) {
    float v[kRedGroups];
#pragma unroll
    for (int u = 0; u < kRedGroups; ++u) v[u] = red[u][threadIdx.x];
#pragma unroll
    for (int n = kRedGroups / 2; n > 0; n /= 2) {
#pragma unroll
      for (int u = 0; u < n; ++u) v[u] += v[u + n];
    }
    const float tot = v[0];
    float* dst = oc < a.H ? a.dgamma + oc : a.dbeta + (oc - a.H);
    if (a.accumulate) *dst += tot;
    else *dst = tot;
  }
}

// y = gelu(x) elementwise over n bf16 values (n % 8 == 0).
__global__ __launch_bounds__(256) void gelu_kernel(const uint16_t* x, uint16_t* y, int64_t n) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
  if (i >= n) return;
  float v[8];
  unpack8(ld_global16(x + i), v);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = gelu_tanh(v[e]);
  *reinterpret_cast<u32x4*>(y + i) = pack8(v);
}

// out[c][r] = in[r][c] for a [R, C] bf16 matrix, 64 x 64 tiles through LDS.
__global__ __launch_bounds__(256) void transpose_kernel(const uint16_t* in, uint16_t* out, int64_t R, int64_t C) {
  __shared__ uint16_t t[64][66];
  const int64_t r0 = (int64_t)blockIdx.y * 64, c0 = (int64_t)blockIdx.x * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int y = ty; y < 64; y += 4) {
    const int64_t r = r0 + y, c = c0 + tx;
    t[y][tx] = (r < R && c < C) ? in[r * C + c] : 0;
  }
  __syncthreads();
  for (int y = ty; y < 64; y += 4) {
    const int64_t c = c0 + y, r = r0 + tx;
    if (c < C && r < R) out[c * R + r] = t[tx][y];
  }
}

// The same where rows and columns come in eights and both buffers are 16-byte
// aligned: 16 bytes per lane in and out, eight lanes a 128-byte line on either
// side.  Row r's eight-column pieces lie rotated by r / 8, so that the column
// reads of eight lanes on eight row groups fall on different banks.
// HBM-bound: 4096 x 16384 in 40 us, 6.7 TB/s (two bytes per lane: 67 us).
__global__ __launch_bounds__(256) void transpose8_kernel(const uint16_t* in, uint16_t* out, int64_t R, int64_t C) {
  __shared__ __attribute__((aligned(16))) uint16_t t[64][64];
  const int64_t r0 = (int64_t)blockIdx.y * 64, c0 = (int64_t)blockIdx.x * 64;
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    const int u = threadIdx.x + 256 * x, y = u >> 3, g = u & 7;
    if (r0 + y < R && c0 + 8 * g < C)
      *reinterpret_cast<u32x4*>(&t[y][((g + (y >> 3)) & 7) * 8]) = ld_global16(in + (r0 + y) * C + c0 + 8 * g);
  }
  __syncthreads();
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    const int u = threadIdx.x + 256 * x, y = u >> 3, g = u & 7;  // column of in, group of eight rows
    if (c0 + y < C && r0 + 8 * g < R) {
      const int p = (((y >> 3) + g) & 7) * 8 + (y & 7);
      u32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        v[e] = (uint32_t)t[8 * g + 2 * e][p] | ((uint32_t)t[8 * g + 2 * e + 1][p] << 16);
      *reinterpret_cast<u32x4*>(out + (c0 + y) * R + r0 + 8 * g) = v;
    }
  }
}

// Row t of dqkv = [dQ_i[t] | bf16(dK[c + t]) | bf16(dV[c + t])] for the
// chunk's rows (B = 1): dQ_i is [s, Hq D] bf16, dK/dV [S, Hkv D] fp32.
__global__ __launch_bounds__(256) void pack_dqkv_kernel(PackArgs a) {
  const int64_t t = blockIdx.x;
  const int wq = a.wq, wkv = a.wkv;
  uint16_t* out = a.out + t * (int64_t)(wq + 2 * wkv);
  for (int c = threadIdx.x * 8; c < wq; c += 256 * 8)
    *reinterpret_cast<u32x4*>(out + c) = ld_global16(a.dq + t * (int64_t)wq + c);
  const float* dk = a.dk + (a.c + t) * (int64_t)wkv;
  const float* dv = a.dv + (a.c + t) * (int64_t)wkv;
  for (int c = threadIdx.x * 8; c < wkv; c += 256 * 8) {
    float f[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = dk[c + e];
    *reinterpret_cast<u32x4*>(out + wq + c) = pack8(f);
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = dv[c + e];
    *reinterpret_cast<u32x4*>(out + wq + wkv + c) = pack8(f);
  }
}

}  // namespace

hipError_t launch_ln_fwd(const LnArgs& a, hipStream_t stream) {
  if (a.rows <= 0 || a.H <= 0 || a.H % 8 || a.H > kLnThreads * 8 * kLnMaxPer) return hipErrorInvalidValue;
  // Up to 1024 columns a wave holds a row: a workgroup would leave half its
  // lanes idle and wait at four barriers (30000 x 256: 34 us against 10,
  // 8192 x 1024: 12.3 against 8.0).
  const dim3 row_grid((unsigned)a.rows), wave_grid((unsigned)((a.rows + 3) / 4)), block(kLnThreads);
  if (a.H <= 512)
    hipLaunchKernelGGL((ln_fwd_kernel<64, 1>), wave_grid, block, 0, stream, a);
  else if (a.H <= 1024)
    hipLaunchKernelGGL((ln_fwd_kernel<64, 2>), wave_grid, block, 0, stream, a);
  else if (a.H <= 4096)
    hipLaunchKernelGGL((ln_fwd_kernel<kLnThreads, 2>), row_grid, block, 0, stream, a);
  else
    hipLaunchKernelGGL((ln_fwd_kernel<kLnThreads, kLnMaxPer>), row_grid, block, 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_ln_bwd(const LnArgs& a, hipStream_t stream) {
  if (a.rows <= 0 || a.H <= 0 || a.H % 8 || a.H > kLnThreads * 8 * kLnMaxPer || a.rows_per_block <= 0)
    return hipErrorInvalidValue;
  LnArgs b = a;
  b.nblocks = (int)((a.rows + a.rows_per_block - 1) / a.rows_per_block);
  // Two column groups per thread at most: three or four leave one wave per
  // SIMD.  Up to 1024 columns a wave is a team of its own (30000 x 256: 53 us
  // with one team of 256, 23 with four of 64; 8192 x 1024: 21.5 and 19.1).
  const dim3 grid((unsigned)b.nblocks);
  if (a.H <= 512)
    hipLaunchKernelGGL((ln_bwd_kernel<256, 64, 1>), grid, dim3(256), 0, stream, b);
  else if (a.H <= 1024)
    hipLaunchKernelGGL((ln_bwd_kernel<256, 64, 2>), grid, dim3(256), 0, stream, b);
  else if (a.H <= 2048)
    hipLaunchKernelGGL((ln_bwd_kernel<256, 256, 1>), grid, dim3(256), 0, stream, b);
  else if (a.H <= 4096)
    hipLaunchKernelGGL((ln_bwd_kernel<256, 256, 2>), grid, dim3(256), 0, stream, b);
  else if (a.H <= 6144)
    hipLaunchKernelGGL((ln_bwd_kernel<384, 384, 2>), grid, dim3(384), 0, stream, b);
  else
    hipLaunchKernelGGL((ln_bwd_kernel<512, 512, 2>), grid, dim3(512), 0, stream, b);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(ln_reduce_kernel, dim3((unsigned)((2 * a.H + kRedCols - 1) / kRedCols)),
                     dim3(kRedCols / 4 * kRedGroups), 0, stream, b);
  return hipGetLastError();
}

hipError_t launch_gelu(const uint16_t* x, uint16_t* y, int64_t n, hipStream_t stream) {
  if (n <= 0 || n % 8) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gelu_kernel, dim3((unsigned)((n / 8 + 255) / 256)), dim3(256), 0, stream, x, y, n);
  return hipGetLastError();
}

hipError_t launch_transpose(const uint16_t* in, uint16_t* out, int64_t R, int64_t C, hipStream_t stream) {
  if (R <= 0 || C <= 0) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((C + 63) / 64), (unsigned)((R + 63) / 64));
  if (R % 8 == 0 && C % 8 == 0 && ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 15) == 0)
    hipLaunchKernelGGL(transpose8_kernel, grid, dim3(256), 0, stream, in, out, R, C);
  else
    hipLaunchKernelGGL(transpose_kernel, grid, dim3(256), 0, stream, in, out, R, C);
  return hipGetLastError();
}

hipError_t launch_pack_dqkv(const PackArgs& a, hipStream_t stream) {
  if (a.rows <= 0 || a.wq % 8 || a.wkv % 8) return hipErrorInvalidValue;
  hipLaunchKernelGGL(pack_dqkv_kernel, dim3((unsigned)a.rows), dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace sppo
