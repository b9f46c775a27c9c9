// fp32 forward and backward of one chunk of sequence-chunked causal
// attention on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32: fp32
// products and fp32 accumulation), with the device library's expf / logf.  The
// fp32 configuration is held to 1e-4 absolute error, and its problems are
// small, so latency and idle compute units bound it rather than the matrix
// pipes.
//
// Same chunk semantics as the bf16 path: queries [c0, c1) attend to keys
// [0, c1), causally masked on the diagonal (Sec. 5.1 of SPPO); backward
// accumulates dK/dV over the reverse chunk walk (Sec. 5.2).
//   fwd   : one workgroup per 16 query rows of a head; its waves take the
//           key blocks in turn, each with its own running max, sum and O.
//   pre   : Delta_r = <dO_r, O_r>.
//   dq    : one workgroup per 16 query rows of a head, waves over key blocks.
//   dkdv  : one workgroup per 16 keys of a KV head, waves over the query
//           blocks of every head of the GQA group.
// The waves' results are added through LDS in wave order.  A block's wave
// depends on its position in the sequence (dkdv: in the chunk) alone, so a
// row's (key's) sum does not depend on the range a launch covers.
//
// Why so: with one thread per row, a 256-row chunk of one head ran on 4 of
// the 1024 SIMDs and took 526 us (forward), 525 us (dq) and 427 us (dkdv) at
// 1024 tokens x 1 head x 64; 16-row tiles times 8 waves spread the same work
// over 128 waves and the matrix units: 13.5, 15.6 and 12.7 us.  At 4096 tokens
// x 8 heads x 128 in 4 chunks the whole walk went from 351 to 2.8 ms (21
// TFLOP/s).  Operands go straight from global memory to registers in
// MFMA layout (no wave shares a block with another of its workgroup, so LDS
// staging would only add a pass); every load is 16 bytes per lane.
//
// MFMA layout (16x16x4, wave64, g = lane / 16, i = lane % 16): A[i][k] and
// B[k][j] hold row / column i at k-slot g, C[r][j] holds column i, rows
// 4 g + v.  The k-slot -> k map is free as long as A and B agree:
//   natural     (k = head dim): step (j, t) uses d = 16 j + 4 g + t, so a lane
//               loads 16 bytes of a row;
//   transposed  (k = row of a block): step t uses row 4 g + t, which is where
//               a C tile keeps it; a lane loads 16 bytes at d = 64 h + 4 i,
//               and component c feeds the C tile (h, c) whose rows are
//               d = 64 h + 4 (row) + c.
#include "sppo_kernels.h"

namespace sppo {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kB = 16;  // rows (keys) per block

__device__ __forceinline__ f32x4 mfma16(float a, float b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// Reductions over the four 16-lane groups that hold one column.
__device__ __forceinline__ float group_max(float x) {
  x = fmaxf(x, __shfl_xor(x, 16));
  return fmaxf(x, __shfl_xor(x, 32));
}
__device__ __forceinline__ float group_sum(float x) {
  x += __shfl_xor(x, 16);
  return x + __shfl_xor(x, 32);
}

// Natural operand: row `row` of a [.., D] tensor, 16 bytes per step group.
template <int D>
__device__ __forceinline__ void ld_nat(const float* row, int g, f32x4 (&x)[D / 16]) {
#pragma unroll
  for (int j = 0; j < D / 16; ++j) x[j] = ld4(row + 16 * j + 4 * g);
}
template <int D>
__device__ __forceinline__ f32x4 dot_nat(const f32x4 (&a)[D / 16], const f32x4 (&b)[D / 16]) {
  // two chains: half the dependent MFMAs
  f32x4 c0 = {0.f, 0.f, 0.f, 0.f}, c1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < D / 16; j += 2) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      c0 = mfma16(a[j][t], b[j][t], c0);
      c1 = mfma16(a[j + 1][t], b[j + 1][t], c1);
    }
  }
  return c0 + c1;
}
// acc[h][c] += (transposed block)(p): x[t][h] is row 4 g + t at d = 64 h + 4 i.
template <int D>
__device__ __forceinline__ void mul_tr(const f32x4 (&x)[4][D / 64], const f32x4& p, f32x4 (&acc)[D / 64][4]) {
#pragma unroll
  for (int t = 0; t < 4; ++t) {
#pragma unroll
    for (int h = 0; h < D / 64; ++h) {
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[h][c] = mfma16(x[t][h][c], p[t], acc[h][c]);
    }
  }
}
template <int D>
__device__ __forceinline__ bool any_nonfinite(const f32x4 (&x)[4][D / 64]) {
  bool bad = false;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
#pragma unroll
    for (int h = 0; h < D / 64; ++h) {
#pragma unroll
      for (int c = 0; c < 4; ++c) bad |= !(fabsf(x[t][h][c]) < INFINITY);
    }
  }
  return __any(bad);
}
// mul_tr over a block on the diagonal.  A masked pair has p = 0, which the
// MFMA would multiply with the row it must not see: harmless unless that row
// holds an infinity or a NaN.  Such blocks go one pair at a time and leave
// masked pairs out.  base + r * stride: row r of the block (r <= rmax);
// seen(r): whether this lane's column sees row r.
template <int D, class F>
__device__ __forceinline__ void mul_tr_masked(const f32x4 (&x)[4][D / 64], const f32x4& p, f32x4 (&acc)[D / 64][4],
                                              const float* base, int64_t stride, int rmax, F seen) {
  if (!any_nonfinite<D>(x)) {
    mul_tr<D>(x, p, acc);
    return;
  }
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  for (int r = 0; r < kB; ++r) {
    const float pv = r % 4 == 0 ? p[0] : r % 4 == 1 ? p[1] : r % 4 == 2 ? p[2] : p[3];
    const float pr = __shfl(pv, 16 * (r / 4) + i);
    if (!seen(r)) continue;
    const float* row = base + (r < rmax ? r : rmax) * stride;
#pragma unroll
    for (int h = 0; h < D / 64; ++h) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[h][c][v] = fmaf(pr, row[64 * h + 16 * g + 4 * v + c], acc[h][c][v]);
      }
    }
  }
}

// LDS image of one wave's [16 columns][D] result, rows padded by 4 floats.
template <int D>
__device__ __forceinline__ void put_tile(float* t, const f32x4 (&acc)[D / 64][4], int i, int g) {
#pragma unroll
  for (int h = 0; h < D / 64; ++h) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
      *reinterpret_cast<f32x4*>(t + i * (D + 4) + 64 * h + 16 * g + 4 * v) =
          f32x4{acc[h][0][v], acc[h][1][v], acc[h][2][v], acc[h][3][v]};
  }
}

template <int D>
__global__ __launch_bounds__(512) void fwd_f32_kernel(ChunkArgs a) {
  constexpr int W = 8, KB = D == 64 ? 2 : 1;  // waves; key blocks per iteration (32 K and 32 V registers)
  __shared__ __attribute__((aligned(16))) float Os[W][kB * (D + 4)];
  __shared__ float Ms[W][kB], Ls[W][kB];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, i = lane & 15, g = lane >> 4;
  const int h = blockIdx.y;
  const int64_t b = blockIdx.z;
  const int hk = h / (a.Hq / a.Hkv);
  const int64_t c0 = a.c0, c1 = a.c1, s = c1 - c0;
  const int64_t q0 = c0 + (int64_t)(gridDim.x - 1 - blockIdx.x) * kB;  // longest rows first
  const int64_t r = q0 + i, rc = r < c1 ? r : c1 - 1;
  const int64_t kend = (q0 + kB < c1) ? q0 + kB : c1;
  f32x4 q[D / 16];
  ld_nat<D>(static_cast<const float*>(a.q) + ((b * s + (rc - c0)) * a.Hq + h) * D, g, q);
  f32x4 o[D / 64][4];
#pragma unroll
  for (int x = 0; x < D / 64; ++x) {
#pragma unroll
    for (int c = 0; c < 4; ++c) o[x][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  float m = -INFINITY, l = 0.f;
  const float* kb = static_cast<const float*>(a.k) + (b * a.S * a.Hkv + hk) * D;
  const float* vb = static_cast<const float*>(a.v) + (b * a.S * a.Hkv + hk) * D;
  const int64_t stride = (int64_t)a.Hkv * D;
  // Rows past the last visible key are read as that key and masked.
  auto ld_k = [&](int64_t k0, f32x4 (&x)[KB][D / 16]) {
#pragma unroll
    for (int n = 0; n < KB; ++n) {
      const int64_t j = k0 + kB * n + i;
      ld_nat<D>(kb + (j < kend ? j : kend - 1) * stride, g, x[n]);
    }
  };
  constexpr int64_t kIt = (int64_t)KB * kB;
  f32x4 kx[KB][D / 16];
  if (w * kIt < kend) ld_k(w * kIt, kx);
  for (int64_t k0 = w * kIt; k0 < kend; k0 += W * kIt) {
    f32x4 vx[KB][4][D / 64];
#pragma unroll
    for (int n = 0; n < KB; ++n) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int64_t j = k0 + kB * n + 4 * g + t;
        const float* row = vb + (j < kend ? j : kend - 1) * stride;
#pragma unroll
        for (int x = 0; x < D / 64; ++x) vx[n][t][x] = ld4(row + 64 * x + 4 * i);
      }
    }
    f32x4 sv[KB];
#pragma unroll
    for (int n = 0; n < KB; ++n) sv[n] = dot_nat<D>(kx[n], q);
    if (k0 + W * kIt < kend) ld_k(k0 + W * kIt, kx);
    float mx = -INFINITY;
#pragma unroll
    for (int n = 0; n < KB; ++n) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        sv[n][v] *= a.scale;
        if (k0 + kB * n + 4 * g + v > r) sv[n][v] = -INFINITY;
        mx = fmaxf(mx, sv[n][v]);
      }
    }
    const float mn = fmaxf(m, group_max(mx));
    const float ms = mn == -INFINITY ? 0.f : mn;  // no visible key yet: P = exp(-inf) = 0
    const float corr = expf(m - ms);
    m = mn;
    l *= corr;
#pragma unroll
    for (int x = 0; x < D / 64; ++x) {
#pragma unroll
      for (int c = 0; c < 4; ++c) o[x][c] *= corr;
    }
#pragma unroll
    for (int n = 0; n < KB; ++n) {
      f32x4 p;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        p[v] = expf(sv[n][v] - ms);
        l += p[v];
      }
      const int64_t kn = k0 + kB * n;
      if (kn + kB - 1 <= q0) {
        mul_tr<D>(vx[n], p, o);
      } else if (kn < kend) {
        mul_tr_masked<D>(vx[n], p, o, vb + kn * stride, stride, (int)(kend - 1 - kn),
                         [&](int rr) { return kn + rr <= r; });
      }
    }
  }
  l = group_sum(l);
  put_tile<D>(Os[w], o, i, g);
  if (g == 0) {
    Ms[w][i] = m;
    Ls[w][i] = l;
  }
  __syncthreads();
  // out = sum_w exp(m_w - m) O_w / sum_w exp(m_w - m) l_w
  constexpr int TPR = 512 / kB;  // threads per row
  const int row = tid / TPR, d0 = tid % TPR;
  const int64_t ro = q0 + row;
  if (ro >= c1) return;
  float mm = -INFINITY;
#pragma unroll
  for (int x = 0; x < W; ++x) mm = fmaxf(mm, Ms[x][row]);
  float f[W], lt = 0.f;
#pragma unroll
  for (int x = 0; x < W; ++x) {
    f[x] = Ms[x][row] == -INFINITY ? 0.f : expf(Ms[x][row] - mm);
    lt += f[x] * Ls[x][row];
  }
  const float inv = 1.f / lt;
  float* orow = static_cast<float*>(a.o) + ((b * s + (ro - c0)) * a.Hq + h) * D;
#pragma unroll
  for (int d = d0; d < D; d += TPR) {
    float acc = 0.f;
#pragma unroll
    for (int x = 0; x < W; ++x) {
      if (f[x] != 0.f) acc += f[x] * Os[x][row * (D + 4) + d];
    }
    orow[d] = acc * inv;
  }
  if (d0 == 0) a.lse[(b * a.Hq + h) * s + (ro - c0)] = mm + logf(lt);
}

// Delta_r = <dO_r, O_r>, a wave per 16 (batch, row, head) rows: the diagonal
// of O dO^T, formed by the MFMA sequence that forms dP in dq and dkdv.  Where
// O_r is one V row (the first row of a sequence) dP - Delta is then exactly 0.
template <int D>
__global__ __launch_bounds__(256) void pre_f32_kernel(ChunkArgs a) {
  const int64_t s = a.c1 - a.c0, n = a.B * s * a.Hq;
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  const int64_t blocks = (n + kB - 1) / kB;
  for (int64_t blk = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); blk < blocks; blk += (int64_t)gridDim.x * 4) {
    const int64_t item = blk * kB + i, ic = item < n ? item : n - 1;
    f32x4 x[D / 16], y[D / 16];
    ld_nat<D>(static_cast<const float*>(a.o) + ic * D, g, x);
    ld_nat<D>(static_cast<const float*>(a.dout) + ic * D, g, y);
    const f32x4 c = dot_nat<D>(x, y);
    if (i / 4 == g && item < n) {  // this lane's column i is among its rows 4 g + v
      const int64_t h = item % a.Hq, rr = (item / a.Hq) % s, b = item / (a.Hq * s);
      a.delta[(b * a.Hq + h) * s + rr] = i % 4 == 0 ? c[0] : i % 4 == 1 ? c[1] : i % 4 == 2 ? c[2] : c[3];
    }
  }
}

// One workgroup's dQ tile: tile x of nx, query head h, batch entry b.
template <int D>
__device__ __forceinline__ void dq_tile(const ChunkArgs& a, int x, int nx, int h, int64_t b,
                                        float (*Qs)[kB * (D + 4)]) {
  constexpr int W = 8;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, i = lane & 15, g = lane >> 4;
  const int hk = h / (a.Hq / a.Hkv);
  const int64_t c0 = a.c0, c1 = a.c1, s = c1 - c0;
  const int64_t q0 = c0 + (int64_t)(nx - 1 - x) * kB;
  const int64_t r = q0 + i, rc = r < c1 ? r : c1 - 1;
  const int64_t kend = (q0 + kB < c1) ? q0 + kB : c1;
  const int64_t off = ((b * s + (rc - c0)) * a.Hq + h) * D;
  f32x4 q[D / 16], dout[D / 16], dq[D / 64][4];
  ld_nat<D>(static_cast<const float*>(a.q) + off, g, q);
  ld_nat<D>(static_cast<const float*>(a.dout) + off, g, dout);
#pragma unroll
  for (int x = 0; x < D / 64; ++x) {
#pragma unroll
    for (int c = 0; c < 4; ++c) dq[x][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const float lse = a.lse[(b * a.Hq + h) * s + (rc - c0)];
  const float delta = a.delta[(b * a.Hq + h) * s + (rc - c0)];
  const float* kb = static_cast<const float*>(a.k) + (b * a.S * a.Hkv + hk) * D;
  const float* vb = static_cast<const float*>(a.v) + (b * a.S * a.Hkv + hk) * D;
  const int64_t stride = (int64_t)a.Hkv * D;
  for (int64_t k0 = w * kB; k0 < kend; k0 += W * kB) {
    f32x4 kx[D / 16], vx[D / 16], kt[4][D / 64];
    const int64_t j = k0 + i < kend ? k0 + i : kend - 1;
    ld_nat<D>(kb + j * stride, g, kx);
    ld_nat<D>(vb + j * stride, g, vx);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int64_t jt = k0 + 4 * g + t < kend ? k0 + 4 * g + t : kend - 1;
#pragma unroll
      for (int x = 0; x < D / 64; ++x) kt[t][x] = ld4(kb + jt * stride + 64 * x + 4 * i);
    }
    const f32x4 qk = dot_nat<D>(kx, q), dp = dot_nat<D>(vx, dout);
    f32x4 ds;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float p = expf(qk[v] * a.scale - lse);
      ds[v] = k0 + 4 * g + v > r ? 0.f : p * (dp[v] - delta);
    }
    if (k0 + kB - 1 <= q0) {
      mul_tr<D>(kt, ds, dq);
    } else {
      mul_tr_masked<D>(kt, ds, dq, kb + k0 * stride, stride, (int)(kend - 1 - k0),
                       [&](int rr) { return k0 + rr <= r; });
    }
  }
  put_tile<D>(Qs[w], dq, i, g);
  __syncthreads();
  constexpr int TPR = 512 / kB;
  const int row = tid / TPR, d0 = tid % TPR;
  if (q0 + row >= c1) return;
  float* out = static_cast<float*>(a.dq) + ((b * s + (q0 + row - c0)) * a.Hq + h) * D;
#pragma unroll
  for (int d = d0; d < D; d += TPR) {
    float acc = Qs[0][row * (D + 4) + d];
#pragma unroll
    for (int y = 1; y < W; ++y) acc += Qs[y][row * (D + 4) + d];
    out[d] = acc * a.scale;
  }
}
template <int D>
__global__ __launch_bounds__(512) void dq_f32_kernel(ChunkArgs a) {
  __shared__ __attribute__((aligned(16))) float Qs[8][kB * (D + 4)];
  dq_tile<D>(a, blockIdx.x, gridDim.x, blockIdx.y, blockIdx.z, Qs);
}

// Waves: 8 for D = 64; 4 for D = 128, whose fragments, accumulators and
// operands (about 260 registers) leave room for one wave per SIMD.
template <int D>
constexpr int kDkdvWaves = D == 64 ? 8 : 4;
// One workgroup's dK/dV tile: tile x from kv0, KV head hk, batch entry b.
template <int D>
__device__ __forceinline__ void dkdv_tile(const ChunkArgs& a, int x, int hk, int64_t b, float (*Ks)[kB * (D + 4)]) {
  constexpr int W = kDkdvWaves<D>, T = 64 * W;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, i = lane & 15, g = lane >> 4;
  const int G = a.Hq / a.Hkv;
  const int64_t c0 = a.c0, c1 = a.c1, s = c1 - c0;
  const int64_t k0 = a.kv0 + (int64_t)x * kB;
  const int64_t j = k0 + i, jc = j < a.kv1 ? j : a.kv1 - 1;
  const int64_t kvoff = ((b * a.S + jc) * a.Hkv + hk) * D;
  f32x4 kx[D / 16], vx[D / 16], dk[D / 64][4], dv[D / 64][4];
  ld_nat<D>(static_cast<const float*>(a.k) + kvoff, g, kx);
  ld_nat<D>(static_cast<const float*>(a.v) + kvoff, g, vx);
#pragma unroll
  for (int x = 0; x < D / 64; ++x) {
#pragma unroll
    for (int c = 0; c < 4; ++c) dk[x][c] = dv[x][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const int64_t klast = k0 + kB - 1 < a.kv1 - 1 ? k0 + kB - 1 : a.kv1 - 1;
  // Query blocks (chunk-local, 16 rows from c0) from the first that sees a
  // key here; block n of head hh goes to wave (hh * nqb + n) % W.
  const int64_t nqb = (s + kB - 1) / kB;
  const int64_t first = k0 > c0 ? (k0 - c0) / kB : 0;
  const int64_t rs = (int64_t)a.Hq * D;  // elements between consecutive query rows
  for (int hh = 0; hh < G; ++hh) {
    const int h = hk * G + hh;
    const float* qb = static_cast<const float*>(a.q) + (b * s * a.Hq + h) * D;
    const float* ob = static_cast<const float*>(a.dout) + (b * s * a.Hq + h) * D;
    const float* lb = a.lse + (b * a.Hq + h) * s;
    const float* eb = a.delta + (b * a.Hq + h) * s;
    const int64_t lead = (hh * nqb + first) % W;
    for (int64_t n = first + (w - lead + W) % W; n < nqb; n += W) {
      const int64_t r0 = n * kB, last = s - 1;  // chunk-local rows
      f32x4 qx[D / 16], ox[D / 16], qt[4][D / 64], ot[4][D / 64];
      const int64_t rn = r0 + i < last ? r0 + i : last;
      ld_nat<D>(qb + rn * rs, g, qx);
      ld_nat<D>(ob + rn * rs, g, ox);
      float lse[4], del[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int64_t rt = r0 + 4 * g + t < last ? r0 + 4 * g + t : last;
        lse[t] = lb[rt];
        del[t] = eb[rt];
#pragma unroll
        for (int x = 0; x < D / 64; ++x) {
          qt[t][x] = ld4(qb + rt * rs + 64 * x + 4 * i);
          ot[t][x] = ld4(ob + rt * rs + 64 * x + 4 * i);
        }
      }
      const f32x4 qk = dot_nat<D>(qx, kx), dp = dot_nat<D>(ox, vx);
      auto seen = [&](int rr) { return r0 + rr <= last && c0 + r0 + rr >= j; };
      f32x4 p, ds;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        p[v] = seen(4 * g + v) ? expf(qk[v] * a.scale - lse[v]) : 0.f;
        ds[v] = seen(4 * g + v) ? p[v] * (dp[v] - del[v]) : 0.f;
      }
      if (c0 + r0 >= klast && r0 + kB - 1 <= last) {
        mul_tr<D>(ot, p, dv);
        mul_tr<D>(qt, ds, dk);
      } else {
        const int rmax = (int)(last - r0 < kB - 1 ? last - r0 : kB - 1);
        mul_tr_masked<D>(ot, p, dv, ob + r0 * rs, rs, rmax, seen);
        mul_tr_masked<D>(qt, ds, dk, qb + r0 * rs, rs, rmax, seen);
      }
    }
  }
  // dK, then dV, through the same LDS image.
  constexpr int TPR = T / kB;
  const int row = tid / TPR, d0 = tid % TPR;
  const int64_t obase = ((b * a.S + k0 + row) * a.Hkv + hk) * D;
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    if (pass) __syncthreads();
    put_tile<D>(Ks[w], pass ? dv : dk, i, g);
    __syncthreads();
    if (k0 + row < a.kv1) {
      float* out = (pass ? a.dv : a.dk) + obase;
#pragma unroll
      for (int d = d0; d < D; d += TPR) {
        float acc = Ks[0][row * (D + 4) + d];
#pragma unroll
        for (int x = 1; x < W; ++x) acc += Ks[x][row * (D + 4) + d];
        if (!pass) acc *= a.scale;
        out[d] = a.accumulate ? out[d] + acc : acc;
      }
    }
  }
}
template <int D>
__global__ __launch_bounds__(64 * kDkdvWaves<D>) void dkdv_f32_kernel(ChunkArgs a) {
  __shared__ __attribute__((aligned(16))) float Ks[kDkdvWaves<D>][kB * (D + 4)];
  dkdv_tile<D>(a, blockIdx.x, blockIdx.y, blockIdx.z, Ks);
}

// Both of a chunk's gradient kernels as one launch (D = 64, where their
// workgroups are alike): neither needs the other's results, and one after the
// other each leaves the card idle for a small grid or at its end.  dQ tiles
// first; dqx and kx tiles in x.
__global__ __launch_bounds__(512) void pair_f32_kernel(ChunkArgs a, int dqx, int kx) {
  constexpr int D = 64;
  __shared__ __attribute__((aligned(16))) float mem[8][kB * (D + 4)];
  const int ndq = dqx * a.Hq * (int)a.B, n = blockIdx.x;
  if (n < ndq) {
    dq_tile<D>(a, n % dqx, dqx, n / dqx % a.Hq, n / (dqx * a.Hq), mem);
  } else {
    const int m = n - ndq;
    dkdv_tile<D>(a, m % kx, m / kx % a.Hkv, m / (kx * a.Hkv), mem);
  }
}

}  // namespace

hipError_t launch_fwd_f32(const ChunkArgs& a, hipStream_t stream) {
  const int64_t s = a.c1 - a.c0;
  dim3 grid((unsigned)((s + kB - 1) / kB), (unsigned)a.Hq, (unsigned)a.B);
  if (a.D == 64) {
    hipLaunchKernelGGL(fwd_f32_kernel<64>, grid, dim3(512), 0, stream, a);
  } else if (a.D == 128) {
    hipLaunchKernelGGL(fwd_f32_kernel<128>, grid, dim3(512), 0, stream, a);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_bwd_pre_f32(const ChunkArgs& a, hipStream_t stream) {
  const int64_t s = a.c1 - a.c0;
  const int64_t blocks = (a.B * s * a.Hq + 4 * kB - 1) / (4 * kB), most = 1 << 20;
  dim3 grid((unsigned)(blocks < most ? blocks : most));
  if (a.D == 64) {
    hipLaunchKernelGGL(pre_f32_kernel<64>, grid, dim3(256), 0, stream, a);
  } else if (a.D == 128) {
    hipLaunchKernelGGL(pre_f32_kernel<128>, grid, dim3(256), 0, stream, a);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// One launch, or for more than 1.3e8 keys several: a launch's tiles and so
// its results are those of one over all of them.
hipError_t launch_bwd_dkdv_f32(const ChunkArgs& a, hipStream_t stream) {
  if (a.kv0 < 0 || a.kv1 > a.c1 || a.kv0 >= a.kv1) return hipErrorInvalidValue;
  if (a.D != 64 && a.D != 128) return hipErrorInvalidValue;
  const int threads = 64 * (a.D == 64 ? kDkdvWaves<64> : kDkdvWaves<128>);
  const int64_t most = kMaxWorkItems / threads * kB;
  hipError_t e = hipSuccess;
  ChunkArgs p = a;
  for (; p.kv0 < a.kv1 && e == hipSuccess; p.kv0 = p.kv1) {
    p.kv1 = a.kv1 - p.kv0 > most ? p.kv0 + most : a.kv1;
    const dim3 grid((unsigned)((p.kv1 - p.kv0 + kB - 1) / kB), (unsigned)a.Hkv, (unsigned)a.B);
    if (a.D == 64) hipLaunchKernelGGL(dkdv_f32_kernel<64>, grid, dim3(threads), 0, stream, p);
    else hipLaunchKernelGGL(dkdv_f32_kernel<128>, grid, dim3(threads), 0, stream, p);
    e = hipGetLastError();
  }
  return e;
}

hipError_t launch_bwd_dq_f32(const ChunkArgs& a, hipStream_t stream) {
  const int64_t s = a.c1 - a.c0;
  dim3 grid((unsigned)((s + kB - 1) / kB), (unsigned)a.Hq, (unsigned)a.B);
  if (a.D == 64) {
    hipLaunchKernelGGL(dq_f32_kernel<64>, grid, dim3(512), 0, stream, a);
  } else if (a.D == 128) {
    hipLaunchKernelGGL(dq_f32_kernel<128>, grid, dim3(512), 0, stream, a);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Where the workgroups are alike, at any size that one dimension of a grid
// holds (us, pre + dK/dV + dQ, one after the other -> pair: 4 heads, rows [0,
// 256) 23.9 -> 15.2, [768, 1024) 38.2 -> 26.6; 8 heads, rows [1000, 2000) 196
// -> 189; 16 heads, 2048 rows 542 -> 543).
bool bwd_pair_f32(const ChunkArgs& a) {
  if (a.D != 64) return false;
  const int64_t s = a.c1 - a.c0;
  const int64_t groups = (s + kB - 1) / kB * a.Hq * a.B + (a.kv1 - a.kv0 + kB - 1) / kB * a.Hkv * a.B;
  return groups <= kMaxWorkItems / 512 && !dq_overwrites_inputs(a, 4);
}

hipError_t launch_bwd_pair_f32(const ChunkArgs& a, hipStream_t stream) {
  if (a.kv0 < 0 || a.kv1 > a.c1 || a.kv0 >= a.kv1 || !bwd_pair_f32(a)) return hipErrorInvalidValue;
  const int64_t s = a.c1 - a.c0, dqx = (s + kB - 1) / kB, kx = (a.kv1 - a.kv0 + kB - 1) / kB;
  const dim3 grid((unsigned)(dqx * a.Hq * a.B + kx * a.Hkv * a.B));
  hipLaunchKernelGGL(pair_f32_kernel, grid, dim3(512), 0, stream, a, (int)dqx, (int)kx);
  return hipGetLastError();
}

}  // namespace sppo
