// TN product of few k-blocks with a write-only epilogue (the weight gradient of
// a chunk of up to a thousand tokens, written and not added):  C[M, N] =
// sum_k A[k, m] B[k, n], A stored [K, M], B stored [K, N], M and N multiples of
// 256, C bf16 or fp32.
//
// Workgroup tile 256 x 256, 8 waves (4 along M x 2 along N, each 64 x 128 =
// 2 x 4 MFMA tiles of 32 x 32), k-block 64, two LDS stages: the DMA of k-block
// kb+1 runs under the MFMAs of k-block kb.
//
// Bound by writing C.  The wave-group schedule of gemm_bf16.hip is the faster
// from about 20 k-blocks on, but with few of them its C^T stores (16 bytes per
// lane, 16 rows an instruction) run at 4 TB/s; here a lane has a column and a
// store covers 32 of them in two rows.  Measured in turn (us, this kernel /
// that one): fp32 6144 x 9984 x 106 51 / 62, 11520 x 1024 x 272 17 / 21, 8192 x
// 1536 x 601 25 / 27, 5888 x 3072 x 814 53 / 53; bf16 1792 x 12544 x 143 25 /
// 32, 9984 x 4352 x 206 42 / 51.
#include "mfma32.h"
#include "sppo_kernels.h"

namespace sppo {
namespace {

constexpr int GBM = 256, GBN = 256, GBK = 64;

template <int EPI>
__global__ __launch_bounds__(512, 1) void gemm_tn_short_kernel(GemmArgs g) {
  // Stage s: A tile then B tile, [64 k-rows][256] as two [64][128] halves.
  constexpr int TILE = GBM * GBK;  // elements per operand tile
  __shared__ __attribute__((aligned(1024))) uint16_t A0[TILE], B0[TILE], A1[TILE], B1[TILE];
  using T = Tile32<128>;

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, gh = lane >> 5;
  const int wm = w & 3, wn = w >> 2;  // wave tile rows 64 wm.., cols 128 wn..
  const int64_t m0 = (int64_t)blockIdx.y * GBM, n0 = (int64_t)blockIdx.x * GBN;

  // ---- DMA: 32 wave instructions (1 KiB each) per operand tile, 4 per wave;
  // instruction u covers rows 4 (u % 16).. of half u / 16.  Rows past K arrive
  // as zeros.
  int da[4], db[4];
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    const int u = w * 4 + x, half = u >> 4;
    da[x] = T::dma(lane, u & 15, g.lda) + half * 128 * 2;
    db[x] = T::dma(lane, u & 15, g.ldb) + half * 128 * 2;
  }
  auto issue = [&](int64_t k0, uint16_t* sa, uint16_t* sb) {
    const int64_t vk = g.K - k0;
    const int nk = vk < GBK ? (int)vk : GBK;
    const auto ra = uniform_rsrc(reinterpret_cast<uint64_t>(g.a + k0 * g.lda + m0), nk * (int)(g.lda * 2));
    const auto rb = uniform_rsrc(reinterpret_cast<uint64_t>(g.b + k0 * g.ldb + n0), nk * (int)(g.ldb * 2));
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int u = w * 4 + x;
      lds_dma16(ra, sa + (u >> 4) * (GBK * 128) + (u & 15) * 512, da[x]);
      lds_dma16(rb, sb + (u >> 4) * (GBK * 128) + (u & 15) * 512, db[x]);
    }
  };

  // ---- operand reads: A of M tile mt, B of N tile nt, k-step kk (16 wide)
  int tro[4][2];
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    tro[d][0] = T::tr(lane, d, 0);
    tro[d][1] = T::tr(lane, d, 1);
  }
  auto a_op = [&](const uint16_t* sa, int mt, int kk) {
    const int ml = wm * 64 + 32 * mt;  // column in the [64][256] tile
    const uint16_t* hb = sa + (ml >> 7) * (GBK * 128);
    const int d = (ml & 127) >> 5;
    return ld_tr(hb, tro[d][0] + 16 * kk * 128, tro[d][1] + 16 * kk * 128);
  };
  auto b_op = [&](const uint16_t* sb, int nt, int kk) {
    const uint16_t* hb = sb + wn * (GBK * 128);
    return ld_tr(hb, tro[nt][0] + 16 * kk * 128, tro[nt][1] + 16 * kk * 128);
  };

  f32x16 acc[2][4];
#pragma unroll
  for (int mt = 0; mt < 2; ++mt) {
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) acc[mt][nt] = f32x16{};
  }
  // Four k-steps per stage, eight MFMAs each; the six operand reads of k-step
  // kk+1 are issued before the MFMAs of k-step kk (register double buffer),
  // and the second wave on the SIMD covers what latency remains.
  auto compute = [&](const uint16_t* sa, const uint16_t* sb) {
    bf16x8 ao[2][2], bo[2][4];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) ao[0][mt] = a_op(sa, mt, 0);
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) bo[0][nt] = b_op(sb, nt, 0);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int cur = kk & 1, nxt = cur ^ 1;
      if (kk < 3) {
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) ao[nxt][mt] = a_op(sa, mt, kk + 1);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) bo[nxt][nt] = b_op(sb, nt, kk + 1);
      }
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) acc[mt][nt] = mfma32(ao[cur][mt], bo[cur][nt], acc[mt][nt]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // k-blocks in pairs (buffers 0, 1), then an odd last one: the loop has a
  // single exit, so the accumulators stay in place.
  const int nkb = (int)((g.K + GBK - 1) / GBK);
  issue(0, A0, B0);
  int kb = 0;
  for (; kb + 2 <= nkb; kb += 2) {
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __syncthreads();  // k-block kb landed; every wave is done with kb-1
    issue((int64_t)(kb + 1) * GBK, A1, B1);
    compute(A0, B0);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __syncthreads();
    if (kb + 2 < nkb) issue((int64_t)(kb + 2) * GBK, A0, B0);
    compute(A1, B1);
  }
  if (kb < nkb) {
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __syncthreads();
    compute(A0, B0);
  }

  // ---- epilogue, lane <-> column n, v <-> row m (8 (v/4) + 4 (l/32) + v%4).
  // Element offsets from C fit 32 bits (checked by the C ABI).
  const uint32_t cs = (uint32_t)g.ldc;
#pragma unroll
  for (int mt = 0; mt < 2; ++mt) {
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      __builtin_amdgcn_sched_barrier(0);
      const int64_t n = n0 + wn * 128 + 32 * nt + l32, mb = m0 + wm * 64 + 32 * mt + 4 * gh;
      const uint32_t cb = (uint32_t)(mb * g.ldc + n);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const uint32_t ic = cb + (8 * (v / 4) + (v % 4)) * cs;
        if constexpr (EPI == kEpiF32) static_cast<float*>(g.c)[ic] = acc[mt][nt][v];
        else static_cast<__bf16*>(g.c)[ic] = (__bf16)acc[mt][nt][v];
      }
    }
  }
}

}  // namespace

hipError_t launch_gemm_tn_short(const GemmArgs& g, hipStream_t stream) {
  if (!g.tn || g.M % GBM || g.N % GBN || (g.epi != kEpiBf16 && g.epi != kEpiF32)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(g.N / GBN), (unsigned)(g.M / GBM));
  if (g.epi == kEpiF32) hipLaunchKernelGGL(gemm_tn_short_kernel<kEpiF32>, grid, dim3(512), 0, stream, g);
  else hipLaunchKernelGGL(gemm_tn_short_kernel<kEpiBf16>, grid, dim3(512), 0, stream, g);
  return hipGetLastError();
}

}  // namespace sppo
