// Dense bf16 GEMM on MFMA (fp32 accumulation) for the projections and the
// MLP of a full transformer layer chunk:  C[M, N] (op)= sum_k A(m, k) B(k, n).
//
// Two operand layouts, both read by LDS-DMA into the swizzled tiles of
// tile_common.h:
//   NT  A [M, K], B [N, K] row-major (k contiguous in both; natural operand
//       reads).  The forward projections x W use the transposed weight W^T
//       [out, in] as B; the data gradients dY W^T use the weight W [in, out]
//       as B.
//   TN  A stored [K, M], B stored [K, N] row-major (k = row; transposed
//       operand reads): the weight gradients X^T dY, accumulated in fp32.
// Both operands of a product read the same k-slot map (natural or
// transposed), so their k values pair up.
//
// Every product is v_mfma_f32_16x16x32_bf16 with B as its first operand, so
// the accumulators hold C^T and a lane stores runs of consecutive columns.
// k-steps are added in order whatever the tile, so the tile size never changes
// a result's bits (but TN products of up to 16 k-blocks that write C without
// reading it have a kernel of their own on 32x32x16 MFMAs, gemm_tn_short.hip).
//
// gemm_bf16_kernel: workgroup tile 256 x 256, k-block 64, 8 waves in two groups
// of four that take turns: a k-block is four phases, each [operand reads and
// one half-tile DMA] then [16 MFMAs, a 64 x 32 quadrant], and the second group
// runs half a phase behind, so on every SIMD one wave's MFMAs cover the other's
// reads and DMA issue.  Bound by the matrix pipes at the power limit: 0.91 us
// per k-block on an otherwise idle chip, 94% of the MFMA issue rate; on a full
// one MFMA busy 0.64-0.76 at 1.8 GHz (counters; the epilogues are the rest, the
// plain one 0.76).  Against 8 waves in step on one
// barrier per k-block with 32x32x16 MFMAs (the previous kernel), TFLOP/s at
// 8192 rows: NT 4096 x 4096 1218 -> 1431, GELU 16384 x 4096 1064 -> 1350,
// residual 4096 x 16384 1163 -> 1426, TN 4096 x 16384 accumulate 1083 -> 1282.
// The phases alone gave 1334 / 1120 / 1371 / 1208, the logistic GELU 1272 and
// the 16x16x32 MFMA (less energy per flop) the rest.  An XCD-grouped tile order
// (bands of 2, 4 or 8 tile rows) moved the shapes by -4% to +2%: plain order.
//
// gemm_small_kernel: 128 x 128 and 64 x 64 tiles for products that 256 x 256
// tiles would spread over too few CUs (1000 x 1024 x 4096: 16 tiles, 82 us;
// 256 tiles of 64 x 64, 17 us).
#include "sppo_kernels.h"
#include "tile_common.h"

namespace sppo {
namespace {

constexpr int GBM = 256, GBN = 256, GBK = 64;

constexpr int kWaitLds = 0xC07F;  // s_waitcnt lgkmcnt(0), the other counters at their maxima

// Epilogue of a wave's [16 MI rows][32 columns] at (m0, n0).  acc holds C^T, so
// a lane has row m = l % 16 of a 16-row tile and, of the 32 columns, NT:
// 8 g + 0..7 (nat_perm), TN: 4 g + 0..3 and 16 + 4 g + 0..3, as runs of four.
// Old values (residual, pre-activation, fp32 accumulator) are all loaded
// before any result is stored.  Element offsets from C / aux fit 32 bits, and
// N, ldc, ldaux are multiples of 4 (checked by the C ABI), so a run of four is
// all inside N or all outside and 8-byte (fp32: 16-byte) aligned.
template <int TN, int EPI, int MI>
__device__ __forceinline__ void store_tile(const GemmArgs& g, int64_t m0, int64_t n0, f32x4 (&acc)[MI][2]) {
  constexpr bool kAux = EPI == kEpiAddBf16 || EPI == kEpiDGelu, kAcc = EPI == kEpiAccF32;
  constexpr int kRun = TN ? 16 : 4;  // from the first run of four to the second
  typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
  const int l16 = threadIdx.x & 15, gh = (threadIdx.x & 63) >> 4;
  const int64_t m = m0 + l16, n = n0 + (TN ? 4 : 8) * gh;
  const int mrem = (int)(g.M - m < 16 * MI ? g.M - m : 16 * MI), nrem = (int)(g.N - n < 32 ? g.N - n : 32);
  const uint32_t cb = (uint32_t)(m * g.ldc + n), ab = (uint32_t)(m * g.ldaux + n);
  const uint32_t cs = 16 * (uint32_t)g.ldc, as = 16 * (uint32_t)g.ldaux;
  f32x4 in[MI][2];
  if constexpr (kAux || kAcc) {
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
      for (int nj = 0; nj < 2; ++nj) {
        in[mi][nj] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (16 * mi < mrem && kRun * nj < nrem) {
          if constexpr (kAcc) {
            in[mi][nj] = *reinterpret_cast<const f32x4*>(static_cast<const float*>(g.c) + (cb + mi * cs + kRun * nj));
          } else {
            const bf16x4_t t =
                *reinterpret_cast<const bf16x4_t*>(static_cast<const __bf16*>(g.aux) + (ab + mi * as + kRun * nj));
#pragma unroll
            for (int e = 0; e < 4; ++e) in[mi][nj][e] = (float)t[e];
          }
        }
      }
    }
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
    for (int nj = 0; nj < 2; ++nj) {
      if (16 * mi < mrem && kRun * nj < nrem) {
        const uint32_t ic = cb + mi * cs + kRun * nj;
        f32x4 r = acc[mi][nj];
        if constexpr (kAcc || EPI == kEpiAddBf16) r += in[mi][nj];
        if constexpr (EPI == kEpiDGelu) {
#pragma unroll
          for (int e = 0; e < 4; ++e) r[e] *= gelu_tanh_grad(in[mi][nj][e]);
        }
        if constexpr (EPI == kEpiAccF32 || EPI == kEpiF32) {
          *reinterpret_cast<f32x4*>(static_cast<float*>(g.c) + ic) = r;
        } else {
          bf16x4_t o = {(__bf16)r[0], (__bf16)r[1], (__bf16)r[2], (__bf16)r[3]};
          if constexpr (EPI == kEpiGelu) {
            *reinterpret_cast<bf16x4_t*>(static_cast<__bf16*>(g.aux) + (ab + mi * as + kRun * nj)) = o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (__bf16)gelu_tanh((float)o[e]);
          }
          *reinterpret_cast<bf16x4_t*>(static_cast<__bf16*>(g.c) + ic) = o;
        }
      }
    }
  }
}

template <int TN, int EPI>
__global__ __launch_bounds__(512, 1) void gemm_bf16_kernel(GemmArgs g) {
  // Half-tile slots [stage][A0, A1, B0, B1].  NT: [128 rows][64]; TN:
  // [64 k-rows][128].
  constexpr int HT = 128 * GBK;  // elements per half tile
  __shared__ __attribute__((aligned(1024))) uint16_t lds[2][4][HT];
  using T = Tile<TN ? 128 : 64>;

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w >> 2, wn = w & 3;  // rows 64 wm.. of each A half, cols 32 wn.. of each B half
  const int64_t m0 = (int64_t)blockIdx.y * GBM, n0 = (int64_t)blockIdx.x * GBN;
  const int nkb = (int)((g.K + GBK - 1) / GBK);

  // ---- DMA: 16 wave instructions (1 KiB each) per half tile, 2 per wave.
  int da[2], db[2];
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    da[x] = T::dma(lane, 2 * w + x, g.lda);
    db[x] = T::dma(lane, 2 * w + x, g.ldb);
  }
  // Half tile `half` of operand A (or B) of k-block kb; k-blocks past the end
  // (and rows past M, N or K) arrive as zeros.
  auto issue = [&](auto isb, int kb, int half, uint16_t* dst) {
    constexpr bool B = decltype(isb)::value != 0;
    const uint16_t* base = B ? g.b : g.a;
    const int64_t ld = B ? g.ldb : g.lda, o0 = (B ? n0 : m0) + 128 * half;
    const int64_t k0 = (int64_t)kb * GBK;
    int64_t valid = TN ? g.K - k0 : (B ? g.N : g.M) - o0;
    const int most = TN ? GBK : 128;
    if (kb >= nkb || valid < 0) valid = 0;
    const int n = valid < most ? (int)valid : most;
    const auto r = uniform_rsrc(reinterpret_cast<uint64_t>(base + (TN ? k0 * ld + o0 : o0 * ld + k0)), n * (int)(ld * 2));
#pragma unroll
    for (int x = 0; x < 2; ++x) lds_dma16(r, dst + (2 * w + x) * 512, B ? db[x] : da[x]);
  };

  // ---- operand reads
  int oa[TN ? 4 : 2], ob[TN ? 2 : 4];  // NT: A [k-step], B [tile][k-step]; TN: [16-column tile]
  if constexpr (!TN) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      oa[kk] = T::nat(lane, kk, wm * 64);  // + 16 mi rows: the swizzle's r4 flips with mi (below)
#pragma unroll
      for (int nj = 0; nj < 2; ++nj) ob[2 * nj + kk] = T::nat_perm(lane, kk, wn * 32, nj);
    }
  } else {
#pragma unroll
    for (int mi = 0; mi < 4; ++mi) oa[mi] = T::tr(lane, 4 * wm + mi);
#pragma unroll
    for (int nj = 0; nj < 2; ++nj) ob[nj] = T::tr(lane, 2 * wn + nj);
  }
  bf16x8 ao[4][2], bo[2][2][2];  // A: [16-row tile][k-step]; B: [half][16-column tile][k-step]
  auto read_a = [&](const uint16_t* t) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
      for (int mi = 0; mi < 4; ++mi) {
        // rows 16 mi on: r4 = mi & 1 flips chunk bit 2, i.e. swaps the two
        // k-steps' addresses
        if constexpr (!TN) ao[mi][kk] = ld_nat(t + 16 * mi * 64, oa[kk ^ (mi & 1)]);
        else ao[mi][kk] = ld_tr(t, oa[mi] + 32 * kk * 128, oa[mi] + (32 * kk + 16) * 128);
      }
    }
  };
  auto read_b = [&](const uint16_t* t, auto half) {
    constexpr int H = decltype(half)::value;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
      for (int nj = 0; nj < 2; ++nj) {
        if constexpr (!TN) bo[H][nj][kk] = ld_nat(t, ob[2 * nj + kk]);
        else bo[H][nj][kk] = ld_tr(t, ob[nj] + 32 * kk * 128, ob[nj] + (32 * kk + 16) * 128);
      }
    }
  };

  f32x4 acc[2][4][2][2];  // [A half][16-row tile][B half][16-column tile]
#pragma unroll
  for (int ha = 0; ha < 2; ++ha) {
#pragma unroll
    for (int mi = 0; mi < 4; ++mi) {
#pragma unroll
      for (int x = 0; x < 4; ++x) acc[ha][mi][x >> 1][x & 1] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  // Phase order.  With F the B half the k-block starts with and S the other:
  //   phase        0              1            2              3
  //   reads        A0             B_S          A1             B_S of kb + 1
  //   loads        A1 of kb + 1   B_F, kb + 2  A0, kb + 2     B_S, kb + 2
  //   quadrant     (A0, B_F)      (A0, B_S)    (A1, B_S)      (A1, B_F)
  // A phase is two barrier intervals, and the groups are one interval apart.
  // Slots: what phase P reads is in registers, in both groups, by the end of
  // the first group's interval 2 P + 2 (the lgkmcnt(0) that ends the MFMAs);
  // its slot is refilled from phase P + 2 (interval 2 P + 4 at the earliest).
  // Loads: what phase P + 1 reads was issued in phase P - 5; the vmcnt(10)
  // before phase P's first barrier leaves only the ten later instructions (two
  // per half tile) in flight, and the other group's wait ends an interval
  // before the first read.
  auto barrier = [] {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // The second half of a phase: the sixteen MFMAs of quadrant (ha, hb).
  auto mma = [&](auto HA, auto HB) {
    constexpr int ha = decltype(HA)::value, hb = decltype(HB)::value;
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(10));
    barrier();
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
      for (int mi = 0; mi < 4; ++mi) {
#pragma unroll
        for (int nj = 0; nj < 2; ++nj) acc[ha][mi][hb][nj] = mfma16(bo[hb][nj][kk], ao[mi][kk], acc[ha][mi][hb][nj]);
      }
    }
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_s_waitcnt(kWaitLds);  // also for reads that a later phase uses
    barrier();
  };
  // The four phases of k-block kb in stage PAR = kb % 2.  F is the B half it
  // starts with (read in the last phase of the k-block before).
  auto block = [&](int kb, auto par) {
    constexpr int PAR = decltype(par)::value, F = PAR, S = 1 - PAR;
    read_a(lds[PAR][0]);
    issue(IC<0>{}, kb + 1, 1, lds[1 - PAR][1]);
    mma(IC<0>{}, IC<F>{});
    read_b(lds[PAR][2 + S], IC<S>{});
    issue(IC<1>{}, kb + 2, F, lds[PAR][2 + F]);
    mma(IC<0>{}, IC<S>{});
    read_a(lds[PAR][1]);
    issue(IC<0>{}, kb + 2, 0, lds[PAR][0]);
    mma(IC<1>{}, IC<S>{});
    read_b(lds[1 - PAR][2 + S], IC<S>{});  // k-block kb + 1 starts with half S
    issue(IC<1>{}, kb + 2, S, lds[PAR][2 + S]);
    mma(IC<1>{}, IC<F>{});
  };

  // The loads of phases -7..-1, in order.
  issue(IC<1>{}, 0, 0, lds[0][2]);
  issue(IC<0>{}, 0, 0, lds[0][0]);
  issue(IC<1>{}, 0, 1, lds[0][3]);
  issue(IC<0>{}, 0, 1, lds[0][1]);
  issue(IC<1>{}, 1, 1, lds[1][3]);
  issue(IC<0>{}, 1, 0, lds[1][0]);
  issue(IC<1>{}, 1, 0, lds[1][2]);
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(10));
  barrier();
  read_b(lds[0][2], IC<0>{});
  __builtin_amdgcn_s_waitcnt(kWaitLds);
  if (w >= 4) barrier();  // the second group starts one interval later
  int kb = 0;
  for (; kb + 2 <= nkb; kb += 2) {
    block(kb, IC<0>{});
    block(kb + 1, IC<1>{});
  }
  if (kb < nkb) block(kb, IC<0>{});
  if (w < 4) barrier();
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));  // no LDS-DMA in flight past the end

#pragma unroll
  for (int ha = 0; ha < 2; ++ha) {
#pragma unroll
    for (int hb = 0; hb < 2; ++hb) {
      f32x4 c[4][2];
#pragma unroll
      for (int mi = 0; mi < 4; ++mi) {
#pragma unroll
        for (int nj = 0; nj < 2; ++nj) c[mi][nj] = acc[ha][mi][hb][nj];
      }
      store_tile<TN, EPI, 4>(g, m0 + 128 * ha + 64 * wm, n0 + 128 * hb + 32 * wn, c);
    }
  }
}

// The same product on BT x BT tiles (128 or 64), one k-block per barrier, NS
// stages of LDS.  128: 8 waves (2 x 4) of 64 x 32; 64: 4 waves (2 x 2) of
// 32 x 32.  Few waves per SIMD leave the instruction stream as the bound: the
// next k-block's operand reads sit between this one's MFMAs (0.50 -> 0.39 us
// per k-block for 128, 0.25 -> 0.23 for 64, on an otherwise idle chip).
template <int TN, int EPI, int BT>
__global__ __launch_bounds__(BT == 128 ? 512 : 256, 1) void gemm_small_kernel(GemmArgs g) {
  constexpr int NW = BT == 128 ? 8 : 4, WN = BT / 32, MI = BT == 128 ? 4 : 2;
  constexpr int NS = BT == 128 ? 5 : 10;  // 160 KiB
  constexpr int TILE = BT * GBK, DPW = TILE / 512 / NW;  // DMA instructions per wave, operand and k-block
  __shared__ __attribute__((aligned(1024))) uint16_t lds[NS][2][TILE];
  using T = Tile<TN ? BT : 64>;

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w / WN, wn = w % WN;
  const int64_t m0 = (int64_t)blockIdx.y * BT, n0 = (int64_t)blockIdx.x * BT;
  const int nkb = (int)((g.K + GBK - 1) / GBK);
  int da[DPW], db[DPW];
#pragma unroll
  for (int x = 0; x < DPW; ++x) {
    da[x] = T::dma(lane, DPW * w + x, g.lda);
    db[x] = T::dma(lane, DPW * w + x, g.ldb);
  }
  // K-blocks are loaded in order, so scalar state walks A and B.  Rows past M
  // or N (NT) and K (TN), and k-blocks past the end, arrive as zeros.
  uint64_t pa = uniform_u64(reinterpret_cast<uint64_t>(g.a + (TN ? m0 : m0 * g.lda)));
  uint64_t pb = uniform_u64(reinterpret_cast<uint64_t>(g.b + (TN ? n0 : n0 * g.ldb)));
  const uint64_t sa_step = (uint64_t)(TN ? GBK * g.lda : GBK) * 2, sb_step = (uint64_t)(TN ? GBK * g.ldb : GBK) * 2;
  const int ra = (int)(g.lda * 2), rb = (int)(g.ldb * 2);  // bytes per row
  const int na = (int)(g.M - m0 < BT ? g.M - m0 : BT) * ra, nb = (int)(g.N - n0 < BT ? g.N - n0 : BT) * rb;
  int left = (int)g.K;  // k not yet loaded
  int slot_in = 0;      // element offset of the slot the next k-block goes to
  uint16_t* const base = &lds[0][0][0];
  auto issue = [&] {
    const int nk = left < GBK ? (left < 0 ? 0 : left) : GBK;
    const auto rsa = uniform_rsrc(pa, TN ? nk * ra : (left > 0 ? na : 0));
    const auto rsb = uniform_rsrc(pb, TN ? nk * rb : (left > 0 ? nb : 0));
    uint16_t* dst = base + slot_in;
#pragma unroll
    for (int x = 0; x < DPW; ++x) {
      lds_dma16(rsa, dst + (DPW * w + x) * 512, da[x]);
      lds_dma16(rsb, dst + TILE + (DPW * w + x) * 512, db[x]);
    }
    pa += sa_step;
    pb += sb_step;
    left -= GBK;
    slot_in = slot_in == (NS - 1) * 2 * TILE ? 0 : slot_in + 2 * TILE;
  };
  // Operand offsets, as in the large kernel.  Transposed reads of a [64][64]
  // tile: rows 16.. of each 32 (r4 = 1) flip chunk bit 2, i.e. column block 2.
  int oa[TN ? MI : 2], ob[TN ? 2 : 4], oah[TN ? MI : 1], obh[TN ? 2 : 1];
  if constexpr (!TN) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      oa[kk] = T::nat(lane, kk, wm * 16 * MI);
#pragma unroll
      for (int nj = 0; nj < 2; ++nj) ob[2 * nj + kk] = T::nat_perm(lane, kk, wn * 32, nj);
    }
  } else {
    constexpr int flip = BT == 64 ? 2 : 0;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
      oa[mi] = T::tr(lane, MI * wm + mi);
      oah[mi] = T::tr(lane, (MI * wm + mi) ^ flip) + 16 * BT;
    }
#pragma unroll
    for (int nj = 0; nj < 2; ++nj) {
      ob[nj] = T::tr(lane, 2 * wn + nj);
      obh[nj] = T::tr(lane, (2 * wn + nj) ^ flip) + 16 * BT;
    }
  }
  f32x4 acc[MI][2];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) acc[mi][0] = acc[mi][1] = f32x4{0.f, 0.f, 0.f, 0.f};

  bf16x8 ao[2][MI][2], bo[2][2][2];
  int slot_rd = 0;
  auto read = [&](auto set) {  // operands of the next k-block
    constexpr int X = decltype(set)::value;
    const uint16_t* sa = base + slot_rd;
    const uint16_t* sb = sa + TILE;
    slot_rd = slot_rd == (NS - 1) * 2 * TILE ? 0 : slot_rd + 2 * TILE;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) {
        if constexpr (!TN) ao[X][mi][kk] = ld_nat(sa + 16 * mi * 64, oa[kk ^ (mi & 1)]);
        else ao[X][mi][kk] = ld_tr(sa, oa[mi] + 32 * kk * BT, oah[mi] + 32 * kk * BT);
      }
#pragma unroll
      for (int nj = 0; nj < 2; ++nj) {
        if constexpr (!TN) bo[X][nj][kk] = ld_nat(sb, ob[2 * nj + kk]);
        else bo[X][nj][kk] = ld_tr(sb, ob[nj] + 32 * kk * BT, obh[nj] + 32 * kk * BT);
      }
    }
  };
  // K-block kb, its operands in set X: those of kb + 1 are read under its
  // MFMAs.  At its start kb + 1 has landed (up to NS - 3 later k-blocks may
  // still be loading), and every wave is done with kb - 1, whose slot takes
  // kb + NS - 1.
  auto step = [&](auto set) {
    constexpr int X = decltype(set)::value;
    __builtin_amdgcn_s_waitcnt(waitcnt_vm((NS - 3) * 2 * DPW));
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    issue();
    read(IC<1 - X>{});
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
        for (int nj = 0; nj < 2; ++nj) acc[mi][nj] = mfma16(bo[X][nj][kk], ao[X][mi][kk], acc[mi][nj]);
      }
    }
    constexpr int kReads = (TN ? 2 : 1) * (2 * MI + 4);
#pragma unroll
    for (int x = 0; x < 4 * MI; ++x) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, (kReads + 4 * MI - 1) / (4 * MI), 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int x = 0; x < NS - 1; ++x) issue();
  __builtin_amdgcn_s_waitcnt(waitcnt_vm((NS - 2) * 2 * DPW));
  __syncthreads();
  read(IC<0>{});
  int kb = 0;
  for (; kb + 2 <= nkb; kb += 2) {
    step(IC<0>{});
    step(IC<1>{});
  }
  if (kb < nkb) step(IC<0>{});
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));  // no LDS-DMA in flight past the end
  store_tile<TN, EPI, MI>(g, m0 + 16 * MI * wm, n0 + 32 * wn, acc);
}

template <int TN, int EPI>
hipError_t launch_tile(const GemmArgs& g, int bt, hipStream_t stream) {
  const dim3 grid((unsigned)((g.N + bt - 1) / bt), (unsigned)((g.M + bt - 1) / bt));
  if (bt == 256) hipLaunchKernelGGL((gemm_bf16_kernel<TN, EPI>), grid, dim3(512), 0, stream, g);
  else if (bt == 128) hipLaunchKernelGGL((gemm_small_kernel<TN, EPI, 128>), grid, dim3(512), 0, stream, g);
  else hipLaunchKernelGGL((gemm_small_kernel<TN, EPI, 64>), grid, dim3(256), 0, stream, g);
  return hipGetLastError();
}

template <int TN>
hipError_t launch_epi(const GemmArgs& g, int bt, hipStream_t stream) {
  switch (g.epi) {
    case kEpiBf16: return launch_tile<TN, kEpiBf16>(g, bt, stream);
    case kEpiAddBf16: return launch_tile<TN, kEpiAddBf16>(g, bt, stream);
    case kEpiGelu: return launch_tile<TN, kEpiGelu>(g, bt, stream);
    case kEpiDGelu: return launch_tile<TN, kEpiDGelu>(g, bt, stream);
    case kEpiAccF32: return launch_tile<TN, kEpiAccF32>(g, bt, stream);
    case kEpiF32: return launch_tile<TN, kEpiF32>(g, bt, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_gemm_bf16(const GemmArgs& g, hipStream_t stream) {
  if (g.M <= 0 || g.N <= 0 || g.K <= 0) return hipErrorInvalidValue;
  // The tile with the least estimated time: rounds of tiles over the CUs (one
  // workgroup each, by LDS) times (k-blocks x time per k-block + prologue and
  // epilogue), in ns as measured.  At 256 CUs: 1000 x 1024 x 4096 takes 69 /
  // 31 / 17 us on 256 / 128 / 64 tiles, 1000 x 4096 x 1024 (GELU) 34 / 17 / 24,
  // 2500 x 9216 x 2304 105 / 130 / 220, 4000 x 2048 x 8192 133 / 140 / 212.
  // Tile rows are a grid's second dimension, which holds kMaxGridYZ of them.
  struct Option { int bt; double kb, fixed; };
  constexpr Option kTiles[3] = {{256, 1000, 8000}, {128, 500, 6000}, {64, 230, 2500}};
  const double cus = device_cus(), nkb = (double)((g.K + GBK - 1) / GBK);
  int bt = 0;
  double best = 0;
  for (const Option& t : kTiles) {
    if (bt && (g.M + t.bt - 1) / t.bt > kMaxGridYZ) continue;
    const double tiles = (double)((g.M + t.bt - 1) / t.bt) * (double)((g.N + t.bt - 1) / t.bt);
    const double ns = __builtin_ceil(tiles / cus) * (nkb * t.kb + t.fixed);
    if (!bt || ns < best) {
      bt = t.bt;
      best = ns;
    }
  }
  // Few k-blocks of TN with a write-only epilogue on 256 tiles are bound by
  // their stores (gemm_tn_short.hip has the figures; even at about 16).
  if (g.tn && bt == 256 && nkb <= 16 && (g.epi == kEpiBf16 || g.epi == kEpiF32)) return launch_gemm_tn_short(g, stream);
  return g.tn ? launch_epi<1>(g, bt, stream) : launch_epi<0>(g, bt, stream);
}

}  // namespace sppo
