// Backward of one chunk of sequence-chunked causal attention, bf16 in / fp32
// accumulate, for gfx950 (MI355X).  The reverse walk over chunks (Sec. 5.2
// of SPPO) calls this for i = N-1..0; dK/dV accumulate across calls in fp32.
//
// Three kernels, all on the caller's stream:
//   bwd_pre   -Delta_r = -<dO_r, O_r> and LSE2_r = LSE_r * log2(e) into the
//             context's workspace (HBM-bound); -Delta is the initial value
//             of the dP accumulators, so the MFMAs produce dP - Delta
//   bwd_dkdv  one workgroup per 128 keys of one KV head at a time (4 waves x
//             32 keys, lane <-> key, K/V fragments in registers); the chunk's
//             query rows of every head of the GQA group stream through LDS in
//             32-row sub-blocks, and per sub-block
//               S = Q K^T, dP = dO V^T, P = exp2(S C - LSE2), dS = P (dP - Delta)
//               dV^T += dO^T P,  dK^T += Q^T dS
//             The kernel is persistent (as many workgroups as the CUs
//             hold at once, one per CU at its register use): each XCD
//             takes key tiles from its own queue, in the XCD-grouped order,
//             and once it is empty from the other XCDs' queues, so XCDs that
//             run faster than others do more of the work.
//   bwd_dq    one workgroup per 128 query rows of one head (lane <-> query);
//             keys stream through LDS in 32-key sub-blocks, and per sub-block
//               S^T = K Q^T, dP^T = V dO^T, dS^T as above, dQ^T += K^T dS^T
// Both stream their sub-blocks through a six-slot LDS ring by LDS-DMA, five
// sub-blocks ahead, one barrier per sub-block, and software-pipeline them:
// the MFMAs of sub-block n+1's S and dP run while the VALU forms sub-block
// n's P and dS, then the gradient MFMAs of sub-block n run.  The order of
// every step is fixed with sched_barrier, so operand reads sit a few MFMAs
// ahead of their use.  Sub-blocks that need the causal mask are done one at
// a time, outside the pipeline.  Grids too small for the chip take the split
// kernels further down.
//
// The products here are 16x16x32 MFMAs; the wide kernels of head size 128, and
// dQ of 64 with one workgroup on most CUs, are in attn_bwd_bf16_mfma32.hip on
// 32x32x16.  Both occupy the matrix pipe for as many cycles a step.  The
// smaller form takes less energy, so the clock rises, but a wave alone on its
// SIMD issues twice the MFMAs: at D = 64, with half the MFMAs per exponential,
// that gains (dK/dV 1-5%, dQ over several passes up to 5%), at 128 it loses.
// What is left is the one wave's instruction stream: moving half the
// exponentials from the S/dP phase to the gradient phase changed nothing.
#include "bwd_tiles.h"
#include "sppo_kernels.h"
#include "tile_common.h"

namespace sppo {
namespace {

// S or dP of a 32 x 32 sub-block: 16 x 16 tiles, [row tile][column tile].
struct S4 {
  f32x4 x[2][2];
};

// ------------------------------------------------------------------ Delta
template <int D>
__global__ __launch_bounds__(256) void bwd_pre_bf16_kernel(ChunkArgs a) {
  constexpr int LPI = D / 8;  // lanes per (b, r, h) row, 8 bf16 each
  const int64_t s = a.c1 - a.c0;
  const int64_t nrows = a.B * s * a.Hq;
  const int64_t item = ((int64_t)blockIdx.x * 256 + threadIdx.x) / LPI;
  const int sub = threadIdx.x % LPI;
  // A backward call's queues start from zero (the dK/dV launches leave them
  // so; cleared here as well, ahead of every call's first dK/dV launch).
  if (blockIdx.x == 0 && threadIdx.x < 9) atomicExch(a.tiles + threadIdx.x, 0);
  float acc = 0.f;
  if (item < nrows) {
    const u32x4 ov = ld_global16(static_cast<const uint16_t*>(a.o) + item * D + 8 * sub);
    const u32x4 dv = ld_global16(static_cast<const uint16_t*>(a.dout) + item * D + 8 * sub);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc += __uint_as_float(ov[e] << 16) * __uint_as_float(dv[e] << 16);
      acc += __uint_as_float(ov[e] & 0xffff0000u) * __uint_as_float(dv[e] & 0xffff0000u);
    }
  }
#pragma unroll
  for (int off = LPI / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if (item < nrows && sub == 0) {
    const int64_t h = item % a.Hq;
    const int64_t rr = (item / a.Hq) % s;
    const int64_t b = item / (a.Hq * s);
    const int64_t idx = (b * a.Hq + h) * s + rr;
    a.delta[idx] = -acc;
    a.lse2[idx] = a.lse[idx] * kLog2e;
  }
}

// ------------------------------------------------------------------ dK dV
__global__ __launch_bounds__(256, 1) void bwd_dkdv_bf16_kernel(ChunkArgs a) {
  constexpr int D = 64;
  using T = Tile<D>;
  constexpr int P = T::P, NK = D / 32, ND = D / 16;  // k-steps of S and dP, d tiles
  constexpr int IPWQ = (kSB / T::RPI) / 4;  // DMA instructions per wave per tensor per sub-block
  static_assert(IPWQ >= 1 && IPWQ * 4 * T::RPI == kSB, "sub-block splits over 4 waves");
  constexpr int DMA_PER_SB = 2 * IPWQ + 1;  // Q, dO, and one for the [LSE2 | -Delta] record
  // One LDS object per ring slot, [Q rows | dO rows], and the slots' records,
  // [LSE2 (32 floats) | -Delta (32 floats)], in an array of their own at the
  // bottom of LDS, where the broadcast reads take their offsets as immediates.
  constexpr int SLOT = 2 * kSB * P;
  __shared__ __attribute__((aligned(1024))) float REC[kRing][64];
  __shared__ __attribute__((aligned(1024))) uint16_t R0[SLOT], R1[SLOT], R2[SLOT], R3[SLOT], R4[SLOT], R5[SLOT];
  auto slot = [&](auto I) -> uint16_t* {
    constexpr int i = decltype(I)::value;
    if constexpr (i == 0) return R0; else if constexpr (i == 1) return R1; else if constexpr (i == 2) return R2;
    else if constexpr (i == 3) return R3; else if constexpr (i == 4) return R4; else return R5;
  };
  auto qbuf = [&](auto I) -> uint16_t* { return slot(I); };
  auto obuf = [&](auto I) -> uint16_t* { return slot(I) + kSB * P; };
  auto lbuf = [&](auto I) -> float* { return REC[decltype(I)::value]; };

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  // Key tiles in the XCD-grouped order (the tiles of a KV head one after
  // another): XCD x owns positions [x T / 8, (x+1) T / 8) of the T tiles.
  // Thread 0 takes the next position from this XCD's queue, or when that
  // is used up from the next XCD's, and hands it to the workgroup through
  // LDS; -1 when every queue is used up.
  const int nx = (int)((a.kv1 - a.kv0 + kKvKeys - 1) / kKvKeys), ny = a.Hkv;
  const int total = nx * ny * (int)a.B;
  __shared__ int s_tile;
  uint32_t xcc;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
  for (;;) {
  if (tid == 0) {
    int t = -1;
    for (int y = 0; y < 8 && t < 0; ++y) {
      const int x = (int)((xcc + y) & 7);
      const int lo = (int)((int64_t)x * total / 8), hi = (int)((int64_t)(x + 1) * total / 8);
      if (lo < hi) {
        const int n = atomicAdd(a.tiles + x, 1);
        if (lo + n < hi) t = lo + n;
      }
    }
    s_tile = t;
  }
  __syncthreads();
  const int tile = s_tile;
  if (tile < 0) break;
  const GridPos gp{tile % nx, (tile / nx) % ny, tile / (nx * ny)};
  const int hk = gp.y;
  const int64_t b = gp.z;
  const int G = a.Hq / a.Hkv;
  const int64_t c0 = a.c0, c1 = a.c1, s = c1 - c0;
  const int64_t kv1 = a.kv1;
  const int64_t k0 = a.kv0 + (int64_t)gp.x * kKvKeys;
  const int64_t j = k0 + 32 * w + l16;  // this lane's keys: j and j + 16
  const float C = a.scale * kLog2e;

  // Query sub-blocks (chunk-local, 32 rows from c0): [sb_begin, sb_u) need
  // the mask, [sb_u, nsb) see every key of the workgroup.
  const int nsb = (int)((s + kSB - 1) / kSB);
  const int sb_begin = k0 > c0 ? (int)((k0 - c0) / kSB) : 0;
  int sb_u = (int)((k0 + kKvKeys - c0 + kSB - 1) / kSB);
  if (sb_u > nsb) sb_u = nsb;
  if (sb_u < sb_begin) sb_u = sb_begin;
  const int N = nsb - sb_u;  // unmasked sub-blocks per head

  int nat[NK];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) nat[kk] = T::nat(lane, kk, 0);
  int tro[ND];
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) tro[dt] = T::tr(lane, dt);
  const int64_t qstride = (int64_t)a.Hq * D;
  int dmaq[IPWQ];
#pragma unroll
  for (int x = 0; x < IPWQ; ++x) dmaq[x] = T::dma(lane, w * IPWQ + x, qstride);
  // The [LSE2 | -Delta] record: waves 0, 1 load LSE2 rows 0..15, 16..31,
  // waves 2, 3 -Delta, 16 lanes each.
  const int dmal = (16 * (w & 1) + (lane & 15)) * 4;
  const float* lsrc = (w < 2) ? a.lse2 : a.delta;
  const int ldst = 32 * (w >> 1) + 16 * (w & 1);

  bf16x8 kf[2][NK], vf[2][NK];
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
    const int64_t jk = j + 16 * kt;
    const int64_t off = ((b * a.S + jk) * a.Hkv + hk) * D;
    const uint16_t* krow = static_cast<const uint16_t*>(a.k) + off;
    const uint16_t* vrow = static_cast<const uint16_t*>(a.v) + off;
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      kf[kt][kk] = jk < kv1 ? as_bf16x8(ld_global16(krow + 32 * kk + 8 * g)) : bf16x8{};
      vf[kt][kk] = jk < kv1 ? as_bf16x8(ld_global16(vrow + 32 * kk + 8 * g)) : bf16x8{};
    }
  }
  f32x4 dk[ND][2], dv[ND][2];  // dK^T, dV^T: [d tile][key tile]
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) dk[dt][0] = dk[dt][1] = dv[dt][0] = dv[dt][1] = f32x4{0.f, 0.f, 0.f, 0.f};

  // DMA of query sub-block sb of head h into a slot; rows past the chunk load
  // zeros, so every call issues DMA_PER_SB instructions per wave.
  auto issue = [&](int h, int sb, uint16_t* qd, uint16_t* od, float* ld) {
    const int64_t r0 = (int64_t)sb * kSB;
    const int64_t valid = s - r0;
    const int64_t tile0 = (b * s + r0) * a.Hq + h;
    const auto rq = tile_rsrc(static_cast<const uint16_t*>(a.q) + tile0 * D, valid, kSB, qstride);
    const auto ro = tile_rsrc(static_cast<const uint16_t*>(a.dout) + tile0 * D, valid, kSB, qstride);
#pragma unroll
    for (int x = 0; x < IPWQ; ++x) {
      lds_dma16(rq, qd + (w * IPWQ + x) * 512, dmaq[x]);
      lds_dma16(ro, od + (w * IPWQ + x) * 512, dmaq[x]);
    }
    const int64_t nrec = valid <= 0 ? 0 : (valid < kSB ? valid : kSB);
    const uint64_t lb = reinterpret_cast<uint64_t>(lsrc + (b * a.Hq + h) * s + r0);
    const uint64_t lbu = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(lb >> 32)) << 32) |
                         (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)lb);
    const auto rl = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<float*>(lbu), (short)0,
                                                      __builtin_amdgcn_readfirstlane((int)(nrec * 4)), kBufferFlags);
    if (lane < 16) lds_dma4(rl, ld + ldst, dmal);
  };
  // The unmasked stream of a head issues its sub-blocks in order, so the
  // scalar state below walks Q, dO and the record one sub-block per call
  // (no per-call index arithmetic).  Past the chunk end the byte counts drop
  // to zero and the DMA fills zeros.
  const int64_t sbb = (int64_t)kSB * qstride * 2;  // bytes per sub-block of Q or dO
  const int qrow_bytes = (int)(qstride * 2);
  uint64_t qa = 0, oa = 0, la = 0;
  int rem = 0;
  auto stream_begin = [&](int h) {
    const int64_t r0 = (int64_t)sb_u * kSB;
    const int64_t tile0 = (b * s + r0) * a.Hq + h;
    qa = uniform_u64(reinterpret_cast<uint64_t>(static_cast<const uint16_t*>(a.q) + tile0 * D));
    oa = uniform_u64(reinterpret_cast<uint64_t>(static_cast<const uint16_t*>(a.dout) + tile0 * D));
    la = uniform_u64(reinterpret_cast<uint64_t>(lsrc + (b * a.Hq + h) * s + r0));
    rem = (int)(s - r0);
  };
  auto stream_issue = [&](uint16_t* qd, uint16_t* od, float* ld) {
    const int n = rem <= 0 ? 0 : (rem < kSB ? rem : kSB);
    const auto rq = uniform_rsrc(qa, n * qrow_bytes);
    const auto ro = uniform_rsrc(oa, n * qrow_bytes);
#pragma unroll
    for (int x = 0; x < IPWQ; ++x) {
      lds_dma16(rq, qd + (w * IPWQ + x) * 512, dmaq[x]);
      lds_dma16(ro, od + (w * IPWQ + x) * 512, dmaq[x]);
    }
    const auto rl = uniform_rsrc(la, n * 4);
    if (lane < 16) lds_dma4(rl, ld + ldst, dmal);
    qa += sbb;
    oa += sbb;
    la += kSB * 4;
    rem -= kSB;
  };
  // Natural operand of the 16 rows 16 t.. of a sub-block, k-step kk, and
  // transposed operand of its 32 rows, d tile dt (rows 16.. swap the two
  // k-steps' chunks and column blocks dt, dt ^ 2).
  auto nat_rd = [&](const uint16_t* X, int t, int kk) { return ld_nat(X + 16 * t * P, nat[kk ^ t]); };
  auto tr_rd = [&](const uint16_t* X, int dt) { return ld_tr(X, tro[dt], tro[dt ^ 2] + 16 * P); };
  // LSE2 and -Delta (the initial value of the dP accumulators) of this lane's
  // rows 16 qt + 4 g + 0..3 of a sub-block, from its record.
  auto rec_rd = [&](const float* ld, int qt) { return *reinterpret_cast<const f32x4*>(ld + 16 * qt + 4 * g); };
  // S = Q K^T and dP - Delta = dO V^T - Delta of one sub-block (lane <-> key).
  auto sdp = [&](const uint16_t* Qs, const uint16_t* Os, const f32x4 (&nd)[2], S4& sv, S4& dp) {
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
        const bf16x8 qx = nat_rd(Qs, qt, kk), ox = nat_rd(Os, qt, kk);
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
          sv.x[qt][kt] = mfma16(qx, kf[kt][kk], kk == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sv.x[qt][kt]);
          dp.x[qt][kt] = mfma16(ox, vf[kt][kk], kk == 0 ? nd[qt] : dp.x[qt][kt]);
        }
      }
    }
  };
  // dV^T += dO^T P, dK^T += Q^T dS of one sub-block.
  auto grads = [&](const uint16_t* Qs, const uint16_t* Os, const bf16x8 (&pb)[2], const bf16x8 (&dsb)[2]) {
#pragma unroll
    for (int dt = 0; dt < ND; ++dt) {
      const bf16x8 ox = tr_rd(Os, dt), qx = tr_rd(Qs, dt);
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        dv[dt][kt] = mfma16(ox, pb[kt], dv[dt][kt]);
        dk[dt][kt] = mfma16(qx, dsb[kt], dk[dt][kt]);
      }
    }
  };

  // Heads of the GQA group one after another, each in row order: the masked
  // sub-blocks one at a time, then the unmasked stream.  A key's dK/dV thus
  // sums its rows in the same order whatever range of keys a launch covers
  // (rows before a key add exact zeros).
  for (int hh = 0; hh < G; ++hh) {
    const int h = hk * G + hh;
    // ---- sub-blocks with the causal mask, one at a time (slot 0)
    for (int sb = sb_begin; sb < sb_u; ++sb) {
      __syncthreads();
      issue(h, sb, qbuf(IC<0>{}), obuf(IC<0>{}), lbuf(IC<0>{}));
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
      __syncthreads();
      const float* ld = lbuf(IC<0>{});
      const f32x4 nd[2] = {rec_rd(ld + 32, 0), rec_rd(ld + 32, 1)}, lg[2] = {rec_rd(ld, 0), rec_rd(ld, 1)};
      S4 sv, dp;
      sdp(qbuf(IC<0>{}), obuf(IC<0>{}), nd, sv, dp);
      const int64_t r0g = c0 + (int64_t)sb * kSB;  // global row of the sub-block's first row
      bf16x8 pb[2], dsb[2];
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        float p[8], ds[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int qt = e >> 2, v = e & 3;
          float pv = fast_exp2(sv.x[qt][kt][v] * C - lg[qt][v]);
          if (j + 16 * kt > r0g + 16 * qt + 4 * g + v) pv = 0.f;  // key j sees row r iff j <= r
          p[e] = pv;
          ds[e] = pv * dp.x[qt][kt][v];
        }
        pb[kt] = pack_bf16x8(p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7]);
        dsb[kt] = pack_bf16x8(ds[0], ds[1], ds[2], ds[3], ds[4], ds[5], ds[6], ds[7]);
      }
      grads(qbuf(IC<0>{}), obuf(IC<0>{}), pb, dsb);
    }

    // ---- unmasked stream, software pipelined
    if (N == 0) continue;
    __syncthreads();  // every slot is free
    stream_begin(h);
    stream_issue(qbuf(IC<0>{}), obuf(IC<0>{}), lbuf(IC<0>{}));
    stream_issue(qbuf(IC<1>{}), obuf(IC<1>{}), lbuf(IC<1>{}));
    stream_issue(qbuf(IC<2>{}), obuf(IC<2>{}), lbuf(IC<2>{}));
    stream_issue(qbuf(IC<3>{}), obuf(IC<3>{}), lbuf(IC<3>{}));
    stream_issue(qbuf(IC<4>{}), obuf(IC<4>{}), lbuf(IC<4>{}));
    // Sub-blocks 0 and 1 land before the loop and step 0's first natural
    // operands are read here; later steps get theirs from the end of the
    // previous B phase.
    __builtin_amdgcn_s_waitcnt(waitcnt_vm((kAhead - 2) * DMA_PER_SB));
    __syncthreads();
    S4 sa, da, sb2, db2;
    f32x4 nd[2] = {rec_rd(lbuf(IC<0>{}) + 32, 0), rec_rd(lbuf(IC<0>{}) + 32, 1)};
    sdp(qbuf(IC<0>{}), obuf(IC<0>{}), nd, sa, da);
    // Natural operand o of a sub-block's A phase: k-step o / 4, row tile
    // (o / 2) % 2, Q (o even) or dO (o odd).
    auto nat_of = [&](const uint16_t* Qx, const uint16_t* Ox, int o) {
      return nat_rd((o & 1) ? Ox : Qx, (o >> 1) & 1, o >> 2);
    };
    bf16x8 opn[4];
    f32x4 lg[2] = {rec_rd(lbuf(IC<0>{}), 0), rec_rd(lbuf(IC<0>{}), 1)};
#pragma unroll
    for (int o = 0; o < 4; ++o) opn[o] = nat_of(qbuf(IC<1>{}), obuf(IC<1>{}), o);
    nd[0] = rec_rd(lbuf(IC<1>{}) + 32, 0);
    nd[1] = rec_rd(lbuf(IC<1>{}) + 32, 1);
    // Step n in slot I: A(n) reads slot I+1 (natural); B(n) reads slot I
    // (transposed) and, in its last slots, A(n+1)'s first natural operands and
    // -Delta from slot I+2 and LSE2 of sub-block n+1.  At its start sub-blocks
    // n+1 and n+2 have landed (only n+3, n+4 may still be loading); then
    // sub-block n+5 goes to slot I+5 = I-1, free since step n-1.  nd holds
    // -Delta of sub-block n+1 and lg LSE2 of sub-block n on entry.
    auto step = [&](auto sl, S4& scur, S4& dcur, S4& snext, S4& dnext) {
      constexpr int I = decltype(sl)::value;
      constexpr int I1 = (I + 1) % kRing, I2 = (I + 2) % kRing, I5 = (I + kAhead) % kRing;
      __builtin_amdgcn_s_waitcnt(waitcnt_vm((kAhead - 3) * DMA_PER_SB));
      __syncthreads();
      stream_issue(qbuf(IC<I5>{}), obuf(IC<I5>{}), lbuf(IC<I5>{}));
      const uint16_t* Qn = qbuf(IC<I1>{});
      const uint16_t* On = obuf(IC<I1>{});
      const uint16_t* Qc = qbuf(IC<I>{});
      const uint16_t* Oc = obuf(IC<I>{});
      // A(n): operand o (NA of them) feeds the two MFMAs (key tiles) of S(n+1)
      // (o even) or dP(n+1) (o odd); it is read four operands ahead.  The VALU
      // turns the 16 elements of S(n), dP(n) into P(n), dS(n) (key tile by key
      // tile), element i beside operand i / (16 / NA).
      constexpr int NA = 4 * NK, EPM = 16 / NA;
      bf16x8 op[NA];
#pragma unroll
      for (int o = 0; o < 4; ++o) op[o] = opn[o];
      float p[16], ds[16];
      uint32_t pk[4][4];  // P and dS of key tile 0, then 1, packed in pairs
      bf16x8 pb[2], dsb[2];
      // B(n): operand jj feeds the two MFMAs of dV (jj even) or dK (jj odd) for
      // d tile jj / 2; it is read three operands ahead (the first three in the
      // last slots of A(n), which read nothing else).
      constexpr int NB = 2 * ND;
      auto tr_op = [&](int jj) { return tr_rd((jj & 1) ? Qc : Oc, jj >> 1); };
      bf16x8 top[NB];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int o = i / EPM;
        auto a_mfma = [&](int kt) {
          const int kk = o >> 2, qt = (o >> 1) & 1;
          if (o & 1) dnext.x[qt][kt] = mfma16(op[o], vf[kt][kk], kk == 0 ? nd[qt] : dnext.x[qt][kt]);
          else snext.x[qt][kt] = mfma16(op[o], kf[kt][kk], kk == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : snext.x[qt][kt]);
        };
        if (i % EPM == 0) a_mfma(0);
        __builtin_amdgcn_sched_barrier(0);
        // Element i's exp, element i-1's dS: an exp's result is not read by the
        // next instruction (that would cost a wait state).
        const int kt = i >> 3, qt = (i >> 2) & 1, v = i & 3;
        p[i] = fast_exp2(scur.x[qt][kt][v] * C - lg[qt][v]);
        if (i % EPM == EPM / 2) {
          __builtin_amdgcn_sched_barrier(0);
          a_mfma(1);
          __builtin_amdgcn_sched_barrier(0);
          if (o + 4 < NA) op[o + 4] = nat_of(Qn, On, o + 4);
          else if (o + 4 - NA < 3) top[o + 4 - NA] = tr_op(o + 4 - NA);
        }
        if (i > 0) ds[i - 1] = p[i - 1] * dcur.x[((i - 1) >> 2) & 1][(i - 1) >> 3][(i - 1) & 3];
        if (i >= 8 && i < 12) {  // P and dS of key tile 0 to bf16, two elements of each a slot
          const int e = 2 * (i - 8);
          pk[0][i - 8] = pack_bf16x2(p[e], p[e + 1]);
          pk[1][i - 8] = pack_bf16x2(ds[e], ds[e + 1]);
        }
        if (i >= 12) {
          const int e = 8 + 2 * (i - 12);
          if (e + 1 < i) pk[2][i - 12] = pack_bf16x2(p[e], p[e + 1]);
          if (e + 1 < i) pk[3][i - 12] = pack_bf16x2(ds[e], ds[e + 1]);
        }
        if (i % EPM == EPM - 1) __builtin_amdgcn_sched_barrier(0);
      }
      pb[0] = as_bf16x8(u32x4{pk[0][0], pk[0][1], pk[0][2], pk[0][3]});
      dsb[0] = as_bf16x8(u32x4{pk[1][0], pk[1][1], pk[1][2], pk[1][3]});
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int jj = 0; jj < NB; ++jj) {
        const int dt = jj >> 1;
        auto b_mfma = [&](int kt) {
          if (jj & 1) dk[dt][kt] = mfma16(top[jj], dsb[kt], dk[dt][kt]);
          else dv[dt][kt] = mfma16(top[jj], pb[kt], dv[dt][kt]);
        };
        b_mfma(0);
        __builtin_amdgcn_sched_barrier(0);
        if (jj == 0) {  // the rest of key tile 1
          pk[2][3] = pack_bf16x2(p[14], p[15]);
          pb[1] = as_bf16x8(u32x4{pk[2][0], pk[2][1], pk[2][2], pk[2][3]});
          ds[15] = p[15] * dcur.x[1][1][3];
        }
        if (jj == 1) {
          pk[3][3] = pack_bf16x2(ds[14], ds[15]);
          dsb[1] = as_bf16x8(u32x4{pk[3][0], pk[3][1], pk[3][2], pk[3][3]});
        }
        __builtin_amdgcn_sched_barrier(0);
        b_mfma(1);
        __builtin_amdgcn_sched_barrier(0);
        if (jj + 3 < NB) {
          top[jj + 3] = tr_op(jj + 3);
        } else {  // A(n+1)'s first natural operands and -Delta, from sub-block n+2; LSE2 of n+1
          const int m0 = jj + 3 - NB;
          opn[m0] = nat_of(qbuf(IC<I2>{}), obuf(IC<I2>{}), m0);
          if (m0 < 2) lg[m0] = rec_rd(lbuf(IC<I1>{}), m0);
          if (m0 == 2) {
            opn[3] = nat_of(qbuf(IC<I2>{}), obuf(IC<I2>{}), 3);
            nd[0] = rec_rd(lbuf(IC<I2>{}) + 32, 0);
            nd[1] = rec_rd(lbuf(IC<I2>{}) + 32, 1);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // Past the last sub-block A still computes S, dP of the (zero) next slot;
    // they are never used.
    for (int n = 0; n < N; n += kRing) {
      step(IC<0>{}, sa, da, sb2, db2);
      if (n + 1 >= N) break;
      step(IC<1>{}, sb2, db2, sa, da);
      if (n + 2 >= N) break;
      step(IC<2>{}, sa, da, sb2, db2);
      if (n + 3 >= N) break;
      step(IC<3>{}, sb2, db2, sa, da);
      if (n + 4 >= N) break;
      step(IC<4>{}, sa, da, sb2, db2);
      if (n + 5 >= N) break;
      step(IC<5>{}, sb2, db2, sa, da);
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));  // no LDS-DMA in flight past the stream
  }

  // Write back rows [k0, k0+128) n [kv0, kv1): lane <-> key, 16 bytes of d
  // per access.  In accumulate mode a key tile's old values are all loaded
  // before any is stored (dK and dV are distinct buffers, which the C ABI
  // checks), so the loads share one memory round trip (the sum is old + dK *
  // scale in one fused multiply-add).
  float* __restrict__ gdk = a.dk;
  float* __restrict__ gdv = a.dv;
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
    const int64_t jk = j + 16 * kt;
    if (jk < kv1) {
      const int64_t base = ((b * a.S + jk) * a.Hkv + hk) * D + 4 * g;
      f32x4 ok[ND], ov[ND];
      if (a.accumulate) {
#pragma unroll
        for (int dt = 0; dt < ND; ++dt) {
          ok[dt] = *reinterpret_cast<const f32x4*>(gdk + base + 16 * dt);
          ov[dt] = *reinterpret_cast<const f32x4*>(gdv + base + 16 * dt);
        }
      }
#pragma unroll
      for (int dt = 0; dt < ND; ++dt) {
        f32x4 xk, xv;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          xk[v] = a.accumulate ? __builtin_fmaf(dk[dt][kt][v], a.scale, ok[dt][v]) : dk[dt][kt][v] * a.scale;
          xv[v] = a.accumulate ? ov[dt][v] + dv[dt][kt][v] : dv[dt][kt][v];
        }
        *reinterpret_cast<f32x4*>(gdk + base + 16 * dt) = xk;
        *reinterpret_cast<f32x4*>(gdv + base + 16 * dt) = xv;
      }
    }
  }
  __syncthreads();  // every wave is past s_tile and the ring before the next tile
  }
  // The last workgroup out resets the queues for the next launch (every
  // other one has taken its last tile before it counts itself out).
  if (tid == 0) {
    __threadfence();
    if (atomicAdd(a.tiles + 8, 1) == (int)gridDim.x - 1) {
      for (int x = 0; x < 9; ++x) atomicExch(a.tiles + x, 0);
    }
  }
}

// --------------------------------------------------------------------- dQ
__global__ __launch_bounds__(256, 1) void bwd_dq_bf16_kernel(ChunkArgs a) {
  constexpr int D = 64;
  using T = Tile<D>;
  constexpr int P = T::P, NK = D / 32, ND = D / 16;  // k-steps of S and dP, d tiles
  constexpr int IPWK = (kSB / T::RPI) / 4;  // DMA instructions per wave per tensor per sub-block
  static_assert(IPWK >= 1 && IPWK * 4 * T::RPI == kSB, "sub-block splits over 4 waves");
  constexpr int DMA_PER_SB = 2 * IPWK;
  // One LDS object per ring slot: [K rows | V rows].
  constexpr int SLOT = 2 * kSB * P;
  __shared__ __attribute__((aligned(1024))) uint16_t R0[SLOT], R1[SLOT], R2[SLOT], R3[SLOT], R4[SLOT], R5[SLOT];
  auto slot = [&](auto I) -> uint16_t* {
    constexpr int i = decltype(I)::value;
    if constexpr (i == 0) return R0; else if constexpr (i == 1) return R1; else if constexpr (i == 2) return R2;
    else if constexpr (i == 3) return R3; else if constexpr (i == 4) return R4; else return R5;
  };
  auto slot_rt = [&](int i) -> uint16_t* {
    return i == 0 ? R0 : i == 1 ? R1 : i == 2 ? R2 : i == 3 ? R3 : i == 4 ? R4 : R5;
  };

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const GridPos gp = xcd_grouped();  // the query tiles of a head behind one L2
  const int t = gridDim.x - 1 - gp.x;  // longest (latest) query tiles first
  const int h = gp.y;
  const int64_t b = gp.z;
  const int hk = h / (a.Hq / a.Hkv);
  const int64_t c0 = a.c0, c1 = a.c1, s = c1 - c0;
  const int64_t q0 = c0 + (int64_t)t * kDqRows;
  const int64_t r = q0 + 32 * w + l16;  // this lane's rows: r and r + 16
  const int64_t kend = (q0 + kDqRows < c1) ? q0 + kDqRows : c1;
  const int nsub = (int)((kend + kSB - 1) / kSB);
  const int N = (int)(q0 / kSB);  // key sub-blocks every row of the workgroup sees in full
  const float C = a.scale * kLog2e;

  int nat[NK];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) nat[kk] = T::nat(lane, kk, 0);
  int tro[ND];
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) tro[dt] = T::tr(lane, dt);
  const int64_t kvstride = (int64_t)a.Hkv * D;
  int dmak[IPWK];
#pragma unroll
  for (int x = 0; x < IPWK; ++x) dmak[x] = T::dma(lane, w * IPWK + x, kvstride);
  const uint16_t* kbase = static_cast<const uint16_t*>(a.k) + (b * a.S * a.Hkv + hk) * D;
  const uint16_t* vbase = static_cast<const uint16_t*>(a.v) + (b * a.S * a.Hkv + hk) * D;

  bf16x8 qf[2][NK], df[2][NK];
  float lse2[2];
  f32x4 ninit[2];  // -Delta of the row: the initial value of each dP^T accumulator, so the MFMAs produce dP^T - Delta
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    const int64_t rq = r + 16 * qt;
    float ndl = 0.f;
    lse2[qt] = INFINITY;  // a padding row gets P = 0
    if (rq < c1) {
      const int64_t off = ((b * s + (rq - c0)) * a.Hq + h) * D;
      const uint16_t* qrow = static_cast<const uint16_t*>(a.q) + off;
      const uint16_t* drow = static_cast<const uint16_t*>(a.dout) + off;
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) {
        qf[qt][kk] = as_bf16x8(ld_global16(qrow + 32 * kk + 8 * g));
        df[qt][kk] = as_bf16x8(ld_global16(drow + 32 * kk + 8 * g));
      }
      lse2[qt] = a.lse2[(b * a.Hq + h) * s + (rq - c0)];
      ndl = a.delta[(b * a.Hq + h) * s + (rq - c0)];
    } else {
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) qf[qt][kk] = df[qt][kk] = bf16x8{};
    }
    ninit[qt] = f32x4{ndl, ndl, ndl, ndl};
  }
  f32x4 dq[ND][2];  // dQ^T: [d tile][query tile]
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) dq[dt][0] = dq[dt][1] = f32x4{0.f, 0.f, 0.f, 0.f};

  // DMA of K/V sub-block u (keys [32u, 32u+32)) into a slot; keys past the
  // chunk end load zeros, so every call issues DMA_PER_SB instructions.
  // Sub-blocks are issued in key order, so scalar state walks K and V one
  // sub-block per call.
  const int64_t sbb = (int64_t)kSB * kvstride * 2;  // bytes per sub-block of K or V
  const int krow_bytes = (int)(kvstride * 2);
  uint64_t ka = uniform_u64(reinterpret_cast<uint64_t>(kbase)), va = uniform_u64(reinterpret_cast<uint64_t>(vbase));
  int remk = (int)c1;  // keys [k0, c1) are valid
  auto issue_next = [&](uint16_t* dst) {
    const int n = remk <= 0 ? 0 : (remk < kSB ? remk : kSB);
    const auto rk = uniform_rsrc(ka, n * krow_bytes);
    const auto rv = uniform_rsrc(va, n * krow_bytes);
#pragma unroll
    for (int x = 0; x < IPWK; ++x) {
      lds_dma16(rk, dst + (w * IPWK + x) * 512, dmak[x]);
      lds_dma16(rv, dst + kSB * P + (w * IPWK + x) * 512, dmak[x]);
    }
    ka += sbb;
    va += sbb;
    remk -= kSB;
  };
  auto nat_rd = [&](const uint16_t* X, int t, int kk) { return ld_nat(X + 16 * t * P, nat[kk ^ t]); };
  auto tr_rd = [&](const uint16_t* X, int dt) { return ld_tr(X, tro[dt], tro[dt ^ 2] + 16 * P); };
  // Natural operand o of a sub-block: k-step o / 4, key tile (o / 2) % 2, K (o even) or V (o odd).
  auto nat_of = [&](const uint16_t* K, int o) { return nat_rd((o & 1) ? K + kSB * P : K, (o >> 1) & 1, o >> 2); };
  // The MFMA of query tile qt that operand o feeds: S^T = K Q^T or dP^T - Delta = V dO^T - Delta (lane <-> query).
  auto sdp_one = [&](const bf16x8& x, int o, int qt, S4& sv, S4& dp) {
    const int kk = o >> 2, kt = (o >> 1) & 1;
    if (o & 1) dp.x[kt][qt] = mfma16(x, df[qt][kk], kk == 0 ? ninit[qt] : dp.x[kt][qt]);
    else sv.x[kt][qt] = mfma16(x, qf[qt][kk], kk == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sv.x[kt][qt]);
  };
  constexpr int NA = 4 * NK;
  auto sdp = [&](const uint16_t* K, S4& sv, S4& dp) {
#pragma unroll
    for (int o = 0; o < NA; ++o) {
      const bf16x8 x = nat_of(K, o);
      sdp_one(x, o, 0, sv, dp);
      sdp_one(x, o, 1, sv, dp);
    }
  };

  // Prologue: sub-blocks 0..4 (which also covers every diagonal sub-block
  // when N is 0).
  issue_next(R0);
  issue_next(R1);
  issue_next(R2);
  issue_next(R3);
  issue_next(R4);

  if (N > 0) {
    __builtin_amdgcn_s_waitcnt(waitcnt_vm((kAhead - 2) * DMA_PER_SB));
    __syncthreads();
    S4 sa, da, sb2, db2;
    sdp(R0, sa, da);
    bf16x8 opn[4];
#pragma unroll
    for (int o = 0; o < 4; ++o) opn[o] = nat_of(R1, o);
    // Step n in slot I: A(n) reads slot I+1 (natural K, V); B(n) reads slot I
    // (transposed K) and, in its last slots, A(n+1)'s first natural operands
    // from slot I+2.  At its start sub-blocks n+1 and n+2 have landed; then
    // sub-block n+5 goes to slot I+5 = I-1, free since step n-1.
    auto step = [&](auto sl, S4& scur, S4& dcur, S4& snext, S4& dnext) {
      constexpr int I = decltype(sl)::value;
      constexpr int I1 = (I + 1) % kRing, I2 = (I + 2) % kRing, I5 = (I + kAhead) % kRing;
      __builtin_amdgcn_s_waitcnt(waitcnt_vm((kAhead - 3) * DMA_PER_SB));
      __syncthreads();
      issue_next(slot(IC<I5>{}));  // sub-block n + kAhead
      const uint16_t* Kn = slot(IC<I1>{});
      const uint16_t* Kc = slot(IC<I>{});
      // A(n): operand o (NA of them) feeds two MFMAs of S^T(n+1) or dP^T(n+1);
      // it is read four operands ahead.  The VALU turns the 16 elements of
      // S^T(n), dP^T(n) into dS^T(n) (query tile by query tile), element i
      // beside operand i / (16 / NA).
      constexpr int EPM = 16 / NA;
      bf16x8 op[NA];
#pragma unroll
      for (int o = 0; o < 4; ++o) op[o] = opn[o];
      float pv[16], ds[16];
      uint32_t pk[2][4];  // dS of query tile 0, then 1, packed in pairs
      bf16x8 dsb[2];
      // B(n): operand jj feeds the two MFMAs of dQ^T d tile jj; it is read three
      // operands ahead (the first three in the last slots of A(n)).
      constexpr int NB = ND;
      bf16x8 top[NB];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int o = i / EPM;
        if (i % EPM == 0) sdp_one(op[o], o, 0, snext, dnext);
        __builtin_amdgcn_sched_barrier(0);
        // Element i's exp, element i-1's dS (no exp result read right away).
        const int qt = i >> 3, kt = (i >> 2) & 1, v = i & 3;
        pv[i] = fast_exp2(scur.x[kt][qt][v] * C - lse2[qt]);
        if (i % EPM == EPM / 2) {
          __builtin_amdgcn_sched_barrier(0);
          sdp_one(op[o], o, 1, snext, dnext);
          __builtin_amdgcn_sched_barrier(0);
          if (o + 4 < NA) op[o + 4] = nat_of(Kn, o + 4);
          else if (o + 4 - NA < 3) top[o + 4 - NA] = tr_rd(Kc, o + 4 - NA);
        }
        if (i > 0) ds[i - 1] = pv[i - 1] * dcur.x[((i - 1) >> 2) & 1][(i - 1) >> 3][(i - 1) & 3];
        if (i >= 8 && i < 12) pk[0][i - 8] = pack_bf16x2(ds[2 * (i - 8)], ds[2 * (i - 8) + 1]);
        if (i >= 12 && 8 + 2 * (i - 12) + 1 < i) pk[1][i - 12] = pack_bf16x2(ds[8 + 2 * (i - 12)], ds[9 + 2 * (i - 12)]);
        if (i % EPM == EPM - 1) __builtin_amdgcn_sched_barrier(0);
      }
      dsb[0] = as_bf16x8(u32x4{pk[0][0], pk[0][1], pk[0][2], pk[0][3]});
      ds[15] = pv[15] * dcur.x[1][1][3];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int jj = 0; jj < NB; ++jj) {
        dq[jj][0] = mfma16(top[jj], dsb[0], dq[jj][0]);
        __builtin_amdgcn_sched_barrier(0);
        if (jj == 0) {
          pk[1][3] = pack_bf16x2(ds[14], ds[15]);
          dsb[1] = as_bf16x8(u32x4{pk[1][0], pk[1][1], pk[1][2], pk[1][3]});
        }
        __builtin_amdgcn_sched_barrier(0);
        dq[jj][1] = mfma16(top[jj], dsb[1], dq[jj][1]);
        __builtin_amdgcn_sched_barrier(0);
        if (jj + 3 < NB) {
          top[jj + 3] = tr_rd(Kc, jj + 3);
        } else {  // A(n+1)'s first natural operands, from sub-block n+2
          const int m0 = jj + 3 - NB;
          opn[m0] = nat_of(slot(IC<I2>{}), m0);
          if (m0 == 2) opn[3] = nat_of(slot(IC<I2>{}), 3);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    for (int n = 0; n < N; n += kRing) {
      step(IC<0>{}, sa, da, sb2, db2);
      if (n + 1 >= N) break;
      step(IC<1>{}, sb2, db2, sa, da);
      if (n + 2 >= N) break;
      step(IC<2>{}, sa, da, sb2, db2);
      if (n + 3 >= N) break;
      step(IC<3>{}, sb2, db2, sa, da);
      if (n + 4 >= N) break;
      step(IC<4>{}, sa, da, sb2, db2);
      if (n + 5 >= N) break;
      step(IC<5>{}, sb2, db2, sa, da);
    }
  }

  // Diagonal sub-blocks [N, nsub) (at most five): already in the ring, since
  // the steady loop loaded five ahead and the prologue covers N = 0.
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
  __syncthreads();
  for (int u = N; u < nsub; ++u) {
    const uint16_t* K = slot_rt(u % kRing);
    S4 sv, dp;
    sdp(K, sv, dp);
    const int rel = (int)(r - (int64_t)u * kSB);  // keys past row r are masked
    bf16x8 dsb[2];
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
      float ds[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int kt = e >> 2, v = e & 3;
        float p = fast_exp2(sv.x[kt][qt][v] * C - lse2[qt]);
        if (16 * kt + 4 * g + v > rel + 16 * qt) p = 0.f;
        ds[e] = p * dp.x[kt][qt][v];
      }
      dsb[qt] = pack_bf16x8(ds[0], ds[1], ds[2], ds[3], ds[4], ds[5], ds[6], ds[7]);
    }
#pragma unroll
    for (int dt = 0; dt < ND; ++dt) {
      const bf16x8 kx = tr_rd(K, dt);
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) dq[dt][qt] = mfma16(kx, dsb[qt], dq[dt][qt]);
    }
  }

#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    const int64_t rq = r + 16 * qt;
    if (rq < c1) {
      uint16_t* qrow = static_cast<uint16_t*>(a.dq) + ((b * s + (rq - c0)) * a.Hq + h) * D;
#pragma unroll
      for (int dt = 0; dt < ND; ++dt)
        *reinterpret_cast<u32x2*>(qrow + 16 * dt + 4 * g) =
            pack_bf16x4(dq[dt][qt][0] * a.scale, dq[dt][qt][1] * a.scale, dq[dt][qt][2] * a.scale,
                        dq[dt][qt][3] * a.scale);
    }
  }
}

// dQ for grids that leave compute units idle: a workgroup is RG groups of 32
// query rows of one head times four parts of the keys (part ks has the 32-key
// sub-blocks u = ks, ks + 4, ...), a wave each; the parts are added through LDS
// in part order.  A sub-block's part depends on its position in the sequence
// alone, so a row's result depends neither on RG nor, as long as every chunk's
// launch takes this kernel, on the chunking.
// bwd_dq_split is one workgroup's work: position gp of a grid nx tiles wide, in
// the kDqSplitBytes bytes of LDS at mem.
constexpr int kDqParts = 4;
template <int D, int RG>
constexpr int kDqSplitBytes = 2 * kDqParts * 2 * kSB * Tile<D>::P * 2 > kDqParts * 32 * RG * (D + 4) * 4
                                  ? 2 * kDqParts * 2 * kSB * Tile<D>::P * 2
                                  : kDqParts * 32 * RG * (D + 4) * 4;
template <int D, int RG>
__device__ __forceinline__ void bwd_dq_split(const ChunkArgs& a, const GridPos gp, int nx, unsigned char* mem) {
  using T = Tile<D>;
  constexpr int P = T::P, NK = D / 32, ND = D / 16, KS = kDqParts, R = 32 * RG;
  constexpr int IPW = 32 / T::RPI / RG;  // DMA instructions per wave for each of K and V
  constexpr int SB = 2 * kSB * P;        // elements of a sub-block's K and V
  constexpr int OP = D + 4;              // row pitch of the partial dQ's, floats

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4, rg = w % RG, ks = w / RG;
  const int h = gp.y;
  const int64_t b = gp.z;
  const int hk = h / (a.Hq / a.Hkv);
  const int64_t c0 = a.c0, c1 = a.c1, s = c1 - c0;
  const int64_t q0 = c0 + (int64_t)(nx - 1 - gp.x) * R;
  const int64_t qw = q0 + 32 * rg, r = qw + l16;  // this lane's rows: r and r + 16
  const int64_t kend = q0 + R < c1 ? q0 + R : c1;
  const int nsub = (int)((kend + kSB - 1) / kSB), nstep = (nsub + KS - 1) / KS;
  const float C = a.scale * kLog2e;

  int nat[NK], tro[ND];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) nat[kk] = T::nat(lane, kk, 0);
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) tro[dt] = T::tr(lane, dt);
  const int64_t kvstride = (int64_t)a.Hkv * D;
  int dma[IPW];
#pragma unroll
  for (int x = 0; x < IPW; ++x) dma[x] = T::dma(lane, rg * IPW + x, kvstride);
  bf16x8 qf[2][NK], df[2][NK];
  float lse2[2];
  f32x4 ninit[2];
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    const int64_t rq = r + 16 * qt, rc = rq < c1 ? rq : c1 - 1;
    const int64_t off = ((b * s + (rc - c0)) * a.Hq + h) * D;
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      qf[qt][kk] = as_bf16x8(ld_global16(static_cast<const uint16_t*>(a.q) + off + 32 * kk + 8 * g));
      df[qt][kk] = as_bf16x8(ld_global16(static_cast<const uint16_t*>(a.dout) + off + 32 * kk + 8 * g));
    }
    lse2[qt] = rq < c1 ? a.lse2[(b * a.Hq + h) * s + (rc - c0)] : INFINITY;  // a padding row gets P = 0
    const float ndl = a.delta[(b * a.Hq + h) * s + (rc - c0)];
    ninit[qt] = f32x4{ndl, ndl, ndl, ndl};
  }
  const uint16_t* kbase = static_cast<const uint16_t*>(a.k) + (b * a.S * a.Hkv + hk) * D;
  const uint16_t* vbase = static_cast<const uint16_t*>(a.v) + (b * a.S * a.Hkv + hk) * D;
  uint16_t* const kv = reinterpret_cast<uint16_t*>(mem) + ks * SB;  // this part's slot, buffer 0
  auto issue = [&](int i) {  // keys past the chunk arrive as zeros
    const int64_t j0 = ((int64_t)i * KS + ks) * kSB;
    uint16_t* dst = kv + (i & 1) * KS * SB;
    const auto rk = tile_rsrc(kbase + j0 * kvstride, c1 - j0, kSB, kvstride);
    const auto rv = tile_rsrc(vbase + j0 * kvstride, c1 - j0, kSB, kvstride);
#pragma unroll
    for (int x = 0; x < IPW; ++x) {
      lds_dma16(rk, dst + (rg * IPW + x) * 512, dma[x]);
      lds_dma16(rv, dst + kSB * P + (rg * IPW + x) * 512, dma[x]);
    }
  };
  f32x4 dq[ND][2];
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) dq[dt][0] = dq[dt][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto block = [&](int u, const uint16_t* K) {
    // Operands are read a few ahead of their MFMAs (left to the compiler, each
    // read was waited for right after it was issued): o is k-step o / 4, key
    // tile (o / 2) % 2, K (o even) or V (o odd).
    constexpr int NA = 4 * NK, kNat = 6, kTr = 4;
    bf16x8 op[NA], top[ND];
    auto rd = [&](int o) {
      const int kk = o >> 2, kt = (o >> 1) & 1;
      return ld_nat(K + ((o & 1) ? kSB * P : 0) + 16 * kt * P, nat[D == 64 ? kk ^ kt : kk]);
    };
    auto rd_tr = [&](int dt) { return ld_tr(K, tro[dt], tro[D == 64 ? dt ^ 2 : dt] + 16 * P); };
    S4 sv, dp;
#pragma unroll
    for (int o = 0; o < kNat; ++o) op[o] = rd(o);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int o = 0; o < NA; ++o) {
      const int kk = o >> 2, kt = (o >> 1) & 1;
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
        if (o & 1) dp.x[kt][qt] = mfma16(op[o], df[qt][kk], kk == 0 ? ninit[qt] : dp.x[kt][qt]);
        else sv.x[kt][qt] = mfma16(op[o], qf[qt][kk], kk == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sv.x[kt][qt]);
      }
      if (o + kNat < NA) op[o + kNat] = rd(o + kNat);
      else if (o + kNat - NA < kTr) top[o + kNat - NA] = rd_tr(o + kNat - NA);
      __builtin_amdgcn_sched_barrier(0);
    }
    const int rel = (int)(r - (int64_t)u * kSB);  // keys past row r are masked
    float p[2][8];
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
#pragma unroll
      for (int e = 0; e < 8; ++e) p[qt][e] = fast_exp2(sv.x[e >> 2][qt][e & 3] * C - lse2[qt]);
    }
    if ((int64_t)u * kSB + kSB - 1 > qw) {
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if (16 * (e >> 2) + 4 * g + (e & 3) > rel + 16 * qt) p[qt][e] = 0.f;
        }
      }
    }
    bf16x8 dsb[2];
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
      float ds[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) ds[e] = p[qt][e] * dp.x[e >> 2][qt][e & 3];
      dsb[qt] = pack_bf16x8(ds[0], ds[1], ds[2], ds[3], ds[4], ds[5], ds[6], ds[7]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int dt = 0; dt < ND; ++dt) {
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) dq[dt][qt] = mfma16(top[dt], dsb[qt], dq[dt][qt]);
      if (dt + kTr < ND) top[dt + kTr] = rd_tr(dt + kTr);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  issue(0);
  for (int i = 0; i < nstep; ++i) {
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __syncthreads();  // step i landed; every wave is done with step i - 1
    if (i + 1 < nstep) issue(i + 1);
    const int u = i * KS + ks;
    if ((int64_t)u * kSB <= qw + 31) block(u, kv + (i & 1) * KS * SB);  // else past this wave's rows
  }

  __syncthreads();
  float* const os = reinterpret_cast<float*>(mem);  // [part][row][D], over the K/V slots
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
      *reinterpret_cast<f32x4*>(os + (ks * R + 32 * rg + 16 * qt + l16) * OP + 16 * dt + 4 * g) = dq[dt][qt];
  }
  __syncthreads();
  constexpr int TPR = 64 * RG * KS / R, EPT = D / TPR;  // threads per row, elements per thread
  const int row = tid / TPR, d0 = (tid % TPR) * EPT;
  if (q0 + row >= c1) return;
  uint16_t* qrow = static_cast<uint16_t*>(a.dq) + ((b * s + (q0 + row - c0)) * a.Hq + h) * D + d0;
#pragma unroll
  for (int e = 0; e < EPT; e += 4) {
    f32x4 acc = *reinterpret_cast<const f32x4*>(os + row * OP + d0 + e);
#pragma unroll
    for (int x = 1; x < KS; ++x) acc += *reinterpret_cast<const f32x4*>(os + (x * R + row) * OP + d0 + e);
    *reinterpret_cast<u32x2*>(qrow + e) =
        pack_bf16x4(acc[0] * a.scale, acc[1] * a.scale, acc[2] * a.scale, acc[3] * a.scale);
  }
}
template <int D>
__global__ __launch_bounds__(512) void bwd_dq_split_kernel(ChunkArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char mem[kDqSplitBytes<D, 2>];
  bwd_dq_split<D, 2>(a, xcd_grouped(), gridDim.x, mem);
}

// dK/dV for grids that leave compute units idle: KG groups of 32 keys of one KV
// head times QS parts of the chunk's query sub-blocks (32 rows; sub-block n of
// the group's head hh is number hh * nsb + n, and part qs has numbers qs, qs +
// QS, ...); the parts are added through LDS in part order.  A sub-block's part
// depends on its position in the chunk alone, so a key's sum does not depend on
// the range of keys a launch covers.  D = 128: 4 waves, one per SIMD by their
// accumulators and K/V fragments; D = 64: 8.
template <int D, int KG, int QS>
constexpr int kDkdvSplitBytes = 2 * QS * 2 * kSB * Tile<D>::P * 2 > QS * 32 * KG * (D + 4) * 4
                                    ? 2 * QS * 2 * kSB * Tile<D>::P * 2
                                    : QS * 32 * KG * (D + 4) * 4;
template <int D, int KG, int QS>
__device__ __forceinline__ void bwd_dkdv_split(const ChunkArgs& a, const GridPos gp, unsigned char* mem) {
  using T = Tile<D>;
  constexpr int P = T::P, NK = D / 32, ND = D / 16, NT = 64 * KG * QS, R = 32 * KG;
  constexpr int IPW = 32 / T::RPI / KG;  // DMA instructions per wave for each of Q and dO
  static_assert(IPW >= 1 && IPW * KG * T::RPI == 32, "a sub-block splits over KG waves");
  constexpr int SB = 2 * kSB * P;  // elements of a sub-block's Q and dO
  constexpr int OP = D + 4;        // row pitch of the partial sums, floats

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4, kg = w % KG, qs = w / KG;
  const int hk = gp.y, G = a.Hq / a.Hkv;
  const int64_t b = gp.z;
  const int64_t c0 = a.c0, c1 = a.c1, s = c1 - c0, kv1 = a.kv1;
  const int64_t kw = a.kv0 + (int64_t)gp.x * R;  // the workgroup's first key
  const int64_t k0 = kw + 32 * kg, j = k0 + l16;  // this lane's keys: j and j + 16
  const float C = a.scale * kLog2e;
  const int nsb = (int)((s + kSB - 1) / kSB);
  const int sb_begin = kw > c0 ? (int)((kw - c0) / kSB) : 0;  // the first sub-block that sees a key here

  int nat[NK], tro[ND];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) nat[kk] = T::nat(lane, kk, 0);
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) tro[dt] = T::tr(lane, dt);
  const int64_t qstride = (int64_t)a.Hq * D;
  int dma[IPW];
#pragma unroll
  for (int x = 0; x < IPW; ++x) dma[x] = T::dma(lane, kg * IPW + x, qstride);
  bf16x8 kf[2][NK], vf[2][NK];
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
    const int64_t jk = j + 16 * kt;
    const int64_t off = ((b * a.S + jk) * a.Hkv + hk) * D;
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      kf[kt][kk] = jk < kv1 ? as_bf16x8(ld_global16(static_cast<const uint16_t*>(a.k) + off + 32 * kk + 8 * g)) : bf16x8{};
      vf[kt][kk] = jk < kv1 ? as_bf16x8(ld_global16(static_cast<const uint16_t*>(a.v) + off + 32 * kk + 8 * g)) : bf16x8{};
    }
  }
  f32x4 dk[ND][2], dv[ND][2];  // dK^T, dV^T: [d tile][key tile]
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) dk[dt][0] = dk[dt][1] = dv[dt][0] = dv[dt][1] = f32x4{0.f, 0.f, 0.f, 0.f};

  // A step is QS consecutive numbers, the first being sub-block n of head hh;
  // steps whose sub-blocks all lie before sb_begin are passed over.
  struct Pos { int hh, n, i; };
  const int total = (G * nsb + QS - 1) / QS;  // steps
  auto settle = [&](Pos& p) {
    for (;;) {
      while (p.n >= nsb) {
        p.n -= nsb;
        ++p.hh;
      }
      if (p.n + QS - 1 >= sb_begin || p.i >= total) return;
      p.n += QS;
      ++p.i;
    }
  };
  auto own = [&](Pos p) {  // this part's number of the step
    p.n += qs;
    while (p.n >= nsb) {
      p.n -= nsb;
      ++p.hh;
    }
    return p;
  };
  auto active = [&](const Pos& p) { return p.hh < G && p.n >= sb_begin; };
  uint16_t* const slot = reinterpret_cast<uint16_t*>(mem) + qs * SB;  // this part's, buffer 0
  f32x4 lg[2], nd[2], lgn[2], ndn[2];  // LSE2 and -Delta of rows 16 qt + 4 g + 0..3, this step's and the next's
  auto issue = [&](const Pos& step, int buf) {
    const Pos p = own(step);
    const int64_t r0 = (int64_t)p.n * kSB;
    const int h = hk * G + (p.hh < G ? p.hh : 0);
    const int64_t valid = active(p) ? s - r0 : 0;
    const int64_t tile0 = (b * s + r0) * a.Hq + h;
    const auto rq = tile_rsrc(static_cast<const uint16_t*>(a.q) + tile0 * D, valid, kSB, qstride);
    const auto ro = tile_rsrc(static_cast<const uint16_t*>(a.dout) + tile0 * D, valid, kSB, qstride);
    uint16_t* dst = slot + buf * QS * SB;
#pragma unroll
    for (int x = 0; x < IPW; ++x) {
      lds_dma16(rq, dst + (kg * IPW + x) * 512, dma[x]);
      lds_dma16(ro, dst + kSB * P + (kg * IPW + x) * 512, dma[x]);
    }
    const int64_t rec = (b * a.Hq + h) * s;
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t rr = r0 + 16 * qt + 4 * g + v;
        const bool ok = rr < s && p.hh < G;  // rows past the chunk: zeros
        lgn[qt][v] = ok ? a.lse2[rec + rr] : 0.f;
        ndn[qt][v] = ok ? a.delta[rec + rr] : 0.f;
      }
    }
  };
  auto block = [&](const Pos& p, const uint16_t* Qs) {
    const uint16_t* Os = Qs + kSB * P;
    // As in the split dQ kernel: natural operand o is k-step o / 4, row tile
    // (o / 2) % 2, Q (o even) or dO (o odd); transposed operand jj is d tile
    // jj / 2 of dO (jj even) or Q (jj odd).
    constexpr int NA = 4 * NK, NB = 2 * ND, kNat = 6, kTr = 4;
    bf16x8 op[NA], top[NB];
    auto rd = [&](int o) {
      const int kk = o >> 2, qt = (o >> 1) & 1;
      return ld_nat(((o & 1) ? Os : Qs) + 16 * qt * P, nat[D == 64 ? kk ^ qt : kk]);
    };
    auto rd_tr = [&](int jj) {
      const int dt = jj >> 1;
      return ld_tr((jj & 1) ? Qs : Os, tro[dt], tro[D == 64 ? dt ^ 2 : dt] + 16 * P);
    };
    S4 sv, dp;
#pragma unroll
    for (int o = 0; o < kNat; ++o) op[o] = rd(o);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int o = 0; o < NA; ++o) {
      const int kk = o >> 2, qt = (o >> 1) & 1;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        if (o & 1) dp.x[qt][kt] = mfma16(op[o], vf[kt][kk], kk == 0 ? nd[qt] : dp.x[qt][kt]);
        else sv.x[qt][kt] = mfma16(op[o], kf[kt][kk], kk == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sv.x[qt][kt]);
      }
      if (o + kNat < NA) op[o + kNat] = rd(o + kNat);
      else if (o + kNat - NA < kTr) top[o + kNat - NA] = rd_tr(o + kNat - NA);
      __builtin_amdgcn_sched_barrier(0);
    }
    const int64_t r0g = c0 + (int64_t)p.n * kSB;  // global row of the sub-block's first row
    float pr[2][8];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
      for (int e = 0; e < 8; ++e) pr[kt][e] = fast_exp2(sv.x[e >> 2][kt][e & 3] * C - lg[e >> 2][e & 3]);
    }
    if (k0 + 31 > r0g) {
      const int rel = (int)(j - r0g);  // key j sees row r iff j <= r
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if (rel + 16 * kt > 16 * (e >> 2) + 4 * g + (e & 3)) pr[kt][e] = 0.f;
        }
      }
    }
    bf16x8 pb[2], dsb[2];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      float ds[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) ds[e] = pr[kt][e] * dp.x[e >> 2][kt][e & 3];
      pb[kt] = pack_bf16x8(pr[kt][0], pr[kt][1], pr[kt][2], pr[kt][3], pr[kt][4], pr[kt][5], pr[kt][6], pr[kt][7]);
      dsb[kt] = pack_bf16x8(ds[0], ds[1], ds[2], ds[3], ds[4], ds[5], ds[6], ds[7]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int jj = 0; jj < NB; ++jj) {
      const int dt = jj >> 1;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        if (jj & 1) dk[dt][kt] = mfma16(top[jj], dsb[kt], dk[dt][kt]);
        else dv[dt][kt] = mfma16(top[jj], pb[kt], dv[dt][kt]);
      }
      if (jj + kTr < NB) top[jj + kTr] = rd_tr(jj + kTr);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  Pos cur{0, 0, 0};
  settle(cur);
  int buf = 0;
  if (cur.i < total) issue(cur, 0);
  while (cur.i < total) {
    Pos nxt{cur.hh, cur.n + QS, cur.i + 1};
    settle(nxt);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __syncthreads();  // this step landed; every wave is done with the one before
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
      lg[qt] = lgn[qt];
      nd[qt] = ndn[qt];
    }
    if (nxt.i < total) issue(nxt, buf ^ 1);
    const Pos p = own(cur);
    if (active(p) && k0 <= c0 + (int64_t)p.n * kSB + kSB - 1) block(p, slot + buf * QS * SB);
    cur = nxt;
    buf ^= 1;
  }

  float* const os = reinterpret_cast<float*>(mem);  // [part][key][D], over the slots
  constexpr int V4 = R * D / 4;                     // 16-byte pieces of the result
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    __syncthreads();
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
      for (int dt = 0; dt < ND; ++dt)
        *reinterpret_cast<f32x4*>(os + (qs * R + 32 * kg + 16 * kt + l16) * OP + 16 * dt + 4 * g) =
            pass ? dv[dt][kt] : dk[dt][kt];
    }
    __syncthreads();
#pragma unroll
    for (int x = 0; x < V4 / NT; ++x) {
      const int e = (x * NT + tid) * 4, row = e / D, d = e % D;
      if (kw + row < kv1) {
        f32x4 acc = *reinterpret_cast<const f32x4*>(os + row * OP + d);
#pragma unroll
        for (int y = 1; y < QS; ++y) acc += *reinterpret_cast<const f32x4*>(os + (y * R + row) * OP + d);
        f32x4* out = reinterpret_cast<f32x4*>((pass ? a.dv : a.dk) + ((b * a.S + kw + row) * a.Hkv + hk) * D + d);
        const f32x4 old = a.accumulate ? *out : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v] = pass ? old[v] + acc[v] : __builtin_fmaf(acc[v], a.scale, old[v]);
        *out = acc;
      }
    }
  }
}
template <int D, int KG, int QS>
__global__ __launch_bounds__(64 * KG * QS) void bwd_dkdv_split_kernel(ChunkArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char mem[kDkdvSplitBytes<D, KG, QS>];
  bwd_dkdv_split<D, KG, QS>(a, xcd_grouped(), mem);
}

// Both of a chunk's split kernels as one launch: neither needs the other's
// results, and one after the other each leaves most of the card idle.  The
// kind with the longer workgroups comes first (dq_first).
struct PairGrid {
  int dq_first, ndq, dqx, ndkdv, dkdvx;  // workgroups of each kind, and tiles in x
};
template <int D, int KG, int QS>
__global__ __launch_bounds__(64 * KG * QS) void bwd_pair_kernel(ChunkArgs a, PairGrid p) {
  constexpr int RG = KG * QS / kDqParts, nq = kDqSplitBytes<D, RG>, nk = kDkdvSplitBytes<D, KG, QS>;
  static_assert(RG * kDqParts == KG * QS, "both kinds have the same waves");
  __shared__ __attribute__((aligned(1024))) unsigned char mem[nq > nk ? nq : nk];
  const int n = blockIdx.x, lead = p.dq_first ? p.ndq : p.ndkdv;
  const bool dq = p.dq_first ? n < lead : n >= lead;
  const int m = n < lead ? n : n - lead;
  if (dq)
    bwd_dq_split<D, RG>(a, xcd_grouped(m, p.dqx, a.Hq, (uint32_t)a.B), p.dqx, mem);
  else
    bwd_dkdv_split<D, KG, QS>(a, xcd_grouped(m, p.dkdvx, a.Hkv, (uint32_t)a.B), mem);
}

}  // namespace

hipError_t launch_bwd_pre_bf16(const ChunkArgs& a, hipStream_t stream) {
  if (!a.tiles) return hipErrorInvalidValue;
  const int64_t s = a.c1 - a.c0;
  const int64_t threads = a.B * s * a.Hq * (a.D / 8);
  dim3 grid((unsigned)((threads + 255) / 256));
  if (a.D == 128) {
    hipLaunchKernelGGL(bwd_pre_bf16_kernel<128>, grid, dim3(256), 0, stream, a);
  } else if (a.D == 64) {
    hipLaunchKernelGGL(bwd_pre_bf16_kernel<64>, grid, dim3(256), 0, stream, a);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Workgroups of the persistent dK/dV kernel that one CU holds at once (its
// registers allow one; asked of the runtime once).
static int dkdv_groups_per_cu() {
  static const int n = [] {
    int b = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, reinterpret_cast<const void*>(&bwd_dkdv_bf16_kernel), 256,
                                                     0) != hipSuccess || b < 1) {
      b = 1;
    }
    return b;
  }();
  return n;
}

// Which kernels a chunk's backward takes.  Drawn by the whole chunk's rows and
// keys, so that launches over parts of [0, c1), and one launch for both
// gradients or two, give the same results.
struct SplitPlan {
  int dkdv;   // 0 the wide kernel, 1 split with 32 keys a workgroup, 2 split with 64
  bool dq;    // the split kernel
  bool pair;  // both in one launch, if dQ overwrites nothing that dK/dV reads
};

// dK/dV: the split kernels where their workgroups all run at once (one a CU):
// 32 keys times four parts, then 64 times two (D = 64: 64 times four).
// Measured (us, wide kernel -> split, event times): 4 heads, rows [1536, 2048)
// 32 -> 17 (256 workgroups of 32 keys); 8 heads, rows [1024, 2048) 47 -> 38
// (256 of 64); D = 64, GQA 32/8, 2048 rows 145 -> 113; but 4 heads, rows [7168,
// 8192) 67 -> 70 (512 of 64), D = 64, 8/2 x batch 2, rows [3334, 5001) 126 ->
// 153 (316).  Two parts halve a workgroup's chain of sub-blocks, which makes
// up for the unpipelined step only while the chain is short: with more than
// 4096 query rows to a key 64 times two is the slower on its own (whole
// backward, wide -> split: 8/2 heads, rows [6656, 8192) 252 -> 263, [4096,
// 8192) 543 -> 599; 16/4 heads, rows [1024, 4096) 394 -> 427; at 4400 rows
// even), but not in one launch with dQ (rows [3500, 4800) 199 -> 151).
// dQ: the split kernel where its workgroups (64 rows) all run at once, one a
// CU.  Measured (us, wide -> split): 4 heads, rows [1536, 2048) 45 -> 29 (32
// workgroups); GQA 16/4, rows [3072, 4096) 80 -> 53 (256); but 32 heads, 1024
// rows 30 -> 34 (512).  D = 64 has room for two a CU: twice the wide kernel's
// workgroups then stream the keys, which pays while an XCD has one head and up
// to 12288 keys of it (3 MiB of K and V in its L2) or two heads and 4096: 8
// heads, rows [2000, 6096) 76 -> 64 (512 workgroups), [7000, 11096) 137 -> 125,
// 16 heads, rows [2000, 3536) 46 -> 44 (384); but 8 heads, rows [12000, 14176)
// 155 -> 160 (272), 16 heads, rows [7000, 8088) 91 -> 98, 32 heads, rows [14000,
// 14768) 163 -> 189 (384), 64/8 heads, 448 rows 12 -> 15.5 (512).  With the pair
// it always does.
// Both in one launch if both take the split kernels and their workgroups are
// at most two to a place on the card (us, pre + dK/dV + dQ, one after the other
// -> pair): 4 heads, rows [0, 512) 27.9 -> 16.5, [1536, 2048) 43.3 -> 28.6 (320
// workgroups on 256 CUs); 8 heads, rows [1024, 2048) 64.1 -> 53.9 (512); D = 64,
// 8/2 x batch 2, rows [1667, 3334) 138 -> 115; but GQA 16/4, rows [3072, 4096)
// 166 -> 183 and 8/2, rows [2048, 4096) 182 -> 192 (768).
static SplitPlan split_plan(const ChunkArgs& a) {
  const bool d64 = a.D == 64;
  const int64_t s = a.c1 - a.c0, heads = a.Hq * a.B, n_cu = a.n_cu;
  const int64_t k64 = (a.c1 + 63) / 64 * a.Hkv * a.B, k32 = (a.c1 + 31) / 32 * a.Hkv * a.B;
  const int64_t q64 = (s + 63) / 64 * heads, q32 = (s + 31) / 32 * heads;
  const int mode = !d64 && k32 <= n_cu ? 1 : k64 <= n_cu ? 2 : 0;
  SplitPlan p;
  const bool at_once = q64 <= n_cu * (d64 ? 2 : 1);
  const int64_t heads_xcd = (heads + 7) / 8;
  p.pair = mode && at_once && (d64 ? q64 : q32) + (mode == 1 ? k32 : k64) <= n_cu * (d64 ? 4 : 2);
  p.dq = p.pair || q64 <= n_cu || (d64 && at_once && a.c1 <= (heads_xcd == 1 ? 12288 : heads_xcd == 2 ? 4096 : 0));
  p.dkdv = d64 || mode == 1 || p.pair || a.Hq / a.Hkv * s <= 4096 ? mode : 0;
  return p;
}

hipError_t launch_bwd_dkdv_bf16(const ChunkArgs& a, hipStream_t stream) {
  if (a.kv0 < 0 || a.kv1 > a.c1 || a.kv0 >= a.kv1 || !a.tiles || a.n_cu < 1) return hipErrorInvalidValue;
  if (a.D != 128 && a.D != 64) return hipErrorInvalidValue;
  const int64_t tiles = (a.kv1 - a.kv0 + kKvKeys - 1) / kKvKeys * a.Hkv * a.B;
  if (tiles > 0x7fffffff) return hipErrorInvalidValue;
  const int mode = split_plan(a).dkdv;
  if (mode) {
    const int r = mode == 2 ? 64 : 32;
    const dim3 grid((unsigned)((a.kv1 - a.kv0 + r - 1) / r), (unsigned)a.Hkv, (unsigned)a.B);
    if (a.D == 64) hipLaunchKernelGGL((bwd_dkdv_split_kernel<64, 2, 4>), grid, dim3(512), 0, stream, a);
    else if (mode == 1) hipLaunchKernelGGL((bwd_dkdv_split_kernel<128, 1, 4>), grid, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL((bwd_dkdv_split_kernel<128, 2, 2>), grid, dim3(256), 0, stream, a);
    return hipGetLastError();
  }
  if (a.D == 128) return launch_bwd_dkdv_mfma32(a, tiles, stream);
  // persistent: as many workgroups as the CUs hold at once
  const int64_t slots = (int64_t)a.n_cu * dkdv_groups_per_cu();
  hipLaunchKernelGGL(bwd_dkdv_bf16_kernel, dim3((unsigned)(tiles < slots ? tiles : slots)), dim3(256), 0, stream, a);
  return hipGetLastError();
}

// The wide kernel of D = 64: 32x32x16 while most CUs hold one workgroup of 128
// rows, 16x16x32 where two overlap on most (figures beside the former: 4 heads,
// rows [10000, 20000), a load of 0.93, 311 / 323 us; 16 heads, rows [8192,
// 12288), 1.67, 253 / 249).
hipError_t launch_bwd_dq_bf16(const ChunkArgs& a, hipStream_t stream) {
  if (a.D != 128 && a.D != 64) return hipErrorInvalidValue;
  const int64_t s = a.c1 - a.c0, wide = (s + kDqRows - 1) / kDqRows * a.Hq * a.B;
  if (split_plan(a).dq) {
    const dim3 grid((unsigned)((s + 63) / 64), (unsigned)a.Hq, (unsigned)a.B);
    if (a.D == 128) hipLaunchKernelGGL(bwd_dq_split_kernel<128>, grid, dim3(512), 0, stream, a);
    else hipLaunchKernelGGL(bwd_dq_split_kernel<64>, grid, dim3(512), 0, stream, a);
  } else if (a.D == 128 || wide <= a.n_cu || load_per_cu(wide, a.c0, a.c1, a.n_cu) < 0.95) {
    return launch_bwd_dq_mfma32(a, stream);
  } else {
    const dim3 grid((unsigned)((s + kDqRows - 1) / kDqRows), (unsigned)a.Hq, (unsigned)a.B);
    hipLaunchKernelGGL(bwd_dq_bf16_kernel, grid, dim3(256), 0, stream, a);
  }
  return hipGetLastError();
}

bool bwd_pair_bf16(const ChunkArgs& a) {
  return (a.D == 128 || a.D == 64) && split_plan(a).pair && !dq_overwrites_inputs(a, 2);
}

hipError_t launch_bwd_pair_bf16(const ChunkArgs& a, hipStream_t stream) {
  if (a.kv0 < 0 || a.kv1 > a.c1 || a.kv0 >= a.kv1 || !bwd_pair_bf16(a)) return hipErrorInvalidValue;
  const int mode = split_plan(a).dkdv;
  const int64_t s = a.c1 - a.c0, rows = a.D == 64 ? 64 : 32, keys = mode == 2 ? 64 : 32;
  const int64_t dqx = (s + rows - 1) / rows, dkdvx = (a.kv1 - a.kv0 + keys - 1) / keys;
  const int64_t ndq = dqx * a.Hq * a.B, ndkdv = dkdvx * a.Hkv * a.B;
  const int64_t parts = a.D == 128 && mode == 2 ? 2 : 4;
  const int dq_first = a.c1 / kDqParts >= a.Hq / a.Hkv * s / parts;
  const PairGrid p{dq_first, (int)ndq, (int)dqx, (int)ndkdv, (int)dkdvx};
  const dim3 grid((unsigned)(ndq + ndkdv));
  if (a.D == 64) hipLaunchKernelGGL((bwd_pair_kernel<64, 2, 4>), grid, dim3(512), 0, stream, a, p);
  else if (mode == 1) hipLaunchKernelGGL((bwd_pair_kernel<128, 1, 4>), grid, dim3(256), 0, stream, a, p);
  else hipLaunchKernelGGL((bwd_pair_kernel<128, 2, 2>), grid, dim3(256), 0, stream, a, p);
  return hipGetLastError();
}

}  // namespace sppo
