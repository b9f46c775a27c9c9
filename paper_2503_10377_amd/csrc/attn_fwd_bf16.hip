// Forward of one chunk of sequence-chunked causal attention, bf16 in / fp32
// accumulate, for gfx950 (MI355X).
//
// Chunk i's queries (rows [c0, c1)) attend to keys [0, c1): every earlier
// chunk fully, the diagonal block causally (two-level activation management,
// Sec. 5.1 of SPPO: K/V of all earlier subsequences stay resident on the GPU).
//
// One workgroup = 4 waves = 128 query rows of one head; each wave owns 32
// rows (lane <-> query, two 16-row tiles, so row statistics are in-lane plus an
// exchange between the four 16-lane groups, made only when a running max
// moves).  Keys stream through LDS by LDS-DMA: K in a ring of four 32-key
// sub-block buffers, V in two 64-key tile buffers, one barrier per 64-key
// tile.  Per 32-key sub-block u each wave computes
//   S^T(u) = K(u) Q^T          (16x v_mfma_f32_16x16x32_bf16, D = 128)
//   P^T(u) = exp2(S^T C - m)   (online softmax in base 2, lazy rescale)
//   O^T   += V(u)^T P^T(u)     (16 MFMAs, P^T fed from S^T's registers)
// software pipelined: the MFMAs of S^T(u+1) run while the VALU turns S^T(u)
// into P^T(u), and the row max of S^T(u+1) is reduced while the PV MFMAs of
// u run.  Key tiles that reach the workgroup's own rows (the causal mask) are
// done afterwards, one at a time.  The epilogue writes O = O^T / l (bf16)
// and LSE = ln2 * (m + log2 l).
//
// Bound by power (the chip holds 1.8 of its 2.4 GHz) and by the softmax between
// the MFMAs.  With two workgroups on most compute units 16x16x32 MFMAs, the row
// max left in-lane, take 3-6% less time than 32x32x16 ones: 32 heads, rows
// [122880, 131072) 15.64 -> 14.97 ms, GQA 32/8, rows [12288, 16384) 840 -> 795
// us, D = 64, 32 heads, rows [8192, 16384) 875 -> 850.  Where most units hold
// one, attn_fwd_bf16_mfma32.hip is the faster; grids that leave units idle take
// the split kernel further down.
#include "sppo_kernels.h"
#include "tile_common.h"

namespace sppo {
namespace {

constexpr int kFwdBR = 128;      // query rows per workgroup (4 waves x 32)
constexpr int kFwdBC = 64;       // keys per V tile (two K sub-blocks)
constexpr float kLazyMax = 8.f;  // log2 headroom before the running max moves

#define SGB(mask, n) __builtin_amdgcn_sched_group_barrier(mask, n, 0)
constexpr int kSgMFMA = 0x008, kSgVALU = 0x002, kSgDSRead = 0x100, kSgTrans = 0x400;

template <int D>
__global__ __launch_bounds__(256, 2) void fwd_bf16_kernel(ChunkArgs a) {
  constexpr int BR = kFwdBR, BC = kFwdBC;
  using T = Tile<D>;
  constexpr int P = T::P;
  constexpr int NK = D / 32;  // k-steps of K Q^T
  constexpr int ND = D / 16;  // 16-wide d tiles of O^T
  constexpr int IPWK = (32 / T::RPI) / 4, IPWV = (BC / T::RPI) / 4;  // DMA instructions per wave
  static_assert(IPWK >= 1 && IPWK * 4 * T::RPI == 32 && IPWV * 4 * T::RPI == BC, "tiles split over 4 waves");
  __shared__ __attribute__((aligned(1024))) uint16_t K0[32 * P];
  __shared__ __attribute__((aligned(1024))) uint16_t K1[32 * P];
  __shared__ __attribute__((aligned(1024))) uint16_t K2[32 * P];
  __shared__ __attribute__((aligned(1024))) uint16_t K3[32 * P];
  __shared__ __attribute__((aligned(1024))) uint16_t V0[BC * P];
  __shared__ __attribute__((aligned(1024))) uint16_t V1[BC * P];
  auto kbuf = [&](auto I) -> uint16_t* {
    if constexpr (decltype(I)::value == 0) return K0;
    else if constexpr (decltype(I)::value == 1) return K1;
    else if constexpr (decltype(I)::value == 2) return K2;
    else return K3;
  };
  auto vbuf = [&](auto I) -> uint16_t* {
    if constexpr (decltype(I)::value == 0) return V0;
    else return V1;
  };
  auto kbuf_rt = [&](int i) -> uint16_t* { return i == 0 ? K0 : i == 1 ? K1 : i == 2 ? K2 : K3; };

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const GridPos gp = xcd_grouped();
  const int t = gridDim.x - 1 - gp.x;  // longest (latest) query tiles first
  const int h = gp.y;
  const int64_t b = gp.z;
  const int hk = h / (a.Hq / a.Hkv);
  const int64_t c0 = a.c0, c1 = a.c1, s = c1 - c0;
  const int64_t q0 = c0 + (int64_t)t * BR;
  const int64_t r = q0 + w * 32 + l16;  // this lane's rows: r and r + 16
  const int64_t kend = (q0 + BR < c1) ? q0 + BR : c1;
  const int nkv = (int)((kend + BC - 1) / BC);
  const int nsub = 2 * nkv;
  const int nfull = (int)(q0 / BC);  // tiles every row of the workgroup sees in full
  const float C = a.scale * kLog2e, iC = 1.f / C;

  int nat[NK];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) nat[kk] = T::nat(lane, kk, 0);
  int tro[ND];
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) tro[dt] = T::tr(lane, dt);
  const int64_t kvstride = (int64_t)a.Hkv * D;
  int dmak[IPWK], dmav[IPWV];
#pragma unroll
  for (int x = 0; x < IPWK; ++x) dmak[x] = T::dma(lane, w * IPWK + x, kvstride);
#pragma unroll
  for (int x = 0; x < IPWV; ++x) dmav[x] = T::dma(lane, w * IPWV + x, kvstride);

  bf16x8 qf[2][NK];
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    const int64_t rq = r + 16 * qt;
    const uint16_t* qrow = static_cast<const uint16_t*>(a.q) + ((b * s + (rq - c0)) * a.Hq + h) * D;
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) qf[qt][kk] = rq < c1 ? as_bf16x8(ld_global16(qrow + 32 * kk + 8 * g)) : bf16x8{};
  }
  const uint16_t* kbase = static_cast<const uint16_t*>(a.k) + (b * a.S * a.Hkv + hk) * D;
  const uint16_t* vbase = static_cast<const uint16_t*>(a.v) + (b * a.S * a.Hkv + hk) * D;

  // The next K sub-block (32 keys) or V tile (64 keys) into LDS; keys past
  // the chunk end load as zeros.  Both are issued in key order, so scalar
  // state walks K and V (no per-call index arithmetic).
  const int krow_bytes = (int)(kvstride * 2);
  uint64_t ka = uniform_u64(reinterpret_cast<uint64_t>(kbase)), va = uniform_u64(reinterpret_cast<uint64_t>(vbase));
  int remk = (int)c1, remv = (int)c1;  // keys left from the next sub-block / tile
  auto issue_k = [&](uint16_t* dst) {
    const int n = remk <= 0 ? 0 : (remk < 32 ? remk : 32);
    const auto rk = uniform_rsrc(ka, n * krow_bytes);
#pragma unroll
    for (int x = 0; x < IPWK; ++x) lds_dma16(rk, dst + (w * IPWK + x) * 512, dmak[x]);
    ka += (uint64_t)32 * krow_bytes;
    remk -= 32;
  };
  auto issue_v = [&](uint16_t* dst) {
    const int n = remv <= 0 ? 0 : (remv < BC ? remv : BC);
    const auto rv = uniform_rsrc(va, n * krow_bytes);
#pragma unroll
    for (int x = 0; x < IPWV; ++x) lds_dma16(rv, dst + (w * IPWV + x) * 512, dmav[x]);
    va += (uint64_t)BC * krow_bytes;
    remv -= BC;
  };
  // K operand of 16-key tile kt, k-step kk; V^T operand of d tile dt (32 keys).
  auto ld_k = [&](const uint16_t* K, int kt, int kk) {
    return ld_nat(K + 16 * kt * P, nat[D == 64 ? kk ^ kt : kk]);  // D = 64: rows 16.. swap the k-steps' chunks
  };
  auto ld_vt = [&](const uint16_t* V, int dt) { return ld_tr(V, tro[dt], tro[D == 64 ? dt ^ 2 : dt] + 16 * P); };

  f32x4 o[ND][2];
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) o[dt][0] = o[dt][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  // Running max (base 2), its limit in units of S, and this lane's share of the row sum.
  float m[2] = {-INFINITY, -INFINITY}, lim[2] = {-INFINITY, -INFINITY}, lsum[2] = {0.f, 0.f};

  // S^T of a 32-key sub-block: [16-key tile][16-query tile].
  struct S4 { f32x4 x[2][2]; };
  auto max8 = [](const S4& sv, int qt) {
    const f32x4 &x = sv.x[0][qt], &y = sv.x[1][qt];
    return max_nc(max3_nc(max3_nc(x[0], x[1], x[2]), max3_nc(x[3], y[0], y[1]), y[2]), y[3]);
  };
  // The running max m moves only when some row of the wave sees a max more
  // than kLazyMax above it (then O and l are rescaled); otherwise the stale m
  // is kept, so P = exp2(x - m) stays <= 2^kLazyMax -- exact in fp32 and in
  // range for bf16 -- and the O rescale is skipped.  mx: this lane's maximum of
  // S, over its own keys; the rows' maxima are only formed when one moves.
  auto rescale_if_needed = [&](float mx0, float mx1) {
    if (__any(mx0 > lim[0] || mx1 > lim[1])) {
      const float mx[2] = {max_groups(mx0) * C, max_groups(mx1) * C};
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
        const float mnew = fmaxf(m[qt], mx[qt]);
        const float alpha = fast_exp2(m[qt] - mnew);  // m = -inf on the first tile: 0
        m[qt] = mnew;
        lim[qt] = (mnew + kLazyMax) * iC;
        lsum[qt] *= alpha;
#pragma unroll
        for (int dt = 0; dt < ND; ++dt) o[dt][qt] *= alpha;
      }
    }
  };

  // One steady sub-block step: A then B.
  //   A: S^T(u+1) = K(u+1) Q^T (MFMA) | P^T(u) = exp2(S^T(u) C - m), bf16 pack (VALU)
  //   B: O^T += V(u)^T P^T(u)   (MFMA) | row sums of P(u), row max of S^T(u+1) (VALU)
  // Knext: sub-block u+1's K buffer; Vh: sub-block u's 32 V rows.
  auto step = [&](const S4& scur, S4& snext, const uint16_t* Knext, const uint16_t* Vh, float (&mx)[2]) {
    bf16x8 kop[2][NK];
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      kop[0][kk] = ld_k(Knext, 0, kk);
      kop[1][kk] = ld_k(Knext, 1, kk);
    }
    bf16x8 vop[ND];
#pragma unroll
    for (int dt = 0; dt < ND; ++dt) vop[dt] = ld_vt(Vh, dt);
    float p[2][8];
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
#pragma unroll
      for (int v = 0; v < 8; ++v) p[qt][v] = fast_exp2(scur.x[v >> 2][qt][v & 3] * C - m[qt]);
    }
    bf16x8 pb[2];
#pragma unroll
    for (int qt = 0; qt < 2; ++qt)
      pb[qt] = pack_bf16x8(p[qt][0], p[qt][1], p[qt][2], p[qt][3], p[qt][4], p[qt][5], p[qt][6], p[qt][7]);
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
        for (int qt = 0; qt < 2; ++qt)
          snext.x[kt][qt] = mfma16(kop[kt][kk], qf[qt][kk], kk == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : snext.x[kt][qt]);
      }
    }
#pragma unroll
    for (int dt = 0; dt < ND; ++dt) {
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) o[dt][qt] = mfma16(vop[dt], pb[qt], o[dt][qt]);
    }
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
      lsum[qt] += ((p[qt][0] + p[qt][1]) + (p[qt][2] + p[qt][3])) + ((p[qt][4] + p[qt][5]) + (p[qt][6] + p[qt][7]));
      mx[qt] = max8(snext, qt);
    }
    // A: four K reads and four exponent FMAs up front, then per MFMA one more
    // read, the exps (the scheduling groups count transcendental ops apart from
    // other VALU ops) and two VALU ops; B: the first PV MFMA, the remaining V
    // reads, then the other PV MFMAs with the sums and the max.  Groups of two
    // or four MFMAs, and all K reads up front, were 1-4% slower.
    SGB(kSgDSRead, 4);
    SGB(kSgVALU, 4);
#pragma unroll
    for (int i = 0; i < 4 * NK; ++i) {
      SGB(kSgMFMA, 1);
      SGB(kSgDSRead, 1);
      SGB(kSgTrans, 16 / (4 * NK));
      if (i < 4 * NK - 2) SGB(kSgVALU, 2);
    }
    SGB(kSgMFMA, 1);
    SGB(kSgDSRead, 8);
    SGB(kSgVALU, 2);
#pragma unroll
    for (int i = 1; i < 2 * ND; ++i) {
      SGB(kSgMFMA, 1);
      SGB(kSgVALU, 2);
    }
  };

  // Prologue: K sub-blocks 0..2 and V tile 0.
  issue_k(K0);
  issue_v(V0);
  if (1 < nsub) issue_k(K1);
  if (2 < nsub) issue_k(K2);
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
  __syncthreads();
  int klast = nsub < 3 ? nsub - 1 : 2, vlast = 0;  // last K sub-block / V tile issued

  auto first_s = [&](const uint16_t* K, S4& sv) {
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        const bf16x8 kx = ld_k(K, kt, kk);
#pragma unroll
        for (int qt = 0; qt < 2; ++qt)
          sv.x[kt][qt] = mfma16(kx, qf[qt][kk], kk == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sv.x[kt][qt]);
      }
    }
  };
  if (nfull > 0) {
    const int U = 2 * nfull;
    S4 sa, sb;
    first_s(K0, sa);
    rescale_if_needed(max8(sa, 0), max8(sa, 1));
    __syncthreads();  // every wave is done with K0 before sub-block 4 lands there
    if (3 < nsub) issue_k(K3);
    if (4 < nsub) issue_k(K0);
    if (1 < nkv) issue_v(V1);
    // Tile j, parity PAR (every LDS base an immediate): sub-blocks 2j (S^T in
    // sa) and 2j+1 (S^T in sb).  At its start K sub-blocks <= 2j+2 and V tile
    // j have landed; sub-blocks 2j-1, 2j and V tile j-1 are free for
    // sub-blocks 2j+3, 2j+4 and V tile j+1.
    auto tile = [&](int j, auto par) {
      constexpr int PAR = decltype(par)::value;
      if (j > 0) {
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
        __syncthreads();
        if (2 * j + 3 < nsub) issue_k(kbuf(IC<(2 * PAR + 3) & 3>{}));
        if (2 * j + 4 < nsub) issue_k(kbuf(IC<(2 * PAR) & 3>{}));
        if (j + 1 < nkv) issue_v(vbuf(IC<(PAR + 1) & 1>{}));
      }
      const uint16_t* V = vbuf(IC<PAR>{});
      float mx[2];
      step(sa, sb, kbuf(IC<(2 * PAR + 1) & 3>{}), V, mx);
      rescale_if_needed(mx[0], mx[1]);
      step(sb, sa, kbuf(IC<(2 * PAR + 2) & 3>{}), V + 32 * P, mx);
      if (2 * j + 2 < U) rescale_if_needed(mx[0], mx[1]);  // past the last steady tile it is not a real max
    };
    int j = 0;
    for (; j + 2 <= nfull; j += 2) {
      tile(j, IC<0>{});
      tile(j + 1, IC<1>{});
    }
    if (j < nfull) tile(j, IC<0>{});
    klast = 2 * nfull + 2 < nsub - 1 ? 2 * nfull + 2 : nsub - 1;
    vlast = nfull < nkv - 1 ? nfull : nkv - 1;
  }

  // Diagonal tiles [nfull, nkv), with the causal mask, one 64-key tile at a
  // time; the first was loaded ahead by the steady loop (or the prologue).
  for (int j = nfull; j < nkv; ++j) {
    if (j > nfull) {
      __syncthreads();  // every wave is done with tile j-1
      for (int u = klast + 1; u <= 2 * j + 1 && u < nsub; ++u) issue_k(kbuf_rt(u & 3));
      if (2 * j + 1 > klast) klast = 2 * j + 1 < nsub - 1 ? 2 * j + 1 : nsub - 1;
      if (j > vlast) {
        issue_v((j & 1) ? V1 : V0);
        vlast = j;
      }
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __syncthreads();
    const int64_t k0 = (int64_t)j * BC;
    const uint16_t* V = (j & 1) ? V1 : V0;
    S4 sv[2];
    const int rel = (int)(r - k0);  // key offset within the tile of row r
#pragma unroll
    for (int jb = 0; jb < 2; ++jb) {
      first_s(kbuf_rt((2 * j + jb) & 3), sv[jb]);
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            if (32 * jb + 16 * kt + 4 * g + v > rel + 16 * qt) sv[jb].x[kt][qt][v] = -INFINITY;
          }
        }
      }
    }
    rescale_if_needed(max_nc(max8(sv[0], 0), max8(sv[1], 0)), max_nc(max8(sv[0], 1), max8(sv[1], 1)));
#pragma unroll
    for (int jb = 0; jb < 2; ++jb) {
      bf16x8 pb[2];
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
        float p[8];
#pragma unroll
        for (int v = 0; v < 8; ++v) {
          p[v] = fast_exp2(sv[jb].x[v >> 2][qt][v & 3] * C - m[qt]);
          lsum[qt] += p[v];
        }
        pb[qt] = pack_bf16x8(p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7]);
      }
#pragma unroll
      for (int dt = 0; dt < ND; ++dt) {
        const bf16x8 vx = ld_vt(V + 32 * jb * P, dt);
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) o[dt][qt] = mfma16(vx, pb[qt], o[dt][qt]);
      }
    }
  }

#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    const float lt = sum_groups(lsum[qt]);
    const int64_t rq = r + 16 * qt;
    if (rq < c1) {
      const float inv = 1.f / lt;
      uint16_t* orow = static_cast<uint16_t*>(a.o) + ((b * s + (rq - c0)) * a.Hq + h) * D;
#pragma unroll
      for (int dt = 0; dt < ND; ++dt)
        *reinterpret_cast<u32x2*>(orow + 16 * dt + 4 * g) =
            pack_bf16x4(o[dt][qt][0] * inv, o[dt][qt][1] * inv, o[dt][qt][2] * inv, o[dt][qt][3] * inv);
      if (g == 0) a.lse[(b * a.Hq + h) * s + (rq - c0)] = (m[qt] + fast_log2(lt)) * kLn2;
    }
  }
}

// The same for grids that leave compute units idle: a workgroup is 8 waves, two
// groups of 32 query rows of one head times four parts of the keys (part ks has
// the 32-key sub-blocks u = ks, ks + 4, ...), each wave with its own running
// max, sum and O; the parts are added through LDS in part order.  A sub-block's
// part depends on its position in the sequence alone, so with chunk boundaries
// on multiples of 32 rows (a wave's rows move their running maxima together) a
// row's result does not depend on the chunking, as long as every chunk's launch
// takes this kernel.  Bound by the latency of a step (four sub-blocks,
// about 1.05 us against 0.42 us for each one in the kernel above); four groups
// times two parts took the same time a step and gained nothing, one group times
// eight parts is bound by L2 (every 32 rows stream K and V).
template <int D>
__global__ __launch_bounds__(512) void fwd_split_kernel(ChunkArgs a) {
  using T = Tile<D>;
  constexpr int P = T::P, NK = D / 32, ND = D / 16, RG = 2, KS = 4, R = 32 * RG;
  constexpr int IPW = 32 / T::RPI / RG;  // DMA instructions per wave for each of K and V
  static_assert(IPW >= 1 && IPW * RG * T::RPI == 32, "a sub-block splits over RG waves");
  constexpr int SB = 2 * 32 * P;     // elements of a sub-block's K and V
  constexpr int OP = D + 4;          // row pitch of the partial O's, floats
  constexpr int kBytes = 2 * KS * SB * 2 > KS * R * OP * 4 ? 2 * KS * SB * 2 : KS * R * OP * 4;
  __shared__ __attribute__((aligned(1024))) unsigned char mem[kBytes];
  __shared__ float Ms[KS][R], Ls[KS][R];

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4, rg = w % RG, ks = w / RG;
  const GridPos gp = xcd_grouped();
  const int h = gp.y;
  const int64_t b = gp.z;
  const int hk = h / (a.Hq / a.Hkv);
  const int64_t c0 = a.c0, c1 = a.c1, s = c1 - c0;
  const int64_t q0 = c0 + (int64_t)(gridDim.x - 1 - gp.x) * R;
  const int64_t qw = q0 + 32 * rg, r = qw + l16;  // this lane's rows: r and r + 16
  const int64_t kend = q0 + R < c1 ? q0 + R : c1;
  const int nsub = (int)((kend + 31) / 32), nstep = (nsub + KS - 1) / KS;
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
  bf16x8 qf[2][NK];
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    const int64_t rq = r + 16 * qt;
    const uint16_t* qrow = static_cast<const uint16_t*>(a.q) + ((b * s + (rq - c0)) * a.Hq + h) * D;
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) qf[qt][kk] = rq < c1 ? as_bf16x8(ld_global16(qrow + 32 * kk + 8 * g)) : bf16x8{};
  }
  const uint16_t* kbase = static_cast<const uint16_t*>(a.k) + (b * a.S * a.Hkv + hk) * D;
  const uint16_t* vbase = static_cast<const uint16_t*>(a.v) + (b * a.S * a.Hkv + hk) * D;
  uint16_t* const kv = reinterpret_cast<uint16_t*>(mem) + ks * SB;  // this part's slot, buffer 0
  auto issue = [&](int i) {  // keys past the chunk arrive as zeros
    const int64_t j0 = ((int64_t)i * KS + ks) * 32;
    uint16_t* dst = kv + (i & 1) * KS * SB;
    const auto rk = tile_rsrc(kbase + j0 * kvstride, c1 - j0, 32, kvstride);
    const auto rv = tile_rsrc(vbase + j0 * kvstride, c1 - j0, 32, kvstride);
#pragma unroll
    for (int x = 0; x < IPW; ++x) {
      lds_dma16(rk, dst + (rg * IPW + x) * 512, dma[x]);
      lds_dma16(rv, dst + 32 * P + (rg * IPW + x) * 512, dma[x]);
    }
  };

  f32x4 o[ND][2];
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) o[dt][0] = o[dt][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m[2] = {-INFINITY, -INFINITY}, lsum[2] = {0.f, 0.f};
  auto block = [&](int u, const uint16_t* K) {
    const uint16_t* V = K + 32 * P;
    // Every K operand up front, the first V^T operands under the softmax, the
    // others kAhead ahead of their MFMAs (left to the compiler, each read was
    // waited for right after it was issued).
    constexpr int kAhead = 4;
    bf16x8 kx[NK][2], vx[ND];
    auto rd_v = [&](int dt) { return ld_tr(V, tro[dt], tro[D == 64 ? dt ^ 2 : dt] + 16 * P); };
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) kx[kk][kt] = ld_nat(K + 16 * kt * P, nat[D == 64 ? kk ^ kt : kk]);
    }
    __builtin_amdgcn_sched_barrier(0);
    f32x4 sv[2][2];
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
        for (int qt = 0; qt < 2; ++qt)
          sv[kt][qt] = mfma16(kx[kk][kt], qf[qt][kk], kk == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sv[kt][qt]);
      }
    }
#pragma unroll
    for (int dt = 0; dt < kAhead; ++dt) vx[dt] = rd_v(dt);
    __builtin_amdgcn_sched_barrier(0);
    if ((int64_t)u * 32 + 31 > qw) {
      const int rel = (int)(r - (int64_t)u * 32);
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            if (16 * kt + 4 * g + v > rel + 16 * qt) sv[kt][qt][v] = -INFINITY;
          }
        }
      }
    }
    float mx[2];
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
      const f32x4 &x = sv[0][qt], &y = sv[1][qt];
      mx[qt] = max_nc(max3_nc(max3_nc(x[0], x[1], x[2]), max3_nc(x[3], y[0], y[1]), y[2]), y[3]) * C;
    }
    if (__any(mx[0] > m[0] + kLazyMax || mx[1] > m[1] + kLazyMax)) {
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
        const float mnew = fmaxf(m[qt], max_groups(mx[qt]));
        // a row that has seen no key yet (m = -inf) has nothing to rescale
        const float alpha = m[qt] == -INFINITY ? 0.f : fast_exp2(m[qt] - mnew);
        m[qt] = mnew;
        lsum[qt] *= alpha;
#pragma unroll
        for (int dt = 0; dt < ND; ++dt) o[dt][qt] *= alpha;
      }
    }
    bf16x8 pb[2];
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
      const float ms = m[qt] == -INFINITY ? 0.f : m[qt];
      float p[8];
#pragma unroll
      for (int v = 0; v < 8; ++v) p[v] = fast_exp2(sv[v >> 2][qt][v & 3] * C - ms);
      lsum[qt] += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
      pb[qt] = pack_bf16x8(p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int dt = 0; dt < ND; ++dt) {
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) o[dt][qt] = mfma16(vx[dt], pb[qt], o[dt][qt]);
      if (dt + kAhead < ND) vx[dt + kAhead] = rd_v(dt + kAhead);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  issue(0);
  for (int i = 0; i < nstep; ++i) {
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __syncthreads();  // step i landed; every wave is done with step i - 1
    if (i + 1 < nstep) issue(i + 1);
    const int u = i * KS + ks;
    if ((int64_t)u * 32 <= qw + 31) block(u, kv + (i & 1) * KS * SB);  // else past this wave's rows
  }

  // The parts, [part][row][D], over the K/V slots.
  const float lt2[2] = {sum_groups(lsum[0]), sum_groups(lsum[1])};
  __syncthreads();
  float* const os = reinterpret_cast<float*>(mem);
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    const int row = 32 * rg + 16 * qt + l16;
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
      *reinterpret_cast<f32x4*>(os + (ks * R + row) * OP + 16 * dt + 4 * g) = o[dt][qt];
    if (g == 0) {
      Ms[ks][row] = m[qt];
      Ls[ks][row] = lt2[qt];
    }
  }
  __syncthreads();
  constexpr int TPR = 512 / R, EPT = D / TPR;  // threads per row, elements of O per thread
  const int row = tid / TPR, d0 = (tid % TPR) * EPT;
  if (q0 + row >= c1) return;
  float mm = Ms[0][row];
#pragma unroll
  for (int x = 1; x < KS; ++x) mm = fmaxf(mm, Ms[x][row]);
  float f[KS], lt = 0.f;
#pragma unroll
  for (int x = 0; x < KS; ++x) {
    f[x] = Ms[x][row] == -INFINITY ? 0.f : fast_exp2(Ms[x][row] - mm);
    lt += f[x] * Ls[x][row];
  }
  const float inv = 1.f / lt;
  uint16_t* orow = static_cast<uint16_t*>(a.o) + ((b * s + (q0 + row - c0)) * a.Hq + h) * D + d0;
#pragma unroll
  for (int e = 0; e < EPT; e += 4) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < KS; ++x) {
      if (f[x] != 0.f) acc += f[x] * *reinterpret_cast<const f32x4*>(os + (x * R + row) * OP + d0 + e);
    }
    *reinterpret_cast<u32x2*>(orow + e) = pack_bf16x4(acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
  }
  if (d0 == 0) a.lse[(b * a.Hq + h) * s + (q0 + row - c0)] = (mm + fast_log2(lt)) * kLn2;
}

}  // namespace

hipError_t launch_fwd_bf16(const ChunkArgs& a, hipStream_t stream) {
  if (a.D != 128 && a.D != 64) return hipErrorInvalidValue;
  const int64_t s = a.c1 - a.c0;
  // The split kernel where its workgroups (64 rows; one a CU by LDS at D = 128,
  // two at D = 64) all run at once.  Forward of 2048 rows x 4 heads x 128 (128
  // workgroups) 33 -> 20 us, of 512 x 32 (256) 9 -> 6.5, but of 1024 x 32 (512)
  // 18 -> 24; D = 64: 1667 x 8 x batch 2 (432) 21 -> 17, 2048 x 32 (1024) even.
  // Up to 64 keys two of its four parts have nothing to do and the sum over
  // them costs more than it saves (64 rows x 16/4 heads 7.5 -> 9.2 us, 32 x 32
  // 7.0 -> 8.4; 128 keys 10.3 -> 9.8).
  // The others by the load of their 128-row workgroups on the compute units:
  // 32x32x16 with no more than one a unit, or where the long ones run alone for
  // most of the launch (8 heads, 5376 rows 92 / 97 us against 16x16x32, 336
  // workgroups at a load of 0.66; rows [3000, 8376) 155 / 157, 0.89; but rows
  // [12000, 16352) 339 / 318, 272 at 0.92).
  const int64_t split = (s + 63) / 64 * a.Hq * a.B, wide = (s + kFwdBR - 1) / kFwdBR * a.Hq * a.B;
  const int cus = device_cus();
  if (a.c1 > 64 && split <= (int64_t)cus * (a.D == 64 ? 2 : 1)) {
    const dim3 grid((unsigned)((s + 63) / 64), (unsigned)a.Hq, (unsigned)a.B);
    if (a.D == 128) hipLaunchKernelGGL(fwd_split_kernel<128>, grid, dim3(512), 0, stream, a);
    else hipLaunchKernelGGL(fwd_split_kernel<64>, grid, dim3(512), 0, stream, a);
  } else if (wide <= cus || load_per_cu(wide, a.c0, a.c1, cus) < 0.9) {
    return launch_fwd_mfma32(a, stream);
  } else {
    const dim3 grid((unsigned)((s + kFwdBR - 1) / kFwdBR), (unsigned)a.Hq, (unsigned)a.B);
    if (a.D == 128) hipLaunchKernelGGL(fwd_bf16_kernel<128>, grid, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL(fwd_bf16_kernel<64>, grid, dim3(256), 0, stream, a);
  }
  return hipGetLastError();
}

}  // namespace sppo
