"""GPU parity at the edges of the kernels' tiles and dispatch rules: sizes one
below, at and one above a tile, remainders in every dimension, and the
smallest sizes, against the fp64 oracle with the gates of parity.py."""
import math
import sys

import numpy as np
import pytest
import torch

import oracle
from oracle import transformer_layer as T
from paper_2503_10377_amd import sppo as L
from paper_2503_10377_amd.chunked import ChunkedAttention
from paper_2503_10377_amd.inputs import make_inputs
from parity import check_all, to_np
from test_gpu_parity import run_case
from test_structured_gates_cpu import bf16_recipe

pytestmark = pytest.mark.gpu


def announce(msg):
    print(f"\n[case] {msg}", file=sys.stderr, flush=True)


def walk(inp, B, S, N, Hq, Hkv, D, dtype, offsets=None):
    ca = ChunkedAttention(B, S, N, Hq, Hkv, D, dtype=dtype, offsets=offsets)
    out = ca.alloc_outputs()
    ca.step(inp, out)
    torch.cuda.synchronize()
    res = {"o": to_np(out["o"]), "lse": to_np(ca.lse_full(out)), "dq": to_np(out["dq"]), "dk": to_np(out["dk"]),
           "dv": to_np(out["dv"])}
    ca.close()
    return res


# 16-row query and key blocks, 8 (D = 64) or 4 waves over them, 32 keys a forward iteration at D = 64.
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("offsets", [[0, 1, 16, 17], [0, 15, 31, 48], [0, 128, 257, 258], [0, 255]])
def test_fp32_blocks(D, offsets):
    gpu, ref, off = run_case(2, offsets[-1], 6, 2, D, "f32", offsets=offsets, seed=17)
    check_all(gpu, ref, "f32", off)


@pytest.mark.parametrize("D", [64, 128])
def test_fp32_nonfinite_rows_stay_behind_the_mask(D):
    """An infinity in V or K of the last key reaches the last row alone, a
    NaN in dO or Q of the first row only the first key: the rows and keys
    beside them in the same blocks keep their values."""
    B, S, Hq, Hkv, N = 1, 61, 2, 1, 2
    offsets = [0, 30, 61]
    announce(f"fp32 non-finite D={D}")
    inp = make_inputs(B, S, Hq, Hkv, D, torch.float32, seed=3, device="cuda")
    ref = walk(inp, B, S, N, Hq, Hkv, D, "f32", offsets)
    bad = {n: t.clone() for n, t in inp.items()}
    bad["v"][:, -1, :, 5] = float("inf")
    bad["k"][:, -1, :, 7] = float("nan")
    got = walk(bad, B, S, N, Hq, Hkv, D, "f32", offsets)
    assert not np.isfinite(got["o"][:, -1]).all()
    for n in ("o", "dq"):
        np.testing.assert_allclose(got[n][:, :-1], ref[n][:, :-1], rtol=0, atol=2e-6, err_msg=n)
    bad = {n: t.clone() for n, t in inp.items()}
    bad["do"][:, 0, :, 3] = float("nan")
    bad["q"][:, 0, :, 9] = float("inf")
    got = walk(bad, B, S, N, Hq, Hkv, D, "f32", offsets)
    assert not np.isfinite(got["dv"][:, 0]).all()
    for n in ("dk", "dv"):
        np.testing.assert_allclose(got[n][:, 1:], ref[n][:, 1:], rtol=0, atol=2e-6, err_msg=n)


def gemm(lay, M, N, K, a, b, epi="bf16", aux=None, c=None):
    lda, ldb = a.shape[1], b.shape[1]
    if c is None:
        c = torch.full((M, N), 7.0, device="cuda", dtype=torch.float32 if "f32" in epi else torch.bfloat16)
    L.sppo_gemm_bf16(lay, M, N, K, a, lda, b, ldb, c, N, epi, aux, N if aux is not None else 0)
    torch.cuda.synchronize()
    return c


# 64, 128 and 256 tiles (the last from 4097 x 4100 on), one k-block, an odd and an even number of them.
@pytest.mark.parametrize("M,N,K", [(63, 68, 64), (65, 60, 192), (64, 1028, 640), (129, 2052, 128), (127, 4100, 64),
                                   (4097, 4100, 64), (4095, 4092, 192)])
def test_gemm_nt_tiles(M, N, K):
    """Every epilogue of NT against the fp64 product; the rows that a product
    of the first 60 rows (another tile) computes have the same bits."""
    announce(f"gemm nt tiles {M}x{N}x{K}")
    g = torch.Generator().manual_seed(M + N + K)
    a, b, x = (torch.randn(*s, generator=g).to(torch.bfloat16) for s in ((M, K), (N, K), (M, N)))
    ad, bd, xd = a.cuda(), b.cuda(), x.cuda()
    ref = to_np(a) @ to_np(b).T
    xr = to_np(x)
    for epi, want in (("bf16", ref), ("add_bf16", ref + xr), ("dgelu", ref * T.gelu_grad(xr)), ("gelu", None),
                      ("f32", ref), ("acc_f32", ref + 7.0)):
        aux = xd.clone() if epi in ("add_bf16", "dgelu", "gelu") else None
        got = gemm("nt", M, N, K, ad, bd, epi, aux)
        sub = gemm("nt", min(M, 60), N, K, ad[:60], bd, epi, None if aux is None else xd[:60].clone())
        assert torch.equal(got[:60], sub), epi
        if epi == "gelu":
            pre = to_np(aux)
            assert np.abs(pre - ref).max() <= 8e-3 * np.abs(ref).max()
            want = T.gelu(pre)
        tol = 1e-5 if "f32" in epi else 8e-3
        assert np.abs(to_np(got) - want).max() <= tol * np.abs(want).max() + 1e-6, epi


@pytest.mark.parametrize("M,N,K", [(256, 256, 64), (512, 768, 129), (1024, 4096, 63), (4096, 4352, 150)])
def test_gemm_tn_tiles(M, N, K):
    announce(f"gemm tn tiles {M}x{N}x{K}")
    g = torch.Generator().manual_seed(M + N + K)
    a, b = (torch.randn(K, n, generator=g).to(torch.bfloat16) for n in (M, N))
    ref = to_np(a).T @ to_np(b)
    got = gemm("tn", M, N, K, a.cuda(), b.cuda(), "f32")
    assert np.abs(to_np(got) - ref).max() <= 1e-5 * np.abs(ref).max() + 1e-6
    got = gemm("tn", M, N, K, a.cuda(), b.cuda(), "acc_f32", c=got)
    assert np.abs(to_np(got) - 2 * ref).max() <= 1e-5 * np.abs(2 * ref).max() + 1e-6
    got = gemm("tn", M, N, K, a.cuda(), b.cuda(), "bf16")
    assert np.abs(to_np(got) - ref).max() <= 8e-3 * np.abs(ref).max()


# TN that is written and not added, up to 16 k-blocks on 256 tiles: one row, odd and even numbers of k-blocks, a last
# one with rows missing, and beside the limit; C's rows longer than N stay as they were past it.
@pytest.mark.parametrize("M,N,K", [(4096, 4352, 1), (4352, 4096, 64), (4096, 4352, 65), (5120, 4096, 190), (4096, 4096, 1024),
                                   (4096, 4096, 1025)])
@pytest.mark.parametrize("epi", ["f32", "bf16"])
def test_gemm_tn_short(M, N, K, epi):
    announce(f"gemm tn short {epi} {M}x{N}x{K}")
    g = torch.Generator().manual_seed(M + N + K)
    a, b = (torch.randn(K, n, generator=g).to(torch.bfloat16) for n in (M, N))
    ld = N + 8
    c = torch.full((M, ld), 7.0, device="cuda", dtype=torch.float32 if epi == "f32" else torch.bfloat16)
    ad, bd = a.cuda(), b.cuda()
    L.sppo_gemm_bf16("tn", M, N, K, ad, M, bd, N, c, ld, epi)
    torch.cuda.synchronize()
    ref = to_np(a).T @ to_np(b)
    got = to_np(c)
    assert (got[:, N:] == 7.0).all()
    assert np.abs(got[:, :N] - ref).max() <= (1e-5 if epi == "f32" else 8e-3) * np.abs(ref).max() + 1e-6


# The split attention kernels (64 query rows, 32 or 64 keys a workgroup, four or two parts) and the wide ones beside
# them: one row, one below, at and above a sub-block (32), a workgroup (64) and a wide tile (128), chunk boundaries off
# all of them, GQA; the last two have enough heads for the wide kernels in some launches and the split ones in others.
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,Hq,Hkv,offsets", [(1, 2, 1, [0, 1, 2]), (2, 2, 2, [0, 31, 63, 96]), (1, 6, 2, [0, 33, 130, 300]),
                                              (1, 4, 1, [0, 64, 192, 449]), (1, 3, 3, [0, 127, 255, 700]),
                                              (2, 32, 8, [0, 257, 600]), (1, 64, 16, [0, 300, 333, 1100])])
def test_bf16_split_and_wide(D, B, Hq, Hkv, offsets):
    gpu, ref, off = run_case(B, offsets[-1], Hq, Hkv, D, "bf16", offsets=offsets, seed=19)
    check_all(gpu, ref, "bf16", off)


# The wide kernels under the mask, with enough heads that no launch of a kind is split: one chunk of 1024 rows x 64 heads
# is 512 workgroups of 128 rows (16x16x32 forward; D = 64: dQ too), two of 512 are 256 each (32x32x16; D = 64: split).
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("kind", ["sharp_self", "sharp_future", "zero_q"])
def test_bf16_structured_wide(kind, D):
    """The first and the last KV group against the oracle, within twice the error
    that the bf16 rounding points alone make on these inputs (computed beside it;
    at D = 64 sharp_self they exceed the gates derived for D = 128).  A mask off
    by one key moves O, LSE and dV by O(1)."""
    B, S, Hq, Hkv = 1, 1024, 64, 32
    inp = make_inputs(B, S, Hq, Hkv, D, torch.bfloat16, seed=6, device="cuda", kind=kind)
    qh, kh = [0, 1, 62, 63], [0, 31]
    host = {n: to_np(t[:, :, qh if n in ("q", "do") else kh]) for n, t in inp.items()}
    args = (host["q"], host["k"], host["v"], host["do"], 1.0 / math.sqrt(D))
    ref, rounded = oracle.attention(*args), bf16_recipe(*args)
    for N in (1, 2):
        announce(f"structured wide {kind} D={D} N={N}")
        got = walk(inp, B, S, N, Hq, Hkv, D, "bf16")
        assert np.abs(got["lse"][:, qh] - ref["lse"]).max() <= 1e-3
        for n in ("o", "dq", "dk", "dv"):
            err = np.abs(got[n][:, :, qh if n in ("o", "dq") else kh] - ref[n])
            base = np.abs(rounded[n] - ref[n])
            assert err.max() <= 2 * base.max() + 1e-6 and err.mean() <= 2 * base.mean() + 1e-7, (n, N, err.max(), base.max())


@pytest.mark.parametrize("D", [64, 128])
def test_bf16_ragged_wide_accumulates(D):
    """dK/dV of the wide kernels added over chunks at boundaries off every tile
    (the launches of the later chunks are past the split kernels' sizes)."""
    gpu, ref, off = run_case(2, 1111, 64, 32, D, "bf16", offsets=[0, 301, 700, 1111], seed=29)
    check_all(gpu, ref, "bf16", off)


def test_bf16_mfma32_dq_of_head_size_64():
    """The 32x32x16 dQ of head size 64 (17 heads, 1000 rows: 272 workgroups of 64
    rows, three heads an XCD) at boundaries off its tiles."""
    gpu, ref, off = run_case(1, 1333, 17, 17, 64, "bf16", offsets=[0, 1001, 1333], seed=31)
    check_all(gpu, ref, "bf16", off)


@pytest.mark.parametrize("Hq,S,N,same", [(32, 8192, 4, True), (4, 8192, 8, False)])
def test_chunking_and_the_choice_of_kernels(Hq, S, N, same):
    """Chunk boundaries on the tile grid leave O, LSE and dQ bit for bit where
    every launch takes the same kernels (here the wide ones).  Where the chunks
    are small enough for the split kernels and the whole is not, the keys are
    summed in another order and against other running maxima: O and dQ differ
    by roundings of P (or dS) and of the result to bf16, 2^-9 each on either
    side; LSE by fp32 sums."""
    inp = make_inputs(1, S, Hq, Hq, 128, torch.bfloat16, seed=37, device="cuda")
    announce(f"chunking Hq={Hq} S={S} N={N}")
    one, many = (walk(inp, 1, S, n, Hq, Hq, 128, "bf16") for n in (1, N))
    for n in ("o", "dq"):
        if same:
            assert np.array_equal(one[n], many[n]), n
        else:
            assert np.linalg.norm(one[n] - many[n]) <= 4 * 2.0**-9 * np.linalg.norm(one[n]), n
    assert np.abs(one["lse"] - many["lse"]).max() <= (0 if same else 2e-5)
    for n in ("dk", "dv"):  # the order of fp32 sums, and (split) the same roundings
        assert np.linalg.norm(one[n] - many[n]) <= (1e-5 if same else 4 * 2.0**-9) * np.linalg.norm(one[n]), n


@pytest.mark.parametrize("Hq,Hkv,D,offsets", [(8, 2, 128, [0, 500, 1000, 1777]), (16, 16, 64, [0, 700, 1500])])
def test_bf16_evicting_walk_equals_resident_by_kernel_choice(Hq, Hkv, D, offsets):
    """The evicting walk's last backward runs its dK/dV once per KV chunk: each
    launch covers fewer keys but takes the same kernel, so the bits agree."""
    res = [run_case(1, offsets[-1], Hq, Hkv, D, "bf16", offsets=offsets, seed=23, offload=o)[0]
           for o in ("qkvol", "qkvol_evict")]
    for n in ("o", "lse", "dq", "dk", "dv"):
        assert np.array_equal(res[0][n], res[1][n]), n


# One wave per row up to 1024 columns, then 256 / 384 / 512 threads; the backward's
# workgroups take 16 rows in pairs, and from 8192 rows on more.
@pytest.mark.parametrize("rows,H", [(3, 8), (37, 512), (34, 520), (19, 1024), (18, 1032), (17, 2048), (5, 4104),
                                    (16, 6152), (8192, 64), (8195, 136), (9000, 1040)])
def test_layernorm_teams(rows, H):
    announce(f"layernorm teams rows={rows} H={H}")
    g = torch.Generator().manual_seed(rows * 7 + H)
    x, dy, dres = [(torch.randn(rows, H, generator=g) + b).to(torch.bfloat16) for b in (0.5, 0.0, 0.0)]
    gamma, beta = 1 + 0.1 * torch.randn(H, generator=g), 0.1 * torch.randn(H, generator=g)
    y, dx = torch.empty(rows, H, device="cuda", dtype=torch.bfloat16), dres.cuda()  # dx in place of dres
    mean, rstd = torch.empty(rows, device="cuda"), torch.empty(rows, device="cuda")
    dg, db = torch.full((H,), 2.0, device="cuda"), torch.full((H,), -1.0, device="cuda")
    wsb = L.sppo_layernorm_bwd_workspace(rows, H)
    ws = torch.full((wsb // 4 + 2,), float("nan"), device="cuda")[1:-1]  # a float's alignment, a word free on each side
    xd, gd = x.cuda(), gamma.cuda()
    L.sppo_layernorm_fwd(rows, H, xd, H, gd, beta.cuda(), 1e-5, y, H, mean, rstd)
    L.sppo_layernorm_bwd(rows, H, xd, H, gd, mean, rstd, dy.cuda(), H, dx, H, dx, H, dg, db, ws, wsb, 1)
    torch.cuda.synchronize()
    assert ws._base[0].isnan() and ws._base[-1].isnan(), "wrote outside the workspace"
    x, dy, dres, gamma, beta = [t.double() for t in (x, dy, dres, gamma, beta)]
    mu = x.mean(1, keepdim=True)
    r = (x.var(1, unbiased=False, keepdim=True) + 1e-5).rsqrt()
    xh = (x - mu) * r
    gg = dy * gamma
    wdx = dres + r * (gg - gg.mean(1, keepdim=True) - xh * (gg * xh).mean(1, keepdim=True))
    # bf16 results: half an ulp (2^-9), and 64 fp32 roundings of terms up to the row's largest.
    for got, want in ((y, xh * gamma + beta), (dx, wdx)):
        lim = want.abs() * 2.0**-8 + 64 * 2.0**-24 * want.abs().amax(1, keepdim=True) * (1 + r)
        assert ((got.cpu().double() - want).abs() <= lim).all()
    # fp32 sums over rows: at most 160 additions in any term's chain, and 32 roundings in the term.
    for got, t, base in ((dg, dy * xh, 2.0), (db, dy, -1.0)):
        lim = 192 * 2.0**-24 * (t.abs().sum(0) + abs(base))
        assert ((got.cpu().double() - base - t.sum(0)).abs() <= lim).all()


# 16 bytes per lane where rows and columns come in eights and the buffers are aligned.
@pytest.mark.parametrize("R,C,off", [(8, 8, 0), (64, 64, 0), (72, 264, 0), (200, 56, 0), (64, 64, 1), (64, 72, 4)])
def test_transpose_wide(R, C, off):
    announce(f"transpose {R}x{C} offset {off}")
    x = torch.randn(R * C + off).to(torch.bfloat16).cuda()[off:]
    y = torch.full((R * C + off + 8,), 3.0, device="cuda", dtype=torch.bfloat16)
    L.sppo_transpose_bf16(x, y[off:], R, C)
    torch.cuda.synchronize()
    assert torch.equal(y[off:off + R * C].view(C, R), x.view(R, C).t()) and (y[off + R * C:] == 3.0).all()


# dK/dV and dQ in one launch (small grids; fp32 D = 64 always) against one after the other (with kernel
# timing on, where they are separate launches): the same bits.  dQ in place of dO takes the separate launches.
@pytest.mark.parametrize("dtype,B,S,N,Hq,Hkv,D", [("bf16", 1, 200, 2, 2, 1, 128), ("bf16", 1, 2047, 4, 4, 4, 128),
                                                  ("bf16", 1, 1999, 2, 8, 8, 128), ("bf16", 2, 1001, 3, 4, 2, 64),
                                                  ("bf16", 1, 65, 1, 1, 1, 64), ("f32", 2, 301, 3, 4, 2, 64)])
def test_backward_pair_matches_separate_launches(dtype, B, S, N, Hq, Hkv, D):
    announce(f"backward pair {dtype} B={B} S={S} N={N} H={Hq}/{Hkv} D={D}")
    inp = make_inputs(B, S, Hq, Hkv, D, torch.bfloat16 if dtype == "bf16" else torch.float32, seed=7, device="cuda")
    ca = ChunkedAttention(B, S, N, Hq, Hkv, D, dtype=dtype, offsets=[S * i // N for i in range(N + 1)])
    outs = []
    for timing in (False, True):
        L.sppo_set_kernel_timing(ca.ctx, timing)
        out = ca.alloc_outputs()
        ca.step(inp, out)
        torch.cuda.synchronize()
        outs.append(out)
    times = L.sppo_kernel_times(ca.ctx)
    assert times["bwd_dkdv"]["launches"] == times["bwd_dq"]["launches"] == N
    for key in ("o", "dq", "dk", "dv"):
        assert torch.equal(outs[0][key], outs[1][key]), key
    c0, c1 = ca.offsets[N - 1], ca.offsets[N]
    q, do, o = [t[:, c0:c1].contiguous() for t in (inp["q"], inp["do"], outs[0]["o"])]
    dk, dv = torch.empty_like(outs[0]["dk"]), torch.empty_like(outs[0]["dv"])
    got = []
    for dq in (torch.empty_like(q), do):  # the second call replaces dO
        L.sppo_attn_bwd_chunk_noalloc(B, S, c0, c1, Hq, Hkv, D, dtype, 0.0, 0, q, inp["k"], inp["v"], o,
                                      outs[0]["lse"][N - 1], do, dq, dk, dv)
        torch.cuda.synchronize()
        got.append((dq.clone(), dk.clone(), dv.clone()))
    assert all(torch.equal(x, y) for x, y in zip(*got))
