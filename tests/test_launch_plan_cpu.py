"""Which kernels the launchers choose, and their grids, without a GPU
(launch_plan.cpp records the launches instead of making them)."""
import os
import subprocess

import pytest

from paper_2503_10377_amd import build as B
from paper_2503_10377_amd import sppo as L

ROOT = B.ROOT
WORK_ITEMS = 1 << 32  # HIP takes fewer than this many work items along a dimension
GRID_YZ = 65535


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    L.lib()
    exe = str(tmp_path_factory.mktemp("plan") / "launch_plan")
    cmd = [B.hipcc(), "-O1", "-std=c++17", "--offload-arch=gfx950", os.path.join(ROOT, "tests", "launch_plan.cpp"), "-I", B.INCLUDE,
           "-I", B.CSRC, "-rdynamic", "-o", exe, "-L", B.PKG, "-l:libsppo.so", f"-Wl,-rpath,{B.PKG}"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(cases):
        env = dict(os.environ, HIP_VISIBLE_DEVICES="-1")
        out = subprocess.run([exe], input="\n".join(cases) + "\n", capture_output=True, text=True, env=env)
        assert out.returncode == 0, out.stderr
        lines = out.stdout.splitlines()
        assert len(lines) == len(cases)
        return [x if x in ("none", "error") else [_launch(g) for g in x.split(" ; ")] for x in lines]

    return run


def _launch(group):
    name, *n = group.split()
    n = list(map(int, n))
    return {"kernel": name, "grid": tuple(n[:3]), "threads": n[3], "keys": tuple(n[4:])}


def legal(launches):
    return launches not in ("none", "error") and all(
        0 < x["grid"][0] * x["threads"] < WORK_ITEMS and 0 < x["grid"][1] <= GRID_YZ and 0 < x["grid"][2] <= GRID_YZ
        for x in launches)


def test_fp32_backward_grids_stay_launchable(plan):
    """Sizes whose tiles times threads pass 2^32: the pair of both gradient
    kernels is then not taken, and dK/dV goes out over ranges of keys on the
    tile grid that cover every key once."""
    # batch 65535 x 8 heads x 256 rows: 9.4M workgroups of 512 in one dimension
    big = "f32 65535 8 1 64 256 0 256"
    pair, dkdv, dq = plan(["pair " + big, "dkdv " + big, "dq " + big])
    assert pair == "none" and legal(dkdv) and legal(dq)
    # one below the line and one at it
    for n, taken in ((2**22 - 1, True), (2**22, False)):  # n tiles of each kind
        p, = plan([f"pair f32 1 1 1 64 {16 * n} 0 {16 * n}"])
        assert (p != "none") == taken and (not taken or legal(p))
    for D in (64, 128):
        for S, c0 in ((140_000_001, 140_000_000), (268_435_457, 268_435_000), (1000, 990)):
            d, = plan([f"dkdv f32 1 1 1 {D} {S} {c0} {S}"])
            assert legal(d)
            at = 0
            for x in d:
                assert x["keys"][0] == at and at % 16 == 0
                at = x["keys"][1]
                assert x["grid"][0] == (at - x["keys"][0] + 15) // 16
            assert at == S and (len(d) == 1) == ((S + 15) // 16 * x["threads"] < WORK_ITEMS)


@pytest.mark.parametrize("tn", [0, 1])
def test_gemm_tiles_fit_the_grid(plan, tn):
    """Tall products whose time estimate favours small tiles keep to a tile
    whose rows fit a grid dimension."""
    cases = [f"gemm {tn} 0 {M} {N} {K}" for M in (65532 * 64, 65536 * 64, 256 * 23438, 65538 * 128, 65535 * 256)
             for N in (256 if tn else 4, 256) for K in (64, 1664, 4096, 16384)]
    plans = plan(cases)
    for c, p in zip(cases, plans):
        assert legal(p) and len(p) == 1, c
    if not tn:  # the small tile is the choice up to the limit
        assert plan(["gemm 0 0 4194240 64 4096"])[0][0]["grid"][1] == 65535


def kernels(p):
    return [x["kernel"] for x in p]


@pytest.mark.parametrize("heads", ["4 4", "8 2", "16 4", "32 8", "32 32"])
def test_wide_backward_by_head_size(plan, heads):
    """Wide dK/dV and dQ launches of several passes take the 32x32x16 kernels at
    head size 128 and the 16x16x32 ones at 64."""
    for c0, c1 in ((0, 30000), (10000, 26000), (114688, 131072)):
        for D, kind in ((128, "mfma32"), (64, "bf16")):
            dkdv, dq = plan([f"{op} bf16 1 {heads} {D} {c1} {c0} {c1}" for op in ("dkdv", "dq")])
            assert legal(dkdv) and f"bwd_dkdv_{kind}_kernel" in kernels(dkdv)[0] and dkdv[0]["grid"][0] <= 256
            assert legal(dq) and f"bwd_dq_{kind}_kernel" in kernels(dq)[0]


# 256 compute units.  Rows [c0, c1) of heads Hq/Hkv: the kernels of dK/dV, dQ and the pair ("none": separate launches).
@pytest.mark.parametrize("B,Hq,Hkv,D,c0,c1,dkdv,dq,pair", [
    (1, 4, 4, 128, 1536, 2048, "dkdv_split_kernelILi128ELi1ELi4E", "dq_split", "pair_kernelILi128ELi1ELi4E"),
    (1, 8, 8, 128, 1024, 2048, "dkdv_split_kernelILi128ELi2ELi2E", "dq_split", "pair_kernelILi128ELi2ELi2E"),
    (1, 16, 4, 128, 3072, 4096, "dkdv_split_kernelILi128ELi2ELi2E", "dq_split", "none"),  # 4096 query rows to a key
    (1, 16, 4, 128, 3071, 4096, "dkdv_mfma32", "dq_mfma32", "none"),  # 4100
    (1, 8, 2, 128, 6144, 8192, "dkdv_mfma32", "dq_split", "none"),
    (1, 8, 2, 128, 3500, 4800, "dkdv_split_kernelILi128ELi2ELi2E", "dq_split", "pair_kernelILi128ELi2ELi2E"),  # 5200
    (1, 8, 2, 128, 0, 7680, "dkdv_mfma32", "dq_mfma32", "none"),
    (1, 1, 1, 128, 2000, 10192, "dkdv_split_kernelILi128ELi2ELi2E", "dq_split", "pair_kernelILi128ELi2ELi2E"),
    (1, 16, 16, 64, 3000, 4000, "dkdv_bf16_kernel", "dq_split", "none"),  # 256 workgroups of 64 rows
    (1, 16, 16, 64, 2560, 4096, "dkdv_bf16_kernel", "dq_split", "none"),  # 384, 2 x 4096 keys an XCD
    (1, 16, 16, 64, 2561, 4097, "dkdv_bf16_kernel", "dq_mfma32", "none"),
    (1, 8, 8, 64, 8192, 12288, "dkdv_bf16_kernel", "dq_split", "none"),
    (1, 8, 8, 64, 10000, 12289, "dkdv_bf16_kernel", "dq_mfma32", "none"),
    (1, 17, 17, 64, 1000, 2000, "dkdv_bf16_kernel", "dq_mfma32", "none"),  # 3 heads an XCD
    (2, 32, 8, 64, 1000, 1500, "dkdv_bf16_kernel", "dq_mfma32", "none"),
    (1, 32, 8, 64, 0, 1024, "dkdv_split_kernelILi64ELi2ELi4E", "dq_split", "pair_kernelILi64ELi2ELi4E"),
])
def test_backward_kernels_of_small_grids(plan, B, Hq, Hkv, D, c0, c1, dkdv, dq, pair):
    args = f"bf16 {B} {Hq} {Hkv} {D} {c1} {c0} {c1}"
    got = plan([f"{op} {args}" for op in ("dkdv", "dq", "pair")])
    for p, want in zip(got, (dkdv, dq, pair)):
        assert (p == "none") if want == "none" else (legal(p) and want in kernels(p)[0]), (p, want)
    mid = c1 // 2 + 13  # a part of the keys: the same kernel
    for lo, hi in ((0, mid), (mid, c1)):
        part, = plan([f"dkdv {args} {lo} {hi}"])
        assert kernels(part) == kernels(got[0])


@pytest.mark.parametrize("Hq,c0,c1,one", [(1, 0, 32768, True), (1, 7000, 24408, True), (1, 7000, 41000, True), (1, 46000, 80000, True),
                                          (4, 10000, 20000, True), (8, 0, 4097, True), (8, 0, 6000, True), (12, 2000, 4730, True),
                                          (12, 8000, 11000, False), (32, 4096, 8192, False), (8, 0, 8192, False)])
def test_wide_dq_of_head_size_64_by_load(plan, Hq, c0, c1, one):
    """The 32x32x16 kernel while most compute units hold one workgroup (no more
    workgroups of 128 rows than 256, or short tiles among them)."""
    p, = plan([f"dq bf16 1 {Hq} {Hq} 64 {c1} {c0} {c1}"])
    assert legal(p) and ("bwd_dq_mfma32_kernelILi64E" if one else "bwd_dq_bf16_kernel") in kernels(p)[0]


@pytest.mark.parametrize("Hq,D,c0,c1,want", [
    (2, 128, 0, 64, "fwd_mfma32"), (2, 64, 63, 64, "fwd_mfma32"), (2, 128, 0, 65, "fwd_split"),
    (4, 128, 0, 4096, "fwd_split"), (4, 128, 0, 4097, "fwd_mfma32"), (4, 128, 6000, 12000, "fwd_mfma32"),
    (16, 128, 6000, 8048, "fwd_mfma32"), (16, 128, 14000, 16049, "fwd_bf16"),  # 256 workgroups, 272 at a load of 0.99
    (8, 128, 0, 5376, "fwd_mfma32"), (8, 128, 3000, 8376, "fwd_mfma32"), (8, 128, 12000, 16352, "fwd_bf16"),
    (32, 128, 0, 2048, "fwd_bf16"), (8, 64, 0, 4096, "fwd_split"), (8, 64, 0, 6000, "fwd_mfma32"),
    (16, 64, 8192, 12288, "fwd_bf16"), (32, 64, 0, 131072, "fwd_bf16")])
def test_forward_by_load(plan, Hq, D, c0, c1, want):
    p, = plan([f"fwd bf16 1 {Hq} {Hq} {D} {c1} {c0} {c1}"])
    assert legal(p) and want in kernels(p)[0] and f"ILi{D}E" in kernels(p)[0]


@pytest.mark.parametrize("epi,short", [(0, True), (5, True), (4, False), (1, False)])
def test_gemm_tn_of_few_k_blocks(plan, epi, short):
    """Weight gradients that are written, over up to 16 k-blocks on 256 tiles;
    those that are added, longer or smaller ones and NT keep their kernels."""
    cases = [(1, 6144, 9984, 106), (1, 6144, 9984, 1024), (1, 6144, 9984, 1025), (1, 256, 256, 64), (0, 6144, 9984, 128)]
    got = plan([f"gemm {tn} {epi} {M} {N} {K}" for tn, M, N, K in cases])
    for (tn, M, N, K), p in zip(cases, got):
        want = short and tn and M > 256 and K <= 1024
        assert legal(p) and ("gemm_tn_short" in kernels(p)[0]) == bool(want), (M, N, K, p)
        if want:
            assert p[0]["grid"] == (N // 256, M // 256, 1)
