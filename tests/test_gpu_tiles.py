"""GPU parity at the edges of the kernels' tiles and dispatch rules: sizes one
below, at and one above a tile, remainders in every dimension, and the
smallest sizes, against the fp64 oracle with the gates of parity.py."""
import sys

import numpy as np
import pytest
import torch

from paper_2503_10377_amd.chunked import ChunkedAttention
from paper_2503_10377_amd.inputs import make_inputs
from parity import check_all, to_np
from test_gpu_parity import run_case

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
