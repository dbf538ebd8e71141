"""The tiled attention kernel's streaming loop and its geometries, and the path
with a maximum that moves from the start, at the key counts where they change:
one to five whole 64-key tiles a key split with and without a ragged one (a
split without whole tiles, or without any), widths with and without the sparse
tile and the row of ones, with statistics, large logits (the fallback, and rows
whose maximum grows along the keys), zero and negative scale.  Against the fp64
oracle with the parity suite's bound."""
import numpy as np
import pytest

import oracle
import paper_2304_11267_amd as sd
from paper_2304_11267_amd import workloads as wl

from parity_util import assert_close, to_device, to_host64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _needs_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sd.load_library()


def check(B, H, Lq, Lk, D, seed, dtype="f16", scale=None, q_mult=1.0, grow=False):
    import torch
    q, k, v = wl.make_qkv(B, H, Lq, Lk, D, seed, dtype, q_mult)
    if grow:   # every key's logits outgrow the earlier ones'
        k = (k.astype(np.float32) * np.linspace(0.2, 4.0, Lk, dtype=np.float32)[:, None]).astype(np.float16)
    scale = float(np.float32(1 / np.sqrt(D))) if scale is None else scale
    rows = None if Lq * Lk * B * H <= 1 << 23 else wl.sample_rows(B, H, Lq, 40, seed)
    r, rl, rs, dev = oracle.attention(q, k, v, scale, dtype="bf16" if dtype == "bf16" else None, rows=rows,
                                     want_dev=True)
    qd, kd, vd = (to_device(t, dtype) for t in (q, k, v))
    for stats in (False, True):
        out = torch.full_like(qd, 7.0)
        ls = torch.full((B, H, Lq, 2), 7.0, dtype=torch.float32, device="cuda") if stats else None
        sd.forward_ex(qd, kd, vd, out, scale, ls=ls)
        torch.cuda.synchronize()
        g = to_host64(out)
        g = g if rows is None else g.reshape(-1, D)[rows]
        assert_close(g.reshape(r.shape), r, dtype=dtype, dev=dev,
                     what=f"{B}x{H}x{Lq}x{Lk}x{D} {dtype} stats={stats}")
        if stats:
            got = ls.cpu().numpy().astype(np.float64).reshape(-1, 2)
            got = got if rows is None else got[rows]
            # L: an fp32 sum of D products (each at most |q| |k| by Cauchy-Schwarz);
            # S: the weights' rounding, and L's error in the exponent
            norm = [np.linalg.norm(to_host64(t), axis=-1).max() for t in (qd, kd)]
            tol = D * 2.0 ** -23 * abs(scale) * norm[0] * norm[1]
            assert np.all(np.abs(got[:, 0] - rl.reshape(-1)) <= tol)
            eps = {"f16": 2.0 ** -10, "bf16": 2.0 ** -7}[dtype]
            assert np.all(np.abs(got[:, 1] / rs.reshape(-1) - 1) <= eps + tol)


# 2 key splits of 64-key tiles in the 128-row geometry (a ring of three buffers)
@pytest.mark.parametrize("Lk", [129, 192, 255, 256, 257, 449, 640, 705, 1031])
@pytest.mark.parametrize("D", [40, 56, 64])
def test_stream_128_rows(D, Lk):
    check(2, 8, 2048, Lk, D, 900 + D + Lk)


# and in 256 rows (D = 64 at any key count, the others from 1024 on): five buffers
# (D = 40), three (D = 64), or two and no stream (D = 48)
@pytest.mark.parametrize("Lk", [130, 321, 640, 1000, 1024, 1030, 1100, 1313])
@pytest.mark.parametrize("D", [40, 48, 64])
def test_stream_256_rows(D, Lk):
    check(2, 8, 4096, Lk, D, 1900 + D + Lk)


@pytest.mark.parametrize("Lk", [130, 200, 448])
def test_stream_64_rows(Lk):
    check(1, 3, 70, Lk, 40, 2900 + Lk)


# between one round of 64-row workgroups and the 128-row grid
def test_stream_partial_grid():
    check(1, 8, 2300, 600, 40, 3900)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("D", [40, 80, 160])
def test_large_logits(D, dtype):
    check(1, 4, 200, 333, D, 4900 + D, dtype, q_mult=4.0)
    check(2, 8, 2048, 320, D, 4950 + D, dtype, q_mult=4.0)


@pytest.mark.parametrize("D,Lk", [(40, 700), (80, 500), (80, 1000), (160, 500), (160, 1000)])
def test_growing_keys(D, Lk):
    check(1, 4, 150, Lk, D, 5900 + D + Lk, grow=True)
    check(2, 8, 2048, Lk, D, 5950 + D + Lk, grow=True)


@pytest.mark.parametrize("scale", [0.0, -0.2, 1e-20, 1e-36])
@pytest.mark.parametrize("D", [40, 80])
def test_scales(D, scale):
    check(1, 4, 150, 400, D, 6900 + D, scale=float(np.float32(scale)))
    check(2, 8, 2048, 300, D, 6950 + D, scale=float(np.float32(scale)))


# four key splits of 64 rows, the last one without keys (9 tiles: 3 + 3 + 3 + 0) or
# with a ragged tile only; scale 0 gives an empty split no weight of its own
@pytest.mark.parametrize("scale", [None, 0.0, 1e-36])
@pytest.mark.parametrize("Lk", [576, 577, 650])
@pytest.mark.parametrize("D", [32, 40, 64, 80])
def test_four_splits_with_an_empty_one(D, Lk, scale):
    check(1, 4, 150, Lk, D, 7900 + D + Lk, scale=None if scale is None else float(np.float32(scale)))


# past one round of 128-row workgroups: two of them on a CU at D = 56 and 64 (two
# buffers, no stream), with short, empty and ragged splits, and their fallback
@pytest.mark.parametrize("Lk", [129, 192, 200, 320, 641])
@pytest.mark.parametrize("D", [56, 64])
def test_two_workgroups_a_cu(D, Lk):
    check(1, 300, 128, Lk, D, 8900 + D + Lk)
    if Lk in (200, 320):
        check(3, 100, 70, Lk, D, 8950 + D + Lk, "bf16")
        check(1, 260, 128, Lk, D, 8970 + D + Lk, q_mult=4.0)
        check(1, 260, 128, Lk, D, 8990 + D + Lk, scale=0.0)


# NaN and infinite inputs: wherever the definition gives NaN or Inf so does every
# path (streaming in each geometry, four splits, two buffers, a maximum that
# moves), and other heads keep their bits.  The kernels' maxima are compiled for
# finite scores: this is what shows that nothing else takes a NaN for a number.
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("shape", [(1, 4, 150, 300, 40), (1, 4, 150, 600, 40), (1, 4, 150, 600, 64),
                                   (2, 8, 2048, 330, 40), (2, 8, 4096, 1030, 40), (1, 16, 2048, 300, 64),
                                   (1, 300, 128, 200, 64), (1, 4, 150, 320, 80), (1, 4, 150, 1000, 160),
                                   (2, 8, 2048, 300, 160)],
                         ids=lambda s: "x".join(map(str, s)))
def test_nan_and_infinity_stay(shape, dtype):
    import torch
    B, H, Lq, Lk, D = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(Lk + D)
    dt = torch.float16 if dtype == "f16" else torch.bfloat16
    clean = [torch.randn(B, H, n, D, device="cuda", generator=g).to(dt) for n in (Lq, Lk, Lk)]
    scale = float(np.float32(1 / np.sqrt(D)))

    def run(q, k, v, stats):
        out = torch.full_like(q, 7.0)
        ls = torch.full((B, H, Lq, 2), 7.0, dtype=torch.float32, device="cuda") if stats else None
        sd.forward_ex(q, k, v, out, scale, ls=ls)
        torch.cuda.synchronize()
        return out, ls

    nan, inf = float("nan"), float("inf")
    # which of q, k, v; row; column; value
    for where, row, col, bad in ((0, Lq - 1, 3, nan), (0, 5, D - 1, inf), (1, 0, 0, nan), (1, Lk - 1, D - 1, nan),
                                 (1, Lk // 2, 1, -inf), (2, Lk - 1, 0, nan), (2, 1, D - 1, inf)):
        ins = [t.clone() for t in clean]
        ins[where][0, 1, row, col] = bad
        q, k, v = (t[0, 1].double() for t in ins)
        a = (q @ k.t().contiguous()) * scale
        p = torch.softmax(a, dim=1)
        ref = p @ v
        for stats in (False, True):
            out, ls = run(*ins, stats)
            got = out[0, 1].double()
            assert not torch.isfinite(got[~torch.isfinite(ref)]).any(), (where, row, bad, stats)
            if stats:
                lost = ~torch.isfinite(p).all(dim=1)
                assert not torch.isfinite(ls[0, 1][lost][:, 1]).any(), (where, row, bad)
            same, same_ls = run(*clean, stats)
            keep = torch.ones(B, H, dtype=torch.bool, device="cuda")
            keep[0, 1] = False
            assert torch.equal(out[keep], same[keep])
            if stats:
                assert torch.equal(ls[keep], same_ls[keep])
