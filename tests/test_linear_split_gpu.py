"""The projections' split-K kernel (few tiles or few token rows): edges of its
32/64-row and 32/64-channel tiles, channel counts that leave waves with short
or empty runs, and equal bits with the shared-tile kernel that longer inputs
take, against the fp64 oracle with the bound of an fp32 sum of K products."""
import numpy as np
import pytest

import oracle
import paper_2304_11267_amd as sd

from parity_util import to_device, to_host64, ulp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _needs_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sd.load_library()


SHAPES = [
    # (L, K, N): too few channels for the rule; 32x32 tiles; 32x64; 64x64; past the rule
    (1, 8, 8), (31, 56, 24),
    (33, 520, 40), (32, 584, 32), (65, 648, 72), (100, 1096, 136), (32, 1280, 1288),
    (257, 528, 640), (512, 1280, 1280), (1000, 776, 520),
    (64, 520, 32768), (50, 584, 32712),
    (1664, 648, 640),
]


@pytest.mark.parametrize("heads", [False, True], ids=["rows", "heads"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_split_product_matches_oracle(shape, heads):
    import torch
    L, K, N = shape
    rng = np.random.default_rng(7200 + L + K + N)
    x = rng.standard_normal((1, L, K), dtype=np.float32).astype(np.float16)
    w = (rng.standard_normal((N, K), dtype=np.float32) / np.float32(np.sqrt(K))).astype(np.float16)
    b = rng.standard_normal(N, dtype=np.float32).astype(np.float16)
    H = N // 8
    y = torch.full((1, H, L, 8) if heads else (1, L, N), 7.0, dtype=torch.float16, device="cuda")
    sd.linear(to_device(x), to_device(w), y, bias=to_device(b), heads=H,
              y_layout=sd.LAYOUT_HEADS if heads else sd.LAYOUT_ROWS)
    torch.cuda.synchronize()
    g = to_host64(y)
    g = g.transpose(0, 2, 1, 3).reshape(1, L, N) if heads else g
    r = oracle.linear(x, w, b)
    bound = (K + 2) * 2.0 ** -22 * (np.abs(x.astype(np.float64)) @ np.abs(w.astype(np.float64)).T) + ulp(r)
    assert np.all(np.abs(g - r) <= bound), float(np.max(np.abs(g - r) / bound))


# 520: runs of 3, 3, 3 and no slices; 584: 3, 3, 3 and 1 of 8 channels; up to 512
# channels no call splits
@pytest.mark.parametrize("K", [40, 320, 520, 584, 768, 1280])
def test_split_product_has_the_shared_tiles_bits(K):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(K)
    x = torch.randn(1, 8192, K, device="cuda", generator=g).half()
    w = (torch.randn(320, K, device="cuda", generator=g) / K ** 0.5).half()
    tall = torch.empty(1, 8192, 320, dtype=torch.float16, device="cuda")
    sd.linear(x, w, tall)                       # 320 shared tiles
    for rows in (1, 154, 1024):                 # 32x32 and (1024 rows) 32x64 split tiles
        part = torch.empty(1, rows, 320, dtype=torch.float16, device="cuda")
        sd.linear(x[:, :rows].contiguous(), w, part)
        assert torch.equal(part, tall[:, :rows]), rows
