"""Group normalisation of runs that do not start on 16 bytes, and of runs too
long for registers: group lengths from one value up, channels shorter than a
chunk, one, two and four workgroups a group, in place, against the fp64 oracle
with the bound of test_norm_act_gpu."""
import numpy as np
import pytest

import paper_2304_11267_amd as sd
from paper_2304_11267_amd import workloads as wl

from test_norm_act_gpu import check_gn

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _needs_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sd.load_library()


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("shape", [
    (1, 5, 3, 5),            # value by value: groups of three values
    (3, 21, 7, 7),           # channels shorter than a chunk, three to a group
    (4, 160, 63, 32),
    (9, 64, 65, 32),
    (2, 1332, 3, 2),         # 1998 values: the last so
    (2, 1336, 3, 2),         # 2004: in chunks, channels shorter than one
    (3, 640, 7, 2),
    (2, 320, 33 * 62, 32),   # four workgroups a group
    (4, 640, 125, 32),       # two
    (9, 640, 249, 32),       # 288 groups of 4980: value by value
    (9, 640, 251, 32),       # of 5020: in chunks, one workgroup a group
    (17, 640, 323, 32),      # 544 groups of 6460 and 6500
    (17, 640, 325, 32),
    (1, 96, 16381, 32),      # 49143 values: past the registers only by alignment
    (1, 96, 16384, 32),      # 49152: the last that fits
    (2, 96, 18001, 32),      # 54003: three reads, misaligned
    (2, 96, 18432, 32),      # 55296: three reads
], ids=lambda s: "x".join(map(str, s)))
def test_runs(shape, in_place):
    B, C, HW, G = shape
    x, gamma, beta = wl.make_norm(B, C, HW, 8300 + B + C + HW)
    check_gn(x, gamma, beta, G, 1e-5, in_place=in_place)


def test_runs_bf16():
    x, gamma, beta = wl.make_norm(2, 320, 33 * 62, 8400, dtype="bf16")
    check_gn(x, gamma, beta, 32, 1e-5, dtype="bf16")
