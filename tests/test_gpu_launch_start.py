"""The start of a matrix-core launch: dictionary operands and first loads with the whole dictionary (no look at the list),
with fewer atoms than the instantiation holds, and with a kept list and scales; the tile walk over one tile per image,
one tile per row, grids that are and are not a multiple of the eight shares, and images many to a call.  Against the
oracle with the bounds of test_gpu_parity.py."""
import numpy as np
import pytest
import torch

import paper_2303_08999_amd as sr
import sr_synth
from test_gpu_parity import MFMA, check_full

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    sr.load()


@pytest.mark.parametrize("n, c, h, w, scale, L, k, coeff, kept", [
    (1, 1, 2, 32, 2, 72, 5, "f32", None),       # one tile
    (11, 1, 2, 32, 2, 72, 5, "f32", None),      # one tile per image, eleven images: one share
    (16, 3, 3, 40, 2, 70, 5, "f16", None),      # two tiles per image, 32 workgroups: eight shares; two atoms of padding
    (3, 3, 37, 24, 4, 72, 5, "f16", None),      # one tile per row
    (2, 3, 30, 64, 3, 128, 7, "f16", None),     # two matrix blocks per slot
    (1, 3, 20, 64, 4, 72, 7, "f8", None),
    (5, 1, 9, 48, 3, 72, 5, "bf16", None),
    (2, 3, 21, 64, 3, 72, 5, "f16", 65),        # a kept list that fills all but one group
    (2, 3, 21, 64, 3, 72, 5, "f32", 9),
    (2, 3, 21, 64, 2, 40, 3, "f8", 8),
])
def test_launch_start(oracle, n, c, h, w, scale, L, k, coeff, kept):
    wl = sr_synth.Workload("start", 40, n, c, h, w, scale, L, k, coeff, "f32")
    rng = np.random.default_rng(L + k)
    lst = None if kept is None else rng.permutation(L)[:kept].astype(np.int32)      # any order
    gamma = None if kept is None else rng.uniform(0.5, 1.5, size=kept).astype(np.float32)
    check_full(oracle, wl, MFMA, kept=lst, gamma=gamma)
