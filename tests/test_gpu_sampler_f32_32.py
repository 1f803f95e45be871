"""FP32 sampler at bond 32: a single term runs two waves per side, two terms of
a combination side by side run one, and a batch two.  Their dot products are
added in one order, so amplitudes and decisions agree bit for bit."""
import os

import numpy as np
import pytest
import torch

import test_gpu_sampler_layouts as layouts
from paper_2604_22718_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_22718_amd import rtt
    return rtt


@pytest.mark.parametrize("N,Rr,W", [(1, 1, 3), (2, 1, 16), (9, 2, 37), (17, 3, 65)])
def test_two_terms_one_of_weight_zero_equal_one(R, N, Rr, W):
    print(f"[case] f32 bond 32 N={N} R={Rr} W={W}", flush=True)
    # (column checkpoints off: their number, and with it the bonds where rows
    # and columns meet, depends on the number of terms)
    os.environ["RTT_CHAIN_CHECKPOINTS"] = "0"
    try:
        one, other = layouts.make(R, N, Rr, 32, "f32", 1, 900 + N), layouts.make(R, N, Rr, 32, "f32", 1, 900 + N)
        two = R.RTT.lincomb([one, other], np.array([1.0, 0.0]))
    finally:
        del os.environ["RTT_CHAIN_CHECKPOINTS"]
    bits = wl.random_spins(W, N, 901)
    for a, b in zip(layouts.chain(R, one, bits, 2, 2), layouts.chain(R, two, bits, 2, 2)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("T,N,tile", [(1, 7, "16"), (1, 7, "32"), (2, 1, "16"), (2, 9, "32"), (3, 6, "16")])
def test_batch_equals_single_state(R, T, N, tile):
    os.environ["RTT_BATCH_TILE"] = tile
    try:
        layouts.test_terms_side_by_side_equal_one_by_one(R, 32, "f32", T, N)
    finally:
        del os.environ["RTT_BATCH_TILE"]
