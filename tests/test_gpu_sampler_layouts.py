"""The sampler's block shapes agree bit for bit where they overlap: 32 walkers
per block against 16 (each group of 16 keeps its own starting bonds, so the
shape may not change a decision or a last bit), and two terms of a combination
side by side against one after the other (the persistent batch form)."""
import os

import numpy as np
import pytest
import torch

from helpers import case
from paper_2604_22718_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_22718_amd import rtt
    return rtt


def make(R, N, Rr, chi, dtype, T, seed):
    pi = wl.path_site_plus_perms(N, Rr, seed)
    bond = wl.open_bonds(N * Rr, chi)
    terms = [R.RTT.create(N, pi, wl.gaussian_cores(bond, seed + 1 + t), dtype) for t in range(T)]
    return terms[0] if T == 1 else R.RTT.lincomb(terms, np.array([1.0, -0.6, 0.8, 0.3])[:T])


def chain(R, psi, bits, calls, sweeps):
    W = bits.shape[0]
    spins = R.spins_to_device(wl.pack_spins(bits))
    la = torch.empty(W, dtype=torch.float64, device="cuda")
    sg = torch.empty(W, dtype=torch.int8, device="cuda")
    acc = torch.zeros(W, dtype=torch.int32, device="cuda")
    for c in range(calls):
        psi.sweep(spins, seed=91, rng_stream=4, sweep0=c * sweeps, n_sweeps=sweeps, logabs=la, sign=sg, accepts=acc)
    torch.cuda.synchronize()
    return spins, la, sg, acc


@pytest.mark.parametrize("N,Rr,chi,dtype,T", [(7, 2, 256, "fp8", 2), (6, 3, 256, "fp8", 4), (5, 2, 256, "fp8", 1),
                                              (9, 2, 128, "bf16", 1), (8, 2, 128, "fp8", 2), (1, 1, 128, "bf16", 1)])
def test_two_groups_per_block_equal_one(R, N, Rr, chi, dtype, T):
    print(f"[case] {dtype} bond {chi} N={N} T={T}", flush=True)
    psi = make(R, N, Rr, chi, dtype, T, 500 + N + chi)
    W = 32 * torch.cuda.get_device_properties(0).multi_processor_count + 21  # two groups, a ragged last block
    bits = wl.random_spins(W, N, 501)
    many = chain(R, psi, bits, 2, 2)
    few = chain(R, psi, bits[:85], 2, 2)
    for a, b in zip(many, few):
        assert torch.equal(a[:85], b)
    assert int(many[3].sum()) > 0


@pytest.mark.parametrize("chi,dtype,T,N", [(32, "bf16", 2, 6), (64, "bf16", 3, 9), (64, "f32", 3, 8), (16, "f32", 3, 1),
                                           (64, "fp8", 8, 5), (128, "f32", 2, 6), (128, "bf16", 3, 5)])
def test_terms_side_by_side_equal_one_by_one(R, chi, dtype, T, N):
    print(f"[case] {dtype} bond {chi} T={T} N={N}", flush=True)
    os.environ["RTT_CHAIN_CHECKPOINTS"] = "0"   # as the persistent form
    try:
        psi = (lambda t: t[0] if T == 1 else R.RTT.lincomb(t, np.linspace(1.0, -0.7, T)))(
            [R.RTT.create(N, wl.path_site_plus_perms(N, 2, 7), wl.gaussian_cores(wl.open_bonds(2 * N, chi), 8 + t), dtype)
             for t in range(T)])
    finally:
        del os.environ["RTT_CHAIN_CHECKPOINTS"]
    bits = wl.random_spins(37, N, 9)
    spins = R.spins_to_device(wl.pack_spins(bits))
    ref = spins.clone()
    ham = R.TFIM(N, 1, 1.0, 2.0)
    batch = R.Batch([psi], [ham], [spins], seed=17)
    for rep in range(2):
        batch.step(n_sweeps=2)
        psi.sweep(ref, seed=17, rng_stream=0, sweep0=2 * rep, n_sweeps=2)
        torch.cuda.synchronize()
        assert torch.equal(batch.spins[0], ref)
    batch.close()
