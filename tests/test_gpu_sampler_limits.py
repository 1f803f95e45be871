"""Where the sampler's blocks change from 16 to 32 walkers: the first count past
16 for every compute unit, and for FP8 cores at bond 256, whose blocks of 32
keep their prefixes in global memory, a train whose state fits 16 walkers per
block but not 32, and a first sweep inside a stream capture, which may not
allocate for them."""
import numpy as np
import pytest
import torch

from paper_2604_22718_amd import workloads as wl
from test_gpu_sampler_layouts import chain, make

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_22718_amd import rtt
    return rtt


def many_walkers():
    return 32 * torch.cuda.get_device_properties(0).multi_processor_count + 21


def test_train_past_a_block_of_32(R):
    N, L = 1024, 5890   # 93 words of positions and 16 of spins: one more than 32 walkers leave room for
    print(f"[case] fp8 bond 256 N={N} L={L}", flush=True)
    pi = np.arange(L, dtype=np.int32) % 6   # the other spins are read by no position
    bond = np.full(L + 1, 2, dtype=np.int32)
    bond[[0, L]], bond[L // 3] = 1, 160
    psi = R.RTT.create(N, pi, wl.gaussian_cores(bond, 700, std=0.7), "fp8")
    bits = wl.random_spins(many_walkers(), N, 701)
    few = bits[:53]
    la, sg = psi.amplitudes(R.spins_to_device(wl.pack_spins(bits)))
    lf, sf = psi.amplitudes(R.spins_to_device(wl.pack_spins(few)))
    assert torch.equal(la[:53], lf) and torch.equal(sg[:53], sf) and bool(torch.isfinite(la).all())
    for a, b in zip(chain(R, psi, bits, 1, 1), chain(R, psi, few, 1, 1)):
        assert torch.equal(a[:53], b)


def test_first_sweep_inside_a_capture(R):
    print("[case] fp8 bond 256, first sweep captured", flush=True)
    N, T = 5, 1
    psi, ref = (make(R, N, 2, 256, "fp8", T, 800) for _ in range(2))
    words = wl.pack_spins(wl.random_spins(many_walkers(), N, 801))
    spins, want = R.spins_to_device(words), R.spins_to_device(words)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        psi.sweep(spins, seed=5, n_sweeps=1)
    for _ in range(3):
        graph.replay()
        ref.sweep(want, seed=5, n_sweeps=1)
        torch.cuda.synchronize()
        assert torch.equal(spins, want)
    # outside the capture the same handle allocates and goes on
    psi.sweep(spins, seed=6, n_sweeps=2)
    ref.sweep(want, seed=6, n_sweeps=2)
    graph.replay()
    ref.sweep(want, seed=5, n_sweeps=1)
    torch.cuda.synchronize()
    assert torch.equal(spins, want)


@pytest.mark.parametrize("chi,dtype,T", [(128, "f32", 1), (128, "bf16", 2), (128, "fp8", 1), (256, "fp8", 1), (256, "fp8", 2)])
@pytest.mark.parametrize("past", [0, 1])
def test_walkers_at_the_change_of_shape(R, chi, dtype, T, past):
    W = 16 * torch.cuda.get_device_properties(0).multi_processor_count + past
    print(f"[case] {dtype} bond {chi} T={T} W={W}", flush=True)
    psi = make(R, 6, 2, chi, dtype, T, 820 + T)
    bits = wl.random_spins(W, 6, 821)
    for a, b in zip(chain(R, psi, bits, 2, 1), chain(R, psi, bits[:33], 2, 1)):   # (a walker's draws go by its index)
        assert torch.equal(a[:33], b)
    la, sg = psi.amplitudes(R.spins_to_device(wl.pack_spins(bits)))
    lf, sf = psi.amplitudes(R.spins_to_device(wl.pack_spins(bits[-33:])))
    assert torch.equal(la[-33:], lf) and torch.equal(sg[-33:], sf)
