"""The wave-resident flip-ratio passes (BF16 and FP8 up to bond 64): at bond 64
equal bit for bit to the form with rows in LDS, which fewer walkers take; at
bond 32, where no other form is left, against the FP64 oracle.  Sizes at the
edges of row tiles, spins split into row groups, ragged last blocks."""
import numpy as np
import pytest
import torch

from helpers import case
from paper_2604_22718_amd import workloads as wl
from test_gpu_parity import assert_parity, run_eval

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_22718_amd import rtt
    return rtt


@pytest.mark.parametrize("N,Rr,dtype,T", [(1, 1, "bf16", 1), (15, 2, "bf16", 1), (16, 2, "fp8", 2), (31, 1, "bf16", 2),
                                          (48, 2, "bf16", 1), (64, 2, "fp8", 1), (66, 2, "bf16", 1), (90, 2, "bf16", 1)])
def test_wave_form_equals_rows_in_lds(R, N, Rr, dtype, T):
    print(f"[case] {dtype} bond 64 N={N} R={Rr} T={T}", flush=True)
    pi, bond = wl.path_site_plus_perms(N, Rr, 31 + N), wl.open_bonds(N * Rr, 64)
    terms = [R.RTT.create(N, pi, wl.gaussian_cores(bond, 40 + N + t), dtype) for t in range(T)]
    psi = terms[0] if T == 1 else R.RTT.lincomb(terms, np.array([1.0, -0.6])[:T])
    ham = R.TFIM(N, 1, 1.0, 2.0)
    W = 4 * torch.cuda.get_device_properties(0).multi_processor_count + 3
    bits = wl.random_spins(W, N, 41)
    many = psi.evaluate(R.spins_to_device(wl.pack_spins(bits)), ham)
    few = psi.evaluate(R.spins_to_device(wl.pack_spins(bits[-39:])), ham)
    torch.cuda.synchronize()
    for k in few:
        assert torch.equal(many[k][-39:], few[k]), k


@pytest.mark.parametrize("N,Rr,dtype,W", [(1, 1, "bf16", 2), (15, 2, "bf16", 5), (16, 2, "fp8", 3), (33, 2, "bf16", 9),
                                          (64, 2, "bf16", 5), (64, 2, "fp8", 1), (70, 2, "bf16", 6)])
def test_bond_32_matches_oracle(R, N, Rr, dtype, W):
    print(f"[case] {dtype} bond 32 N={N} R={Rr} W={W}", flush=True)
    pi, bond, cores = case(N, Rr, 32, "perm", seed=60 + N)
    bits = wl.random_spins(W, N, 61)
    _, qc, out = run_eval(R, pi, bond, cores, N, bits, dtype)
    assert_parity(out, qc, pi, bits, dtype, "uniform", min_well=0)
