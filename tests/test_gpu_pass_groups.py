"""Wave-resident flip-ratio passes (BF16 and FP8 up to bond 64) where the spins
are split into two row groups of at most 80 rows, so that most steps of a group
have no odd row: at bond 64 equal bit for bit to the form with rows in LDS,
which fewer walkers take; at bond 32 against the FP64 oracle.  And batch classes
whose members take different forms, against each state evaluated by itself."""
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


def make(R, N, Rr, chi, dtype, T, seed):
    pi, bond = wl.path_site_plus_perms(N, Rr, seed), wl.open_bonds(N * Rr, chi)
    terms = [R.RTT.create(N, pi, wl.gaussian_cores(bond, seed + 1 + t), dtype) for t in range(T)]
    return terms[0] if T == 1 else R.RTT.lincomb(terms, np.array([1.0, -0.6])[:T])


@pytest.mark.parametrize("N,Rr,dtype,T,groups,nslot", [(144, 2, "bf16", 1, 2, 80), (158, 2, "fp8", 1, 2, 80),
                                                       (150, 3, "bf16", 2, 2, 80), (158, 1, "bf16", 1, 1, 80)])
def test_wave_form_equals_rows_in_lds(R, N, Rr, dtype, T, groups, nslot):
    print(f"[case] {dtype} bond 64 N={N} R={Rr} T={T}", flush=True)
    psi = make(R, N, Rr, 64, dtype, T, 31 + N)
    assert (psi.info["groups"], psi.info["nslot"]) == (groups, nslot)
    simds = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    W, few = simds + 3, 39
    assert few * T * groups < simds   # a pass per SIMD is where the wave form begins
    ham = R.TFIM(N, 1, 1.0, 2.0)
    bits = wl.random_spins(W, N, 41)
    many = psi.evaluate(R.spins_to_device(wl.pack_spins(bits)), ham)
    some = psi.evaluate(R.spins_to_device(wl.pack_spins(bits[-few:])), ham)
    torch.cuda.synchronize()
    for k in some:
        assert torch.equal(many[k][-few:], some[k]), k


@pytest.mark.parametrize("N,dtype", [(130, "bf16"), (158, "fp8")])
def test_bond_32_two_groups_match_oracle(R, N, dtype):
    print(f"[case] {dtype} bond 32 N={N}", flush=True)
    pi, bond, cores = case(N, 2, 32, "perm", seed=60 + N)
    bits = wl.random_spins(3, N, 61)
    psi, qc, out = run_eval(R, pi, bond, cores, N, bits, dtype)
    assert (psi.info["groups"], psi.info["nslot"]) == (2, 80)
    assert_parity(out, qc, pi, bits, dtype, "uniform", min_well=0)


@pytest.mark.parametrize("chi,dtype,T", [(64, "bf16", 1), (64, "fp8", 2), (32, "bf16", 2)])
def test_batch_class_of_both_forms(R, chi, dtype, T):
    print(f"[case] batch {dtype} bond {chi} T={T}", flush=True)
    sizes = [(36, 2, 410), (100, 2, 150), (16, 2, 37), (144, 2, 60)]   # rows: 48, 112 (in LDS), 32, two groups of 80
    rtts = [make(R, N, Rr, chi, dtype, T, 70 + N) for N, Rr, _ in sizes]
    slots = [p.info["nslot"] for p in rtts]
    assert max(slots) > 80 and sum(s <= 80 for s in slots) == 3, slots
    hams = [R.TFIM(N, 1, 1.0, 2.0) for N, _, _ in sizes]
    spins = [R.spins_to_device(wl.pack_spins(wl.random_spins(W, N, 80 + N))) for N, _, W in sizes]
    batch = R.Batch(rtts, hams, spins, seed=9)
    for rep in range(3):
        batch.step(n_sweeps=1)
        for i, (psi, ham) in enumerate(zip(rtts, hams)):
            want = psi.evaluate(batch.spins[i], ham, ratios=False)["eloc"]
            torch.cuda.synchronize()
            assert torch.equal(batch.eloc[i], want), (rep, i)
    batch.close()
