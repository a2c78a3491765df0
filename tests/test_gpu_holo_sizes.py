"""Sizes at which the complex model's kernels change shape: 16, 32 and 64 lanes per
local energy over pairs of samples (odd batches), one wave per ln psi, and one, two
and three hidden units per lane with several segments in one sampler launch.

Bars as for the other tests of this model: decisions exact, local energies within
1e-10 and ln psi within 1e-12 (FP64 sums of at most 65 + 130 and products of at most
130 terms: some 500 roundings of 1.1e-16 would give 5.5e-14).
"""
import numpy as np
import pytest

import synth
from oracle import core, holo

pytestmark = pytest.mark.gpu

BASE = synth.WORKLOADS["tfim1d_n10"].replace(precision="c128")


def make(L, alpha, chains, S, sweep):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible HIP device")
    from paper_2112_10526_amd.nqs import VMCState
    w = BASE.replace(L=L, alpha=alpha, sigma=0.05, samples_per_chain=S, sweep_size=sweep)
    print(f"[case] L={L} alpha={alpha} chains={chains} S={S} sweep={sweep}", flush=True)
    return VMCState.from_workload(w, n_chains=chains), w, torch


@pytest.mark.parametrize("L", [3, 15, 16, 17, 31, 32, 33, 63, 64, 65])
@pytest.mark.parametrize("alpha,n", [(1, 1), (2, 33)])
def test_log_psi_and_local_energy(L, alpha, n):
    st, w, torch = make(L, alpha, 8, 4, L)
    s = synth.random_configs(n, L, 5 + L)
    rbm = holo.RbmC(w.n_sites, w.n_hidden, w.params())
    ham = core.Hamiltonian.tfim(w.n_sites, w.bonds(), w.J, w.h)
    sd = torch.from_numpy(s).cuda()
    lp, ref = st.log_psi(sd).cpu().numpy(), np.asarray(holo.log_psi(rbm, s))
    scale = np.maximum(np.abs(ref), 1.0)
    assert (np.abs(lp.real - ref.real) / scale).max() <= 1e-12
    assert (np.abs(np.angle(np.exp(1j * (lp.imag - ref.imag)))) / scale).max() <= 1e-12
    e, eref = st.local_energy(sd).cpu().numpy(), np.asarray(holo.local_energy(rbm, ham, s))
    assert (np.abs(e - eref) / np.maximum(np.abs(eref), 1.0)).max() <= 1e-10
    st.close()


@pytest.mark.parametrize("L,alpha,chains,S,sweep,discard", [
    (3, 1, 1, 1, 1, 0),       # one proposal, one wave of a block
    (10, 1, 5, 3, 65, 2),     # a segment longer than one draw of 64
    (65, 2, 6, 2, 64, 1),     # M = 130: a third, nearly empty slot of the four
])
def test_segments_of_one_launch(L, alpha, chains, S, sweep, discard):
    st, w, _ = make(L, alpha, chains, S, sweep)
    ch = st.get_chains()
    smp, acc, rate = st.sample(n_discard=discard, log_accepts=True)
    rbm = holo.RbmC(w.n_sites, w.n_hidden, w.params())
    margin = 1.0
    if discard:
        d = holo.sample(rbm, ch, discard, sweep, w.chain_seed, 0, mode="cached")
        ch, margin = d.chains, d.margins.min()
    ref = holo.sample(rbm, ch, S, sweep, w.chain_seed, discard * sweep, mode="cached",
                      log_accepts=True)
    assert min(margin, ref.margins.min()) > 1e-12
    np.testing.assert_array_equal(acc.cpu().numpy(), ref.accepts)
    np.testing.assert_array_equal(smp.cpu().numpy(), ref.samples)
    np.testing.assert_array_equal(st.get_chains(), ref.chains)
    assert abs(rate - ref.n_accepted.sum() / ref.accepts.size) < 1e-15
    st.close()
