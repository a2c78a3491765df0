"""Local energies at the edges of the kernel's split: 64 items per chunk, 128 per wave,
four waves of items per block, hidden units in twos (FP64) and fours (FP32), logarithms
every 64, odd batches, and batches large enough for eight samples per wave.

Bars as for the other local energies: 1e-10 relative in FP64, 1e-4 in FP32.  The split
over samples changes no sample's operations, so a sample's energy in a large batch
equals the one it has in a small batch to the last bit.
"""
import numpy as np
import pytest

import synth
from oracle import core

pytestmark = pytest.mark.gpu


def state(kind, N, n_bonds, M, prec, n):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible HIP device")
    from paper_2112_10526_amd.nqs import VMCState
    print(f"[case] {kind} N={N} bonds={n_bonds} M={M} {prec} n={n}", flush=True)
    rng = np.random.default_rng(N + 7 * n_bonds + M)
    bonds = [[b % N, (b % N + 1 + b // N) % N] for b in range(n_bonds)]
    params = rng.normal(size=N + M + N * M) * 0.05
    st = VMCState(model=kind, n_sites=N, bonds=bonds, J=0.7, h=1.3, n_hidden=M, precision=prec,
                  n_chains=n, samples_per_chain=1, sweep_size=N, seed=3, params=params)
    ham = (core.Hamiltonian.tfim(N, bonds, 0.7, 1.3) if kind == "tfim"
           else core.Hamiltonian.heisenberg(N, bonds, 0.7))
    return st, core.Rbm(N, M, params), ham, torch


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("fp32", 1e-4)])
@pytest.mark.parametrize("kind,N,n_bonds,M,n", [
    ("tfim", 2, 1, 1, 1),
    ("tfim", 64, 64, 3, 5),
    ("tfim", 65, 130, 62, 33),
    ("tfim", 128, 128, 64, 4),
    ("tfim", 129, 200, 65, 3),
    ("tfim", 520, 520, 5, 7),       # more item groups than a block has waves
    ("heisenberg", 64, 64, 126, 9),
    ("heisenberg", 64, 65, 4, 2),
    ("heisenberg", 100, 257, 130, 6),
    ("heisenberg", 260, 514, 66, 3),
])
def test_against_the_oracle(kind, N, n_bonds, M, n, prec, tol):
    st, rbm, ham, torch = state(kind, N, n_bonds, M, prec, n)
    s = synth.random_configs(n, N, 5 + N)
    e = st.local_energy(torch.from_numpy(s).cuda()).cpu().numpy()
    ref = core.local_energy(rbm, ham, s)
    assert (np.abs(e - ref) / np.maximum(np.abs(ref), 1.0)).max() <= tol
    st.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("kind,N,n_bonds,n", [("tfim", 65, 65, 65541), ("heisenberg", 200, 385, 16391)])
def test_batch_size_changes_nothing(kind, N, n_bonds, n, prec):
    st, _, _, torch = state(kind, N, n_bonds, 7, prec, n)
    s = torch.from_numpy(synth.random_configs(n, N, 9)).cuda()
    e = st.local_energy(s)
    for k in (0, 1000, n - 13):
        assert torch.equal(e[k:k + 13], st.local_energy(s[k:k + 13].contiguous()))
    st.close()
