"""The one-launch CG of small FP64 systems against a dense solve, at the edges of the
sizes it takes (one and two 16-wide tiles each way, one to four 64-sample groups per
wave, a single sample, the work limit), and the three drivers of a step.

A solve stopped at relative residual tol is off by at most tol |f| / shift (S >= 0);
rounding adds about 1e-13 of the direction's size."""
import numpy as np
import pytest

import synth
from oracle import core

pytestmark = pytest.mark.gpu
SHIFT, TOL = 0.01, 1e-12


def _state(N, M, n, vb=True, hb=True, chains=None):
    from paper_2112_10526_amd.nqs import VMCState
    p = synth.rbm_params(N, M, 5, 0.1, vb, hb)
    chains = chains or n
    st = VMCState(model="tfim", n_sites=N, bonds=synth.chain_bonds(N), J=1.0, h=1.0, n_hidden=M,
                  visible_bias=vb, hidden_bias=hb, precision="fp64", n_chains=chains,
                  samples_per_chain=n // chains, sweep_size=N, seed=3, params=p)
    return st, core.Rbm(N, M, p, vb, hb)


@pytest.mark.parametrize("N,M,n,vb,hb", [
    (3, 1, 1, True, True), (3, 2, 70, True, True), (15, 15, 512, True, True),
    (10, 10, 513, True, False), (10, 12, 1024, False, True),
    (10, 10, 1025, True, True), (16, 16, 100, True, True),  # (these two: iteration kernels)
    (15, 31, 500, True, True), (12, 24, 512, True, True), (31, 15, 512, True, True),
    (20, 10, 300, False, False)])
def test_direction(N, M, n, vb, hb):
    import torch
    print(f"[case] {N} {M} {n} {vb} {hb}", flush=True)
    st, rbm = _state(N, M, n, vb, hb)
    s = synth.random_configs(n, N, 11)
    st.load_samples(torch.from_numpy(s).cuda())
    _, g = st.expect_and_grad()
    d, info = st.sr_update(diag_shift=SHIFT, lr=0.0, tol=TOL, maxiter=4000)
    ham = core.Hamiltonian.tfim(N, synth.chain_bonds(N), 1.0, 1.0)
    O = core.jacobian(rbm, s)
    f = core.force(O, core.local_energy(rbm, ham, s))
    assert np.abs(g.cpu().numpy() - f).max() <= 1e-11 * max(np.abs(f).max(), 1e-3)
    assert info.converged
    x = core.cholesky_solve(core.qgt_dense(O), f, SHIFT)
    tol = TOL * np.linalg.norm(f) / SHIFT + 1e-11 * np.abs(x).max() + 1e-13
    assert np.linalg.norm(d.cpu().numpy() - x) <= tol * (1 + np.sqrt(x.size))


def test_maxiter_and_the_drivers_agree():
    from paper_2112_10526_amd.nqs import batch_step, step_begin, step_poll
    cfg = dict(diag_shift=SHIFT, lr=0.02, tol=1e-8, maxiter=2000)
    runs = []
    for how in ("step", "batch", "async"):
        st, _ = _state(10, 10, 256, chains=64)
        for _ in range(3):
            if how == "step":
                rep = st.vmc_step(**cfg)
            elif how == "batch":
                rep = batch_step([st], [cfg])[0]
            else:
                step_begin(st, cfg)
                rep = step_poll([st])[0]
        runs.append((rep.energy["mean"], rep.sr.iterations, st.get_params()))
    for r in runs[1:]:
        assert r[:2] == runs[0][:2]
        np.testing.assert_array_equal(r[2], runs[0][2])
    st, _ = _state(10, 10, 256, chains=64)
    st.sample()
    st.expect_and_grad()
    _, info = st.sr_update(diag_shift=SHIFT, lr=0.0, tol=1e-14, maxiter=3, allow_notconv=True)
    assert info.iterations == 3 and not info.converged
