"""ln psi in blocks of 32, 64 and 128 rows (batches of 16,385 rows and more) with more
hidden tiles than a block has waves, and in its register forms for 161 to 271 sites.

The large batches' rows are compared with the oracle, and bit for bit with the same rows
in batches of 1,000 (blocks of 16 rows): a row's sums do not depend on its block.
Tolerances: FP64 1e-12 of the number of terms; FP32: theta is a sum of N + 1 terms
with |theta| <= 2 here, each rounded by 2^-24, weighted by |tanh theta| <= 1.
"""
import numpy as np
import pytest

import synth
from oracle import core

pytestmark = pytest.mark.gpu


def _state(N, M, precision):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible HIP device")
    from paper_2112_10526_amd.nqs import VMCState
    p = synth.rbm_params(N, M, 5, 0.05)
    st = VMCState(model="tfim", n_sites=N, bonds=synth.chain_bonds(N), J=1.0, h=1.0, n_hidden=M,
                  precision=precision, n_chains=8, samples_per_chain=1, sweep_size=N, seed=3,
                  params=p)
    return st, core.Rbm(N, M, p)


def _tol(N, M, precision):
    return 1e-12 * (N + M) if precision == "fp64" else M * 2 * (N + 1) * 2.0**-24


@pytest.mark.parametrize("N,M,n", [(7, 140, 16385), (10, 131, 32800), (5, 300, 65601)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_large_batches(N, M, n, precision):
    import torch
    print(f"[case] {N} {M} {n} {precision}", flush=True)
    st, rbm = _state(N, M, precision)
    s = synth.random_configs(n, N, 8)
    sd = torch.from_numpy(s).cuda()
    y = st.log_psi(sd).cpu().numpy()
    np.testing.assert_allclose(y, core.log_psi(rbm, s), rtol=0, atol=_tol(N, M, precision))
    for k in range(0, n, 1000):
        np.testing.assert_array_equal(y[k:k + 1000], st.log_psi(sd[k:k + 1000]).cpu().numpy())
    st.close()


@pytest.mark.parametrize("N", [161, 170, 192, 207, 224, 240, 260, 271])
@pytest.mark.parametrize("M,n", [(33, 70), (200, 16400)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_register_forms(N, M, n, precision):
    import torch
    print(f"[case] {N} {M} {n} {precision}", flush=True)
    st, rbm = _state(N, M, precision)
    s = synth.random_configs(n, N, 9)
    y = st.log_psi(torch.from_numpy(s).cuda()).cpu().numpy()
    k = np.unique(np.concatenate([np.arange(min(n, 300)), np.arange(max(0, n - 300), n)]))
    np.testing.assert_allclose(y[k], core.log_psi(rbm, s[k]), rtol=0, atol=_tol(N, M, precision))
    st.close()
