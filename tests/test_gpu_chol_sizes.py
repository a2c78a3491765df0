"""The Cholesky solve at the edges of its panels (32 columns), tiles (32 up to 2,048,
64 above) and backward forms (one workgroup with one or two columns per thread, one
launch per block above 2,048).  The tolerance is that of test_gpu_chol: the oracle's
direction to 1e-10 of its largest entry (condition number below 1e4 here)."""
import numpy as np
import pytest

import synth
from oracle import core
from test_gpu_chol import plain_state, rel_close

pytestmark = pytest.mark.gpu


# P = L + M + L M: 24, 35, 63 (last panel of 31), 99, 440, 1080, 1224, 2144
@pytest.mark.parametrize("L,alpha,n", [(4, 1, 64), (5, 1, 64), (7, 1, 96), (9, 1, 128), (20, 1, 96),
                                       (23, 2, 256), (24, 2, 128), (32, 2, 256)])
def test_direction_at_the_edges(L, alpha, n):
    import torch
    st, w = plain_state(L, alpha, n, 1)
    s = synth.random_configs(n, w.n_sites, 5 + L)
    st.load_samples(torch.from_numpy(s).cuda())
    st.expect_and_grad()
    d, info = st.sr_update(qgt="jacobian_dense", diag_shift=0.01, lr=0.0)
    assert info.converged and info.iterations == 0
    rbm = core.Rbm(w.n_sites, w.n_hidden, w.params())
    ham = core.Hamiltonian.tfim(w.n_sites, w.bonds(), 1.0, 1.0)
    O = core.jacobian(rbm, s)
    f = core.force(O, core.local_energy(rbm, ham, s))
    x = core.cholesky_solve(core.qgt_dense(O), f, 0.01)
    rel_close(d.cpu().numpy(), x, 1e-10, np.abs(x).max())
