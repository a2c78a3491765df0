"""The product of the stored QGT from its upper triangle (G above 32 MiB): 256 and 512
columns per block, P no multiple of a tile or of a block, and the whole product where
the Jacobian's buffer is too small for the partial sums.

The direction's residual |(J^T J + eps) x - f| is formed in FP64 from the public
Jacobian.  FP64: CG stops at 1e-10 |f| of its recursive residual and the true one
differs by some 1e-16 |G| |x| per iteration, below 1e-9 |f| with eps = |G|_F / 10.
FP32: J's entries and the n-term sums of G carry at most (n + 4) 2^-24 of
|J|^T |J| <= |J|_F^2 each.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,prec,n", [
    (33, 63, "fp64", 256),    # P = 2,175: 256 columns per block
    (32, 90, "fp32", 256),    # P = 3,002
    (33, 63, "fp64", 16),     # too little scratch
    (64, 320, "fp32", 512),   # P = 20,864: 512 columns per block
])
def test_direction_residual(N, M, prec, n):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible HIP device")
    from paper_2112_10526_amd.nqs import VMCState
    print(f"[case] N={N} M={M} {prec} n={n}", flush=True)
    P = N + M + N * M
    rng = np.random.default_rng(N + M)
    st = VMCState(model="tfim", n_sites=N, bonds=[[i, (i + 1) % N] for i in range(N)], J=1.0, h=1.0,
                  n_hidden=M, precision=prec, n_chains=n // 4, samples_per_chain=4, sweep_size=N,
                  seed=5, params=rng.normal(size=P) * 0.05, qgt="jacobian_dense")
    st.thermalize(2)
    s = st.sample()[0]
    _, f = st.expect_and_grad()
    J = st.jacobian(s.reshape(-1, N), center=True).double()
    fro2 = float((J * J).sum())
    x, info = st.sr_update(qgt="jacobian_dense", diag_shift=0.1 * fro2, lr=0.0, tol=1e-10)
    r = J.T @ (J @ x) + 0.1 * fro2 * x - f
    bound = 1e-9 * float(f.norm())
    if prec == "fp32":
        bound += (n + 4) * 2.0**-24 * fro2 * float(x.norm())
    assert info.converged
    assert float(r.norm()) <= bound
    st.close()
