"""Backward error of the direct solve where the Gram matrix is singular to working
precision (fewer samples than parameters, or few distinct samples) and only the shift
keeps it definite.

The residual |(J^H J + eps) x - f| is formed in 80-bit arithmetic from the public
Jacobian and force.  A backward stable solve leaves at most (3 P + 1) 2^-53 |A| |x|
(factor, forward and backward substitution), the Gram's sums of n terms another
n 2^-53 |J|_F^2 |x|.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,n,prec", [
    (6, 6, 30, "fp64"), (6, 6, 300, "fp64"), (5, 15, 200, "fp64"), (10, 10, 60, "fp64"),
    (4, 4, 20, "c128"), (6, 6, 40, "c128"),
])
@pytest.mark.parametrize("eps", [1e-6, 1e-10])
def test_residual_of_a_nearly_singular_system(N, M, n, prec, eps):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible HIP device")
    from paper_2112_10526_amd.nqs import VMCState
    print(f"[case] N={N} M={M} n={n} {prec} eps={eps}", flush=True)
    P = N + M + N * M
    ld = np.clongdouble if prec == "c128" else np.longdouble
    for seed in range(8):
        rng = np.random.default_rng(seed)
        p = rng.normal(size=P) * 0.1
        if prec == "c128":
            p = p + 1j * rng.normal(size=P) * 0.1
        st = VMCState(model="tfim", n_sites=N, bonds=[[i, (i + 1) % N] for i in range(N)], J=1.0,
                      h=1.0, n_hidden=M, precision=prec, n_chains=n, samples_per_chain=1,
                      sweep_size=2 * N, seed=seed, params=p, qgt="jacobian_dense",
                      dense_solver="cholesky")
        s = st.sample()[0].reshape(-1, N)
        _, f = st.expect_and_grad()
        J = st.jacobian(s).cpu().numpy().astype(ld)
        x, _ = st.sr_update(qgt="jacobian_dense", diag_shift=eps, lr=0.0)
        x, f = x.cpu().numpy(), f.cpu().numpy()
        st.close()
        J = (J - J.mean(0)) / np.sqrt(np.longdouble(n))
        r = J.conj().T @ (J @ x.astype(ld)) + eps * x - f
        A = float((abs(J) ** 2).sum()) + eps
        got = float(np.sqrt((abs(r) ** 2).sum())) / (2.0**-53 * A * float(np.linalg.norm(x)))
        assert got <= n + 3 * P + 1, (seed, got)
