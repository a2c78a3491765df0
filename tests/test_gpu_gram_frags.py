"""The BF16 form's Gram over its three tile sizes, with batches that end inside a block of
32 samples (one, an odd and an even number of blocks) and columns that end inside a tile.

As for the other stored-QGT products, the direction's residual |(J^T J + eps) x - f| is
formed in FP64 from the public Jacobian.  An entry of J kept as hi + lo loses 2^-17 of
itself and the product lo.lo another 2^-16, and the sums of three products over n samples
carry at most (3 n + 4) 2^-24 of |J|^T |J| <= |J|_F^2.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,n", [
    (2, 1, 1), (3, 15, 31), (10, 20, 32), (9, 25, 33), (16, 16, 65), (20, 41, 1000),
    (64, 43, 96),      # 276 tiles of 128, the lower triangle read or not
    (64, 43, 2016),
    (64, 60, 520),     # 136 tiles of 256
    (63, 67, 1055),
])
def test_direction_residual(N, M, n):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible HIP device")
    from paper_2112_10526_amd.nqs import VMCState
    print(f"[case] N={N} M={M} n={n}", flush=True)
    P = N + M + N * M
    st = VMCState(model="tfim", n_sites=N, bonds=[[i, i + 1] for i in range(N - 1)], J=1.0, h=1.0,
                  n_hidden=M, precision="bf16", n_chains=n, samples_per_chain=1, sweep_size=2 * N,
                  seed=5, params=np.random.default_rng(N + M).normal(size=P) * 0.1,
                  qgt="jacobian_dense")
    s = st.sample()[0]
    _, f = st.expect_and_grad()
    J = st.jacobian(s.reshape(-1, N), center=True).double()
    fro2 = float((J * J).sum())
    eps = 0.1 * fro2 + 1e-3
    x, info = st.sr_update(qgt="jacobian_dense", diag_shift=eps, lr=0.0, tol=1e-10)
    r = J.T @ (J @ x) + eps * x - f
    bound = 1e-9 * float(f.norm()) + (2 * 2.0**-17 + 2.0**-16 + (3 * n + 4) * 2.0**-24) * fro2 * float(x.norm())
    assert info.converged
    assert float(r.norm()) <= bound
    st.close()
