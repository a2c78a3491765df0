"""The FP32 and unsliced FP64 Gram over whole and quartered tiles: batches that end inside
a step of 4 or a group of 32 samples, columns that end inside a tile.

The direction's residual |(J^T J + eps) x - f| in FP64 from the public Jacobian: FP32
sums of n terms carry at most (n + 4) 2^-24 of |J|_F^2 (FP64: the solver's 1e-10).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,n,prec", [
    (2, 1, 1, "fp32"), (3, 15, 31, "fp32"), (10, 20, 33, "fp32"), (9, 25, 5, "fp32"),
    (20, 41, 1002, "fp32"),
    (64, 43, 94, "fp32"),       # 276 whole tiles, lower triangle mirrored
    (64, 43, 1003, "fp32"),     # the same, upper triangle only
    (64, 63, 66, "fp64"),       # 561 tiles: one slice
])
def test_direction_residual(N, M, n, prec):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible HIP device")
    from paper_2112_10526_amd.nqs import VMCState
    print(f"[case] N={N} M={M} n={n} {prec}", flush=True)
    P = N + M + N * M
    st = VMCState(model="tfim", n_sites=N, bonds=[[i, i + 1] for i in range(N - 1)], J=1.0, h=1.0,
                  n_hidden=M, precision=prec, n_chains=n, samples_per_chain=1, sweep_size=2 * N,
                  seed=5, params=np.random.default_rng(N + M).normal(size=P) * 0.1,
                  qgt="jacobian_dense")
    s = st.sample()[0]
    _, f = st.expect_and_grad()
    J = st.jacobian(s.reshape(-1, N), center=True).double()
    fro2 = float((J * J).sum())
    eps = 0.1 * fro2 + 1e-3
    x, info = st.sr_update(qgt="jacobian_dense", diag_shift=eps, lr=0.0, tol=1e-10)
    r = J.T @ (J @ x) + eps * x - f
    bound = 1e-9 * float(f.norm())
    if prec == "fp32":
        bound += (n + 4) * 2.0**-24 * fro2 * float(x.norm())
    assert info.converged
    assert float(r.norm()) <= bound
    st.close()
