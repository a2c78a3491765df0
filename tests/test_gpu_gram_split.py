"""The BF16 form's Gram against the FP64 product of the same pairs, hi.hi + hi.lo + lo.hi.

The pairs are split on the host from the public centred Jacobian (the same FP32 entries),
so only the FP32 sums of 3 n products stand between the two.  A step of entry (p, q)
rounds by at most 2^-24 |J_p| |J_q| (columns); the steps' and the entries' signs are
independent, so row p of the difference times x is about sqrt(3 n) 2^-24 |J_p| times the
length of the vector |J_q| x_q.  The solver adds 1e-9 |f|.  Each case also checks that the bound tells the product from one without its small terms, from
one with a single cross term, and from one without the batch's last 32 samples.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,n", [
    (3, 15, 31), (10, 20, 32), (9, 25, 33), (16, 16, 65), (20, 41, 1000),
    (64, 43, 96),      # 276 tiles of 128, all of G
    (64, 43, 2016),    # the same, upper triangle only
    (64, 60, 520),     # 136 tiles of 256
    (63, 67, 1055),
])
def test_three_products(N, M, n):
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
    J = st.jacobian(s.reshape(-1, N), center=True).cpu()
    fro2 = float((J.double() ** 2).sum())
    eps = 0.1 * fro2
    x, info = st.sr_update(qgt="jacobian_dense", diag_shift=eps, lr=0.0, tol=1e-10)
    st.close()
    assert info.converged
    x, f = x.cpu(), f.cpu()
    hi = J.to(torch.bfloat16).float()
    lo = (J - hi).to(torch.bfloat16).double()
    hi = hi.double()

    def residual(rows, cross):
        h, l = hi[:rows], lo[:rows]
        y = h.T @ (h @ x)
        if cross > 0:
            y += h.T @ (l @ x)
        if cross > 1:
            y += l.T @ (h @ x)
        return float((y + eps * x - f).norm())

    col = J.double().norm(dim=0)
    bound = 1e-9 * float(f.norm()) + np.sqrt(3 * n) * 2.0**-24 * np.sqrt(fro2) * float((col * x).norm())
    assert residual(n, 2) <= bound
    assert residual(n, 1) > bound and residual(n, 0) > bound
    assert residual((n - 1) // 32 * 32, 2) > bound


def test_one_sample():
    """One centred sample is zero, and so are the force and the direction."""
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible HIP device")
    from paper_2112_10526_amd.nqs import VMCState
    for prec in ("bf16", "fp32"):
        st = VMCState(model="tfim", n_sites=2, bonds=[[0, 1]], J=1.0, h=1.0, n_hidden=1,
                      precision=prec, n_chains=1, samples_per_chain=1, sweep_size=4, seed=5,
                      params=np.random.default_rng(3).normal(size=5) * 0.1, qgt="jacobian_dense")
        st.sample()
        _, f = st.expect_and_grad()
        x, _ = st.sr_update(qgt="jacobian_dense", diag_shift=1e-3, lr=0.0, tol=1e-10)
        assert not f.any() and not x.any()
        st.close()
