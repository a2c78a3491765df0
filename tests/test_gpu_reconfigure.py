"""A context that is configured for another model answers as a fresh one does: nothing of
the first model's tile list, table order or product form stays behind.  Same kernels on
the same inputs: the directions and energies are equal bit for bit.
"""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _kwargs(N, M, precision, n):
    return dict(model="tfim", n_sites=N, bonds=[[i, (i + 1) % N] for i in range(N)], J=1.0, h=0.9,
                n_hidden=M, precision=precision, n_chains=n, samples_per_chain=1, sweep_size=N,
                seed=11, qgt="jacobian_dense", allocate=False)


def _solve(st, N, M):
    P = N + M + N * M
    rng = np.random.default_rng(P)
    p = rng.normal(size=P) * 0.1
    if st.complex:
        p = p + 1j * rng.normal(size=P) * 0.1
    st.bind()
    st.set_params(p)
    s = st.sample(n_discard=2)[0]
    e, g = st.expect_and_grad()
    x, info = st.sr_update(qgt="jacobian_dense", diag_shift=0.05, lr=0.0, tol=1e-8)
    assert info.converged
    return s.cpu().numpy(), g.cpu().numpy(), x.cpu().numpy()


# (sites, hidden units, precision, samples): 4,224 BF16 columns take Gram tiles of 256 and
# the triangle product, the others tiles of 128
SMALL = {"c128": (10, 20, "c128", 200), "bf16": (10, 20, "bf16", 200), "fp64": (12, 30, "fp64", 100)}
LARGE = (64, 64, "bf16", 600)


@pytest.mark.parametrize("first,then", [
    (LARGE, SMALL["c128"]), (LARGE, SMALL["bf16"]), (LARGE, SMALL["fp64"]),
    (SMALL["c128"], LARGE), (SMALL["fp64"], SMALL["c128"]),
])
def test_second_model_of_a_context(first, then):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible HIP device")
    from paper_2112_10526_amd import _lib
    from paper_2112_10526_amd.nqs import VMCState
    print(f"[case] {first} then {then}", flush=True)
    fresh = VMCState(**_kwargs(*then))
    want = _solve(fresh, *then[:2])
    fresh.close()
    st = VMCState(**_kwargs(*then))
    old = VMCState(**_kwargs(*first))
    old.ctx, st.ctx = st.ctx, old.ctx  # st holds the context made for `first`
    old.close()
    N, M, precision, n = then
    b = np.ascontiguousarray(_kwargs(*then)["bonds"], dtype=np.int32)
    st._check(st.lib.nqs_set_tfim(st.ctx, N, N, b.ctypes.data_as(ctypes.c_void_p), 1.0, 0.9))
    st._check(st.lib.nqs_set_rbm(st.ctx, M, 1, 1, _lib.PRECISIONS[precision]))
    st._check(st.lib.nqs_set_sampler(st.ctx, _lib.RULES["local"], n, 1, N, 11, 0))
    st._check(st.lib.nqs_set_qgt(st.ctx, _lib.QGTS["jacobian_dense"]))
    st.workspace_bytes = int(st.lib.nqs_workspace_bytes(st.ctx))
    got = _solve(st, N, M)
    st.close()
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a, b)
