"""The complex model's workspace: the Gram matrix's slice partials are bounded (64 MiB, or
about 2,048 tile-slices of 256 KiB), and a workspace without room for all of the slices is
taken, with fewer of them, and gives the same direction up to the sums' rounding.
"""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
MB = 2.0**20


def _state(N, M, n, **kw):
    from paper_2112_10526_amd.nqs import VMCState
    return VMCState(model="tfim", n_sites=N, bonds=[[i, (i + 1) % N] for i in range(N)], J=1.0,
                    h=1.0, n_hidden=M, precision="c128", n_chains=n, samples_per_chain=1,
                    sweep_size=N, seed=3, **kw)


def _sizes(N, M, n):
    P = N + M + N * M
    Pld = (P + 127) // 128 * 128
    t = Pld // 128
    return P, 16 * (n + 8) * Pld + 16 * P * Pld, t * (t + 1) // 2 * MB / 4


@pytest.mark.parametrize("N,M,n,slices", [
    (64, 128, 1000, 1), (64, 64, 2048, 4), (64, 64, 200, 1), (20, 20, 4096, 25), (8, 8, 300, 64),
])
def test_partials_are_bounded(N, M, n, slices):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible HIP device")
    print(f"[case] N={N} M={M} n={n}", flush=True)
    P, matrices, tiles = _sizes(N, M, n)
    st = _state(N, M, n, allocate=False)
    # batch and parameter buffers: activations of chains, samples and a batch of at least
    # 1,024, tables, vectors
    rest = 16 * M * (2 * n + max(n, 1024)) + 4 * N * max(n, 1024) + 400 * (P + 128) + 64 * n + MB
    assert st.workspace_bytes <= matrices + max(64 * MB, slices * tiles) + rest
    st.close()


def test_a_smaller_workspace_binds():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible HIP device")
    N, M, n = 14, 14, 1500
    P, _, tiles = _sizes(N, M, n)
    p = np.random.default_rng(4).normal(size=2 * P).view(complex) * 0.1

    def direction(less):
        st = _state(N, M, n, allocate=False)
        full = st.workspace_bytes
        st.workspace_bytes = full - less
        st.bind()
        st.set_params(p)
        s = st.sample()[0].cpu().numpy()
        st.expect_and_grad()
        x = st.sr_update(diag_shift=0.05, lr=0.0, tol=1e-12)[0].cpu().numpy()
        st.close()
        return s, x

    s0, x0 = direction(0)
    for slices in (1, 5):
        s, x = direction(int(slices * tiles))
        np.testing.assert_array_equal(s, s0)
        np.testing.assert_allclose(x, x0, rtol=0, atol=1e-10 * np.abs(x0).max())
    st = _state(N, M, n, allocate=False)
    full = st.workspace_bytes
    buf = torch.empty(full + 256, dtype=torch.uint8, device="cuda")
    at = buf.data_ptr() + (-buf.data_ptr()) % 256
    bind = st.lib.nqs_bind_workspace
    assert bind(st.ctx, ctypes.c_void_p(at), 16 * P) != 0  # (less than the parameters take)
    assert bind(st.ctx, ctypes.c_void_p(at), full) == 0    # (all slices again)
    st.close()
