"""Parameters from the host and from tensors: equal values give equal states, a tensor
with too few values and one with a value that is not finite are refused and leave the
state as it was.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _state(kind, N=6, M=12):
    from paper_2112_10526_amd.nqs import VMCState
    kw = dict(model="tfim", n_sites=N, bonds=[[i, (i + 1) % N] for i in range(N)], J=1.0, h=1.0,
              n_hidden=M, n_chains=32, samples_per_chain=2, sweep_size=N, seed=3)
    if kind == "symm":
        perms = np.stack([(np.arange(N) + g) % N for g in range(N)]).astype(np.int32)
        return VMCState(precision="fp64", symmetries=perms, alpha=2, **kw)
    return VMCState(precision=kind, **kw)


@pytest.mark.parametrize("kind", ["fp64", "fp32", "bf16", "c128", "symm"])
def test_host_and_device_values(kind):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible HIP device")
    print(f"[case] {kind}", flush=True)
    st = _state(kind)
    P = st.n_params
    rng = np.random.default_rng(1)
    p, q = (0.1 * rng.normal(size=P) + (0.1j * rng.normal(size=P) if kind == "c128" else 0.0)
            for _ in range(2))
    st.set_params(p)
    s = st.sample()[0].reshape(-1, st.n_sites)
    st.load_samples(s)

    def seen():
        e, g = st.expect_and_grad()
        return st.get_params(), e["mean"], g.cpu().numpy(), st.log_psi(s).cpu().numpy()

    want = seen()
    np.testing.assert_array_equal(want[0], p)
    st.set_params(q)
    st.set_params(torch.from_numpy(p).cuda())
    for a, b in zip(seen(), want):
        np.testing.assert_array_equal(a, b)
    with pytest.raises(ValueError):
        st.set_params(torch.from_numpy(q[:-1]).cuda())
    with pytest.raises(ValueError):
        st.set_params(torch.empty(0, dtype=torch.float64))
    bad = q.copy()
    bad[-1] = np.nan
    for v in (bad, torch.from_numpy(bad).cuda()):
        with pytest.raises(Exception, match="finite"):
            st.set_params(v)
    for a, b in zip(seen(), want):
        np.testing.assert_array_equal(a, b)
    st.close()
