"""A context moved from the null stream to another stream: what was queued before (the
tables of new parameters, a sampled batch) is done when the new stream's work reads it.
"""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "bf16", "c128"])
def test_null_stream_to_another(precision):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible HIP device")
    from paper_2112_10526_amd.nqs import VMCState
    print(f"[case] {precision}", flush=True)
    N, M, n = 40, 400, 2048
    P = N + M + N * M
    rng = np.random.default_rng(2)
    ps = [0.05 * rng.normal(size=P) + (0.05j * rng.normal(size=P) if precision == "c128" else 0.0)
          for _ in range(3)]
    kw = dict(model="tfim", n_sites=N, bonds=[[i, (i + 1) % N] for i in range(N)], J=1.0, h=1.0,
              n_hidden=M, precision=precision, n_chains=n, samples_per_chain=1, sweep_size=N, seed=3)
    s = torch.from_numpy(rng.choice([-1, 1], size=(n, N)).astype(np.int8)).cuda()
    ref = VMCState(params=ps[0], **kw)
    want = []
    for p in ps:
        ref.set_params(p)
        want.append(ref.log_psi(s).cpu().numpy())
    ref.close()
    st = VMCState(params=ps[0], **kw)
    assert st.stream.cuda_stream == 0
    st.load_samples(s)
    dev = [torch.from_numpy(p).cuda() for p in ps]
    other = torch.cuda.Stream()
    torch.cuda.synchronize()
    for p, w in zip(dev, want):
        st._check(st.lib.nqs_set_stream(st.ctx, None))
        st.set_params(p)
        st._check(st.lib.nqs_set_stream(st.ctx, ctypes.c_void_p(other.cuda_stream)))
        with torch.cuda.stream(other):
            y = st.log_psi(s)
        other.synchronize()
        np.testing.assert_array_equal(y.cpu().numpy(), w)
    st.close()
