"""The sampler's table rows and its look-ahead: every number of hidden units per lane
(1 to 32, vectors of 1 and 2), one and two chains per wave, both rules, and lattices so
small that consecutive proposals keep hitting the same spins.

Decisions are exact against the oracle for every chain whose smallest |u - ratio^2|
exceeds 1e-12 there.
"""
import numpy as np
import pytest

from oracle import core

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rule,N,M,C,K,S", [
    ("local", 2, 1, 3, 70, 2),
    ("local", 2, 64, 2048, 33, 1),      # pairs, one unit per lane and chain slot
    ("local", 3, 65, 2048, 65, 1),
    ("local", 12, 200, 2050, 12, 1),    # pairs, eight units per lane
    ("local", 12, 200, 64, 12, 3),      # the same model, one chain per wave
    ("local", 5, 257, 7, 40, 2),
    ("local", 5, 600, 4, 40, 1),
    ("local", 4, 1500, 2, 31, 1),
    ("exchange", 2, 3, 2048, 64, 1),
    ("exchange", 4, 130, 2048, 100, 1),
    ("exchange", 6, 300, 5, 65, 2),
])
def test_decisions_fp64(rule, N, M, C, K, S):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible HIP device")
    from paper_2112_10526_amd.nqs import VMCState
    print(f"[case] {rule} N={N} M={M} C={C} K={K} S={S}", flush=True)
    rng = np.random.default_rng(N + M)
    bonds = [[i, (i + 1) % N] for i in range(N if N > 2 else 1)]
    params = rng.normal(size=N + M + N * M) * (0.3 / np.sqrt(M))
    st = VMCState(model="heisenberg" if rule == "exchange" else "tfim", n_sites=N, bonds=bonds,
                  J=1.0, h=1.0, n_hidden=M, precision="fp64", rule=rule, n_chains=C,
                  samples_per_chain=S, sweep_size=K, seed=21, params=params,
                  total_sz_zero=rule == "exchange")
    ch = st.get_chains()
    smp, acc, _ = st.sample(log_accepts=True)
    ref = core.sample(core.Rbm(N, M, params), ch, S, K, 21, 0, rule=rule, bonds=np.array(bonds),
                      mode="cached", log_accepts=True)
    good = ref.margins > 1e-12
    assert good.mean() > 0.99
    np.testing.assert_array_equal(acc.cpu().numpy()[good], ref.accepts[good])
    np.testing.assert_array_equal(smp.cpu().numpy()[good], ref.samples[good])
    st.close()
