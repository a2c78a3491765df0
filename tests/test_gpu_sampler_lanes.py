"""Every lane of a chain takes the same decision.  A chain's log ratio is a sum over its
lanes; if lanes round it differently, a uniform between two of the values makes some of
them accept and others not, and the chain's activations belong to no configuration until
they are recomputed.  That is one FP32 proposal in some tens of millions, so 4,096 chains
make 500 proposals each at seeds where it has happened, and all of their decisions are
replayed: given the chain's own earlier decisions, the proposal is taken exactly where
ln u < 2 ln |psi'/psi| in FP64.

Tolerance: |theta| stays below 3, so an activation's update, rounded a few times by 2^-24,
is off by up to cosh^2 theta = 100 times that; some hundred updates of independent signs
before theta is recomputed, 40 units with |tanh 2W| = 0.2: 6e-4 of 2 ln ratio.  Decisions
within 2e-3 of the threshold are not compared.
"""
import numpy as np
import pytest

from oracle import core

pytestmark = pytest.mark.gpu


def _draws(p, c, seed):
    """Words of draw p of chains c (Philox4x32-10)."""
    mask, sh = np.uint64(0xFFFFFFFF), np.uint64(32)
    x = [np.full(c.shape, v, np.uint64) for v in (p & 0xFFFFFFFF, p >> 32, 0, 0)]
    x[2] = c.astype(np.uint64)
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        a, b = x[0] * np.uint64(0xD2511F53), x[2] * np.uint64(0xCD9E8D57)
        x = [(b >> sh) ^ x[1] ^ np.uint64(k0), b & mask, (a >> sh) ^ x[3] ^ np.uint64(k1), a & mask]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return x


@pytest.mark.parametrize("seed", [24, 13])
def test_replayed_decisions_fp32(seed):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible HIP device")
    from paper_2112_10526_amd.nqs import VMCState
    print(f"[case] seed={seed}", flush=True)
    N, M, C, S, K = 20, 40, 4096, 2, 250
    P = N + M + N * M
    p = np.random.default_rng(seed).normal(size=P) * 0.1
    a, b, W = p[:N], p[N:N + M], p[N + M:].reshape(M, N)
    st = VMCState(model="tfim", n_sites=N, bonds=[[i, (i + 1) % N] for i in range(N)], J=1.0,
                  h=1.0, n_hidden=M, precision="fp32", n_chains=C, samples_per_chain=S,
                  sweep_size=K, seed=seed, params=p)
    s = st.get_chains().astype(np.float64)
    smp, acc, _ = st.sample(log_accepts=True)
    smp, acc = smp.cpu().numpy(), acc.cpu().numpy().astype(bool)
    st.close()
    c = np.arange(C)
    assert [int(w[7]) for w in _draws(5, c, seed)] == list(core.philox((5, 0, 7, 0), seed))
    theta = s @ W.T + b
    worst = 0.0
    for q in range(S * K):
        w = _draws(q, c, seed)
        i = (w[0].astype(np.int64) * N) >> 32
        u = ((w[1] >> np.uint64(5)).astype(float) * 67108864.0 +
             (w[2] >> np.uint64(6)).astype(float)) / 9007199254740992.0
        si = s[c, i]
        new = theta - 2.0 * si[:, None] * W[:, i].T
        ln2 = 2.0 * (np.log(np.cosh(new) / np.cosh(theta)).sum(1) - 2.0 * a[i] * si)
        gap = np.log(u) - ln2
        wrong = (gap < 0) != acc[:, q]
        worst = max(worst, float(np.abs(gap[wrong]).max(initial=0.0)))
        m = acc[:, q]
        theta[m] = new[m]
        s[c[m], i[m]] = -si[m]
        if (q + 1) % K == 0:
            np.testing.assert_array_equal(s, smp[:, q // K])
    assert worst <= 2e-3, worst
