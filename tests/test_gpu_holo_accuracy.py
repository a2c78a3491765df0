"""Complex activations against tanh in 80-bit arithmetic: with W = 0 the hidden-bias
columns of the complex Jacobian are tanh(b_j).

In units of 2^-53 |tanh|: hyperbolic and trigonometric functions good to a unit in the
last place, their sum and two quotients, each rounded once, are about 0.8 rms (0.79 to
0.87 was measured with the functions called one by one, 1.06 to 1.14 with the hyperbolic
pair from one exponential and the quotients from a reciprocal); where sinh and cosh
are the same number the real part is exactly 1.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lo,hi,rms", [(1.0, 4.0, 0.95), (4.0, 19.0, 0.85), (25.0, 340.0, 0.05)])
@pytest.mark.parametrize("y", [0.1, 1.5, 3.0])
def test_activations(lo, hi, rms, y):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible HIP device")
    from paper_2112_10526_amd.nqs import VMCState
    print(f"[case] [{lo}, {hi}] y={y}", flush=True)
    N, M = 2, 500
    st = VMCState(model="tfim", n_sites=N, bonds=[[0, 1]], J=1.0, h=1.0, n_hidden=M,
                  precision="c128", n_chains=2, samples_per_chain=1, sweep_size=2, seed=3)
    s = torch.ones((1, N), dtype=torch.int8, device="cuda")
    rng = np.random.default_rng(7)
    sq = []
    for _ in range(50):
        b = (np.exp(rng.uniform(np.log(lo), np.log(hi), M)) * rng.choice([-1.0, 1.0], M)
             + 1j * rng.uniform(-y, y, M))
        st.set_params(np.concatenate([np.zeros(N), b, np.zeros(N * M)]))
        t = st.jacobian(s).cpu().numpy()[0, N:N + M]
        br, bi = b.real.astype(np.longdouble), b.imag.astype(np.longdouble)
        d = 2 * (np.sinh(br) ** 2 + np.cos(bi) ** 2)  # cosh 2x + cos 2y without cancellation
        re, im = np.sinh(2 * br) / d, np.sin(2 * bi) / d
        sq.append(((t.real - re) ** 2 + (t.imag - im) ** 2) / (re * re + im * im))
    st.close()
    assert float(np.sqrt(np.mean(sq))) <= rms * 2.0**-53
