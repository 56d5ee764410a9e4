"""The activation of the closure's training and evaluation kernels,
tanh(x) = (1 - e) / (1 + e) with e = exp(-2 |x|), rounds its quotient
correctly.

The gradient of the second layer's biases shows the activations in FP32: with
zero weights in front of it and one sample, unit j's is c (1 - h_j^2) with the
same c for every unit, and h_0 = tanh(0) = 0 gives c.  For x in [2, 3] h lies in
[0.96, 1), where an ulp is 2^-24.  The roundings on the way are, in ulp: 1 - e
(uniform in +-1/2: rms 0.289), 1 + e, whose ulp is 2^-23 (rms 0.577), and the
quotient (0.289 correctly rounded); the error of e itself enters as 2 e < 0.04 of
it.  Together 0.707, and 0.82 with a quotient that is off by 0.5 ulp rms (the
product with a refined reciprocal).  Bound: 0.76; 9300 values give the rms to
within 1%."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_tanh_quotient_is_correctly_rounded():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_09910_amd import lbm
    rng = np.random.default_rng(5)
    p = np.zeros(1337, np.float32)
    p[1280:1312] = 1 / 32  # third layer; the first two layers' weights stay zero
    p[1319:1325] = 1.0     # input scales
    p[1325:1331], p[1331:1337] = -1e30, 1e30
    x = torch.zeros((1, 6), device="cuda")
    t = torch.full((1,), -1.0, device="cuda")
    err = []
    print("[case] tanh over x in [2, 3]", flush=True)
    for _ in range(300):
        b2 = rng.uniform(2.0, 3.0, 32).astype(np.float32)
        b2[0] = 0.0
        p[1248:1280] = b2
        _, grad = lbm.mlp_loss_grad(torch.tensor(p, device="cuda"), x, t)
        g = grad.cpu().numpy().astype(np.float64)[1248:1280]
        h = np.sqrt(1.0 - g[1:] / g[0])
        err.append((h - np.tanh(b2[1:].astype(np.float64))) * 2.0 ** 24)
    rms = float(np.sqrt(np.mean(np.square(err))))
    print(f"tanh in [2, 3]: rms error {rms:.3f} ulp, largest {np.abs(err).max():.2f}")
    assert rms <= 0.76
