"""The loss gradient adds the partial gradients in FP64: up to 512 tiles of 64
samples each tile is a partial of its own, up to 1024 tiles each pair.

Of every four tiles the first holds one sample with residual +G or -G in turn and
the later ones a residual of 2e-8 G, less than half an ulp beside it: added in FP32
they vanish, and the large ones cancel.  All weights are zero, so that the output
bias' gradient is 2/n sigmoid(b3) times the sum of the residuals, exactly known.
Tolerance 1e-5: the FP32 exponential of sigmoid(-20), whose argument of 28.9 in
base 2 is rounded to 2^-20, and a few roundings more."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles, small", [(8, (1, 2, 3)), (512, (1, 2, 3)), (520, (2, 3)), (1024, (2, 3))])
def test_partials_are_added_in_fp64(tiles, small):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_09910_amd import lbm
    print(f"[case] gradient partials of {tiles} tiles", flush=True)
    n, G, r = 64 * tiles, 2.0 ** 20, np.float32(0.02)
    p = np.zeros(1337, np.float32)
    p[1312] = -20.0
    p[1319:1325] = 1.0
    p[1325:1331], p[1331:1337] = -1e30, 1e30
    params = torch.tensor(p, device="cuda")
    x = torch.zeros((n, 6), device="cuda")
    t = lbm.mlp_forward(params, x).clone().reshape(-1)  # zero residual
    for b in range(tiles // 4):
        t[256 * b + 5] = -G if b % 2 else G
        for k in small:
            t[256 * b + 64 * k + 7 * k] = -float(r)
    _, grad = lbm.mlp_loss_grad(params, x, t)
    got = float(grad[1312])
    want = 2.0 / n / (1.0 + np.exp(20.0)) * float(r) * len(small) * (tiles // 4)
    print(f"{tiles} tiles: {got:.6e}, expected {want:.6e}")
    assert abs(got - want) <= 1e-5 * want
