"""The loss gradient's split of the samples over wavefronts, blocks and partial
sums, at the sizes where it changes: part of a tile of 64, one tile more than a
block's four, and the sizes around 512 blocks of four tiles, where wavefronts
start to loop.  The targets put the whole gradient into a few samples at the
edges of tiles, so that a sample left out or taken twice changes it by a large
part, against the oracle's FP64 gradient of those samples.  (Every other target
is the network's own output as the bfloat16 forward pass gives it, so those
samples carry no gradient; the oracle's FP64 forward pass would see a residual
in each of them.)

Tolerance: a weight gradient is a chain of at most five bfloat16 roundings
(unit roundoff 2^-9: activations of both layers, the delta of layer 2, the
weights it is carried back with, the delta of layer 1), 5 * 2^-9 = 1e-2 of the
few samples that carry it, doubled for the forward pass's own roundings."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 65, 256, 257, 512 * 256 - 1, 512 * 256, 512 * 256 + 1])
def test_gradient_at_the_edges_of_its_partition(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_09910_amd import lbm
    rng = np.random.default_rng(n)
    p = np.concatenate([rng.normal(0, 0.4, 192), rng.normal(0, 0.2, 32), rng.normal(0, 0.2, 1024),
                        rng.normal(0, 0.2, 32), rng.normal(0, 0.3, 32), [-3.0]]).astype(np.float32)
    norm = np.concatenate([rng.normal(0, 0.3, 6), rng.uniform(0.5, 2.0, 6), np.full(6, -1e30),
                           np.full(6, 1e30)]).astype(np.float32)
    x = rng.normal(0, 1.0, (n, 6)).astype(np.float32)
    t = oracle.mlp_forward(p, norm, x, bf16=True).astype(np.float32)
    edges = sorted({k for k in (0, 63, 64, 255, 256, n // 2, n - 2, n - 1) if 0 <= k < n})
    t[edges] += 1.0
    dev = lambda a: torch.tensor(a, device="cuda")  # noqa: E731
    print(f"[case] mlp_loss_grad n={n}", flush=True)
    loss, g = lbm.mlp_loss_grad(dev(np.r_[p, norm]), dev(x), dev(t))
    _, ref = oracle.mlp_loss_grad(p, norm, x[edges], t[edges])
    ref *= len(edges) / n
    g = g.cpu().numpy().astype(np.float64)
    rel = np.linalg.norm(g - ref) / np.linalg.norm(ref)
    print("rel", rel, "loss", float(loss), len(edges) / n)
    assert rel < 2e-2
    assert abs(float(loss) * n / len(edges) - 1.0) < 1e-2  # each edge sample is 1 off, to the forward pass's rounding
