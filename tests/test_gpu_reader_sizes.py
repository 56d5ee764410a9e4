"""The state readers on either side of the size from which their outputs are
written with the streaming hint (256 MB: 2^24 cells of density and velocity,
2^25 populations): the same populations as the gather kernel reads, bit for bit,
and moments equal to their sums up to FP32 rounding (19 terms: 1e-6 of the
largest), after an odd number of steps."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(128, 128, 107), (128, 128, 109), (256, 256, 255), (256, 256, 256)])
def test_readers_around_the_streaming_size(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_09910_amd import lbm
    nx, ny, nz = shape
    n = nx * ny * nz
    print(f"[case] readers {shape}", flush=True)
    g = lbm.Lattice(shape, q=19, tau=0.6, storage="f16")
    gen = torch.Generator(device="cuda").manual_seed(1)
    rho = 1 + 0.01 * torch.rand((nz, ny, nx), dtype=torch.float64, device="cuda", generator=gen)
    u = 0.04 * (torch.rand((3, nz, ny, nx), dtype=torch.float64, device="cuda", generator=gen) - 0.5)
    g.init_equilibrium(rho, u)
    g.step(3)
    cells = np.unique(np.r_[0, n - 1, np.random.default_rng(2).integers(0, n, 4000)])
    f = g.gather(cells)
    at = torch.tensor(cells, device="cuda")
    assert torch.equal(g.get_pdfs().view(19, -1)[:, at].T, f)
    r, v = g.moments()
    d = f.sum(1)
    assert float((r.view(-1)[at].double() - d).abs().max()) <= 1e-6
    jx = f[:, 1] - f[:, 2] + f[:, 7] - f[:, 8] + f[:, 9] - f[:, 10] + f[:, 11] - f[:, 12] + f[:, 13] - f[:, 14]
    assert float((v[0].reshape(-1)[at].double() - jx / d).abs().max()) <= 1e-6
