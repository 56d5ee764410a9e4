"""Totals at sizes around their split into 1024 slices of 512 threads (fewer
cells than slices, one slice cell more or less, ragged rows), after an even and
an odd number of steps and with solid cells, against the sums of the canonical
populations in 64 bits.

Tolerance: a cell's density and momentum are FP32 sums of its q deviations
(q roundings of 2^-24 of their size), added up in FP64, so a total is within
q * 2^-24 * sum |d| of the exact sum of the deviations."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 5, 7), (1023, 1, 1), (32, 32, 1), (41, 5, 5), (130, 63, 65)])
@pytest.mark.parametrize("steps, solids", [(0, False), (1, False), (3, True)])
def test_totals_equal_the_sums_of_the_populations(shape, steps, solids):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_09910_amd import inputs, lbm
    n = shape[0] * shape[1] * shape[2]
    solid = None
    if solids and n > 1:
        solid = (np.random.default_rng(3).random(shape[::-1]) < 0.2).astype(np.uint8)
    print(f"[case] totals {shape} steps={steps} solids={solids}", flush=True)
    g = lbm.Lattice(shape, q=19, tau=0.7, force=(1e-4, 2e-5, 0), solid=solid)
    rho, u = inputs.channel(*shape, u_c=0.05, noise=0.3, seed=n)
    g.init_equilibrium(rho, u)
    g.step(steps)
    mass, mom = g.totals()
    f = g.get_pdfs().cpu().numpy()
    c = np.array([(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0),
                  (-1, -1, 0), (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1), (0, 1, 1),
                  (0, -1, -1), (0, 1, -1), (0, -1, 1)], float)
    w = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)
    d = f - w[:, None, None, None]
    if solid is not None:
        d[:, solid != 0] = 0.0
    fluid = n - (0 if solid is None else int(solid.sum()))
    tol = 19 * 2.0 ** -24 * np.abs(d).sum() + 1e-13
    assert abs(mass - (fluid + d.sum())) <= tol + 1e-15 * fluid
    assert np.all(np.abs(mom - np.einsum("ia,izyx->a", c, d)) <= tol)
