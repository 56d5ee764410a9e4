"""Row lengths at which the launch shape of the dense kernels changes: one more
cell than a segment, multiples of 32 that are not multiples of 64, whole rows in
one workgroup up to 320 cells, half rows, rows of whole 512-cell segments, and rows
longer than a workgroup.  A channel with a body force, D3Q19 in both dense
schemes with TRT and MRT, with solid cells and D3Q27 too, seven steps from a noisy start, against the
oracle: maximum relative population error 1e-5 in FP32 storage (a few FP32
roundings per step and population; the bound of the other parity tests)."""
import numpy as np
import pytest

from test_gpu_parity import max_rel, pair

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

NX = [65, 96, 129, 160, 246, 300, 321, 350, 400, 449, 500, 512, 600, 700, 1000]


@pytest.mark.parametrize("nx", NX)
@pytest.mark.parametrize("q, streaming, solids, collision",
                         [(19, "aa", False, "trt"), (19, "et", False, "trt"), (27, "aa", True, "trt"), (19, "et", True, "trt"),
                          (19, "aa", False, "mrt")])
def test_row_lengths_match_oracle(nx, q, streaming, solids, collision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_09910_amd import inputs
    shape = (nx, 3, 3)
    solid = None
    if solids:
        solid = np.zeros(shape[::-1], np.uint8)
        solid[1, 1, [5, nx // 2, nx - 2]] = 1
    print(f"[case] row length {nx} q={q} {streaming} solids={solids} {collision}", flush=True)
    bc = ("periodic", "periodic", "noslip", "noslip", "periodic", "periodic")
    g, o = pair(shape, q=q, tau=0.6, force=(1e-5, 0, 0), bc=bc, solid=solid, streaming=streaming, collision=collision)
    rho, u = inputs.channel(*shape, u_c=0.05, noise=0.05, seed=nx)
    g.init_equilibrium(rho, u)
    o.init_equilibrium(rho, u)
    g.step(7)
    o.step(7)
    err = max_rel(g.get_pdfs(), o.get_pdfs(), solid)
    print(f"row length {nx} q={q} {streaming}: {err:.2e}")
    assert err <= 1e-5
