"""The FP32 TRT collision gives a cell the same bits in every kernel: lattices of
every size (small ones are compiled without streaming hints, and take other launch
shapes) and the three streaming schemes agree bit for bit.

A periodic flow is stepped alone and 24 times along z (more than 2^23 cells, beyond
the last-level cache), in the AA pattern, the Esoteric Twist and with sparse
addressing; every copy has to hold the same populations as the small AA lattice."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPE, COPIES = (96, 64, 64), 24


def _net():
    r = np.random.default_rng(1)
    p = [r.normal(0, 0.3, 192), r.normal(0, 0.1, 32), r.normal(0, 0.15, 1024), r.normal(0, 0.1, 32),
         r.normal(0, 0.1, 32), [-5.0]]
    return np.concatenate(p + [np.zeros(6), [1e-3, 1e-3, 1e-3, 1e-2, 1e-2, 1.0], np.full(6, -1e30),
                               np.full(6, 1e30)]).astype(np.float32)


def _populations(copies, q, solids, closure, streaming):
    from paper_2305_09910_amd import lbm
    nx, ny, nz = SHAPE
    g = torch.Generator(device="cuda").manual_seed(3)
    u = 0.02 * (2 * torch.rand((3, nz, ny, nx), dtype=torch.float64, device="cuda", generator=g) - 1)
    solid = None
    if solids:
        solid = (torch.rand((nz, ny, nx), device="cuda", generator=g) < 0.1).to(torch.uint8)
        solid = solid.repeat(copies, 1, 1).cpu().numpy()
    lat = lbm.Lattice((nx, ny, nz * copies), q=q, tau=0.55, force=(1e-5, 0, 0), solid=solid, closure=closure,
                      streaming=streaming,
                      bc=("periodic", "periodic", "noslip", "noslip", "periodic", "periodic"))
    if closure == "mlp":
        lat.set_closure_weights(_net())
    lat.init_equilibrium(torch.ones((nz * copies, ny, nx), dtype=torch.float64, device="cuda"), u.repeat(1, copies, 1, 1))
    lat.step(6)
    return lat.get_pdfs().reshape(q, copies, nz, ny, nx)


@pytest.mark.parametrize("solids", [False, True])
@pytest.mark.parametrize("q, closure", [(19, "none"), (19, "smagorinsky"), (19, "mlp"), (27, "none"), (27, "mlp")])
def test_trt_gives_the_same_bits_in_every_kernel(q, closure, solids):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ref = _populations(1, q, solids, closure, "aa")
    for streaming in ("aa", "et", "sparse"):
        for copies in (1, COPIES):
            print(f"[case] TRT bits q={q} {closure} solids={solids} {streaming} copies={copies}", flush=True)
            f = _populations(copies, q, solids, closure, streaming)
            assert torch.equal(f, ref.expand_as(f)), (streaming, copies)
            del f
    torch.cuda.empty_cache()
