"""Workgroups in slabs of planes per XCD against workgroups in the launch's order.

A lattice steps in slabs where a plane is no multiple of eight workgroups; the same
flow eight times along the periodic y axis has eight times the workgroups in a
plane, so it steps in the launch's order.  With solids (FP32) every lattice that
fits the last-level cache steps in slabs, and the other one is repeated until it
does not.  Each cell's arithmetic is the same in both, so that every copy holds the
same populations bit for bit.

rows: the rows per workgroup at that row length; ny is a multiple of them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape, rows", [((40, 4, 2), 4), ((64, 12, 9), 4), ((100, 6, 11), 2), ((65, 10, 40), 2)])
@pytest.mark.parametrize("storage, streaming, collision, solids",
                         [("f32", "aa", "trt", False), ("f32", "et", "mrt", False), ("f16", "aa", "trt", False),
                          ("bf16", "aa", "mrt", False), ("f16", "aa", "hrr", False), ("f32", "aa", "mrt", True),
                          ("f32", "et", "trt", True)])
def test_slabs_against_the_launch_order(shape, rows, storage, streaming, collision, solids):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_09910_amd import inputs
    from paper_2305_09910_amd.lbm import Lattice
    nx, ny, nz = shape
    print(f"[case] slab order {shape} {storage} {streaming} {collision} solids={solids}", flush=True)
    bc = ("periodic",) * 4 + ("noslip", "noslip")
    rho, u = (torch.tensor(np.asarray(v), device="cuda") for v in inputs.channel(*shape, u_c=0.05, noise=0.05, seed=nx))
    solid = None
    if solids:
        solid = np.zeros((nz, ny, nx), np.uint8)
        solid[nz // 2, ny // 2, 3::7] = 1
    per_plane = -(-nx // (128 if 64 < nx < 128 else 64)) * (ny // rows)

    def run(copies):
        lat = Lattice((nx, copies * ny, nz), q=19, tau=0.6, force=(1e-5, 0, 0), bc=bc, storage=storage,
                      streaming=streaming, collision=collision, hrr_sigma=0.995 if collision == "hrr" else None,
                      solid=None if solid is None else np.tile(solid, (1, copies, 1)))
        lat.init_equilibrium(rho.repeat(1, copies, 1), u.repeat(1, 1, copies, 1))
        lat.step(7)
        return lat.get_pdfs().reshape(19, nz, copies, ny, nx), lat.state_bytes()

    one, size = run(1)
    copies = 8
    if solids:  # beyond the cache
        copies = (256 << 20) // size + 1
    many, size = run(copies)
    if solids:
        assert size > 224 << 20
    else:
        wide = 4 if storage == "f32" else 2
        assert per_plane % 8 != 0 and 8 * nx * ny * nz * 19 * wide <= (32 << 20 if wide == 4 else 10 << 20)
    assert torch.equal(many, one.expand_as(many))
    torch.cuda.empty_cache()
