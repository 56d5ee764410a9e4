"""Small lattices whose planes are not a multiple of eight workgroups step in slabs
of planes per XCD.  The same flow eight times along the periodic y axis takes
workgroups in the launch's order.  Each cell's arithmetic is the same in both, so
that every copy holds the same populations bit for bit, whatever the storage."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(40, 5, 2), (64, 17, 9), (100, 7, 11), (65, 9, 40)])
@pytest.mark.parametrize("storage, streaming, collision",
                         [("f32", "aa", "trt"), ("f32", "et", "mrt"), ("f16", "aa", "trt"), ("bf16", "aa", "mrt"), ("f16", "et", "trt"),
                          ("f16", "aa", "hrr")])
def test_slabs_step_as_the_whole_grid(shape, storage, streaming, collision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import numpy as np
    from paper_2305_09910_amd import inputs
    from paper_2305_09910_amd.lbm import Lattice
    nx, ny, nz = shape
    print(f"[case] slabs {shape} {storage} {streaming} {collision}", flush=True)
    bc = ("periodic",) * 4 + ("noslip", "noslip")
    rho, u = inputs.channel(*shape, u_c=0.05, noise=0.05, seed=nx)
    out = []
    for n in (1, 8):
        lat = Lattice((nx, n * ny, nz), q=19, tau=0.6, force=(1e-5, 0, 0), bc=bc, storage=storage, streaming=streaming,
                      collision=collision)
        lat.init_equilibrium(np.concatenate([np.asarray(rho)] * n, axis=-2), np.concatenate([np.asarray(u)] * n, axis=-2))
        lat.step(7)
        out.append(lat.get_pdfs())
    q = out[0].shape[0]
    one, eight = out[0].reshape(q, nz, ny, nx), out[1].reshape(q, nz, n, ny, nx)
    for k in range(n):
        assert torch.equal(one, eight[:, :, k]), f"copy {k}"
