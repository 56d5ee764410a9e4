"""Steps taken one call each and all in one call give the same bits.  A lattice of
more than half of the last-level cache steps with streaming hints in calls of fewer
than four steps (other lattices may step in between) and without them in longer
ones; the arithmetic is the same."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape, storage, streaming, collision, solids",
                         [((128, 128, 100), "f32", "aa", "trt", False), ((130, 101, 100), "f32", "et", "mrt", False),
                          ((128, 128, 100), "f32", "aa", "hrr", False), ((200, 160, 130), "f16", "aa", "trt", False),
                          ((130, 101, 120), "f32", "aa", "trt", True), ((128, 128, 120), "f32", "sparse", "trt", True)])
def test_steps_in_one_call_and_in_many(shape, storage, streaming, collision, solids):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_09910_amd import inputs
    from paper_2305_09910_amd.lbm import Lattice
    print(f"[case] step calls {shape} {storage} {streaming} {collision} solids={solids}", flush=True)
    rho, u = inputs.channel(*shape, u_c=0.05, noise=0.05, seed=3)
    solid = None
    if solids:
        solid = (np.random.default_rng(4).random(shape[::-1]) < 0.02).astype(np.uint8)
    out = []
    for calls in ([8], [1] * 8, [3, 5]):
        lat = Lattice(shape, q=19, tau=0.6, force=(1e-5, 0, 0), storage=storage, streaming=streaming,
                      collision=collision, hrr_sigma=0.995 if collision == "hrr" else None, solid=solid,
                      bc=("periodic", "periodic", "noslip", "noslip", "periodic", "periodic"))
        lat.init_equilibrium(rho, u)
        for n in calls:
            lat.step(n)
        out.append(lat.get_pdfs())
        assert 90 << 20 < lat.state_bytes() < 224 << 20
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])
    torch.cuda.empty_cache()
