"""The inputs that lbm_closure_features returns are bit for bit those that the
fused step gives its network: the trusted range, which the step tests its inputs
against, is set to end exactly at the value of one cell after another, and the
step's count of fallbacks has to be the number of cells beyond it.  (A value that
differed in its last place would change the count whenever it is the boundary's
own.)"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q, storage, streaming", [(19, "f32", "aa"), (27, "f32", "aa"), (19, "f16", "aa"),
                                                   (19, "f32", "et"), (19, "f32", "sparse"), (27, "f32", "et")])
def test_step_sees_the_features_that_are_read(q, storage, streaming):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_09910_amd import inputs, lbm
    shape = (40, 12, 10)
    print(f"[case] closure features against the step, q={q} {storage} {streaming}", flush=True)
    rng = np.random.default_rng(3)
    p = np.concatenate([rng.normal(0, 0.3, 192), rng.normal(0, 0.1, 32), rng.normal(0, 0.15, 1024),
                        rng.normal(0, 0.1, 32), rng.normal(0, 0.1, 32), [-5.0]])
    scale = np.array([1e-3, 1e-3, 1e-3, 1e-2, 1e-2, 1.0])
    lat = lbm.Lattice(shape, q=q, tau=0.51, force=(3e-6, 1e-6, 0), storage=storage, streaming=streaming, closure="mlp",
                      bc=("periodic", "periodic", "noslip", "noslip", "periodic", "periodic"))

    def weights(lo, hi):
        lat.set_closure_weights(np.concatenate([p, np.zeros(6), scale, lo, hi]).astype(np.float32))

    free = np.full(6, 1e30)
    weights(-free, free)
    rho, u = inputs.channel(*shape, u_c=0.08, noise=0.2, seed=11)
    lat.init_equilibrium(rho, u)
    wrong = []
    for steps in (3, 1):
        lat.step(steps)
        state = lat.save_state()
        x = lat.closure_features().cpu().numpy().reshape(-1, 6)
        lat.closure_fallbacks()
        for k in range(6):
            for c in rng.choice(len(x), 24, replace=False):
                hi = free.copy()
                hi[k] = x[c, k]
                weights(-free, hi)
                lat.load_state(*state)
                lat.step(1)
                got, want = lat.closure_fallbacks(), int((x[:, k] > x[c, k]).sum())
                if got != want:
                    wrong.append((steps, k, int(c), got, want))
        weights(-free, free)
        lat.load_state(*state)
    print(f"q={q} {storage} {streaming}: {len(wrong)} of 288 counts differ")
    assert not wrong, wrong[:8]
