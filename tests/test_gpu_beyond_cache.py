"""Lattices beyond the last-level cache.  They run the compilation of the steps that
has streaming hints, and for rows that 64 or 128 do not divide other launch shapes;
the small lattices of the other parity tests run neither.

A channel that repeats along z is stepped alone and, as one lattice beyond the
cache, as often as that takes.  The small lattice is compared with the oracle
(FP32: 1e-5 as in the other parity tests; 16-bit: two steps, three roundings of the
largest deviation), and every copy has to hold its populations bit for bit: a cell's
arithmetic is the same in both."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import BCS

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MRT27 = (1.6, 1.75, 1.55, 1.65, 1.7)
BC = ("periodic", "periodic", "noslip", "noslip", "periodic", "periodic")
CACHE = 256 << 20
FORMS = [(19, "f32", "aa", "trt", "smagorinsky", False), (19, "f32", "aa", "mrt", "smagorinsky", False),
         (19, "f32", "aa", "hrr", "none", False), (27, "f32", "aa", "trt", "none", False),
         (27, "f32", "aa", "trt", "mlp", False), (19, "f32", "et", "mrt", "smagorinsky", False),
         (19, "f32", "et", "trt", "smagorinsky", False), (19, "f32", "sparse", "mrt", "none", True),
         (27, "f32", "sparse", "trt", "smagorinsky", True), (19, "f32", "aa", "trt", "none", True),
         (19, "f32", "aa", "hrr", "none", True), (27, "f32", "aa", "mrt", "none", True),
         (27, "f32", "et", "trt", "none", True), (19, "f16", "aa", "trt", "none", False),
         (19, "f16", "aa", "mrt", "none", False), (19, "bf16", "et", "trt", "none", False),
         (19, "f16", "aa", "trt", "none", True), (27, "f16", "et", "trt", "none", True)]


def _net():
    r = np.random.default_rng(1)
    p = np.concatenate([r.normal(0, 0.3, 192), r.normal(0, 0.1, 32), r.normal(0, 0.15, 1024), r.normal(0, 0.1, 32),
                        r.normal(0, 0.1, 32), [-5.0]])
    norm = np.concatenate([np.zeros(6), [1e-3, 1e-3, 1e-3, 1e-2, 1e-2, 1.0], np.full(6, -1e30), np.full(6, 1e30)])
    return p.astype(np.float32), norm.astype(np.float32)


def _lattice(shape, form, solid):
    from paper_2305_09910_amd import lbm
    q, storage, streaming, collision, closure, _ = form
    lat = lbm.Lattice(shape, q=q, tau=0.6, force=(1e-5, 0, 0), bc=BC, solid=solid, storage=storage, closure=closure,
                      cs=0.1, collision=collision, mrt_rates=MRT27 if q == 27 else None, streaming=streaming,
                      hrr_sigma=0.995 if collision == "hrr" else None)
    if closure == "mlp":
        lat.set_closure_weights(np.concatenate(_net()))
    return lat


@pytest.mark.parametrize("nx", [96, 130, 160, 246, 300, 320, 376, 400, 444, 512, 600, 700, 1000])
@pytest.mark.parametrize("form", FORMS, ids=lambda f: "-".join(str(v) for v in f))
def test_copies_beyond_the_cache_match_the_oracle(nx, form):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_09910_amd import inputs
    q, storage, streaming, collision, closure, solids = form
    shape = (nx, 6, 4)
    print(f"[case] beyond the cache {shape} {form}", flush=True)
    solid = None
    if solids:
        solid = np.zeros(shape[::-1], np.uint8)
        solid[1, 2, [5, nx // 2, nx - 2]] = 1
        solid[3, 4, 7] = 1
    steps = 7 if storage == "f32" else 2
    rho, u = (np.asarray(v) for v in inputs.channel(*shape, u_c=0.05, noise=0.05, seed=nx))
    o = oracle.Sim(q, shape, bc=tuple(BCS[b] for b in BC), tau=0.6, force=(1e-5, 0, 0), solid=solid, cs=0.1,
                   closure={"none": oracle.CL_NONE, "smagorinsky": oracle.CL_SMAG, "mlp": oracle.CL_MLP}[closure])
    if collision == "mrt":
        o.set_mrt(MRT27 if q == 27 else oracle.MRT_DHUMIERES)
    if collision == "hrr":
        o.set_hrr(0.995)
    if closure == "mlp":
        o.set_mlp(*_net())
    o.init_equilibrium(rho, u)
    o.step(steps)
    small = _lattice(shape, form, solid)
    small.init_equilibrium(rho, u)
    small.step(steps)
    got = small.get_pdfs().reshape(q, *shape[::-1])
    ref = o.get_pdfs().reshape(q, *shape[::-1])
    fluid = np.ones(shape[::-1], bool) if solid is None else solid == 0
    err = np.abs(got.cpu().numpy() - ref)[:, fluid]
    if storage == "f32":
        bound = 1e-5 * np.abs(ref)[:, fluid]
    else:
        w = oracle.velocity_set(q)[1]
        dmax = np.abs(ref - w[:, None, None, None])[:, fluid].max()
        bound = 3 * (2.0 ** -11 if storage == "f16" else 2.0 ** -8) * dmax + 1e-7 * np.abs(ref)[:, fluid]
    assert np.all(err <= bound), float((err / np.abs(ref)[:, fluid]).max())

    copies = CACHE * 9 // 8 // small.state_bytes() + 2  # the small sparse store has a part-filled chunk of its own
    many = None if solid is None else np.tile(solid, (copies, 1, 1))
    large = _lattice((nx, shape[1], shape[2] * copies), form, many)
    assert large.state_bytes() > CACHE
    large.init_equilibrium(torch.tensor(rho, device="cuda").repeat(copies, 1, 1),
                           torch.tensor(u, device="cuda").repeat(1, copies, 1, 1))
    large.step(steps)
    f = large.get_pdfs().reshape(q, copies, *shape[::-1])
    assert torch.equal(f, got[:, None].expand_as(f))
    del f, large, small
    torch.cuda.empty_cache()
