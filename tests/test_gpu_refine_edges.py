"""The refinement exchange at the edges of its workgroups of 64 coarse interface
cells along x (one cell, one less than a workgroup, one more), with fine levels
on both sides, which one launch serves, and on one side, against the oracle:
maximum relative population error 1e-5 in FP32 storage, the bound of the other
refinement tests (FP32 rounding of a few steps)."""
import pytest

from test_gpu_refine import TOL32, build, max_rel, random_start, step_both

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q", [19, 27])
@pytest.mark.parametrize("nx, sides", [(1, "both"), (63, "both"), (65, "both"), (65, "hi")])
def test_refine_at_workgroup_edges(q, nx, sides):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gpu, orc = build((nx, 3, 2), 2, 0.65, (1e-5, 0, 0), q=q, lo=sides == "both")
    random_start(gpu, orc, 5)
    step_both(gpu, orc, 3)
    for name in gpu:
        err = max_rel(gpu[name], orc[name])
        print(f"refine edge nx={nx} {sides} q={q} level {name}: {err:.2e}")
        assert err <= TOL32
