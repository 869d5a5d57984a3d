"""The gradient of a set at rest: no particle has a force, so there is no first time step to differentiate and the
steps move nothing; the gradient is that of the loss alone."""
import numpy as np
import pytest

from paper_1906_07925_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("field", ["uniform", "rbf_exp"])
def test_gradient_without_a_force(dim, field):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1906_07925_amd import mpsph as M
    # a normal particle midway between two fixed ones in one search cell, the normal one first: its forces cancel exactly
    x = np.full((3, dim), 0.5, np.float32)
    x[1, 0], x[2, 0] = 0.25, 0.75
    spec = (W.unit_square if dim == 2 else W.unit_cube)(3)
    if field == "rbf_exp":
        spec.update(field="rbf_exp", n_rbf=1, rbf_width=0.3, rbf_centre=np.full((1, dim), 0.5), rbf_coeff=np.array([0.1]))
    state = [torch.from_numpy(a).cuda() for a in (x, np.array([0, 1, 1], np.int32), np.array([0, 3, 3], np.int32))]
    out = []
    for steps in (0, 1, 3):
        R = M.Relaxer(spec, n=3, s0=0.3, cell_log2=1)
        R.load(*state)
        out.append(R.grad(steps, 2, 1.0, n_rbf=1 if field == "rbf_exp" else 0, want_pos=True))
        if steps:
            assert R.metrics()["pairs"] > 0 and R.metrics()["dt1"] == 0.0
            assert torch.equal(R.store()[0], state[0])
        R.close()
    for L, gc, gx in out[1:]:
        assert L == out[0][0] and torch.isfinite(gx).all() and torch.equal(gx, out[0][2])
        if field == "rbf_exp":
            assert np.array_equal(gc, out[0][1])
