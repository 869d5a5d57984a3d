"""Exports after a gradient: every field is that of the last step of the first ckpt_every steps, the mid-point
velocity and the drift with that step's own time steps."""
import numpy as np
import pytest

from paper_1906_07925_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps,ckpt", [(4, 2), (5, 2), (3, 1), (2, 4)])
@pytest.mark.parametrize("debug", [False, True])
def test_exports_are_of_one_step(steps, ckpt, debug):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1906_07925_amd import mpsph as M
    n = 900
    rng = np.random.Generator(np.random.PCG64(12))
    spec = W.rbf_cube(n, n_rbf=4, coeff=rng.normal(0.0, 0.1, size=4))
    x = torch.from_numpy(rng.uniform(size=(n, 3)).astype(np.float32)).cuda()
    col = torch.from_numpy(rng.integers(0, 5, size=n).astype(np.int32)).cuda()
    A, B = (M.Relaxer(spec, n=n, debug=debug) for _ in range(2))
    for R in (A, B):
        R.load(x, col)
    A.grad(steps, ckpt, 1.0, n_rbf=4)
    B.step(min(ckpt, steps))
    for f in ("h", "a", "vt", "x0") + (("rho", "at", "v", "dr") if debug else ()):
        assert torch.equal(A.field(f), B.field(f)), f
    A.close()
    B.close()
