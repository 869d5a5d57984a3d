"""The gradient's record: steps written in place, the last segment recorded as the forward pass runs
it, coefficient sums of a wave of particles over chunks of Gaussians.  Gradients against the float64
oracle at the bounds of the gradient tests, the state afterwards against plain steps."""
import numpy as np
import pytest

from oracle import grad as G
from paper_1906_07925_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return torch


def _case(dim, n_rbf, n, seed=3, **kw):
    rng = np.random.Generator(np.random.PCG64(seed + n_rbf))
    spec = W.rbf_cube(n, n_rbf=n_rbf, coeff=rng.normal(0.0, 0.1, size=n_rbf), s0=float(n) ** (-1.0 / dim), **kw)
    if dim == 2:
        spec.update(dim=2, lo=(0.0, 0.0), hi=(1.0, 1.0), rbf_centre=spec["rbf_centre"][:, :2].copy())
    side = int(np.ceil(n ** (1.0 / dim)))
    x = np.stack(np.meshgrid(*[(np.arange(side) + 0.5) / side] * dim, indexing="ij"), -1).reshape(-1, dim)
    x = np.clip(x[rng.permutation(len(x))[:n]] + rng.uniform(-0.2, 0.2, size=(n, dim)) / side, 0.0, 1.0)
    col = rng.integers(0, 5, size=n).astype(np.int32)
    return spec, x.astype(np.float32), col, np.zeros(n, np.int32)


def _relaxer(torch, spec, x, col, typ, debug=False):
    from paper_1906_07925_amd import mpsph as M
    R = M.Relaxer(spec, n=x.shape[0], debug=debug)
    R.load(torch.from_numpy(x).cuda(), torch.from_numpy(col).cuda(), torch.from_numpy(typ).cuda())
    return R


# table of one entry, ends of a chunk, a second and a full last chunk; particles past a whole wave
@pytest.mark.parametrize("dim,n_rbf,n", [(3, 1, 641), (2, 31, 700), (3, 33, 640), (2, 32, 1021), (3, 64, 700)])
def test_coefficient_chunks_match_oracle(torch_cuda, dim, n_rbf, n):
    spec, x, col, typ = _case(dim, n_rbf, n)
    pr = G.Problem(spec, spec["s0"], col, typ)
    L0, gc0, gx0, _, _, _ = G.run(pr, x.astype(np.float64), spec["rbf_coeff"], 2, 1.0, want_x0_grad=True)
    R = _relaxer(torch_cuda, spec, x, col, typ)
    L, gc, gx = R.grad(2, 2, 1.0, n_rbf=n_rbf, want_pos=True)
    R.close()
    gx = gx.cpu().numpy().astype(np.float64)
    assert abs(L - L0) <= 1e-5 * abs(L0)
    assert np.linalg.norm(gc - gc0) <= 2e-3 * np.linalg.norm(gc0)
    assert np.linalg.norm(gx - gx0) <= 2e-3 * np.linalg.norm(gx0)


@pytest.mark.parametrize("steps,ckpt", [(0, 2), (1, 1), (3, 5), (4, 2), (5, 2)])
@pytest.mark.parametrize("debug", [False, True])
def test_steps_go_on_after_a_gradient(torch_cuda, steps, ckpt, debug):
    torch = torch_cuda
    spec, x, col, typ = _case(3, 8, 900)
    A, B = (_relaxer(torch, spec, x, col, typ, debug) for _ in range(2))
    A.grad(steps, ckpt, 1.0, n_rbf=8, want_pos=True)
    B.step(steps)
    if 0 < steps <= ckpt:   # one segment: the exports refer to its last step, which is the run's
        assert torch.equal(A.cells()[0], B.cells()[0])
        key = lambda p: torch.sort(p[0].long() * 900 + p[1].long()).values
        assert torch.equal(key(A.pairs()), key(B.pairs()))
        for f in ("h", "a", "vt") + (("rho", "at", "v", "dr") if debug else ()):
            assert torch.equal(A.field(f), B.field(f)), f
    for more in (1, 3):
        A.step(more)
        B.step(more)
        assert torch.equal(A.store()[0], B.store()[0])
        assert A.metrics() == B.metrics()
    ga, gb = A.grad(2, 1, 1.0, n_rbf=8), B.grad(2, 2, 1.0, n_rbf=8)
    assert ga[0] == gb[0] and np.array_equal(ga[1], gb[1])
    A.close()
    B.close()


def _tree_candidates(x, reach):
    """The oracle's candidate pairs (all with |x_i - x_j| < max(reach_i, reach_j)) by a k-d tree instead of all n^2."""
    import torch
    from scipy.spatial import cKDTree
    p = cKDTree(x).query_pairs(float(reach.max()) * (1.0 + 1e-9), output_type="ndarray")
    i, j = np.concatenate([p[:, 0], p[:, 1]]), np.concatenate([p[:, 1], p[:, 0]])
    keep = np.linalg.norm(x[i] - x[j], axis=1) < np.maximum(reach[i], reach[j]) * (1.0 + 1e-9)
    o = np.lexsort((j[keep], i[keep]))
    return torch.as_tensor(i[keep][o]), torch.as_tensor(j[keep][o])


@pytest.mark.parametrize("n", [16384, 16385])   # the most particles at 16 lanes, the fewest at 8
def test_lanes_of_the_adjoint_match_oracle(torch_cuda, monkeypatch, n):
    spec, x, col, typ = _case(3, 6, n)
    monkeypatch.setattr(G, "_candidates", _tree_candidates)
    pr = G.Problem(spec, spec["s0"], col, typ)
    L0, gc0, gx0, _, _, _ = G.run(pr, x.astype(np.float64), spec["rbf_coeff"], 1, 1.0, want_x0_grad=True)
    R = _relaxer(torch_cuda, spec, x, col, typ)
    L, gc, gx = R.grad(1, 1, 1.0, n_rbf=6, want_pos=True)
    R.close()
    gx = gx.cpu().numpy().astype(np.float64)
    assert abs(L - L0) <= 1e-5 * abs(L0)
    assert np.linalg.norm(gc - gc0) <= 2e-3 * np.linalg.norm(gc0)
    assert np.linalg.norm(gx - gx0) <= 2e-3 * np.linalg.norm(gx0)
