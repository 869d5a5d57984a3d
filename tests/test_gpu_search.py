"""The search grid of the pair passes, whose rows follow the cut-off and not the cell size: rows of
several cells, of one cell and of half a cell, rows that span a periodic box, particles with more rows
than one chunk of the row table holds.  Single steps against the oracle at the standard bounds."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1906_07925_amd import workloads as W
from tests import parity_util as PU

pytestmark = pytest.mark.gpu


def _periodic(dim, n):
    return dict(dim=dim, geometry="periodic", lo=(0.0,) * dim, hi=(1.0,) * dim, field="uniform", n=n)


# (region, dim, particles, cell_log2, lanes)
CASES = [("box", 2, 3000, 3, 4), ("box", 2, 3000, 8, 8), ("box", 3, 4000, 2, 2), ("box", 3, 4000, 7, 4),
         ("periodic", 2, 1500, 2, 4), ("periodic", 2, 1500, 7, 8), ("periodic", 3, 1200, 1, 4),
         ("periodic", 3, 1200, 3, 8), ("periodic", 3, 1200, 5, 2), ("graded", 3, 6000, -1, 2), ("graded", 3, 6000, 6, 8)]


@pytest.mark.parametrize("region,dim,n,k,lanes", CASES)
def test_search_rows_keep_the_step(region, dim, n, k, lanes):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    rng = np.random.Generator(np.random.PCG64(13 * n + dim))
    x = rng.uniform(0.0, 1.0, size=(n, dim)).astype(np.float32)
    if region == "periodic":
        spec, s0 = _periodic(dim, n), float(n) ** (-1.0 / dim)
    elif region == "box":
        spec, s0 = (W.unit_square if dim == 2 else W.unit_cube)(n), float(n) ** (-1.0 / dim)
    else:   # 1:12, half of the particles around the fine sphere: coarse particles reach hundreds of rows
        spec = W.cube_with_inclusion(n, ratio=12.0)
        u = rng.normal(size=(n // 2, 3))
        x[: n // 2] = 0.5 + (0.25 + 0.05 * rng.uniform(-1, 1, size=(n // 2, 1))) * u / np.linalg.norm(u, axis=1)[:, None]
        s0 = O.OracleParams(dict(spec, n=n)).s0
    col = rng.integers(0, 4, size=n).astype(np.int32)
    PU.check_single_step(spec, s0, x, col, np.zeros(n, np.int32), cell_log2=k, lanes=lanes)


@pytest.mark.parametrize("dim,n,k,lanes", [(2, 900, 5, 4), (2, 2500, -1, 2), (3, 2000, -1, 8), (3, 2000, 4, 4)])
@pytest.mark.parametrize("kappa", [1.3, 1.999, 2.0])
def test_shorter_cut_off_keeps_the_step(dim, n, k, lanes, kappa):
    """kappa = 2 has passes of its own, without the cut-off tests that a shorter one needs."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    rng = np.random.Generator(np.random.PCG64(7 * n + dim))
    spec = dict((W.unit_square if dim == 2 else W.unit_cube)(n), kappa=kappa)
    x = rng.uniform(0.0, 1.0, size=(n, dim)).astype(np.float32)
    col = rng.integers(0, 3, size=n).astype(np.int32)
    typ = rng.choice([0, 0, 0, 1, 2], size=n).astype(np.int32)
    PU.check_single_step(spec, float(n) ** (-1.0 / dim), x, col, typ, cell_log2=k, lanes=lanes)


def test_batch_of_two_cut_offs_keeps_each_domain():
    """A launch with one shorter cut-off takes the general passes for all of its domains: the domain
    with kappa = 2 ends where its own kernels take it, bit for bit."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1906_07925_amd import mpsph as M
    rng = np.random.Generator(np.random.PCG64(3))
    n = 1500
    specs = [dict(W.unit_square(n), n=n, kappa=k) for k in (2.0, 1.4)]
    xs = [rng.uniform(0.0, 1.0, size=(n, 2)).astype(np.float32) for _ in specs]
    col = torch.from_numpy(rng.integers(0, 2, size=n).astype(np.int32)).cuda()

    def run(sel):
        R = M.Relaxer([specs[i] for i in sel], n=[n] * len(sel))
        R.load(torch.from_numpy(np.concatenate([xs[i] for i in sel])).cuda(), col.repeat(len(sel)))
        R.step(5)
        out = R.split(R.store()[0])
        R.close()
        return out
    both = run([0, 1])
    for i in range(2):
        assert torch.equal(both[i], run([i])[0]), i
