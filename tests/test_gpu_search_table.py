"""The search table and order that the pair passes work on, against numpy: cells from the positions, the table
as the lower bound of every cell, the particles of a cell in load order."""
import math

import numpy as np
import pytest

from paper_1906_07925_amd import workloads as W

pytestmark = pytest.mark.gpu

TILE = 4096   # table entries per block of the scan


def search_cells(x, k, rb, xb):
    """Search cell of float32 positions in the unit box at 2^k cells (walls at cells 0 and 2^k - 1)."""
    X = x.astype(np.float64) * (2 ** k - 1)
    c = np.floor(X)
    o = (X - c).astype(np.float32)
    c, o = np.where(o >= 1, c + 1, c).astype(np.int64), np.where(o >= 1, np.float32(0), o)
    cell = (c[:, 0] << xb) + np.floor(o[:, 0].astype(np.float64) * 2 ** xb).astype(np.int64)
    r = np.floor((c + o.astype(np.float64)) * 2.0 ** -rb).astype(np.int64)[:, 1:]
    kr = k - rb
    if r.shape[1] == 1:
        row = r[:, 0]
    else:
        t = min(4, kr)
        lo, hi = r & (2 ** t - 1), r >> t
        row = lo[:, 0] | lo[:, 1] << t | hi[:, 0] << 2 * t | hi[:, 1] << (kr + t)
    return cell + (row << (k + xb)), 2 ** (k + xb + kr * r.shape[1])


# (dim, particles, cell_log2, tiles, domains): one tile ordered by one block (at most 4096 particles) and by two
# launches; two tiles, three half ones of a batch; 16; 64, the most that one launch scans; 128, with a launch for the
# sums of the tiles; rows of many cells, of one and of half a cell
CASES = [(2, 1, 3, 1, 1), (2, 63, 4, 1, 1), (2, 4096, 3, 1, 1), (2, 4097, 3, 1, 1), (3, 4096, 2, 1, 1), (2, 2048, 5, 2, 1),
         (2, 1000, 4, 2, 3), (2, 16384, 6, 16, 1), (2, 65536, 8, 64, 1), (2, 65537, 8, 64, 1), (3, 65536, 6, 64, 1),
         (2, 131072, 8, 128, 1), (3, 140000, 6, 128, 1), (3, 140000, 5, 128, 1), (2, 65536, 8, 192, 3), (3, 20011, -1, None, 1),
         (2, 40, 9, 1, 1), (3, 500, 7, 1, 1)]


@pytest.mark.parametrize("dim,n,k,tiles,ndom", CASES)
def test_search_table_and_order(dim, n, k, tiles, ndom):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1906_07925_amd import mpsph as M
    rng = np.random.Generator(np.random.PCG64(11 * n + dim))
    spec = dict((W.unit_square if dim == 2 else W.unit_cube)(n), n=n)
    x = rng.uniform(0.0, 1.0, size=(ndom * n, dim)).astype(np.float32)
    x[: n // 4] = x[n // 2: n // 2 + n // 4]           # coincident pairs share a cell
    x[: n // 8] = np.round(x[: n // 8])                # walls and corners
    s0 = float(n) ** (-1.0 / dim)
    R = M.Relaxer([spec] * ndom, n=[n] * ndom, s0=[s0] * ndom, cell_log2=k)
    for _ in range(2):                                 # the second load starts from the counts of two steps
        R.load(torch.from_numpy(x).cuda(), torch.zeros(ndom * n, dtype=torch.int32, device="cuda"))
        R.step(1)
        start, order, rb, xb = R.search()
        cell, ncells = search_cells(x, R.cell_log2(), rb, xb)
        cell = cell + np.repeat(np.arange(ndom), n) * ncells
        start, order = start.cpu().numpy().astype(np.int64), order.cpu().numpy()
        assert start.size == ndom * ncells + 1
        if tiles is not None:
            assert -(-ndom * ncells // TILE) == tiles
        assert np.array_equal(order, np.argsort(cell, kind="stable"))
        assert np.array_equal(start, np.searchsorted(np.sort(cell), np.arange(start.size)))
        R.step(1)
        start = R.search()[0].cpu().numpy().astype(np.int64)
        assert start[0] == 0 and start[-1] == ndom * n and np.all(np.diff(start) >= 0)
    R.close()


def _steep(dim, kind, a, b):
    """Size fields with a range beyond 1:8: the distance to a sphere of radius a, graded 1:b; a mesh of nodes a times as
    fine near the centre of the box; a Gaussian of width a that takes the spacing down by exp(b)."""
    s = (W.unit_square if dim == 2 else W.unit_cube)(0)
    if kind == "sphere":
        s.update(field="sphere_distance", fcentre=(0.5,) * dim, fb=a, fa=(b - 1.0) / (math.sqrt(dim) / 2.0 - a))
    elif kind == "mesh":
        ax = np.linspace(0.0, 1.0, b) - 0.5
        r2 = sum(g ** 2 for g in np.meshgrid(*[ax] * dim, indexing="ij")).reshape(-1)
        s.update(field="grid", grid_n=(b,) * dim + (1,) * (3 - dim), grid_s=1.0 - (1.0 - 1.0 / a) * np.exp(-r2 / 0.01))
    else:
        s.update(field="rbf_exp", n_rbf=1, rbf_width=a, rbf_centre=np.full((1, dim), 0.4), rbf_coeff=np.array([-float(b)]))
    return s


def _mean_spacing(s, dim):
    """int s^(1-d) / int s^-d over the unit box at s0 = 1, by midpoints."""
    m = 2000 if dim == 2 else 250
    ax = (np.arange(m) + 0.5) / m
    X = np.meshgrid(*[ax] * dim, indexing="ij")
    if s["field"] == "sphere_distance":
        f = 1.0 + s["fa"] * np.abs(np.sqrt(sum((g - 0.5) ** 2 for g in X)) - s["fb"])
    elif s["field"] == "grid":
        from scipy.ndimage import map_coordinates
        nodes = s["grid_n"][0]
        f = map_coordinates(s["grid_s"].reshape((nodes,) * dim), [g * (nodes - 1) for g in X], order=1)
    else:
        f = np.exp(s["rbf_coeff"][0] * np.exp(-sum((g - 0.4) ** 2 for g in X) / (2 * s["rbf_width"] ** 2)))
    return (f ** (1 - dim)).sum() / (f ** -dim).sum()


@pytest.mark.parametrize("dim,kind,a,b", [(3, "sphere", 0.25, 60), (3, "sphere", 0.05, 60), (3, "sphere", 0.25, 100),
                                          (2, "sphere", 0.05, 200), (3, "mesh", 30.0, 40), (3, "rbf", 0.04, 4)])
def test_rows_follow_the_mean_cut_off_of_steep_fields(dim, kind, a, b):
    """Rows between the mean cut-off over 1.05 and half of it, as everywhere (fields whose mean a coarse lattice misses by
    more than 1.6)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1906_07925_amd import mpsph as M
    n, k = 2000, 7 if dim == 3 else 10
    spec = _steep(dim, kind, a, b)
    cut = 2.6 * _mean_spacing(spec, dim) * (2 ** k - 1) / 1.05          # kappa tau / 1.05, in cells at s0 = 1
    # a field scale that puts it in the middle of a power of two, and the rows above the limit of the table's size
    s0 = 2.0 ** 3.5 / cut
    R = M.Relaxer(dict(spec, n=n), n=n, s0=s0, cell_log2=k)
    rng = np.random.Generator(np.random.PCG64(1))
    R.load(torch.from_numpy(rng.uniform(size=(n, dim)).astype(np.float32)).cuda(), torch.zeros(n, dtype=torch.int32, device="cuda"))
    R.step(1)
    assert R.search()[2] == 3
    R.close()
