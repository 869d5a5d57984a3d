"""The search table and order that the pair passes work on, against numpy: cells from the positions, the table
as the lower bound of every cell, the particles of a cell in load order."""
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
