"""The counting order of the particles by cell key: the cell table and the order inside a cell.

The table must be the lower bound of every cell in the sorted keys, and the order inside a cell must
not depend on the arrival order of the counting atomics: two contexts of the same input stay
identical bit for bit.
"""
import numpy as np
import pytest

from paper_1906_07925_amd import workloads as W

pytestmark = pytest.mark.gpu

# (dim, particles, cell_log2): a table smaller than one scan tile (4096 cells), exactly one, one
# particle more, the last table whose blocks sum their predecessors themselves (16 tiles) and the
# first beyond, crowded cells (one cell per axis and half), and a table of more than 8 cells per
# particle (radix order)
CASES = [(2, 1, -1), (2, 255, 4), (2, 1024, 4), (2, 1025, 4), (2, 16384, 7), (2, 16385, 8), (3, 3000, 1), (3, 20011, -1),
         (2, 40, 9)]


@pytest.mark.parametrize("dim,n,k", CASES)
def test_cell_table_and_order(dim, n, k):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1906_07925_amd import mpsph as M
    rng = np.random.Generator(np.random.PCG64(7 * n + dim))
    spec = (W.unit_square if dim == 2 else W.unit_cube)(n)
    x = rng.uniform(0.0, 1.0, size=(n, dim)).astype(np.float32)
    x[: n // 4] = x[n // 2: n // 2 + n // 4]           # coincident pairs share a cell
    col = rng.integers(0, 4, size=n).astype(np.int32)
    out = []
    for _ in range(2):
        R = M.Relaxer(spec, n=n, s0=0.5 * float(n) ** (-1.0 / dim), cell_log2=k)
        for _ in range(2):                             # a second load starts from clean counts
            R.load(torch.from_numpy(x).cuda(), torch.from_numpy(col).cuda())
            R.step(3)
        keys, cstart, _ = R.cells()
        keys = keys.cpu().numpy().astype(np.uint32).astype(np.int64)
        cstart = cstart.cpu().numpy().astype(np.int64)
        assert np.array_equal(cstart, np.searchsorted(np.sort(keys), np.arange(cstart.size)))
        out.append((R.store(), R.metrics()))
        R.close()
    (xa, ta), ma = out[0]
    (xb, tb), mb = out[1]
    assert torch.equal(xa, xb) and torch.equal(ta, tb) and ma == mb


# tables of one tile, ordered by one block: a lone particle, a wave's edge, the most particles of the
# block and one more (two launches again)
@pytest.mark.parametrize("dim,n,k", [(2, 1, 3), (2, 65, 3), (2, 1023, 3), (2, 4095, 3), (2, 4096, 3), (2, 4097, 3), (3, 4096, 2)])
def test_one_block_order(dim, n, k):
    test_cell_table_and_order(dim, n, k)


# tables of 32, 64 and 128 tiles: the last that one launch scans and the first with a launch for the sums
@pytest.mark.parametrize("dim,n,k", [(2, 60000, 9), (2, 60000, 10), (2, 60000, 11)])
def test_scan_of_many_tiles(dim, n, k):
    test_cell_table_and_order(dim, n, k)
