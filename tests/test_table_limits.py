"""Sizes of the search table (no GPU): the workspace of a batch holds the sum of its domains' tables, whatever their
cells and rows, up to the stated limit of 2^28 cells."""
import pytest

from paper_1906_07925_amd import mpsph as M
from paper_1906_07925_amd import workloads as W


# the most cells a batch may have: 2^28 in domains of 2^16 and 2^15 cells, with rows of half a cell
@pytest.mark.parametrize("dim,k,ndom", [(2, 8, 4096), (3, 5, 4096)])
def test_tables_of_a_batch_add_up(dim, k, ndom):
    spec = dict((W.unit_square if dim == 2 else W.unit_cube)(1), n=1, s0=1e-4)   # a cut-off far below a cell
    one = M.workspace_bytes(spec, 1, cell_log2=k)
    table = 2 ** (k + (dim - 1) * (k + 1))                  # rows of half a cell
    assert one > 2 * 4 * table                              # the table and its counts
    assert M.batch_workspace_bytes([spec] * ndom, [1] * ndom, cell_log2=k) > 2 * 4 * table * ndom
