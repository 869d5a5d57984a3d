"""Size fields whose largest spacing reaches far beyond the cells: the separations keep their 32-bit precision
whatever the bound of the field over the box.  Domains whose separations leave the range of the
fixed-point coordinates load their neighbours' cells as well; those of few cells never do.  Steps and
gradients against the oracle."""
import math

import numpy as np
import pytest

from oracle import grad as G
from oracle import oracle as O
from paper_1906_07925_amd import workloads as W
from tests import parity_util as PU

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return torch


def _uniform_ball(rng, n, dim, c, r):
    u = rng.normal(size=(n, dim))
    return c + r * rng.uniform(size=(n, 1)) ** (1.0 / dim) * u / np.linalg.norm(u, axis=1)[:, None]


def _labels(rng, n, types=(0, 0, 0, 1)):
    return rng.integers(0, 4, size=n).astype(np.int32), rng.choice(types, size=n).astype(np.int32)


def _levelset(n, outside):
    """Uniform spacing inside a ball, `outside` times that on the mesh nodes no particle can see."""
    spec = W.levelset_ball(n)
    m = spec["grid_n"][0]
    ax = np.linspace(0.0, 1.0, m) - 0.5
    r = np.sqrt(ax[:, None, None] ** 2 + ax[None, :, None] ** 2 + ax[None, None, :] ** 2).reshape(-1)
    spec["grid_s"] = np.where(r < 0.4 + 2.0 * math.sqrt(3.0) / (m - 1), 1.0, outside)
    return spec, 0.4 * (4.0 / 3.0 * math.pi / n) ** (1.0 / 3.0)


def _errors(spec, s0, x, col, typ, k, lanes):
    """Relative errors of one step's pair sums against the oracle, in norms over the particles.  The viscous sum
    goes with the time step squared, whose error is one particle's; it is taken per unit of that."""
    _, _, _, r = PU.oracle_step(spec, s0, x, col, typ)
    m, g = PU.gpu_run(spec, s0, x, col, typ, cell_log2=k, lanes=lanes)
    assert abs(m["pairs"] - r["pairs"]) <= r["band_pairs"]
    return {"rho": PU.rel(g["rho"], r["rho"]), "a": PU.rel(g["a"], r["a"]),
            "at": PU.rel(g["at"] / m["dt1"] ** 2, r["at"] / r["dt1"] ** 2)}


@pytest.mark.parametrize("k,lanes", [(-1, None), (4, 2), (6, 8), (7, 4)])   # few cells (the grid bounds separations), many
def test_mesh_spacing_outside_the_region(torch_cuda, k, lanes):
    """No particle sees the outer nodes: only the order of the sums may change with them, so the errors, norms over
    3000 particles of rounding errors of one size, stay what they are without them (half as much again allowed)."""
    n = 3000
    rng = np.random.Generator(np.random.PCG64(5))
    x = _uniform_ball(rng, n, 3, 0.5, 0.399).astype(np.float32)
    col, typ = _labels(rng, n, (0,))
    ref = None
    for outside in (1.0, 1e2, 1e3, 1e6, 1e9):
        e = _errors(*_levelset(n, outside), x, col, typ, k, lanes)
        ref = ref or e
        assert all(e[f] <= 1.5 * ref[f] for f in e), (outside, e, ref)


def _rbf(dim, n, peak):
    """An RBF field that rises to exp(peak) in a corner away from the particles."""
    spec = W.rbf_cube(n, n_rbf=3, width=0.1, coeff=np.array([peak, 0.1, -0.1]), s0=0.5 * n ** (-1.0 / dim))
    spec.update(dim=dim, lo=(0.0,) * dim, hi=(1.0,) * dim,
                rbf_centre=np.array([[0.0, 0.0, 0.0], [0.7, 0.7, 0.7], [0.9, 0.6, 0.8]])[:, :dim].copy())
    return spec


@pytest.mark.parametrize("dim,k,lanes", [(2, -1, None), (2, 7, 2), (2, 9, 8), (3, -1, None), (3, 6, 4), (3, 7, 2)])
@pytest.mark.parametrize("peak", [4.0, 7.0])
def test_rbf_field_of_wide_range(torch_cuda, dim, k, lanes, peak):
    n = 2500
    rng = np.random.Generator(np.random.PCG64(8))
    x = rng.uniform(0.5, 1.0, size=(n, dim)).astype(np.float32)
    spec = _rbf(dim, n, peak)
    PU.check_single_step(spec, spec["s0"], x, *_labels(rng, n), cell_log2=k, lanes=lanes)


@pytest.mark.parametrize("dim,k,n", [(2, 7, 700), (3, 6, 700), (3, 7, 600)])
def test_gradient_of_a_wide_field(torch_cuda, dim, k, n):
    torch = torch_cuda
    from paper_1906_07925_amd import mpsph as M
    rng = np.random.Generator(np.random.PCG64(9))
    spec = _rbf(dim, n, 7.0)
    side = math.ceil(n ** (1.0 / dim))
    x = np.stack(np.meshgrid(*[(np.arange(side) + 0.5) / side] * dim, indexing="ij"), -1).reshape(-1, dim)
    x = 0.5 + 0.5 * np.clip(x[rng.permutation(len(x))[:n]] + rng.uniform(-0.2, 0.2, size=(n, dim)) / side, 0.0, 1.0)
    x = x.astype(np.float32)
    col, typ = rng.integers(0, 5, size=n).astype(np.int32), np.zeros(n, np.int32)
    pr = G.Problem(spec, spec["s0"], col, typ)
    L0, gc0, gx0, _, _, _ = G.run(pr, x.astype(np.float64), spec["rbf_coeff"], 2, 1.0, want_x0_grad=True)
    R = M.Relaxer(spec, n=n, cell_log2=k)
    R.load(torch.from_numpy(x).cuda(), torch.from_numpy(col).cuda(), torch.from_numpy(typ).cuda())
    L, gc, gx = R.grad(2, 2, 1.0, n_rbf=3, want_pos=True)
    R.close()
    gx = gx.cpu().numpy().astype(np.float64)
    assert abs(L - L0) <= 1e-5 * abs(L0)
    assert np.linalg.norm(gc - gc0) <= 2e-3 * np.linalg.norm(gc0)
    assert np.linalg.norm(gx - gx0) <= 2e-3 * np.linalg.norm(gx0)


def _graded_square(n, ratio, rng):
    spec = dict(W.unit_square(n), field="sphere_distance", fcentre=(0.5, 0.5), fb=0.25,
                fa=(ratio - 1.0) / (math.sqrt(0.5) - 0.25))
    x = rng.uniform(0.0, 1.0, size=(n, 2))
    m = 3 * n // 4   # most of them around the fine circle, as the target density has it
    u = rng.normal(size=(m, 2))
    x[:m] = 0.5 + (0.25 + 0.02 * rng.normal(size=(m, 1))) * u / np.linalg.norm(u, axis=1)[:, None]
    return spec, np.clip(x, 0.0, 1.0).astype(np.float32)


@pytest.mark.parametrize("ratio", [12.0, 30.0, 100.0, 200.0])
@pytest.mark.parametrize("k,lanes", [(-1, None), (6, 2), (9, 8)])
def test_strongly_graded_square(torch_cuda, ratio, k, lanes):
    """At the standard bounds up to 1:30.  Beyond, the spacing's own rounding (FP32, 1.2e-5 at 1:100) leaves no room
    for bounds per particle; norms keep theirs."""
    n = 6000
    rng = np.random.Generator(np.random.PCG64(int(ratio)))
    spec, x = _graded_square(n, ratio, rng)
    s0 = O.OracleParams(dict(spec, n=n)).s0
    col, typ = _labels(rng, n, (0,))
    if ratio <= 30.0:
        PU.check_single_step(spec, s0, x, col, typ, cell_log2=k, lanes=lanes)
    else:
        assert max(_errors(spec, s0, x, col, typ, k, lanes).values()) <= 1e-5


# separations beyond the coordinates' range (2^7 and 2^8 cells), half a period of 64 cells within it
@pytest.mark.parametrize("dim,k,lanes", [(2, 6, 4), (2, 7, 2), (2, 8, 8), (3, 7, 4)])
def test_graded_periodic_box(torch_cuda, dim, k, lanes):
    n = 1500
    rng = np.random.Generator(np.random.PCG64(dim + k))
    spec = dict(dim=dim, geometry="periodic", lo=(0.0,) * dim, hi=(1.0,) * dim, field="sphere_distance",
                fcentre=(0.5,) * dim, fb=0.25, fa=6.0 if dim == 2 else 3.0, n=n)
    x = rng.uniform(0.0, 1.0, size=(n, dim)).astype(np.float32)
    PU.check_single_step(spec, 0.04 if dim == 2 else 0.06, x, *_labels(rng, n, (0,)), cell_log2=k, lanes=lanes)


@pytest.mark.parametrize("variant", ["default", "persistent", "tile"])
@pytest.mark.parametrize("n2", [700, 40000])   # the step closed in the viscous pass, and by a launch of its own
def test_batch_of_wide_and_narrow_domains(torch_cuda, variant, n2):
    """Every domain ends bit for bit where a context of its own takes it."""
    torch = torch_cuda
    from paper_1906_07925_amd import mpsph as M
    rng = np.random.Generator(np.random.PCG64(4))
    a, xa = _graded_square(4000, 100.0, rng)
    c, s0c = _levelset(2000, 1e6)
    doms = [(a, 4e-3, xa), (W.unit_square(n2), n2 ** -0.5, rng.uniform(size=(n2, 2))),
            (c, s0c, _uniform_ball(rng, 2000, 3, 0.5, 0.399)), (W.unit_cube(1100), 0.1, rng.uniform(size=(1100, 3)))]
    col = [rng.integers(0, 3, size=len(d[2])).astype(np.int32) for d in doms]

    def run(sel, v):
        R = M.Relaxer([doms[i][0] for i in sel], n=[len(doms[i][2]) for i in sel], s0=[doms[i][1] for i in sel], cell_log2=6)
        R.set_pair_variant(v)
        R.load(torch.from_numpy(np.concatenate([doms[i][2].astype(np.float32).reshape(-1) for i in sel])).cuda(),
               torch.from_numpy(np.concatenate([col[i] for i in sel])).cuda())
        R.step(3)
        out = R.split(R.store()[0].cpu().numpy()), R.domain_metrics()
        R.close()
        return out
    xs, ms = run(range(4), variant)
    for i in range(4):
        (x1,), (m1,) = run([i], "default")
        assert np.array_equal(np.asarray(xs[i]).reshape(-1), np.asarray(x1).reshape(-1)), i
        for key in ("pairs", "interface_pairs", "candidates", "dt1", "dt2"):
            assert ms[i][key] == m1[key], (i, key)


def test_coefficients_that_widen_the_field(torch_cuda):
    """New coefficients may take a context to the other separations and back: captured steps follow, and
    the exports of the step before still hold."""
    torch = torch_cuda
    from paper_1906_07925_amd import mpsph as M
    n = 2500
    rng = np.random.Generator(np.random.PCG64(6))
    x = torch.from_numpy(rng.uniform(0.5, 1.0, size=(n, 3)).astype(np.float32)).cuda()
    col = torch.from_numpy(rng.integers(0, 4, size=n).astype(np.int32)).cuda()
    flat, steep = np.array([0.0, 0.1, -0.1]), np.array([7.0, 0.1, -0.1])

    def relaxer():
        return M.Relaxer(dict(_rbf(3, n, 0.0), rbf_coeff=flat), n=n, cell_log2=6)

    def eager(coeff):
        R = relaxer()
        R.set_field_coeff(coeff)
        R.load(x, col)
        R.step(2)
        out = R.store()[0]
        R.close()
        return out
    R = relaxer()
    for coeff in (flat, steep, flat):
        R.set_field_coeff(coeff)
        for _ in range(2):
            R.load(x, col)
            R.step_graph(2)
            assert torch.equal(R.store()[0], eager(coeff))
    def key():
        i, j = R.pairs()
        return torch.sort(i.long() * n + j.long()).values
    before = key()
    R.set_field_coeff(steep)
    assert torch.equal(before, key())
    R.close()
