"""One launch per kernel for both dimension groups of a batch: every domain ends bit for bit where a
context of its own takes it, with domains of one block and of a partial last block, a periodic one among
them, a shorter cut-off, and with the step closed in the viscous pass (at most 128 blocks per domain) or
by a launch of its own."""
import numpy as np
import pytest

from paper_1906_07925_amd import workloads as W

pytestmark = pytest.mark.gpu


def _domain(dim, n, periodic, kappa, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    if periodic:
        spec = dict(dim=dim, geometry="periodic", lo=(0.0,) * dim, hi=(1.0,) * dim, field="uniform")
    else:
        spec = (W.unit_square if dim == 2 else W.unit_cube)(n)
    x = rng.uniform(0.0, 1.0, size=(n, dim)).astype(np.float32)
    return dict(spec, n=n, kappa=kappa), x, rng.integers(0, 3, size=n).astype(np.int32)


@pytest.mark.parametrize("n2,n3", [((63, 1000), (31, 900)), ((64, 8200), (33, 1500)), ((1,), (4200,))])
@pytest.mark.parametrize("periodic", [0, 2, 3])
@pytest.mark.parametrize("kappa", [2.0, 1.6])
def test_mixed_launch_keeps_each_domain(n2, n3, periodic, kappa):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1906_07925_amd import mpsph as M
    doms = [_domain(2, n, periodic == 2 and n > 500, kappa if k == 0 else 2.0, 10 + k) for k, n in enumerate(n2)]
    doms += [_domain(3, n, periodic == 3 and n > 500, 2.0, 20 + k) for k, n in enumerate(n3)]
    doms = doms[1:] + doms[:1]

    def run(ds):
        R = M.Relaxer([d[0] for d in ds], n=[len(d[1]) for d in ds])
        R.load(torch.from_numpy(np.concatenate([d[1].reshape(-1) for d in ds])).cuda(),
               torch.from_numpy(np.concatenate([d[2] for d in ds])).cuda())
        R.step(4)
        out = R.split(R.store()[0].cpu().numpy()), R.domain_metrics()
        R.close()
        return out
    xs, ms = run(doms)
    for k, d in enumerate(doms):
        (xk,), (mk,) = run([d])
        assert np.array_equal(np.asarray(xs[k]).reshape(-1), np.asarray(xk).reshape(-1)), k
        for key in ("pairs", "interface_pairs", "candidates", "dt1", "dt2"):
            if key in mk:
                assert ms[k][key] == mk[key], (k, key)
