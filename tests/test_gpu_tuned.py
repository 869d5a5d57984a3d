"""What the autotuner returns is what it timed: another context configured with the returned cell exponent and
lanes has the same cells, rows and candidates and takes the same steps, bit for bit."""
import numpy as np
import pytest

from paper_1906_07925_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,scale", [("levelset", 1.0), ("levelset", 0.25), ("cube_inclusion_2m", 0.02), ("annulus_262k", 0.2),
                                        ("square_4k", 1.0), ("rbf_cube_1m", 0.05)])
def test_configured_like_the_tuned_context(name, scale):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1906_07925_amd import mpsph as M
    if name == "levelset":
        cfg = dict(spec=W.levelset_ball(int(scale * (1 << 20))), seed=5, init="random", n_colours=4)
    else:
        cfg = W.config(name, scale=scale)
    x, col, typ = W.make_state(cfg)
    n = x.shape[0]
    spec = dict(cfg["spec"], n=n)
    state = [torch.from_numpy(a).cuda() for a in (x.astype(np.float32), col, typ)]
    A = M.Relaxer(spec, n=n)
    s0 = spec.get("s0")
    k, lanes = A.autotune(*state, probe_steps=2, warm_steps=2)
    B = M.Relaxer(spec, n=n, s0=s0)
    B.configure(k, lanes)
    B.load(*state)
    for R in (A, B):
        R.step(3)
    sa, sb = A.search(), B.search()
    assert sa[2:] == sb[2:], (k, lanes)
    assert torch.equal(sa[0], sb[0]) and torch.equal(sa[1], sb[1])
    assert A.metrics() == B.metrics() and torch.equal(A.store()[0], B.store()[0])
    A.close()
    B.close()
