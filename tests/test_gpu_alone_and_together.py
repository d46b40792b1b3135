"""A result's bits do not depend on what else is in the call: pairs of very
different sizes and extents in a batch, the cosine's three sums and the backward's
two sides give what each gives alone, with either cluster rule."""
import numpy as np
import pytest

from paper_2012_03683_amd import synth

from gpu_util import to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(params=[(0, 1.0, 0.5), (1, 0.5, 1.0)], ids=["octree", "chunks"])
def cvo(request):
    import paper_2012_03683_amd as m
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this environment")
    m.load_library()
    base = m.cvo_get_tuning()
    rule, cell, clus = request.param
    m.cvo_set_tuning(cluster_rule=rule, cluster_max=16, cell_factor=cell, cluster_factor=clus)
    yield m
    m.cvo_set_tuning(**base)


@pytest.mark.parametrize("prm", [dict(ell_init=0.1, ell_min=0.1, max_iter=5, fixed_iters=True),
                                 dict(ell_init=0.1, ell_min=0.05, max_iter=120),
                                 dict(ell_init=0.2, ell_min=0.05, max_iter=25, ell_mode=1)],
                         ids=["fixed", "annealed", "adaptive"])
def test_pairs_of_a_batch(cvo, prm):
    # (pairs rebuild their views at different steps; one finds no overlap)
    ps = [synth.rgbd_pair(seed=60, n=20000, m=3001, lazy=True), synth.rgbd_pair(seed=61, n=8000, m=9023, lazy=True),
          synth.rgbd_pair(seed=62, n=2001, m=1500, lazy=True), synth.random_pair(63, 700, 900, synth.rgbd_pair(
              seed=62, n=16, m=16, lazy=True).spec, extent=30.0)]
    dev = [to_dev(p, torch) for p in ps]
    Ts, reps = cvo.cvo_align_batched(dev, ps[0].spec, prm)
    for (X, Z, U, V), T, r in zip(dev, Ts, reps):
        T1, r1, _ = cvo.cvo_align(X, Z, U, V, ps[0].spec, prm)
        assert np.array_equal(T, T1) and r == r1


@pytest.mark.parametrize("n,m", [(20011, 3000), (6000, 20011), (40, 20011)])
def test_sides_and_sums(cvo, n, m):
    p = synth.rgbd_pair(seed=5, n=n, m=m, lazy=True)
    X, Z, U, V = to_dev(p, torch)
    I = np.eye(4)
    both = cvo.cvo_inner_product_backward(X, Z, I, 0.1, 1.0, U, V, p.spec)
    src = cvo.cvo_inner_product_backward(X, Z, I, 0.1, 1.0, U, V, p.spec, need=("x", "u"))
    tgt = cvo.cvo_inner_product_backward(X, Z, I, 0.1, 1.0, U, V, p.spec, need=("z", "v", "ell"))
    assert torch.equal(both["dX"], src["dX"]) and torch.equal(both["dU"], src["dU"])
    assert torch.equal(both["dZ"], tgt["dZ"]) and torch.equal(both["dV"], tgt["dV"])
    assert both["dell"] == tgt["dell"]
    _, fxz, fxx, fzz = cvo.cvo_cosine(X, Z, I, 0.1, U, V, p.spec)
    assert fxz == cvo.cvo_inner_product(X, Z, I, 0.1, U, V, p.spec)[0]
    assert fxx == cvo.cvo_inner_product(X, X, I, 0.1, U, U, p.spec)[0]
    assert fzz == cvo.cvo_inner_product(Z, Z, I, 0.1, V, V, p.spec)[0]
