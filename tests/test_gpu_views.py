"""View build at the edges of its tiles: clouds of one point up to a few sort
tiles, both cluster rules, with repeated points (blocks that no octree level
splits), evaluated against the FP64 oracle.  |P| is exact; F and the gradient
are within 1e-5 of the larger of the value and its absolute sum, as everywhere
(FP32 pair terms, FP64 sums)."""
import numpy as np
import pytest

import oracle
from paper_2012_03683_amd import synth

from gpu_util import assert_eval_matches, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cvo():
    import paper_2012_03683_amd as m
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this environment")
    m.load_library()
    base = m.cvo_get_tuning()
    yield m
    m.cvo_set_tuning(**base)


@pytest.mark.parametrize("rule,cmax", [(0, 8), (0, 16), (0, 64), (1, 8), (1, 16), (1, 64)])
@pytest.mark.parametrize("n,m", [(1, 1), (1, 1025), (255, 257), (1024, 1023), (1025, 2049), (4097, 63)])
def test_views_at_tile_edges(cvo, n, m, rule, cmax):
    spec = [synth.se_block(3, 0.3), synth.lin_block(2)]
    p = synth.random_pair(1000 * n + m, n, m, spec, extent=0.5)
    # every third query repeats one point, and every fifth reference another
    p.z[::3] = p.z[0]
    p.x[::5] = p.x[n // 2]
    T = synth.random_motion(np.random.default_rng(n + m), 2.0, 0.03)
    X, Z, U, V = to_dev(p, torch)
    cvo.cvo_set_tuning(cluster_rule=rule, cluster_max=cmax, cell_factor=0.5, cluster_factor=0.5)
    g = cvo.cvo_evaluate(X, Z, T, 0.08, U, V, spec)
    o = oracle.evaluate(p.x, p.u, p.z, p.v, spec, 0.08, T=T)
    assert_eval_matches(g, o, what=f"{n} x {m}, rule {rule}, clusters of {cmax}")


def test_view_of_many_tiles_matches_the_view_of_few(cvo):
    """A batch whose sides exceed the digit tables' tiles takes the large sort;
    its pairs register as they do alone, where the tables are used."""
    ps = [synth.rgbd_pair(seed=60 + k, n=n, m=m, lazy=True) for k, (n, m) in enumerate([(60000, 3001), (50000, 1023),
                                                                                     (47001, 40000)])]
    assert sum(p.x.shape[0] for p in ps) > 128 * 1024 > max(p.x.shape[0] for p in ps)
    prm = dict(ell_init=0.1, ell_min=0.1, max_iter=4, fixed_iters=True)
    dev = [to_dev(p, torch) for p in ps]
    Ts, reps = cvo.cvo_align_batched(dev, ps[0].spec, prm)
    for (X, Z, U, V), T, r in zip(dev, Ts, reps):
        T1, r1, _ = cvo.cvo_align(X, Z, U, V, ps[0].spec, prm)
        assert r["n_pairs"] == r1["n_pairs"] and r["total_pairs"] == r1["total_pairs"]
        # four steps of FP64 arithmetic on sums that differ in their order only
        np.testing.assert_allclose(T, T1, rtol=0, atol=1e-9)
