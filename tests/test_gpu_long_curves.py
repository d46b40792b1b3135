"""Clouds whose extent is 10^4 to 10^7 times their cutoff (one point far off), so
that the query order's keys take all their bits and the sort all its passes, with
either cluster rule, alone and with the bits of 40 pairs above them.  |P| is
exact; F and the gradient are within 1e-5 of the larger of the value and its
absolute sum, as everywhere."""
import numpy as np
import pytest

import oracle
from paper_2012_03683_amd import synth

from gpu_util import assert_eval_matches, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
SPEC = [synth.se_block(3, 0.3)]


@pytest.fixture(scope="module")
def cvo():
    import paper_2012_03683_amd as m
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this environment")
    m.load_library()
    base = m.cvo_get_tuning()
    yield m
    m.cvo_set_tuning(**base)


def _pair(seed, n, m, far):
    p = synth.random_pair(seed, n, m, SPEC, extent=1.0)
    p.x[n // 2] = far
    p.z[m // 3] = -far
    return p


@pytest.mark.parametrize("rule", [0, 1], ids=["octree", "chunks"])
@pytest.mark.parametrize("far", [1e3, 1e4, 1e5, 1e6])
def test_one_point_far_off(cvo, rule, far):
    p = _pair(int(far), 1500, 1300, far)
    X, Z, U, V = to_dev(p, torch)
    T = synth.random_motion(np.random.default_rng(3), 1.0, 0.02)
    cvo.cvo_set_tuning(cluster_rule=rule, cluster_max=16, cell_factor=1.0, cluster_factor=0.5)
    g = cvo.cvo_evaluate(X, Z, T, 0.1, U, V, SPEC)
    o = oracle.evaluate(p.x, p.u, p.z, p.v, SPEC, 0.1, T=T)
    assert_eval_matches(g, o, what=f"far {far}, rule {rule}")


@pytest.mark.parametrize("rule", [0, 1], ids=["octree", "chunks"])
def test_forty_pairs_with_a_point_far_off(cvo, rule):
    cvo.cvo_set_tuning(cluster_rule=rule, cluster_max=16, cell_factor=1.0, cluster_factor=0.5)
    ps = [_pair(100 + k, 300 + 7 * k, 280 + 11 * k, 10.0 ** (3 + k % 3)) for k in range(40)]
    dev = [to_dev(p, torch) for p in ps]
    prm = dict(ell_init=0.2, ell_min=0.2, max_iter=3, fixed_iters=True)
    Ts, reps = cvo.cvo_align_batched(dev, SPEC, prm)
    for (X, Z, U, V), T, r in zip(dev, Ts, reps):
        T1, r1, _ = cvo.cvo_align(X, Z, U, V, SPEC, prm)
        assert r["n_pairs"] == r1["n_pairs"] and r["total_pairs"] == r1["total_pairs"]
        # three steps of FP64 arithmetic on sums that differ in their order at most
        np.testing.assert_allclose(T, T1, rtol=0, atol=1e-9)
