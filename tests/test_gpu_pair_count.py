"""|P| is exact where the pairs of one cluster of queries pass 2^31: without a
cutoff every query has every reference point."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_pairs_of_a_cluster_pass_32_bits():
    import paper_2012_03683_amd as cvo
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this environment")
    g = torch.Generator(device="cuda").manual_seed(5)
    n, m = 34_000_000, 70
    X = torch.rand(n, 3, device="cuda", generator=g)
    Z = torch.rand(m, 3, device="cuda", generator=g)
    base = cvo.cvo_get_tuning()
    try:
        # one cluster of 64 queries, and one of 6
        cvo.cvo_set_tuning(cluster_rule=1, cluster_max=64, cluster_factor=2.0)
        r = cvo.cvo_evaluate(X, Z, np.eye(4), 1.0, spec=[], kappa=float("inf"))
    finally:
        cvo.cvo_set_tuning(**base)
    assert 64 * n > 2 ** 31
    assert r["n_pairs"] == n * m
