"""Pieces beyond the linear cost buckets of the dispatch order (a large piece_work:
a cluster's whole neighbourhood in one piece), against the FP64 oracle.  |P| is
exact; F and the gradient are within 1e-5 of the larger of the value and its
absolute sum, as everywhere."""
import numpy as np
import pytest

import oracle
from paper_2012_03683_amd import synth

from gpu_util import assert_eval_matches, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("work", [1 << 16, 1 << 20, 1 << 24])
@pytest.mark.parametrize("n,m", [(600, 700), (6000, 1500)])
def test_heavy_pieces(n, m, work):
    import paper_2012_03683_amd as cvo
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this environment")
    spec = [synth.se_block(3, 0.3)]
    p = synth.random_pair(n, n, m, spec, extent=1.0)
    T = synth.random_motion(np.random.default_rng(n), 2.0, 0.03)
    X, Z, U, V = to_dev(p, torch)
    base = cvo.cvo_get_tuning()
    try:
        cvo.cvo_set_tuning(piece_work=work, cluster_max=64, cluster_rule=1, cluster_factor=2.0)
        g = cvo.cvo_evaluate(X, Z, T, 0.3, U, V, spec)
    finally:
        cvo.cvo_set_tuning(**base)
    assert_eval_matches(g, oracle.evaluate(p.x, p.u, p.z, p.v, spec, 0.3, T=T), what=f"{n} x {m}, work {work}")
