"""The piece plan at the edges of its rule: the candidates of all clusters put
the floor of a piece's candidates at its smallest, in between and at its
largest, with clusters that have none and clusters cut into many pieces,
against the FP64 oracle.  |P| is exact; F and the gradient are within 1e-5 of
the larger of the value and its absolute sum, as everywhere."""
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


# every query sees every reference point (a cloud of extent 0.5, cutoff > 1), so
# clusters x references candidates: floors of 128 (twice), 320 and 512
@pytest.mark.parametrize("n,m,cmax", [(129, 255, 8), (1999, 2050, 8), (4001, 2050, 8), (9001, 2050, 8)])
@pytest.mark.parametrize("far", [0, 64])
def test_piece_floor_edges(cvo, n, m, cmax, far):
    spec = [synth.se_block(3, 0.3)]
    p = synth.random_pair(n + m, n, m, spec, extent=0.5)
    p.z[:far] += 100.0  # clusters without candidates
    T = synth.random_motion(np.random.default_rng(n), 2.0, 0.03)
    X, Z, U, V = to_dev(p, torch)
    cvo.cvo_set_tuning(cluster_rule=1, cluster_max=cmax, cell_factor=0.5, cluster_factor=1.0)
    g = cvo.cvo_evaluate(X, Z, T, 0.6, U, V, spec)
    o = oracle.evaluate(p.x, p.u, p.z, p.v, spec, 0.6, T=T)
    assert_eval_matches(g, o, what=f"{n} x {m}, clusters of {cmax}, {far} far")
