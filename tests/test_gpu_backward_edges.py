"""Backward at the edges of its blocks of 64 queries, one and both sides,
against the FP64 oracle.  Pair terms are FP32 (position gradients sum them in
FP32 over at most 80 terms, then FP64): 1e-5 relative, plus a tenth of that of
the largest element for cancelling sums, as in the other backward tests."""
import numpy as np
import pytest

import oracle
from paper_2012_03683_amd import synth

from gpu_util import to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SPECS = {
    "geometric": [],
    "se5_lin19": [synth.se_block(5, 0.2), synth.lin_block(19)],
    "two_lin": [synth.se_block(2, 0.4), synth.lin_block(3), synth.lin_block(4)],
}


@pytest.fixture(scope="module")
def cvo():
    import paper_2012_03683_amd as m
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this environment")
    m.load_library()
    return m


def _cmp(g, o, name):
    g = g.double().cpu().numpy()
    scale = np.max(np.abs(o)) if o.size else 0.0
    assert np.all(np.abs(g - o) <= 1e-5 * np.abs(o) + 1e-6 * scale + 1e-12), name


@pytest.mark.parametrize("name", list(SPECS))
@pytest.mark.parametrize("n,m", [(1, 1), (63, 65), (64, 64), (129, 1), (65, 700)])
def test_backward_at_block_edges(cvo, n, m, name):
    spec = SPECS[name]
    p = synth.random_pair(n + 7 * m, n, m, spec, extent=0.3)
    T = synth.random_motion(np.random.default_rng(n), 1.5, 0.02)
    X, Z, U, V = to_dev(p, torch)
    o = oracle.backward(p.x, p.u, p.z, p.v, spec, 0.12, T=T)
    both = cvo.cvo_inner_product_backward(X, Z, T, 0.12, 1.0, U, V, spec)
    src = cvo.cvo_inner_product_backward(X, Z, T, 0.12, 1.0, U, V, spec, need=("x", "u"))
    tgt = cvo.cvo_inner_product_backward(X, Z, T, 0.12, 1.0, U, V, spec, need=("z", "v", "ell"))
    for key, ref, one in (("dX", "dx", src), ("dZ", "dz", tgt), ("dU", "du", src), ("dV", "dv", tgt)):
        if both[key] is None:
            continue
        _cmp(both[key], o[ref], key)
        assert torch.equal(both[key], one[key]), key  # a side alone is the same sums
    assert both["dell"] == pytest.approx(o["dell"], rel=1e-5, abs=1e-12)
    assert both["dell"] == tgt["dell"] and src["dell"] is None
