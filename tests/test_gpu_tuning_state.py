"""The tuning a handle reports is all that decides the shape of its views: a handle
whose fields were changed and set back evaluates with the bits of a fresh one,
and each state -- fresh, an octree shape set, set back -- matches the oracle (|P|
exact, F, the gradient and the derivatives within 1e-5, as everywhere)."""
import numpy as np
import pytest

import oracle
from paper_2012_03683_amd import synth

from gpu_util import assert_eval_matches, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture()
def cvo():
    """The module with a fresh handle for the device, and its own one afterwards."""
    import paper_2012_03683_amd as m
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this environment")
    m.load_library()
    dev = torch.cuda.current_device()
    old = m._handles.pop(dev, None)
    yield m
    fresh = m._handles.pop(dev, None)
    if old is not None:
        m._handles[dev] = old
    if fresh is not None:
        m.load_library().cvo_destroy(fresh)


def _calls(cvo, d, p, T, ell):
    X, Z, U, V = d
    e = cvo.cvo_evaluate(X, Z, T, ell, U, V, p.spec)
    c = cvo.cvo_cosine(X, Z, T, ell, U, V, p.spec)
    b = cvo.cvo_inner_product_backward(X, Z, T, ell, 1.0, U, V, p.spec)
    a = cvo.cvo_align(X, Z, U, V, p.spec, dict(ell_init=ell, ell_min=ell, max_iter=3, fixed_iters=True), T)[0]
    return {**{k: np.asarray(v) for k, v in e.items()}, "cos": np.asarray(c), "T": a,
            **{k: np.asarray(v if k == "dell" else v.cpu()) for k, v in b.items()}}


def _same(a, b):
    return all(np.array_equal(a[k], b[k]) for k in a)


def test_shape_follows_the_fields(cvo):
    p = synth.stereo_pair(seed=31, n=3001, m=2500, lazy=True)
    d, T, ell = to_dev(p, torch), np.eye(4), 0.4
    o = oracle.evaluate(p.x, p.u, p.z, p.v, p.spec, ell, T=T)
    ob = oracle.backward(p.x, p.u, p.z, p.v, p.spec, ell, T=T)
    start = cvo.cvo_get_tuning()
    fresh = _calls(cvo, d, p, T, ell)
    cvo.cvo_set_tuning(**start)
    assert _same(fresh, _calls(cvo, d, p, T, ell))  # asked for, as stated
    cvo.cvo_set_tuning(cluster_rule=0, cell_factor=1.0, cluster_factor=0.5)
    octree = _calls(cvo, d, p, T, ell)
    assert not _same(fresh, octree)
    cvo.cvo_set_tuning(**start)
    assert cvo.cvo_get_tuning() == start
    back = _calls(cvo, d, p, T, ell)
    assert _same(fresh, back)
    for g in (fresh, octree, back):
        assert_eval_matches(g, o)
        for k, r in (("dX", "dx"), ("dZ", "dz"), ("dU", "du"), ("dV", "dv")):
            scale = np.abs(ob[r]).max()
            assert np.all(np.abs(g[k] - ob[r]) <= 1e-5 * np.abs(ob[r]) + 1e-6 * scale), k
        assert g["dell"] == pytest.approx(ob["dell"], rel=1e-5)
        assert g["cos"][1] == pytest.approx(o["F"], rel=1e-5)
