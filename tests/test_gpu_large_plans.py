"""Plans that do not fit: one that needs more output slots than there can be ends
in an error before anything is written by it, and evaluations that fit one by
one but not together (the cosine's three sums, the backward's two sides) are
taken one by one, with the bits they have alone."""
import numpy as np
import pytest

from paper_2012_03683_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
INF = float("inf")


@pytest.fixture(scope="module")
def cvo():
    import paper_2012_03683_amd as m
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this environment")
    m.load_library()
    return m


def _cloud(n, D, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.rand(n, 3, device="cuda", generator=g),
            torch.rand(n, D, device="cuda", generator=g) if D else None)


def test_too_many_slots_is_an_error(cvo):
    X, _ = _cloud(1_500_000, 0, 1)
    I = np.eye(4)
    for call in (lambda: cvo.cvo_inner_product(X, X, I, 0.1, spec=[], kappa=INF),
                 lambda: cvo.cvo_cosine(X, X, I, 0.1, spec=[], kappa=INF),
                 lambda: cvo.cvo_inner_product_backward(X, X, I, 0.1, spec=[], kappa=INF)):
        with pytest.raises(Exception, match="output slots"):
            call()
    # the handle goes on working
    F, pairs = cvo.cvo_inner_product(X[:1000], X[:1000], I, 0.1, spec=[], kappa=INF)
    assert pairs == 1000 * 1000 and F > 1000.0


def test_cosine_one_by_one(cvo):
    spec = [synth.se_block(5, 0.2)]
    X, U = _cloud(120_000, 5, 2)
    Z, V = _cloud(118_001, 5, 3)
    I = np.eye(4)
    c, fxz, fxx, fzz = cvo.cvo_cosine(X, Z, I, 0.1, U, V, spec, kappa=INF)
    for f, (A, B, P, Q) in ((fxz, (X, Z, U, V)), (fxx, (X, X, U, U)), (fzz, (Z, Z, V, V))):
        F, pairs = cvo.cvo_inner_product(A, B, I, 0.1, P, Q, spec, kappa=INF)
        assert F == f and pairs == A.shape[0] * B.shape[0]
    assert c == pytest.approx(fxz / np.sqrt(fxx * fzz), rel=1e-15)


def test_backward_one_by_one(cvo):
    spec = [synth.se_block(5, 0.2), synth.lin_block(19)]
    X, U = _cloud(100_000, 24, 4)
    Z, V = _cloud(90_001, 24, 5)
    I = np.eye(4)
    both = cvo.cvo_inner_product_backward(X, Z, I, 0.1, 1.0, U, V, spec, kappa=INF)
    src = cvo.cvo_inner_product_backward(X, Z, I, 0.1, 1.0, U, V, spec, kappa=INF, need=("x", "u"))
    tgt = cvo.cvo_inner_product_backward(X, Z, I, 0.1, 1.0, U, V, spec, kappa=INF, need=("z", "v", "ell"))
    assert torch.equal(both["dX"], src["dX"]) and torch.equal(both["dU"], src["dU"])
    assert torch.equal(both["dZ"], tgt["dZ"]) and torch.equal(both["dV"], tgt["dV"])
    assert both["dell"] == tgt["dell"]
    # F does not change when both clouds move alike
    net = both["dX"].double().sum(0) + both["dZ"].double().sum(0)
    assert torch.all(net.abs() <= 1e-6 * both["dX"].double().abs().sum(0))
