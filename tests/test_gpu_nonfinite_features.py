"""Features that are not finite reach the derivatives of the pairs they are in and
no others: a point without a neighbour has zero gradients whatever its features."""
import numpy as np
import pytest

from paper_2012_03683_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("spec", [[synth.se_block(3, 0.3)], [synth.se_block(3, 0.3), synth.lin_block(2)]],
                         ids=["se", "se_lin"])
def test_point_without_neighbours(spec, bad):
    import paper_2012_03683_amd as cvo
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this environment")
    D = sum(b["dim"] for b in spec)
    g = torch.Generator(device="cuda").manual_seed(3)
    X, Z = (torch.rand(n, 3, device="cuda", generator=g) for n in (200, 150))
    U, V = (torch.rand(n, D, device="cuda", generator=g) for n in (200, 150))
    want = cvo.cvo_inner_product_backward(X, Z, np.eye(4), 0.1, 1.0, U, V, spec)
    far = torch.full((1, 3), 50.0, device="cuda")
    row = torch.full((1, D), bad, device="cuda")
    X1, U1 = torch.cat([X, far]), torch.cat([U, row])
    Z1, V1 = torch.cat([Z, -far]), torch.cat([V, row])
    r = cvo.cvo_inner_product_backward(X1, Z1, np.eye(4), 0.1, 1.0, U1, V1, spec)
    for k, n in (("dX", 200), ("dZ", 150), ("dU", 200), ("dV", 150)):
        assert torch.equal(r[k][n], torch.zeros_like(r[k][n])), k
        # (another cloud's box orders the sums anew: FP32 results of FP64 sums)
        torch.testing.assert_close(r[k][:n], want[k], rtol=1e-5, atol=1e-6 * float(want[k].abs().max()))


def test_pair_with_a_feature_that_is_not_finite():
    """Its own derivatives are not finite, as the weight times an infinite difference."""
    import paper_2012_03683_amd as cvo
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this environment")
    spec = [synth.se_block(3, 0.3)]
    X = torch.zeros(1, 3, device="cuda")
    U, V = torch.zeros(1, 3, device="cuda"), torch.zeros(1, 3, device="cuda")
    V[0, 1] = float("inf")
    r = cvo.cvo_inner_product_backward(X, X, np.eye(4), 0.1, 1.0, U, V, spec)
    assert torch.isnan(r["dV"][0, 1]) and torch.isnan(r["dU"][0, 1])
