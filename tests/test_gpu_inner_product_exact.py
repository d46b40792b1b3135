"""The inner product's pair terms are FP64 where the features are LIN columns alone,
whose signed weights may cancel: its exponential is within 1.9e-9, so F is within
2.5e-9 of its terms' absolute sum of F in 64 bits.  Terms rounded to FP32 leave about
1e-7 of the absolute sum at these few pairs."""
import numpy as np
import pytest

from paper_2012_03683_amd import synth

from gpu_util import to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cvo():
    import paper_2012_03683_amd as m
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this environment")
    m.load_library()
    return m


def _pair(n, m, spec, seed):
    p = synth.random_pair(seed, n, m, spec, extent=0.3)
    rng = np.random.default_rng(seed)
    p.u, p.v = (rng.normal(size=a.shape).astype(np.float32) for a in (p.u, p.v))
    return p, synth.random_motion(rng, 1.5, 0.02)


@pytest.mark.parametrize("lin", [1, 4, 19, 32, 64])
@pytest.mark.parametrize("n,m", [(1, 1), (9, 13), (65, 40), (301, 200)])
def test_inner_product_keeps_64_bits(cvo, n, m, lin):
    spec = [synth.lin_block(lin)]
    p, T = _pair(n, m, spec, 1000 * lin + n)
    X, Z, U, V = to_dev(p, torch)
    F, pairs = cvo.cvo_inner_product(X, Z, T, 0.12, U, V, spec)
    x, z, u, v = (a.astype(np.float64) for a in (p.x, p.z, p.u, p.v))
    s = ((x[None] - (z @ T[:3, :3].T + T[:3, 3])[:, None]) ** 2).sum(-1)
    w = np.exp(-0.5 * s / 0.12 ** 2) * (s <= 0.36 ** 2)
    assert pairs == np.count_nonzero(w)
    assert abs(F - (w * (v @ u.T)).sum()) <= 2.5e-9 * (w * (np.abs(v) @ np.abs(u).T)).sum()
