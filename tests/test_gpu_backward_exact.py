"""The backward's pair terms are FP64 (no SE columns, whose features are rounded
to FP32 when they are scaled): its exponential is within 1.9e-9, so every sum is
within 2.5e-9 of its terms' absolute sum of the same sum in 64 bits, and a
gradient returned in FP32 adds half a unit of its last place (2^-24).  Terms
rounded to FP32 leave about 1e-7 of the absolute sum at these few pairs, which
signed LIN weights let dF/dell keep."""
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


def _sums(p, T, ell):
    """(value, absolute sum of its terms) of every derivative, in 64 bits."""
    x, z = p.x.astype(np.float64), p.z.astype(np.float64)
    zp = z @ T[:3, :3].T + T[:3, 3]
    d = x[None] - zp[:, None]
    s = (d ** 2).sum(-1)
    bare = np.exp(-0.5 * s / ell ** 2) * (s <= (3.0 * ell) ** 2)
    w = bare
    out = {}
    if p.D:
        u, v = p.u.astype(np.float64), p.v.astype(np.float64)
        w = bare * (v @ u.T)
        out["dU"] = bare.T @ v, bare.T @ np.abs(v)
        out["dV"] = bare @ u, bare @ np.abs(u)
    a = bare * (np.abs(v) @ np.abs(u).T) if p.D else bare
    out["dell"] = (w * s).sum() / ell ** 3, (a * s).sum() / ell ** 3
    wd, ad = w[..., None] * d, a[..., None] * np.abs(d)
    R = T[:3, :3]
    out["dX"] = -wd.sum(0) / ell ** 2, ad.sum(0) / ell ** 2
    out["dZ"] = wd.sum(1) @ R / ell ** 2, ad.sum(1) @ np.abs(R) / ell ** 2
    return out


@pytest.mark.parametrize("lin", [0, 3, 19, 32, 64])
@pytest.mark.parametrize("n,m", [(9, 13), (65, 40), (301, 200)])
def test_backward_keeps_64_bits(cvo, n, m, lin):
    spec = [synth.lin_block(lin)] if lin else []
    p = synth.random_pair(1000 * lin + n, n, m, spec, extent=0.3)
    if lin:
        rng = np.random.default_rng(n + lin)
        p.u, p.v = (rng.normal(size=a.shape).astype(np.float32) for a in (p.u, p.v))
    T = synth.random_motion(np.random.default_rng(n), 1.5, 0.02)
    X, Z, U, V = to_dev(p, torch)
    g = cvo.cvo_inner_product_backward(X, Z, T, 0.12, 1.0, U, V, spec)
    for key, (ref, mag) in _sums(p, T, 0.12).items():
        val = np.asarray(g[key] if key == "dell" else g[key].double().cpu().numpy())
        half = 0.0 if key == "dell" else 2.0 ** -24
        assert np.all(np.abs(val - ref) <= 2.5e-9 * mag + half * np.abs(ref) + 1e-38), key
