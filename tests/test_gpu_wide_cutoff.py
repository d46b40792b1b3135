"""Finite cutoffs of many lengthscales, up to one whose product with the
lengthscale overflows: every pair is in P, so the evaluation is that without a
cutoff (the oracle's).  Clouds stand 40 m from the origin: offsets are taken from
the cluster's centre, so FP32 keeps F and the gradient within 1e-5 of the larger of
the value and its absolute sum at a lengthscale of 2 cm, as everywhere, and F (at
which rounding of offsets by the step of a coarser centre would show) within 1e-6."""
import numpy as np
import pytest

import oracle
from paper_2012_03683_amd import synth

from gpu_util import assert_eval_matches, to_dev

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


@pytest.mark.parametrize("kappa,ell,extent,shift", [
    (1e7, 0.02, 0.05, 40.0), (1e4, 0.02, 0.05, 40.0), (50.0, 0.02, 0.05, 40.0),
    (1.7e308, 1.5, 3.0, 40.0), (1.7e308, 0.02, 0.05, 40.0), (1e300, 1e10, 1.0, 0.0)])
def test_cutoff_beyond_the_clouds(cvo, kappa, ell, extent, shift):
    spec = [synth.lin_block(4)]
    p = synth.random_pair(7, 13, 9, spec, extent=extent, noise=0.2 * extent, angle_deg=0.0, trans=0.0)
    p.x += np.float32(shift)
    p.z += np.float32(shift)
    T = np.eye(4)
    T[:3, 3] = 0.1 * extent
    X, Z, U, V = to_dev(p, torch)
    o = oracle.evaluate(p.x, p.u, p.z, p.v, spec, ell, T=T, kappa=INF)
    assert o["n_pairs"] == 13 * 9
    g = cvo.cvo_evaluate(X, Z, T, ell, U, V, spec, kappa=kappa)
    assert_eval_matches(g, o, what=f"kappa {kappa}, ell {ell}")
    assert abs(g["F"] - o["F"]) <= 1e-6 * o["absF"]
