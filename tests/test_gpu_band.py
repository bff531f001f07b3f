"""GPU: the grid summation with the connection coefficients at the edges of its kernels' bin groups
(4 bins per adjoint workgroup, 16 and 32 per contraction, pairs of chunks above), value and gradient against the oracle's shift-stencil form.

Bars: float64 sums of at most 1e5 terms, 1e5 x 2^-53 = 1.1e-11; float32 fields carry 2^-24 per
operation over the ~20 operations between delta and a product and the filters' weights sum to at
most 4 in magnitude per axis, 20 x 2^-24 x 16 = 1.9e-5."""
import functools

import numpy as np
import pytest

from mockgen import random_field
from oracle import adjoint as A
from oracle import estimator as E
from tests._common import assert_grad_close, assert_zeta_close

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {"f64": 1.1e-11, "f32": 1.9e-5}


@functools.lru_cache(maxsize=None)
def _reference(basis, n, nb, lmax):
    """Field (values that float32 holds), cotangent, and the oracle's zeta and dJ/ddelta."""
    box = 10.0 * n
    edges = np.linspace(0.1 * box, 0.35 * box, nb + 1)
    delta = random_field(n, 400 + n + nb).astype(np.float32).astype(np.float64)
    lam = np.random.default_rng(500 + nb).standard_normal((lmax + 1, nb, nb))
    op = E.Plan(n, box, lmax, edges, basis=basis)
    return box, edges, delta, lam, E.zeta_gamma(op, delta), A.zeta_gamma_grad(op, delta, lam)


@pytest.mark.parametrize("basis", ["b3", "d4"])
@pytest.mark.parametrize("n,nb", [(16, 1), (16, 4), (16, 5), (16, 16), (16, 20), (16, 33), (32, 6)])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_gamma_bin_groups(prec, basis, n, nb):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_15209_amd as mp3
    print("[case] gamma bin groups", prec, basis, n, nb, flush=True)
    lmax = 1 if nb <= 5 else 0
    box, edges, delta, lam, zref, gref = _reference(basis, n, nb, lmax)
    plan = mp3.Plan(n, box, lmax, edges, precision=prec, summation="gamma", basis=basis, batch=2)
    rd = torch.float64 if prec == "f64" else torch.float32
    # the second mock: half the field and the negated cotangent (zeta is cubic, the gradient quadratic)
    d = torch.as_tensor(np.stack([delta, 0.5 * delta]), dtype=rd, device="cuda")
    lt = torch.as_tensor(np.stack([lam, -lam]), device="cuda")
    z = plan.zeta(d).cpu().numpy()
    z1, g1, _ = (t if t is None else t.cpu().numpy() for t in plan.zeta_value_and_grad(d, lt))
    g2 = plan.zeta_backward(d, lt)[0].cpu().numpy()
    for j, (a, b) in enumerate([(1.0, 1.0), (0.125, -0.25)]):
        assert_zeta_close(z[j], a * zref, TOL[prec])
        assert_zeta_close(z1[j], a * zref, TOL[prec])
        assert_grad_close(g1[j], b * gref, TOL[prec], "one sweep")
        assert_grad_close(g2[j], b * gref, TOL[prec], "backward")
