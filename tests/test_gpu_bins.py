"""GPU: values at the bin counts where the contractions change form -- one and two 16-bin matrix blocks,
4x4 blocks at 17..20 bins, the vector ALUs beyond (float64 from 17, float32 from 33 bins), one or two bins
per gather lane -- on grids whose items share a launch, against the oracle; the one sweep's and the two
calls' gradients against each other.

Bars: float64 1.1e-11 (1e5 terms x 2^-53); float32 1.9e-5 (20 operations x 2^-24 x 16, the largest sum of
interpolation weights); gradients of the two ways agree to twice that."""
import functools

import numpy as np
import pytest

from mockgen import lognormal_catalogue
from oracle import basis as B
from oracle import estimator as E
from tests._common import assert_zeta_close

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {"f64": 1.1e-11, "f32": 1.9e-5}
LMAX = 2


@functools.lru_cache(maxsize=None)
def _case(n, nb, form):
    box = 10.0 * n
    edges = np.linspace(0.1 * box, 0.35 * box, nb + 1)
    pos, w = lognormal_catalogue(n, box, 1500, 0.05 * box, 601, 602, 603, (0.5, 1.5))
    op = E.Plan(n, box, LMAX, edges)
    if form == "particle":
        return box, edges, pos, w, E.zeta_particle(op, pos, w)
    delta = B.density_contrast(B.deposit(pos, w, n, box), float(np.sum(w.astype(np.float64))))
    return box, edges, pos, w, E.zeta_nodal(op, delta)


@pytest.mark.parametrize("form,n,nb", [("nodal", 16, 1), ("nodal", 16, 16), ("nodal", 16, 17), ("nodal", 16, 32),
                                       ("nodal", 16, 33), ("nodal", 16, 50), ("nodal", 32, 15), ("nodal", 32, 20),
                                       ("particle", 16, 1), ("particle", 16, 2), ("particle", 16, 3),
                                       ("particle", 16, 20), ("particle", 16, 33)])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_bin_counts(prec, form, n, nb):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_15209_amd as mp3
    print("[case] bin counts", prec, form, n, nb, flush=True)
    box, edges, pos, w, ref = _case(n, nb, form)
    plan = mp3.Plan(n, box, LMAX, edges, precision=prec, summation=form)
    pt, wt = torch.as_tensor(pos, device="cuda"), torch.as_tensor(w, device="cuda")
    delta = plan.deposit(pt, wt)
    cat = (pt, wt) if form == "particle" else ()
    lam = torch.as_tensor(np.random.default_rng(604).standard_normal((1, LMAX + 1, nb, nb)), device="cuda")
    assert_zeta_close(plan.zeta(delta, *cat).cpu().numpy()[0], ref, TOL[prec])
    z, g, dw = plan.zeta_value_and_grad(delta, lam, pt, wt)
    assert_zeta_close(z.cpu().numpy()[0], ref, TOL[prec])
    g2, dw2 = plan.zeta_backward(delta, lam, pt, wt)
    for a, b in ((g, g2), (dw, dw2)):
        a, b = a.double().cpu().numpy(), b.double().cpu().numpy()
        assert np.abs(a - b).max() <= 2 * TOL[prec] * np.abs(b).max()


@pytest.mark.parametrize("form,lmax,nb", [("nodal", 1, 3), ("nodal", 2, 16), ("nodal", 3, 20), ("gamma", 1, 3),
                                          ("gamma", 2, 5), ("gamma", 3, 2)])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_paired_multipoles(prec, form, lmax, nb):
    """The m = 0 fields of two multipoles in one transform (one (l, m) per launch, so that the nodal form
    pairs too): value and gradient of mocks with cotangents of their own against the oracle."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_15209_amd as mp3
    from mockgen import random_field
    from oracle import adjoint as A
    from tests._common import assert_grad_close
    print("[case] paired multipoles", prec, form, lmax, nb, flush=True)
    n, box = 16, 160.0
    edges = np.linspace(16.0, 56.0, nb + 1)
    delta = np.stack([random_field(n, 611), random_field(n, 612)]).astype(np.float32).astype(np.float64)
    lam = np.random.default_rng(613).standard_normal((2, lmax + 1, nb, nb))
    plan = mp3.Plan(n, box, lmax, edges, precision=prec, summation=form, batch=2)
    plan.tune_set("item_group", 1)
    d = torch.as_tensor(delta, dtype=torch.float64 if prec == "f64" else torch.float32, device="cuda")
    lt = torch.as_tensor(lam, device="cuda")
    z0 = plan.zeta(d).cpu().numpy()
    z, g, _ = (t if t is None else t.cpu().numpy() for t in plan.zeta_value_and_grad(d, lt))
    g2 = plan.zeta_backward(d, lt)[0].cpu().numpy()
    op = E.Plan(n, box, lmax, edges)
    for j in range(2):
        ref = E.zeta_nodal(op, delta[j]) if form == "nodal" else E.zeta_gamma_quadrature(op, delta[j])
        gref = (A.zeta_nodal_grad if form == "nodal" else A.zeta_gamma_grad)(op, delta[j], lam[j])
        assert_zeta_close(z0[j], ref, TOL[prec])
        assert_zeta_close(z[j], ref, TOL[prec])
        assert_grad_close(g[j], gref, TOL[prec], "one sweep")
        assert_grad_close(g2[j], gref, TOL[prec], "backward")


@pytest.mark.parametrize("lmax,nb", [(1, 3), (2, 16), (3, 20)])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_paired_multipoles_particle(prec, lmax, nb):
    """The same in the particle form (float64 beyond 16 bins stays unpaired): value, dJ/ddelta and dJ/dw at
    the particle gradient's bars (1e-10 float64, 1e-4 float32)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_15209_amd as mp3
    from oracle import adjoint as A
    from tests._common import assert_grad_close
    print("[case] paired multipoles, particle form", prec, lmax, nb, flush=True)
    n, box = 16, 160.0
    tol = {"f64": 1e-10, "f32": 1e-4}[prec]
    edges = np.linspace(16.0, 56.0, nb + 1)
    pos, w = lognormal_catalogue(n, box, 900, 8.0, 621, 622, 623, (0.5, 1.5))
    lam = np.random.default_rng(624).standard_normal((lmax + 1, nb, nb))
    plan = mp3.Plan(n, box, lmax, edges, precision=prec, summation="particle")
    pt, wt = torch.as_tensor(pos, device="cuda"), torch.as_tensor(w, device="cuda")
    delta = plan.deposit(pt, wt)
    lt = torch.as_tensor(lam[None], device="cuda")
    z, g, dw = plan.zeta_value_and_grad(delta, lt, pt, wt)
    g2, dw2 = plan.zeta_backward(delta, lt, pt, wt)
    op = E.Plan(n, box, lmax, edges)
    ref = E.zeta_particle(op, pos, w)
    gref, wref = A.zeta_particle_grad(op, pos, w, lam)
    for zz in (plan.zeta(delta, pt, wt), z):
        assert_zeta_close(zz.cpu().numpy()[0], ref, tol)
    for a, b in ((g, gref), (g2, gref)):
        assert_grad_close(a.cpu().numpy()[0], b, tol, "dJ/ddelta")
    for a in (dw, dw2):
        assert_grad_close(a.cpu().numpy(), wref, tol, "dJ/dw")


def test_paired_multipoles_of_unlike_size():
    """float32 pairs where the two fields differ most: a field smooth on three cells, bins from r = 0, l <= 6 (the
    innermost bin's zeta falls by about a hundred from l to l + 1).  Every multipole by its own norm within the
    float32 bar, and within four times the error of the unpaired items (plus 4 x 2^-24, one field's rounding)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_15209_amd as mp3
    print("[case] pairs of unlike size", flush=True)
    n, lmax, nb = 32, 6, 6
    f = np.fft.fftfreq(n) * 2 * np.pi
    k2 = f[:, None, None] ** 2 + f[None, :, None] ** 2 + f[None, None, :] ** 2
    x = np.fft.fftn(np.random.default_rng(631).standard_normal((4, n, n, n)), axes=(1, 2, 3)) * np.exp(-4.5 * k2)
    x = np.fft.ifftn(x, axes=(1, 2, 3)).real
    d = torch.as_tensor(x / x.std(), dtype=torch.float32, device="cuda")

    def zeta(prec, group):
        plan = mp3.Plan(n, 320.0, lmax, np.linspace(0.0, 80.0, nb + 1), precision=prec, batch=4)
        plan.tune_set("item_group", group)
        return plan.zeta(d.double() if prec == "f64" else d).cpu().numpy()

    ref = zeta("f64", 1024)
    err = {g: np.sqrt(((zeta("f32", g) - ref) ** 2).sum((0, 2, 3)) / (ref ** 2).sum((0, 2, 3))) for g in (1, 1024)}
    assert (err[1] <= TOL["f32"]).all(), err
    assert (err[1] <= 4 * err[1024] + 4 * 2.0 ** -24).all(), err
