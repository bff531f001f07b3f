"""GPU: what the value and the gradient of one sweep owe to the cotangent."""
import numpy as np
import pytest

from mockgen import random_field

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# gradients of two orders of the same float operations (bars as in test_gpu_bins.py)
TOL = {"f64": 1.1e-11, "f32": 1.9e-5}


def _fields(n, nb, lmax, prec, seed):
    """Two mocks and two cotangents on the GPU."""
    rd = torch.float64 if prec == "f64" else torch.float32
    d = np.stack([random_field(n, seed), random_field(n, seed + 1)])
    lam = np.random.default_rng(seed + 2).standard_normal((2, lmax + 1, nb, nb))
    return torch.as_tensor(d, dtype=rd, device="cuda"), torch.as_tensor(lam, device="cuda")


@pytest.mark.parametrize("basis,nb", [("b3", 1), ("b3", 2), ("b3", 5), ("b3", 20), ("b3", 33), ("b3", 64), ("d4", 6)])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_gamma_value_does_not_depend_on_the_cotangent(prec, basis, nb):
    """The grid-Gamma one sweep contracts the plain fields: zeta is mp3_zeta's, bit for bit, and the fields
    turned into the eigenbasis afterwards give mp3_zeta_backward's gradient."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_15209_amd as mp3
    print("[case] gamma value", prec, basis, nb, flush=True)
    n, lmax = 16, 2
    d, lam = _fields(n, nb, lmax, prec, 810)
    plan = mp3.Plan(n, 160.0, lmax, np.linspace(5.0, 60.0, nb + 1), precision=prec, summation="gamma", basis=basis,
                    batch=2)
    z, g, _ = plan.zeta_value_and_grad(d, lam)
    assert torch.equal(z, plan.zeta(d))
    g2 = plan.zeta_backward(d, lam)[0]
    assert (g - g2).abs().max() <= 2 * TOL[prec] * g2.abs().max()


@pytest.mark.parametrize("form", ["nodal", "gamma"])
@pytest.mark.parametrize("exponent", [-600, 600])
def test_gradient_is_linear_in_the_cotangent(form, exponent):
    """A cotangent times 2^+-600 (its entries' squares leave float64) gives the gradient times the same."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_15209_amd as mp3
    print("[case] scaled cotangent", form, exponent, flush=True)
    n, nb, lmax = 16, 5, 2
    d, lam = _fields(n, nb, lmax, "f64", 820)
    plan = mp3.Plan(n, 160.0, lmax, np.linspace(5.0, 60.0, nb + 1), precision="f64", summation=form, batch=2)
    ref, zref = plan.zeta_backward(d, lam)[0], plan.zeta(d)
    z, g, _ = plan.zeta_value_and_grad(d, lam * 2.0 ** exponent)
    for a in (g, plan.zeta_backward(d, lam * 2.0 ** exponent)[0]):
        assert (a * 2.0 ** -exponent - ref).abs().max() <= 2 * TOL["f64"] * ref.abs().max()
    assert (z - zref).abs().max() <= TOL["f64"] * zref.abs().max()


@pytest.mark.parametrize("form", ["nodal", "gamma"])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_non_finite_cotangent(prec, value, form):
    """One entry off the diagonal that is not finite: no finite gradient of its mock, the other mock's as without
    it, and the value as ever."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_15209_amd as mp3
    print("[case] non-finite cotangent", prec, value, form, flush=True)
    n, nb, lmax = 16, 5, 2
    d, lam = _fields(n, nb, lmax, prec, 830)
    plan = mp3.Plan(n, 160.0, lmax, np.linspace(5.0, 60.0, nb + 1), precision=prec, summation=form, batch=2)
    ref, zref = plan.zeta_backward(d, lam)[0], plan.zeta(d)
    lam[0, 1, 3, 1] = value
    z, g, _ = plan.zeta_value_and_grad(d, lam)
    for a in (g, plan.zeta_backward(d, lam)[0]):
        assert not torch.isfinite(a[0]).any()
        assert (a[1] - ref[1]).abs().max() <= 2 * TOL[prec] * ref[1].abs().max()
    assert (z - zref).abs().max() <= TOL[prec] * zref.abs().max()


@pytest.mark.parametrize("basis,prec,nb", [("b3", "f64", 3), ("b3", "f64", 20), ("b3", "f32", 3), ("b3", "f32", 20),
                                           ("b3", "bf16x3", 20), ("d4", "f64", 3), ("d4", "f64", 20), ("d4", "f32", 3),
                                           ("d4", "f32", 20)])
def test_gamma_task_loop(basis, prec, nb):
    """The grid-Gamma contraction with several tasks to a workgroup (contract_wgs 64: 8 or 4 tasks each at 32^3)
    against one task each, and the gradient beside it, which no knob cuts."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_15209_amd as mp3
    print("[case] gamma task loop", basis, prec, nb, flush=True)
    n, lmax = 32, 1
    tol = TOL["f64" if prec == "f64" else "f32"]
    d, lam = _fields(n, nb, lmax, prec, 840)
    out = []
    for wgs in (64, 4096):
        plan = mp3.Plan(n, 320.0, lmax, np.linspace(5.0, 110.0, nb + 1), precision=prec, summation="gamma",
                        basis=basis, batch=2)
        plan.tune_set("contract_wgs", wgs)
        out.append(plan.zeta_value_and_grad(d, lam)[:2])
    for a, b in zip(*out):
        assert (a - b).abs().max() <= tol * b.abs().max()
