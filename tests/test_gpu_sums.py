"""GPU: the length of a workgroup's sums does not reach the value.  A constant field c has
zeta_0[b1][b2] = c^3 for every pair of shell bins (q = 0 alone, where the window is one), and every product of
the contraction is the same number, so that rounding errors of a running sum add up instead of cancelling.

Bar: 64 additions of one pencil and 11 operations on the way to them (window, three factors, scale), u each:
75 x 2^-24 = 4.5e-6 in float32, 75 x 2^-53 = 8.4e-15 in float64, whatever the number of pencils."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nb,lmax,batch,group", [(64, 2, 12, 1, 0), (64, 2, 12, 1, 1), (64, 12, 8, 1, 0),
                                                   (64, 20, 6, 1, 0), (64, 20, 2, 1, 1), (64, 24, 4, 1, 0),
                                                   (64, 24, 2, 1, 1), (64, 40, 4, 1, 0), (128, 12, 8, 16, 0)])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_constant_field(prec, n, nb, lmax, batch, group):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_15209_amd as mp3
    print("[case] constant field", prec, n, nb, lmax, batch, group, flush=True)
    tol = 75 * 2.0 ** (-53 if prec == "f64" else -24)
    plan = mp3.Plan(n, float(n), lmax, np.linspace(0.1 * n, 0.3 * n, nb + 1), precision=prec, batch=batch)
    plan.tune_set("item_group", group)
    lam = torch.eye(nb, dtype=torch.float64, device="cuda").repeat(batch, lmax + 1, 1, 1)
    for c in (0.7, 1.3):
        d = torch.full((batch, n, n, n), c, dtype=plan.real_dtype, device="cuda")
        c3 = float(d[0, 0, 0, 0]) ** 3
        for z in (plan.zeta(d), plan.zeta_value_and_grad(d, lam)[0]):
            assert np.abs(z[:, 0].cpu().numpy() / c3 - 1).max() <= tol
