"""GPU: the particle form's adjoint sources where the scatter's stages change shape -- column blocks of
8 bins, passes of 24 bins, stages of 256 (float32) or 128 (float64) particles that overflow in one dense
cell, tiles without particles -- against the oracle's gradient at the particle form's bars
(1e-10 float64, 1e-4 float32)."""
import functools

import numpy as np
import pytest

from oracle import adjoint as A
from oracle import estimator as E
from tests._common import assert_grad_close

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-10, "f32": 1e-4}
N, BOX, LMAX = 16, 160.0, 1


def _catalogue(kind):
    """"dense": 700 particles in one cell and a few elsewhere; "sparse": 5 particles on the periodic seam."""
    rng = np.random.default_rng(71)
    if kind == "sparse":
        pos = np.array([[0.0, 0.0, 0.0], [159.9, 0.1, 80.0], [159.99, 159.99, 159.99], [40.0, 80.0, 120.0],
                        [79.9, 80.1, 79.9]])
    else:
        pos = np.concatenate([75.0 + 9.0 * rng.random((700, 3)), rng.random((60, 3)) * BOX])
    pos = np.minimum(pos.astype(np.float32), np.float32(159.999))
    return pos, rng.uniform(0.5, 1.5, len(pos)).astype(np.float32)


@functools.lru_cache(maxsize=None)
def _reference(kind, nb):
    pos, w = _catalogue(kind)
    edges = np.linspace(15.0, 56.0, nb + 1)
    lam = np.random.default_rng(72 + nb).standard_normal((LMAX + 1, nb, nb))
    return pos, w, edges, lam, A.zeta_particle_grad(E.Plan(N, BOX, LMAX, edges), pos, w, lam)


@pytest.mark.parametrize("kind,nb", [("dense", 1), ("dense", 8), ("dense", 9), ("dense", 17), ("dense", 24),
                                     ("dense", 25), ("sparse", 3), ("sparse", 20)])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_scatter_stages(prec, kind, nb):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_15209_amd as mp3
    print("[case] scatter stages", prec, kind, nb, flush=True)
    pos, w, edges, lam, (gref, wref) = _reference(kind, nb)
    plan = mp3.Plan(N, BOX, LMAX, edges, precision=prec, summation="particle")
    pt, wt = torch.as_tensor(pos, device="cuda"), torch.as_tensor(w, device="cuda")
    delta = plan.deposit(pt, wt)
    lt = torch.as_tensor(lam[None], device="cuda")
    for g, dw in (plan.zeta_backward(delta, lt, pt, wt), plan.zeta_value_and_grad(delta, lt, pt, wt)[1:]):
        assert_grad_close(g.cpu().numpy()[0], gref, TOL[prec], "dJ/ddelta")
        assert_grad_close(dw.cpu().numpy(), wref, TOL[prec], "dJ/dw")


@pytest.mark.parametrize("nb", [3, 9, 20])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_workgroups_without_particles(prec, nb):
    """Mocks of 20000, 90 and 1 particles in one call: the gather's twenty workgroups per mock leave two and
    nineteen without a particle in the small ones.  Each mock against a call of its own."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_15209_amd as mp3
    print("[case] workgroups without particles", prec, nb, flush=True)
    rng = np.random.default_rng(73)
    off = np.cumsum([0, 20000, 90, 1])
    pos = torch.as_tensor((rng.random((off[-1], 3)) * 159.9).astype(np.float32), device="cuda")
    w = torch.as_tensor(rng.uniform(0.5, 1.5, off[-1]).astype(np.float32), device="cuda")
    lam = torch.as_tensor(rng.standard_normal((3, LMAX + 1, nb, nb)), device="cuda")
    edges = np.linspace(15.0, 56.0, nb + 1)
    plan = mp3.Plan(N, BOX, LMAX, edges, precision=prec, summation="particle", batch=3)
    z, g, dw = plan.zeta_value_and_grad(plan.deposit(pos, w, off), lam, pos, w, off)
    one = mp3.Plan(N, BOX, LMAX, edges, precision=prec, summation="particle")
    for j in range(3):
        p, u = pos[off[j]:off[j + 1]].contiguous(), w[off[j]:off[j + 1]].contiguous()
        z1, g1, dw1 = one.zeta_value_and_grad(one.deposit(p, u), lam[j:j + 1].contiguous(), p, u)
        pairs = [(z[j], z1[0]), (g[j], g1[0])]
        if j < 2:   # one particle's weight does not change its contrast: dJ/dw is zero, a difference of large terms
            pairs.append((dw[off[j]:off[j + 1]], dw1))
        for got, ref in pairs:
            assert (got - ref).abs().max() <= TOL[prec] * ref.abs().max()
