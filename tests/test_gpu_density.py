"""dL/dV(r) of the adjoint, the band densities of a whole filter, against the FP64 oracle adjoint at every box up to 64^3:
spheres up to the radius n / 4 and wider ones, and more band chunks than bands, one band per chunk, and chunks of two of
which the last stay empty."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import grad, matfree  # noqa: E402
from paper_1406_4350_amd import chebfd as cf  # noqa: E402
from paper_1406_4350_amd import workload as wl  # noqa: E402


def _rel(a, b):
    return float(np.linalg.norm(np.ravel(a - b)) / max(np.linalg.norm(np.ravel(b)), 1e-300))


@pytest.mark.parametrize("n,radius,nb", [(8, 2, 6), (12, 3, 6), (12, 4, 6), (16, 4, 8), (24, 7, 8), (32, 8, 8),
                                         (32, 9, 33), (48, 9, 23), (64, 8, 16), (64, 17, 20)])
def test_band_densities(n, radius, nb):
    """Bounds: 1e-8 (FP64) and 1e-3 (mixed) of the norm, those of the other adjoint tests."""
    cfg = wl.SMALL["tiny_paw"].replace(name=f"den{n}_{radius}", n=n, radius=radius, nb=nb, seed_index=500 + n)
    pb = wl.make_problem(cfg)
    ops = matfree.Operators.from_problem(pb)
    lp = matfree.lanczos_upper_bound(ops, pb.v0, 10)[0]
    lm = float(np.max(matfree.rayleigh_quotients(ops, pb.X0)))
    c, r, m, nk = 0.5 * (lp + lm), 0.5 * (lp - lm), 2, 4
    w = np.random.default_rng(11).uniform(0, 1, nk)
    print(f"[case] n={n} R={radius} npw={pb.npw} nb={nb}", flush=True)
    _, _, _, dV, _ = grad.filter_rr_grad(ops, pb.X0, m, c, r, w, pb.D)
    for prec, dtype, tol in [(cf.CHEB_FP64, torch.complex128, 1e-8), (cf.CHEB_MIXED, torch.complex64, 1e-3)]:
        plan = cf.plan_from_problem(pb, prec)
        _, _, gV, _ = plan.filter_rr_backward(cf.to_device_block(pb.X0, dtype), m, c, r, w, 2)
        e = _rel(gV.cpu().numpy(), dV)
        print(f"[check] prec={prec} dV {e:.2e}", flush=True)
        assert e < tol
        plan.close()


@pytest.mark.parametrize("nb", [6, 16, 17, 83])
def test_block_gradient(nb):
    """dL/dD with band counts on either side of the 16 slices that share a block entry. Bounds as above."""
    cfg = wl.SMALL["tiny_paw"].replace(name=f"dd{nb}", n=16, radius=4, nb=nb, seed_index=600 + nb)
    pb = wl.make_problem(cfg)
    ops = matfree.Operators.from_problem(pb)
    lp = matfree.lanczos_upper_bound(ops, pb.v0, 10)[0]
    lm = float(np.max(matfree.rayleigh_quotients(ops, pb.X0)))
    c, r, m, nk = 0.5 * (lp + lm), 0.5 * (lp - lm), 2, 4
    w = np.random.default_rng(13).uniform(0, 1, nk)
    _, _, _, _, dD = grad.filter_rr_grad(ops, pb.X0, m, c, r, w, pb.D)
    print(f"[case] nb={nb} entries={dD.size}", flush=True)
    plan = cf.plan_from_problem(pb, cf.CHEB_FP64)
    _, _, _, gD = plan.filter_rr_backward(cf.to_device_block(pb.X0, torch.complex128), m, c, r, w, 2)
    assert _rel(gD.cpu().numpy(), dD) < 1e-8
    plan.close()
