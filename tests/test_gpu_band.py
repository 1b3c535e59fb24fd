"""The transforms of a band in one launch (boxes up to 16^3): against the three passes, which the plan takes while its
kernel-class timers are on, at every box and several sphere radii, in both precisions, and at the Gamma point; and
the wider spheres that keep the three passes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import matfree  # noqa: E402
from paper_1406_4350_amd import chebfd as cf  # noqa: E402
from paper_1406_4350_amd import workload as wl  # noqa: E402


def _config(n, radius, nb):
    return wl.Config(f"band{n}_{radius}", n, radius, float(max(radius, 2)), "random", 1, 2, "sp", False, nb, 2, 1, 1,
                     140 + n)


@pytest.mark.parametrize("prec", [cf.CHEB_FP64, cf.CHEB_MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("n,radius", [(8, 1), (8, 2), (8, 3), (12, 3), (12, 5), (16, 4), (16, 7), (24, 6)])
def test_one_launch_matches_three_passes_and_oracle(n, radius, prec):
    """The same codelets in the same order: equal up to contraction of the compiler, a few roundings of n^3-point
    sums. Bound: 3 transforms of log2 n levels each way, eps per level."""
    print(f"[case] n={n} R={radius} prec={prec}", flush=True)
    nb = 5
    pb = wl.make_problem(_config(n, radius, nb))
    plan = cf.plan_from_problem(pb, prec)
    X = cf.to_device_block(pb.X0, plan.dtype)
    one = plan.apply_H(X)
    plan.profile_enable(True)
    three = plan.apply_H(X)
    plan.profile_enable(False)
    eps = 1.2e-7 if prec == cf.CHEB_MIXED else 2.3e-16
    tol = 6 * np.log2(n) * eps
    assert float(torch.linalg.vector_norm(one - three) / torch.linalg.vector_norm(three)) < tol
    ref = matfree.Operators.from_problem(pb).apply_H(pb.X0)
    err = np.linalg.norm(cf.to_host_block(one) - ref) / np.linalg.norm(ref)
    assert err < (2e-5 if prec == cf.CHEB_MIXED else 1e-12)
    plan.close()


@pytest.mark.parametrize("nb", [1, 4, 7])
def test_gamma_pairs(nb):
    """Two real bands per transform, an odd last one alone."""
    gp = wl.make_gamma_problem(_config(16, 4, nb))
    plan = cf.plan_from_problem(gp, cf.CHEB_FP64)
    X = torch.empty((nb, gp.npw), dtype=torch.complex128, device="cuda")  # row stride npw for one band too
    X.copy_(torch.from_numpy(np.ascontiguousarray(gp.X0.T)))
    one = plan.apply_H(X)
    plan.profile_enable(True)
    three = plan.apply_H(X)
    plan.profile_enable(False)
    assert float(torch.linalg.vector_norm(one - three) / torch.linalg.vector_norm(three)) < 24 * 2.3e-16
    plan.close()
