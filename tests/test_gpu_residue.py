"""The FP64 projector products that run on the INT8 matrix cores (large plans: residues modulo 15 coprime numbers,
exact integer products): operators against the same products in plain FP64, at widths on and off the edges of the 256
tiles and of the 1024-column pieces, and operands that are left to the FP64 matrix cores."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1406_4350_amd import chebfd as cf  # noqa: E402
from paper_1406_4350_amd import workload as wl  # noqa: E402

# 17 077 plane waves and 832 projectors: both products of 300 bands and more take the INT8 matrix cores
CFG = wl.Config("residue64", 64, 16, 16.0, "sc", 4, 64, "2s2p1d", True, 8, 4, 1, 4, 131)


@pytest.fixture(scope="module")
def problem():
    pb = wl.make_problem(CFG)
    plan = cf.plan_from_problem(pb, cf.CHEB_FP64)
    P = torch.from_numpy(np.ascontiguousarray(pb.P.T)).cuda()
    yield pb, plan, P, torch.from_numpy(pb.Q).cuda()
    plan.close()


def _block(npw, nb, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn((nb, npw), dtype=torch.complex128, device="cuda", generator=g)


def _s(X, P, Q):
    return X + ((X @ P.conj().T) * Q) @ P


@pytest.mark.parametrize("nb", [300, 511, 513, 1024, 1025])
def test_operators_match_plain_fp64(problem, nb):
    """S X and S^-1 S X = X. Either side sums 17 077 and 832 terms in FP64: at most 17 077 eps, about 4e-12, of the
    products' magnitude, in practice a few sqrt(17 077) eps = 3e-14."""
    pb, plan, P, Q = problem
    print(f"[case] residue64 nb={nb}", flush=True)
    X = _block(pb.npw, nb, nb)
    Y = plan.apply_S(X)
    ref = _s(X, P, Q)
    rel = torch.linalg.vector_norm(Y - ref, dim=1) / torch.linalg.vector_norm(ref, dim=1)
    assert float(rel.max()) < 1e-13
    Z = plan.apply_Sinv(Y)
    rel = torch.linalg.vector_norm(Z - X, dim=1) / torch.linalg.vector_norm(X, dim=1)
    assert float(rel.max()) < 1e-12


def test_padded_rows_and_scaled_bands(problem):
    """Rows of a wider tensor (leading dimension above npw), bands from 1e-100 to 1e100, a zero band, and a band whose
    one entry dominates: each band is scaled by itself, a power of two scales its result exactly."""
    pb, plan, P, Q = problem
    nb = 320
    wide = torch.zeros((nb, pb.npw + 37), dtype=torch.complex128, device="cuda")
    X = wide[:, :pb.npw]
    X.copy_(_block(pb.npw, nb, 5))
    base = plan.apply_S(X.contiguous())
    X[1] *= 2.0 ** 332
    X[2] *= 2.0 ** -332
    X[3] = 0.0
    X[4, 7] = 1e12
    Y = torch.empty_like(wide)[:, :pb.npw]
    plan.apply_S(X, Y)
    assert torch.equal(Y[0], base[0]) and torch.equal(Y[5:], base[5:])
    assert torch.equal(Y[1], base[1] * 2.0 ** 332) and torch.equal(Y[2], base[2] * 2.0 ** -332)
    assert float(Y[3].abs().max()) == 0.0
    ref = _s(X[4:5].contiguous(), P, Q)
    assert float(torch.linalg.vector_norm(Y[4:5] - ref) / torch.linalg.vector_norm(ref)) < 1e-13


@pytest.mark.parametrize("value", [float("nan"), float("inf"), 1e200])
def test_unfit_operand_takes_the_fp64_product(problem, value):
    """A band with a NaN, an Inf or entries beyond the integers' range sends the block through the FP64 product: the
    other bands keep FP64 accuracy and the band itself its NaN, or its finite value."""
    pb, plan, P, Q = problem
    X = _block(pb.npw, 320, 9)
    X[17, 11] = complex(value, 0.0)
    Y = plan.apply_S(X)
    keep = [i for i in range(320) if i != 17]
    ref = _s(X[keep], P, Q)
    rel = torch.linalg.vector_norm(Y[keep] - ref, dim=1) / torch.linalg.vector_norm(ref, dim=1)
    assert float(rel.max()) < 1e-13
    if value == 1e200:
        r = _s(X[17:18] * 1e-200, P, Q)
        assert float(torch.linalg.vector_norm(Y[17] * 1e-200 - r) / torch.linalg.vector_norm(r)) < 1e-13
    else:
        assert not bool(torch.isfinite(torch.view_as_real(Y[17])).all())


def test_filter_takes_both_products(problem):
    """The filter on a block wide enough for the INT8 products against the same bands in a narrow block, which the FP64
    products take: both within FP64 rounding amplified by the recurrence."""
    pb, plan, P, Q = problem
    X = _block(pb.npw, 512, 3)
    lp = plan.upper_bound(X[0], 10)
    c, r = 0.55 * lp, 0.45 * lp
    narrow = X[100:116].clone()
    plan.filter(X, 6, c, r)
    plan.filter(narrow, 6, c, r)
    rel = torch.linalg.vector_norm(X[100:116] - narrow, dim=1) / torch.linalg.vector_norm(narrow, dim=1)
    assert float(rel.max()) < 1e-11
