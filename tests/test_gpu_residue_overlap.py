"""INT8 projector products of bands that hardly overlap a projector, or of projections that hardly overlap a plane wave's
row of P: FP64 keeps the digits of such products, whose terms are far below the product of the norms, and the bands
beside them are not touched. 17 077 plane waves, 832 projectors, 1024 bands; H X = P P^H X (no potential, no kinetic
term, D = 1)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1406_4350_amd import chebfd as cf  # noqa: E402

NPROJ, NB, ODD = 832, 1024, 8


def _plan(P, g):
    plan = cf.Plan(g, np.zeros(g.shape[0]), 64, np.arange(0, NPROJ + 1, 13).astype(np.int32), False)
    plan.set_potential(torch.zeros((64,) * 3, dtype=torch.float64))
    plan.set_projectors(P, None)
    plan.set_D(torch.eye(13, dtype=torch.float64).repeat(NPROJ // 13, 1, 1).reshape(-1))
    return plan


def _randn(gen, *shape):
    return torch.randn(shape, dtype=torch.complex128, device="cuda", generator=gen)


def _check(P, g, smooth, odd, rows):
    """odd bands (on the plane waves `rows`): relative error below 1e-12, some sqrt(17 077) eps = 3e-14 of sums that do
    not cancel; the other bands: the same, and the same bits with and without the odd ones beside them."""
    plan = _plan(P, g)
    X = smooth.clone()
    base = plan.apply_H(X)
    X[:ODD] = odd
    Y = plan.apply_H(X)
    assert torch.equal(Y[ODD:], base[ODD:])
    ref = (X[:2 * ODD] @ P.conj().T) @ P
    err = torch.linalg.vector_norm((Y[:2 * ODD] - ref)[:, rows], dim=1) / torch.linalg.vector_norm(ref[:, rows], dim=1)
    print("largest relative error, odd and smooth bands:", float(err[:ODD].max()), float(err[ODD:].max()), flush=True)
    assert float(err.max()) < 1e-12
    plan.close()


def _sphere():
    r = np.arange(-16, 17)
    g = np.stack(np.meshgrid(r, r, r, indexing="ij"), axis=-1).reshape(-1, 3)
    return np.ascontiguousarray(g[(g * g).sum(axis=1) <= 256]).astype(np.int32)


def test_bands_outside_the_projectors():
    """Projectors that decay to 1e-10 at the edge of the sphere, bands that live there."""
    g = _sphere()
    gen = torch.Generator(device="cuda").manual_seed(11)
    g2 = torch.from_numpy((g * g).sum(1)).to("cuda", torch.float64)
    P = _randn(gen, NPROJ, g.shape[0]) * torch.exp(-23.0 * g2 / 256)
    X = _randn(gen, NB, g.shape[0]) / (1.0 + g2 / 16)
    odd = torch.where(g2 > 230, _randn(gen, ODD, g.shape[0]), torch.zeros((), dtype=torch.complex128, device="cuda"))
    _check(P, g, X, odd, torch.arange(g.shape[0], device="cuda"))


def test_projections_outside_the_rows():
    """Half of the projectors is everywhere of order 1 and equal on plane waves 0 and 1, the other half is of order 1e-10
    on the last 5000 plane waves. The difference of the first two plane waves has projections on the second half only,
    which hardly overlap the rows of those 5000."""
    g = _sphere()
    gen = torch.Generator(device="cuda").manual_seed(12)
    P = _randn(gen, NPROJ, g.shape[0])
    P[::2, 1] = P[::2, 0]
    P[1::2, -5000:] *= 1e-10
    X = _randn(gen, NB, g.shape[0])
    odd = torch.zeros((ODD, g.shape[0]), dtype=torch.complex128, device="cuda")
    odd[:, 0] = 2.0 ** torch.arange(ODD, device="cuda")  # products without rounding: the first half cancels exactly
    odd[:, 1] = -odd[:, 0]
    _check(P, g, X, odd, torch.arange(g.shape[0] - 5000, g.shape[0], device="cuda"))
