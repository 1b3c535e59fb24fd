"""Operands that are constant along the contraction: every residue of a modulus is the same, and the int32 accumulators
of the INT8 products are as large as they get. Plane-wave counts on both sides of the longest product taken."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1406_4350_amd import chebfd as cf  # noqa: E402


def _sphere(r2):
    r = np.arange(-40, 41)
    g = np.stack(np.meshgrid(r, r, r, indexing="ij"), axis=-1).reshape(-1, 3)
    return np.ascontiguousarray(g[(g * g).sum(axis=1) <= r2]).astype(np.int32)


@pytest.mark.parametrize("r2,npw", [(1069, 146533), (1081, 148981)])
def test_constant_operands(r2, npw):
    """H X = P D P^H X with P and X constant: every entry is nproj d v^2 npw x. 188566250453174 is, unscaled, an integer
    that the split reduces to 121 modulo 241, so 148 981 squares of it sum to more than 2^31. Tolerance: a sum of equal
    terms carries at most npw eps / 2 in a serial chain, 1.6e-11; the products sum in parts."""
    g = _sphere(r2)
    assert g.shape[0] == npw
    print(f"[case] constant operands npw={npw}", flush=True)
    nproj, nb, v = 832, 512, 188566250453174.0
    plan = cf.Plan(g, np.zeros(npw), 128, np.arange(0, nproj + 1, 13).astype(np.int32), False)
    plan.set_potential(torch.zeros((128,) * 3, dtype=torch.float64))
    plan.set_projectors(torch.full((nproj, npw), v, dtype=torch.complex128, device="cuda"), None)
    plan.set_D(torch.eye(13, dtype=torch.float64).repeat(nproj // 13, 1, 1).reshape(-1) * 2.0 ** -96)
    X = torch.full((nb, npw), v, dtype=torch.complex128, device="cuda")
    X[1::2] *= 2.0 ** 40
    Y = plan.apply_H(X)
    want = nproj * 2.0 ** -96 * v * v * npw * v
    assert float((Y[0::2] / want - 1.0).abs().max()) < 1.6e-11
    assert float((Y[1::2] / (want * 2.0 ** 40) - 1.0).abs().max()) < 1.6e-11
    plan.close()
