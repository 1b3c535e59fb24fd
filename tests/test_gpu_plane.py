"""(K + V) X against numpy's transforms at every box, for spheres on either side of the radius
n / 4 (up to which the plane pass leaves the empty frequency digits out) and for a slab that is narrow in gx but not in
gy, with a sphere whose outermost x-lines hold one column and a slab whose do not."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1406_4350_amd import chebfd as cf  # noqa: E402
from paper_1406_4350_amd import workload as wl  # noqa: E402


@pytest.mark.parametrize("prec", [cf.CHEB_FP64, cf.CHEB_MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("shape", ["quarter", "beyond", "slab"])
@pytest.mark.parametrize("n", [8, 12, 16, 24, 32, 48, 64, 96, 128])
def test_local_part(n, shape, prec):
    """Bound: eps per level and direction, 6 log2 n levels, a factor 6 for the codelets' constants."""
    g = wl.sphere(n // 4 if shape == "quarter" else n // 4 + 1)
    if shape == "slab":
        g = np.ascontiguousarray(g[np.abs(g[:, 0]) <= n // 8])
    print(f"[case] n={n} {shape} prec={prec} npw={g.shape[0]}", flush=True)
    rng = np.random.default_rng(n)
    nb, npw = 3, g.shape[0]
    kin = 0.01 * (g.astype(np.float64) ** 2).sum(axis=1)
    V = rng.normal(size=(n, n, n))
    X = rng.normal(size=(nb, npw)) + 1j * rng.normal(size=(nb, npw))
    plan = cf.Plan(g, kin, n, np.zeros(1, np.int32), False, prec=prec)
    plan.set_potential(torch.from_numpy(V))
    Xd = torch.from_numpy(X).to("cuda", plan.dtype)
    Y = plan.apply_H(Xd).to("cpu", torch.complex128).numpy()
    Xr = Xd.to("cpu", torch.complex128).numpy()
    f = g % n
    for b in range(nb):
        box = np.zeros((n, n, n), dtype=np.complex128)
        box[f[:, 0], f[:, 1], f[:, 2]] = Xr[b]
        ref = np.fft.fftn(np.fft.ifftn(box) * V)[f[:, 0], f[:, 1], f[:, 2]] + kin * Xr[b]
        err = np.linalg.norm(Y[b] - ref) / np.linalg.norm(ref)
        eps = 1.2e-7 if prec == cf.CHEB_MIXED else 2.3e-16
        assert err < 36 * np.log2(n) * eps, (b, err)
    plan.close()
