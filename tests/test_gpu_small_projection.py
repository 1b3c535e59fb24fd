"""S X, H X and S^-1 X where P^H X is a small product whose K is split over blocks and whose partials the projector-space kernel
adds, against NumPy: shortest and longest K of that product, one projector to 1024 (64 blocks of 16 rows, no more are
split), the largest and one more for S^-1 (192), atoms of none and of unequal sizes, Gamma point."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1406_4350_amd import chebfd as cf  # noqa: E402


@pytest.mark.parametrize("q,sizes,nb,gamma", [
    (25, [1], 1, False), (25, [13, 0, 7, 0, 45], 17, False), (36, [13] * 5, 64, False), (36, [13] * 5, 197, False),
    (36, [40, 300, 1], 2, False), (38, [512, 500, 12], 1, False), (38, [200, 824, 1], 1, False),
    (38, [64, 1, 63], 40, False), (36, [192], 8, False), (36, [192, 1], 8, False), (40, [13] * 5, 8, True), (49, [1, 0, 130], 33, True)])
def test_operators_of_a_split_projection(q, sizes, nb, gamma):
    r = np.arange(-7, 8)
    g = np.stack(np.meshgrid(r, r, r, indexing="ij"), axis=-1).reshape(-1, 3)
    q2 = (g * g).sum(axis=1)
    if gamma:
        x, y, z = g.T
        keep = (q2 <= q) & ((x > 0) | ((x == 0) & ((y > 0) | ((y == 0) & (z >= 0)))))
    else:
        keep = q2 <= q
    g = np.ascontiguousarray(g[keep]).astype(np.int32)
    npw = g.shape[0]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    nproj = int(off[-1])
    print(f"[case] npw={npw} nproj={nproj} nb={nb} gamma={gamma}", flush=True)
    kin = 0.02 * (g * g).sum(axis=1).astype(np.float64)
    plan = cf.Plan(g, kin, 32, off, True, gamma=gamma)
    plan.set_potential(torch.zeros((32, 32, 32), dtype=torch.float64, device="cuda"))
    rng = np.random.default_rng(npw + nproj)
    P = (rng.standard_normal((nproj, npw)) + 1j * rng.standard_normal((nproj, npw))) / npw ** 0.5
    X = rng.standard_normal((nb, npw)) + 1j * rng.standard_normal((nb, npw))
    if gamma:  # real functions: a real coefficient at G = 0, the others stand for two plane waves by their sqrt(2)
        zero = int(np.nonzero((g == 0).all(axis=1))[0][0])
        P[:, zero], X[:, zero] = P[:, zero].real, X[:, zero].real
    Q = 0.1 + rng.random(nproj)
    blocks = [(lambda d: (d + d.T) / max(s, 1) ** 0.5)(rng.standard_normal((s, s))) for s in sizes]
    D = np.zeros((nproj, nproj))
    for o, b in zip(off, blocks):
        D[o:o + len(b), o:o + len(b)] = b
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    plan.set_projectors(dev(P), dev(Q))
    plan.set_D(dev(np.concatenate([b.reshape(-1) for b in blocks])))
    Xd = dev(X)
    got_s, got_h = plan.apply_S(Xd).cpu().numpy(), plan.apply_H(Xd).cpu().numpy()
    got_i = plan.apply_Sinv(Xd).cpu().numpy()
    plan.close()
    p = X @ P.conj().T  # rows are bands
    p_abs = np.abs(X) @ np.abs(P).T
    if gamma:
        p = p.real
    for got, local, M in ((got_s, np.ones(npw), np.diag(Q)), (got_h, kin, D)):
        want = X * local + (p @ M.T) @ P
        # each of the three sums loses at most (terms + a few) half ulps of the sum of its magnitudes; three real products
        # per complex one double that. NumPy's own sums are bounded likewise. The transforms of a zero potential give zero.
        bound = 4 * (npw + 2 * nproj + 16) * 2.0 ** -53 * (np.abs(X * local) + (p_abs @ np.abs(M).T) @ np.abs(P))
        assert (np.abs(got - want) <= bound).all(), float((np.abs(got - want) / bound).max())
    # S^-1 X = X - P C^-1 P^H X, C = Q^-1 + P^H P: each band to the same count of roundings of the norms in it, times the
    # condition of the inverse
    C = np.diag(1.0 / Q) + P.conj() @ P.T
    if gamma:
        C = C.real
    Ci = np.linalg.inv(C)
    want = X - (p @ Ci.T) @ P
    norm = np.linalg.norm(X, axis=1) + np.linalg.norm(P, 2) * np.linalg.norm(Ci, 2) * np.linalg.norm(p, axis=1)
    bound = 4 * (npw + 2 * nproj + 16) * 2.0 ** -53 * np.linalg.cond(C) * norm
    err = np.linalg.norm(got_i - want, axis=1)
    assert (err <= bound).all(), float((err / bound).max())
