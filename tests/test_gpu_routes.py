"""The kernels that projector products take (cheb_profile_routes), and the special cases of the INT8 route on blocks that
are shown to take it: padded rows, scaled and zero bands, bands and projectors that are not fit for the integers."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1406_4350_amd import chebfd as cf  # noqa: E402
from paper_1406_4350_amd import workload as wl  # noqa: E402

CFG = wl.Config("routes64", 64, 16, 16.0, "sc", 4, 64, "2s2p1d", True, 8, 4, 1, 4, 151)  # 17 077 plane waves, 832 projectors


@pytest.fixture(scope="module")
def problem():
    pb = wl.make_problem(CFG)
    plan = cf.plan_from_problem(pb, cf.CHEB_FP64)
    yield pb, plan, torch.from_numpy(np.ascontiguousarray(pb.P.T)).cuda(), torch.from_numpy(pb.Q).cuda()
    plan.close()


def _block(npw, nb, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn((nb, npw), dtype=torch.complex128, device="cuda", generator=g)


def _s(X, P, Q):
    return X + ((X @ P.conj().T) * Q) @ P


def _rel(Y, ref):
    return float((torch.linalg.vector_norm(Y - ref, dim=1) / torch.linalg.vector_norm(ref, dim=1)).max())


def _took(plan, fn):
    """(routes of the projections, of the back-projections) of the products inside fn()."""
    a = plan.profile_routes()
    fn()
    b = plan.profile_routes()
    return [{r: b[k][r] - a[k][r] for r in cf.ROUTES if b[k][r] != a[k][r]} for k in ("project", "backproject")]


def _rule(pb, nb):
    v, x, y = ctypes.c_int(), ctypes.c_double(), ctypes.c_double()
    out = []
    for M, K, back in ((CFG.natom * 13, pb.npw, 0), (pb.npw, CFG.natom * 13, 1)):
        cf.load_library().cheb_product_route(M, nb, K, back, ctypes.byref(v), ctypes.byref(x), ctypes.byref(y))
        out.append({"int8" if v.value else "mfma": 1})
    return out


@pytest.mark.parametrize("nb", [16, 300, 320, 511, 512, 513, 768, 1025, 1537])
def test_operators_take_the_route_of_the_rule(problem, nb):
    """S X on either route: sums of 17 077 and 832 terms in FP64, a few sqrt(17 077) eps = 3e-14."""
    pb, plan, P, Q = problem
    print(f"[case] routes64 nb={nb}", flush=True)
    X = _block(pb.npw, nb, nb)
    Y = torch.empty_like(X)
    assert _took(plan, lambda: plan.apply_S(X, Y)) == _rule(pb, nb)
    assert _rel(Y, _s(X, P, Q)) < 1e-13


def test_padded_rows_and_scaled_bands_on_int8(problem):
    """Leading dimension above npw; bands 2^332 and 2^-332 times as large, a zero band, a band whose one entry dominates:
    every band is scaled by itself, so powers of two scale its result exactly and no band changes another's bits."""
    pb, plan, P, Q = problem
    nb = 512
    wide = torch.zeros((nb, pb.npw + 37), dtype=torch.complex128, device="cuda")
    X = wide[:, :pb.npw]
    X.copy_(_block(pb.npw, nb, 5))
    base = plan.apply_S(X.contiguous())
    X[1] *= 2.0 ** 332
    X[2] *= 2.0 ** -332
    X[3] = 0.0
    X[4, 7] = 1e12
    Y = torch.empty_like(wide)[:, :pb.npw]
    assert _took(plan, lambda: plan.apply_S(X, Y)) == [{"int8": 1}, {"int8": 1}]
    assert torch.equal(Y[0], base[0]) and torch.equal(Y[5:], base[5:])
    assert torch.equal(Y[1], base[1] * 2.0 ** 332) and torch.equal(Y[2], base[2] * 2.0 ** -332)
    assert float(Y[3].abs().max()) == 0.0
    assert _rel(Y[4:5], _s(X[4:5].contiguous(), P, Q)) < 1e-13


@pytest.mark.parametrize("value", [float("nan"), float("inf"), 1e200, 1e-200])
def test_unfit_band_on_int8(problem, value):
    """A band with a NaN, an Inf or beyond the integers' range takes the FP64 product inside the call, alone: the other
    bands keep their bits, the band its NaN or, with finite entries, its value."""
    pb, plan, P, Q = problem
    X = _block(pb.npw, 512, 9)
    base = plan.apply_S(X)
    if value == 1e-200:
        X[17] *= value
    else:
        X[17, 11] = complex(value, 0.0)
    Y = torch.empty_like(X)
    assert _took(plan, lambda: plan.apply_S(X, Y)) == [{"int8": 1}, {"int8": 1}]
    keep = [i for i in range(512) if i != 17]
    assert torch.equal(Y[keep], base[keep])
    if value in (1e200, 1e-200):
        assert _rel(Y[17:18] / value, _s(X[17:18] / value, P, Q)) < 1e-13
    else:
        assert not bool(torch.isfinite(torch.view_as_real(Y[17])).all())


@pytest.mark.parametrize("value", [1e200, 1e-200, 0.0])
def test_unfit_projector_turns_the_route_off(problem, value):
    """A projector scaled beyond the integers' range, where every product takes the FP64 matrix cores, and a projector of
    zeros, which is fit: H X = P D P^H X (no kinetic term and potential)."""
    pb, _, P, _ = problem
    plan = cf.Plan(pb.gidx, np.zeros(pb.npw), 64, pb.proj_off, False)
    plan.set_potential(torch.zeros((64,) * 3, dtype=torch.float64))
    Pu = P.clone()
    Pu[100] *= value
    plan.set_projectors(Pu, None)
    D = torch.eye(13, dtype=torch.float64).repeat(CFG.natom, 1, 1)
    if value == 1e200:  # its square would overflow FP64
        D[100 // 13, 100 % 13, 100 % 13] = 0.0
    plan.set_D(D.reshape(-1))
    X = _block(pb.npw, 512, 21)
    Y = torch.empty_like(X)
    route = "int8" if value == 0.0 else "mfma"
    assert _took(plan, lambda: plan.apply_H(X, Y)) == [{route: 1}, {route: 1}]
    Pr = Pu.clone()
    Pr[100] = 0.0
    assert _rel(Y, (X @ Pr.conj().T) @ Pr) < 1e-13
    plan.close()


@pytest.mark.parametrize("nb", [1100, 2100])
def test_shrinking_blocks_keep_the_route(problem, nb):
    """A filter with a degree per band whose active blocks pass through widths above the pieces that the workspace of the
    widest block is laid out for: every product whose block the rule gives to INT8 takes it, and every band equals the
    plain filter of its degree (two filters whose products sum in different orders: 1e-11 after 6 steps)."""
    pb, plan, _, _ = problem
    X = _block(pb.npw, nb, nb)
    width = [nb, nb - 50, 1000 if nb < 2000 else 1900, 900 if nb < 2000 else 1000, 800, 300]  # active at step 1, 2, ...
    deg = np.array([sum(b < k for k in width) for b in range(nb)], dtype=np.int32)
    lp = plan.upper_bound(X[0], 10)
    c, r = 0.55 * lp, 0.45 * lp
    Y = X.clone()
    took = _took(plan, lambda: plan.filter_degrees(Y, deg, c, r))
    want = [{}, {}]
    for k in [nb] + width:  # the projections of the start block and of each step
        route = next(iter(_rule(pb, k)[0]))
        want[0][route] = want[0].get(route, 0) + 1
    for k in width:
        route = next(iter(_rule(pb, k)[1]))
        want[1][route] = want[1].get(route, 0) + 1
    assert took == want and want[0] == {"int8": 7}
    for m in range(1, 7):
        some = [b for b in range(nb) if deg[b] == m][:40]
        Z = X[some].clone()
        plan.filter(Z, m, c, r)
        assert _rel(Y[some], Z) < 1e-11


def test_int8_route_in_a_graph(problem):
    """S X on INT8 captured once and replayed on new inputs, with a band that is unfit in some of them (its flag is set on
    the device): the bits of the eager call each time."""
    pb, plan, _, _ = problem
    X, Y = _block(pb.npw, 512, 41), torch.empty((512, pb.npw), dtype=torch.complex128, device="cuda")
    plan.apply_S(X, Y)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        assert _took(plan, lambda: plan.apply_S(X, Y)) == [{"int8": 1}, {"int8": 1}]
    for k in range(4):
        X.copy_(_block(pb.npw, 512, 42 + k))
        if k % 2:
            X[100 + k, 3] = float("nan")
        graph.replay()
        torch.cuda.synchronize()
        eager = plan.apply_S(X)
        assert torch.equal(Y.isnan(), eager.isnan()) and torch.equal(Y.nan_to_num(0.0), eager.nan_to_num(0.0))
        assert int(Y.isnan().any(1).sum()) == k % 2


def test_plan_without_residue_planes(problem):
    """A plan over the smaller buffer holds no planes, neither do its workspaces, and its products are FP64 ones, equal
    to the INT8 ones up to rounding; a buffer one byte short is refused."""
    pb, plan, P, Q = problem
    lean = cf.Plan(pb.gidx, pb.kin, 64, pb.proj_off, True, residue_planes=False)
    planes = 48 * P.numel()  # of one product; the plan holds those of both
    assert plan.persistent.numel() - lean.persistent.numel() > 2 * planes
    lean.set_potential(torch.from_numpy(np.ascontiguousarray(pb.V)))
    lean.set_projectors(P, Q)
    lean.set_D(torch.from_numpy(pb.D_packed))
    X = _block(pb.npw, 512, 31)
    Y = torch.empty_like(X)
    assert _took(lean, lambda: lean.apply_S(X, Y)) == [{"mfma": 1}, {"mfma": 1}]
    assert _rel(plan.apply_S(X), Y) < 1e-13
    assert plan.workspace(cf.CHEB_OP_SINV, 512).numel() - lean.workspace(cf.CHEB_OP_SINV, 512).numel() > 48 * X.numel()
    h, buf = ctypes.c_void_p(), torch.empty_like(lean.persistent)
    for size, status in ((lean.persistent.numel(), cf.CHEB_OK), (lean.persistent.numel() - 1, cf.CHEB_ERR_WORKSPACE)):
        st = lean.lib.cheb_plan_create(ctypes.byref(lean.desc), buf.data_ptr(), size, None, ctypes.byref(h))
        assert st == status
        if st == cf.CHEB_OK:
            lean.lib.cheb_plan_destroy(h)
    lean.close()


def test_planes_of_one_product(problem):
    """256 projectors: P^H x pays on INT8 at some widths, P w at none, so the plan holds the planes of P^H x only."""
    pb = wl.make_problem(wl.Config("routes64b", 64, 16, 16.0, "sc", 4, 64, "sp", True, 8, 4, 1, 4, 152))
    plan = cf.plan_from_problem(pb, cf.CHEB_FP64)
    lean = cf.Plan(pb.gidx, pb.kin, 64, pb.proj_off, True, residue_planes=False)
    planes = plan.persistent.numel() - lean.persistent.numel()
    assert 48 * pb.P.size < planes < 60 * pb.P.size
    P, Q = torch.from_numpy(np.ascontiguousarray(pb.P.T)).cuda(), torch.from_numpy(pb.Q).cuda()
    X = _block(pb.npw, 513, 51)
    Y = torch.empty_like(X)
    assert _took(plan, lambda: plan.apply_S(X, Y)) == [{"int8": 1}, {"mfma": 1}]
    assert _rel(Y, _s(X, P, Q)) < 1e-13
    assert _rel(plan.apply_Sinv(Y), X) < 1e-12
    plan.close()
    lean.close()


def test_mixed_routes_and_reset(problem):
    """Mixed plans count their FP16 products by tile; profile_enable resets the counts; other classes are refused."""
    pb, _, _, _ = problem
    plan = cf.plan_from_problem(pb, cf.CHEB_MIXED)
    X = _block(pb.npw, 512, 2).to(torch.complex64)
    plan.filter(X, 2, 10.0, 30.0)
    r = plan.profile_routes()
    assert sum(r["project"].values()) == 3 and sum(r["backproject"].values()) == 2
    assert r["project"]["int8"] == r["project"]["mfma"] == r["backproject"]["mfma"] == 0
    assert r["backproject"]["fp16_128"] == 2  # 134 x 4 tiles of 128
    plan.profile_enable(True)
    plan.profile_enable(False)
    assert not any(plan.profile_routes()["project"].values())
    c = (ctypes.c_int64 * 4)()
    assert plan.lib.cheb_profile_routes(plan.handle, cf.TIMERS.index("small"), c) == cf.CHEB_ERR_ARG
    assert plan.lib.cheb_profile_routes(plan.handle, cf.TIMERS.index("project"), None) == cf.CHEB_ERR_ARG
    plan.close()
