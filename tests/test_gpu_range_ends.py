"""Calls at the ends of the ranges that the kernels take: orders at their LDS
limits, arguments at the ends of the exponent range, query buffers in any
order of calls."""
import numpy as np
import pytest

import oracle
from paper_1602_05301_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1602_05301_amd import qbx
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return qbx.Context(0)


def _dev(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


# H_0 and H_1 at omega 2^k and targets at powers of two from one source at the
# origin, so that x is exact: at centres (p = 0) and by the smooth rule.  As
# between the forms of the ordinary range: 4e-15.
def _hankel_at(ctx, which, bound, k, direct=True):
    mp = pytest.importorskip("mpmath")
    from paper_1602_05301_amd import qbx
    omega, d = 2.0 ** k, 2.0 ** np.arange(-3, 4)
    pts = inputs.Points(np.zeros(1), np.zeros(1), np.ones(1), np.ones(1), np.zeros(1), np.full(1, 1e-3),
                        d, 0.0 * d, 1e-3 * d)
    tx = d if bound else -d
    tc = np.arange(d.size, dtype=np.int32) if bound else np.full(d.size, -1, dtype=np.int32)
    geo = qbx.Geometry(ctx, pts, omega, 1e-10, tx, 0.0 * tx, tc, qbx.options(p=0, direct=direct))
    sig = _dev(np.ones((1, 1), dtype=np.complex128))
    sig = (sig if which == "S" else None, sig if which == "D" else None)
    u = geo.eval(*sig).cpu().numpy()[0]
    both = torch.empty((1, tx.size), dtype=torch.complex128, device="cuda:0")
    ctx.eval_batch([geo], [sig[0]], [sig[1]], [both])
    torch.cuda.synchronize()
    assert np.array_equal(both.cpu().numpy()[0], u)
    n = 0 if which == "S" else 1

    def hankel(x):
        x = mp.mpf(x)
        if x < 1e10:
            return mp.besselj(n, x) + 1j * mp.bessely(n, x)
        # Hankel's expansion, the next term below 1e-20
        return mp.sqrt(2 / (mp.pi * x)) * mp.expj(x - n * mp.pi / 2 - mp.pi / 4) * (1 + 1j * (4 * n * n - 1) / (8 * x))
    with mp.workdps(140):
        ref = np.array([complex(0.25j * (mp.mpf(omega) * np.sign(v) if n else 1) * hankel(omega * abs(v))) for v in tx])
    err = np.abs(u - ref) / np.abs(ref)
    print(f"omega 2^{k} {which} bound {bound}: {err.max():.2e}", flush=True)
    assert (err <= 4e-15).all()


# Arguments whose square underflows.
@pytest.mark.parametrize("bound", [True, False])
@pytest.mark.parametrize("which", ["S", "D"])
@pytest.mark.parametrize("k", [-600, -520])
def test_hankel_at_tiny_arguments(ctx, which, bound, k):
    _hankel_at(ctx, which, bound, k)


# Arguments on both sides of 1e14, where the phase takes another reduction, and
# far beyond, by the direct rule and (a tree of one box) by the near field.
@pytest.mark.parametrize("direct", [True, False])
@pytest.mark.parametrize("bound", [True, False])
@pytest.mark.parametrize("which", ["S", "D"])
@pytest.mark.parametrize("k", [45, 47, 52, 60, 300])
def test_hankel_at_huge_arguments(ctx, which, bound, k, direct):
    _hankel_at(ctx, which, bound, k, direct)


# L2QBXL at leaf orders around the bounds where its staging changes: at p = 14
# wide J_n rows up to order 75, 16 centres an item up to 295, 8 up to 405, and
# orders up to 480.  Alone and batched with a geometry of low orders, one and two
# densities, against the oracle: eps is 1e-10, ten times that in l2.
@pytest.mark.parametrize("omega,order", [(20.0, 75), (20.0, 76), (250.0, 231), (250.0, 232), (400.0, 295),
                                         (400.0, 296), (700.0, 455), (700.0, 480)])
def test_l2qbxl_at_high_leaf_orders(ctx, omega, order):
    from paper_1602_05301_amd import qbx
    g = inputs.star(24, 16, lobes=3, amp=0.3)
    tc = np.arange(g.n, dtype=np.int32)

    def opts(p_add):
        return qbx.options(p=14, p_add=p_add, leaf_max=64)
    p_add = order - int(qbx.Plan(g, omega, 1e-10, g.sx, g.sy, tc, opts(0)).orders()[2])
    plan = qbx.Plan(g, omega, 1e-10, g.sx, g.sy, tc, opts(p_add))
    box = plan.boxes()
    lev = box["level"][(box["leaf"] > 0) & (box["nctr"] > 0)]
    assert lev.min() == 2 and plan.orders()[2] == order
    r = np.random.default_rng(order)
    ss, sd = inputs.complex_gaussian(r, (2, g.n)), inputs.complex_gaussian(r, (2, g.n))
    ref = oracle.direct_qbx(omega, 14, g, g.sx, g.sy, ss, sd, tgt_ctr=tc)
    geo = qbx.Geometry(ctx, g, omega, 1e-10, g.sx, g.sy, tc, opts(p_add))
    low = qbx.Geometry(ctx, g, 20.0, 1e-10, g.sx, g.sy, tc, opts(-1))
    u = geo.eval(_dev(ss), _dev(sd))
    err = np.linalg.norm(u.cpu().numpy() - ref) / np.linalg.norm(ref)
    print(f"omega {omega} order {order}: {err:.2e}", flush=True)
    assert err <= 1e-9
    one = geo.eval(_dev(ss[1:]), _dev(sd[1:]))
    both = [torch.empty_like(u), torch.empty_like(u)]
    ctx.eval_batch([low, geo], [_dev(ss)] * 2, [_dev(sd)] * 2, both)
    torch.cuda.synchronize()
    assert torch.equal(one[0], u[1]) and torch.equal(both[1], u)
    assert torch.equal(both[0], low.eval(_dev(ss), _dev(sd)))


# Targets so close to their centre, or to it in wavelengths, that the downward
# recurrence leaves the exponent range in a few steps: what is left of the
# expansion is its order 0, which the coefficients of the same call give, and
# orders +-1 times x / 2, which the tolerance covers (coefficients stay below 10
# here), and rounding.
@pytest.mark.parametrize("p", [0, 1, 5, 14, 40])
def test_evaluation_beside_the_centre(ctx, p):
    from paper_1602_05301_amd import qbx
    r = np.random.default_rng(p)
    ang = r.uniform(0, 2 * np.pi, 5)
    pts = inputs.Points(40 * np.cos(ang), 40 * np.sin(ang), np.ones(5), np.cos(ang), np.sin(ang), np.ones(5),
                        np.zeros(1), np.zeros(1), np.ones(1))
    tx = np.concatenate([[0.0], 10.0 ** -np.arange(12.0, 160.0)])
    geo = qbx.Geometry(ctx, pts, 1.0, 1e-10, tx, 0.0 * tx, np.zeros(tx.size, dtype=np.int32),
                       qbx.options(p=p, direct=True))
    sig = _dev(inputs.complex_gaussian(r, (2, 5)))
    u, coef = (a.cpu().numpy() for a in geo.eval(sig, None, coef=True))
    a0 = coef.reshape(2, 2 * p + 1)[:, p:p + 1]
    assert np.abs(coef).max() < 10.0
    err = np.abs(u - a0)
    print(f"p {p}: {err.max():.2e}", flush=True)
    assert (err <= 1e-15 + 10.0 * tx).all()


# Targets far from their centre, on both sides of the bound of the upward
# recurrence and past the range of an int, against mpmath from the coefficients
# of the same call; alone and batched.  The tolerance is of the sum of moduli,
# |J_n| about sqrt(2 / (pi x)) there (up to 3 times that at n = 40 and x = 99):
# 2e-14 as for nearer targets, and x 1.1e-16 where the recurrence takes x steps.
@pytest.mark.parametrize("p", [0, 1, 14, 40])
def test_evaluation_far_from_the_centre(ctx, p):
    mp = pytest.importorskip("mpmath")
    from paper_1602_05301_amd import qbx
    r = np.random.default_rng(p)
    x = np.array([60.0, 99.0, 101.0, 9999.0, 123456.0, 2.0 ** 31, 5.0 * 2.0 ** 30, 3.0 * 2.0 ** 45, 2.0 ** 60])
    pts = inputs.Points(np.array([40.0]), np.zeros(1), np.ones(1), np.ones(1), np.zeros(1), np.ones(1),
                        np.zeros(1), np.zeros(1), np.ones(1))
    geo = qbx.Geometry(ctx, pts, 1.0, 1e-10, x, 0.0 * x, np.zeros(x.size, dtype=np.int32),
                       qbx.options(p=p, direct=True))
    sig = _dev(inputs.complex_gaussian(r, (1, 1)))
    u, coef = (a.cpu().numpy() for a in geo.eval(sig, None, coef=True))
    a = coef.reshape(2 * p + 1)
    with mp.workdps(60):
        J = []
        for v in x:
            if v < 1e9:
                col = [mp.besselj(n, mp.mpf(v)) for n in range(p + 1)]
            else:                                    # two terms of the expansion, the next below 1e-20
                col = []
                for n in range(2):
                    w = mp.mpf(v) - n * mp.pi / 2 - mp.pi / 4
                    m = 4 * n * n
                    col.append(mp.sqrt(2 / (mp.pi * v)) * (mp.cos(w) - mp.sin(w) * (m - 1) / (8 * mp.mpf(v))))
                while len(col) <= p:
                    n = len(col) - 1
                    col.append(2 * n / mp.mpf(v) * col[n] - col[n - 1])
            J.append([float(c) for c in col[:p + 1]])
    J = np.array(J).T
    l = np.arange(-p, p + 1)
    Jl = J[abs(l)] * np.where((l < 0) & (l % 2 == 1), -1.0, 1.0)[:, None]
    err = np.abs(u[0] - (a[:, None] * Jl).sum(0)) / (np.abs(a).sum() * np.sqrt(2 / (np.pi * x)))
    print(f"p {p}: {err}", flush=True)
    assert (err <= 2e-14 + np.where(x < 100.0, 3.3e-16 * x, 0.0)).all()
    both = torch.empty((1, x.size), dtype=torch.complex128, device="cuda:0")
    ctx.eval_batch([geo], [sig], [None], [both])
    torch.cuda.synchronize()
    assert np.array_equal(both.cpu().numpy(), u)


# The kept blocks of the query calls: small calls first, then larger ones.  The
# largest blocks are the ones kept (the driver's free memory falls by them once
# and stays), and no more than two of at most 16 MiB each.
def test_query_blocks_are_kept_in_any_order(ctx):
    from paper_1602_05301_amd import qbx
    g = inputs.star(40, 16, lobes=5, amp=0.3)

    def geometry(c):
        return qbx.Geometry(c, g, 5.0, 1e-8, g.sx, g.sy, np.arange(g.n, dtype=np.int32), qbx.options(p=8))
    r = np.random.default_rng(3)
    n = 1000000
    x, y, rad = _dev(r.uniform(-1.4, 1.4, n)), _dev(r.uniform(-1.4, 1.4, n)), _dev(np.full(n, -1.0))
    free = lambda: torch.cuda.mem_get_info(0)[0]

    def query(geo, m):
        geo.area_query(x[:m], y[:m], rad[:m])
        torch.cuda.synchronize()
        return free()
    sizes = (10, 20000, n, n, 700000, n)
    warm = geometry(qbx.Context(0))               # torch's own buffers of these sizes
    for m in sizes:
        query(warm, m)
    c = qbx.Context(0)
    geo = geometry(c)
    geo.points_near("sources", x[:10], y[:10], rad[:10])
    query(geo, 10)
    f0 = query(geo, 20000)
    f1 = query(geo, n)
    assert f0 - f1 >= 3 * n                       # n counts of four bytes, less what was freed
    assert query(geo, n) == f1 and query(geo, 700000) == f1 and query(geo, n) == f1
    geo.associate(x[:1000], y[:1000])
    assert f0 - free() <= 2 * (16 << 20)


# Boxes with neither a V nor an X list behind the last V-list entry (two small
# curves far apart: chains of single children below level 2): their locals are
# zero plus the parent's, with no row to look up.  eps is 1e-10, ten times that
# in l2.
@pytest.mark.parametrize("nd", [1, 3])
def test_boxes_behind_the_last_v_list_entry(ctx, nd):
    from paper_1602_05301_amd import qbx
    g = inputs.concat([inputs.star(4, 16, lobes=3, amp=0.1, radius=0.02, center=(0.9, 0.87)),
                       inputs.star(4, 16, lobes=3, amp=0.1, radius=0.02, center=(-0.91, -0.88))])
    tc = np.arange(g.n, dtype=np.int32)
    opts = qbx.options(p=8, leaf_max=48)
    plan = qbx.Plan(g, 5.0, 1e-10, g.sx, g.sy, tc, opts)
    v, x = plan.list(1)[0], plan.list(3)[0]
    behind = (v[:-1] == v[-1]) & (x[1:] == x[:-1])
    assert v[-1] > 0 and behind.sum() > 8
    r = np.random.default_rng(nd)
    ss, sd = inputs.complex_gaussian(r, (nd, g.n)), inputs.complex_gaussian(r, (nd, g.n))
    ref = oracle.direct_qbx(5.0, 8, g, g.sx, g.sy, ss, sd, tgt_ctr=tc)
    geo = qbx.Geometry(ctx, g, 5.0, 1e-10, g.sx, g.sy, tc, opts)
    u = geo.eval(_dev(ss), _dev(sd))
    both = torch.empty_like(u)
    ctx.eval_batch([geo], [_dev(ss)], [_dev(sd)], [both])
    torch.cuda.synchronize()
    assert torch.equal(both, u)
    err = np.linalg.norm(u.cpu().numpy() - ref) / np.linalg.norm(ref)
    print(f"nd {nd}: {err:.2e}", flush=True)
    assert err <= 1e-9


# The near field's item sizes on both sides of their rule: 16 pairs a lane where
# such items are 16 per CU, 8 below.  The items are counted from the plan (near
# lists of the U lists alone, w_direct = 0), as the launch counts them; then the
# FMM against the direct mode at every target, and a batch with a small geometry
# against the call alone.  eps is 1e-8, ten times that in l2.
def _items(plan, limit):
    box = plan.boxes()
    start, idx = plan.list(0)
    total = 0
    for b in np.nonzero((box["leaf"] > 0) & (box["nctr"] > 0))[0]:
        nc, ns, ng = int(box["nctr"][b]), int(box["nsrc"][idx[start[b]:start[b + 1]]].sum()), 1

        def pairs(n):
            cg = max(1, min(n, 64))
            parts = 128 // cg
            return -(-ns // parts) * -(-n // cg)
        while ng < nc and pairs(-(-nc // ng)) > limit:
            ng += 1
        total += ng
    return total


@pytest.mark.parametrize("panels,many", [(2800, False), (3800, True)])
def test_near_field_item_rule(ctx, panels, many):
    from paper_1602_05301_amd import qbx
    g = inputs.star(panels, 16, lobes=7, amp=0.3)
    tc = np.arange(g.n, dtype=np.int32)
    opts = qbx.options(p=10, leaf_max=64, w_direct=0)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    larger = _items(qbx.Plan(g, 40.0, 1e-8, g.sx, g.sy, tc, opts), 16)
    print(f"panels {panels}: {larger / cus:.1f} items per CU", flush=True)
    assert (larger >= 16 * cus) == many and 12 * cus < larger < 20 * cus
    r = np.random.default_rng(panels)
    sig = _dev(inputs.complex_gaussian(r, (1, g.n)))
    geo = qbx.Geometry(ctx, g, 40.0, 1e-8, g.sx, g.sy, tc, opts)
    u = geo.eval(sig, sig)
    ref = qbx.Geometry(ctx, g, 40.0, 1e-8, g.sx, g.sy, tc, qbx.options(p=10, direct=True)).eval(sig, sig)
    err = float(torch.linalg.norm(u - ref) / torch.linalg.norm(ref))
    print(f"panels {panels}: {err:.2e}", flush=True)
    assert err <= 1e-7
    s = inputs.star(40, 16, lobes=3, amp=0.3)
    small = qbx.Geometry(ctx, s, 10.0, 1e-8, s.sx, s.sy, np.arange(s.n, dtype=np.int32), opts)
    ssig = sig[:, :s.n].contiguous()
    both = [torch.empty_like(ssig), torch.empty_like(u)]
    ctx.eval_batch([small, geo], [ssig, sig], [ssig, sig], both)
    torch.cuda.synchronize()
    assert torch.equal(both[1], u) and torch.equal(both[0], small.eval(ssig, ssig))


# Area queries and disk tests on the deepest tree (two coincident sources in
# leaves of one point: 31 levels), from squares about them and about other points,
# against every leaf of the plan.  The stack's bound is 9 + 3 per level.
def test_area_queries_on_the_deepest_tree(ctx):
    from paper_1602_05301_amd import qbx
    g = inputs.star(8, 16, lobes=3, amp=0.3)
    dup = np.array([g.sx[5], g.sx[77]]), np.array([g.sy[5], g.sy[77]])
    cat = lambda a, b: np.concatenate([a, b])
    pts = inputs.Points(cat(g.sx, dup[0]), cat(g.sy, dup[1]), cat(g.w, g.w[:2]), cat(g.nx, g.nx[:2]),
                        cat(g.ny, g.ny[:2]), cat(g.h, g.h[:2]), g.cx, g.cy, g.cr)
    tc = np.arange(g.n, dtype=np.int32)
    opts = qbx.options(p=2, direct=True, leaf_max=1, level_restrict=False)
    plan = qbx.Plan(pts, 1.0, 1e-6, g.sx, g.sy, tc, opts)
    box = plan.boxes()
    assert plan.stats()["n_levels"] == 31
    R0 = plan.stats()["root_radius"]
    leaf = np.nonzero(box["leaf"])[0]
    rb = np.ldexp(R0, -box["level"][leaf])
    bx, by = -R0 + (2 * box["ix"][leaf] + 1) * rb, -R0 + (2 * box["iy"][leaf] + 1) * rb
    r = np.random.default_rng(9)
    n = 600
    at = r.integers(0, pts.sx.size, n)
    at[:200:2], at[1:200:2] = 5, pts.sx.size - 1
    rad = 10.0 ** r.uniform(-11, 0.5, n)
    x, y = pts.sx[at] + 0.3 * rad, pts.sy[at] - 0.2 * rad
    geo = qbx.Geometry(ctx, pts, 1.0, 1e-6, g.sx, g.sy, tc, opts)
    start, leaves = (a.cpu().numpy() for a in geo.area_query(_dev(x), _dev(y), _dev(rad)))
    near = geo.points_near("sources", _dev(x), _dev(y), _dev(rad)).cpu().numpy()
    for i in range(n):
        gap = np.maximum(abs(bx - x[i]), abs(by - y[i])) - rb - rad[i]
        tol = 1e-14 * (R0 + rad[i])
        got = set(leaves[start[i]:start[i + 1]].tolist())
        assert set(leaf[gap < -tol].tolist()) <= got <= set(leaf[gap <= tol].tolist()), i
        d2 = (pts.sx - x[i]) ** 2 + (pts.sy - y[i]) ** 2
        assert near[i] == (d2 <= rad[i] ** 2).any()


# Panel interpolation on both sides of the staging's lower bounds (panels of 8
# nodes, 4 rows), panel counts around a block's: sums of q products of
# unit-variance entries, 1e-12 as in the tests of longer panels.
@pytest.mark.parametrize("panels,q,qs", [(1, 7, 4), (9, 8, 3), (7, 8, 4), (17, 7, 40), (300, 64, 2), (300, 2, 2)])
def test_upsample_of_short_panels(ctx, panels, q, qs):
    r = np.random.default_rng(panels + q)
    L, x = r.standard_normal((qs, q)), inputs.complex_gaussian(r, (panels * q,))
    ys, yd = _dev(np.zeros(panels * qs, dtype=np.complex128)), _dev(np.zeros(panels * qs, dtype=np.complex128))
    ctx.upsample(_dev(L), q, qs, _dev(x), 2.0 - 1.0j, ys=ys, yd=yd)
    ref = (x.reshape(panels, q) @ L.T).ravel()
    assert np.abs(yd.cpu().numpy() - ref).max() <= 1e-12
    assert np.abs(ys.cpu().numpy() - (2.0 - 1.0j) * ref).max() <= 1e-11


# Expansions of order 0 away from their centres: the value is the coefficient
# times J_0, as close as the library's j0 (an ulp or two of its envelope
# sqrt(2 / (pi x)), and the product's rounding): 1e-15 of it.
def test_order_zero_takes_no_sum(ctx):
    mp = pytest.importorskip("mpmath")
    from paper_1602_05301_amd import qbx
    x = np.concatenate([np.linspace(1.0, 40.0, 157), np.linspace(40.3, 99.7, 98)])
    pts = inputs.Points(np.array([40.0]), np.zeros(1), np.ones(1), np.ones(1), np.zeros(1), np.ones(1),
                        np.zeros(1), np.zeros(1), np.ones(1))
    geo = qbx.Geometry(ctx, pts, 1.0, 1e-10, x, 0.0 * x, np.zeros(x.size, dtype=np.int32),
                       qbx.options(p=0, direct=True))
    sig = _dev(np.full((1, 1), 0.75 - 0.5j))
    u, coef = (a.cpu().numpy() for a in geo.eval(sig, None, coef=True))
    with mp.workdps(40):
        J = np.array([float(mp.besselj(0, mp.mpf(float(v)))) for v in x])
    a = coef.reshape(1)[0]
    err = np.abs(u[0] - a * J) / (np.abs(a) * np.sqrt(2 / (np.pi * x)))
    print(f"p 0: {err.max():.2e} at x = {x[err.argmax()]:g}", flush=True)
    assert err.max() <= 1e-15
