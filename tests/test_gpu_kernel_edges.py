"""Kernels at the sizes where their splits and ranges can go wrong, through
the C ABI against the FP64 oracle."""
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


def _densities(g, nd, seed):
    r = inputs.rng_for(seed, inputs.PURPOSE_DENSITY)
    return inputs.complex_gaussian(r, (nd, g.n)), inputs.complex_gaussian(r, (nd, g.n))


# Translation tables hold only the entries that count for a row.  With the
# order increment far above what eps needs, truncation is below rounding, and
# what is left is rounding (1e-13 at these orders) and whatever the dropped
# entries add: 1e-12 for both.  The frequencies take boxes from far below the
# wavelength (scale factors at their lower clamp; at much lower frequencies
# still, such orders overflow) to several wavelengths.
@pytest.mark.parametrize("which", ["S", "D"])
@pytest.mark.parametrize("omega", [2.0, 20.0, 150.0])
def test_translation_rows_keep_what_counts(ctx, omega, which):
    from paper_1602_05301_amd import qbx
    g = inputs.star(80, 16, lobes=5, amp=0.3)
    p = 8
    s, _ = _densities(g, 1, 40)
    ss, sd = (s, None) if which == "S" else (None, s)
    tc = np.arange(g.n, dtype=np.int32)
    ref = oracle.direct_qbx(omega, p, g, g.sx, g.sy, ss, sd, tgt_ctr=tc)
    geo = qbx.Geometry(ctx, g, omega, 1e-13, g.sx, g.sy, tc, qbx.options(p=p, p_add=70, leaf_max=24))
    u = geo.eval(_dev(ss), _dev(sd)).cpu().numpy()
    err = np.linalg.norm(u - ref) / np.linalg.norm(ref)
    print(f"omega {omega} {which}: {err:.2e}", flush=True)
    assert err <= 1e-12


# H_0 and H_1 on both sides of the bound between their two forms, close to
# zero and at a few hundred wavelengths: one source at the
# origin, p = 0, every target at its centre on the axis, so that each value is
# (i/4) H_0(x) or (i/4) H_1(x) with x exact.  The fits are within 1.3e-15 of
# |H|, and a few roundings follow: 4e-15.
@pytest.mark.parametrize("which", ["S", "D"])
def test_hankel_forms_meet(ctx, which):
    mp = pytest.importorskip("mpmath")
    from paper_1602_05301_amd import qbx
    x = np.concatenate([2.0 ** np.arange(-40, 12, 3.0), np.nextafter(4.0, [0.0, 9.0]),
                        np.linspace(0.5, 12.0, 93), np.linspace(100.0, 1000.0, 61)])
    pts = inputs.Points(np.zeros(1), np.zeros(1), np.ones(1), np.ones(1), np.zeros(1), np.ones(1),
                        x, 0.0 * x, 0.25 * x)
    geo = qbx.Geometry(ctx, pts, 1.0, 1e-10, x, 0.0 * x, np.arange(x.size, dtype=np.int32),
                       qbx.options(p=0, direct=True))
    sig = _dev(np.ones((1, 1), dtype=np.complex128))
    u = geo.eval(sig if which == "S" else None, sig if which == "D" else None).cpu().numpy()[0]
    n = 0 if which == "S" else 1
    with mp.workdps(40):
        ref = np.array([complex(mp.mpc(0, 0.25) * (mp.besselj(n, mp.mpf(float(v))) + 1j * mp.bessely(n, mp.mpf(float(v)))))
                        for v in x])
    err = np.abs(u - ref) / np.abs(ref)
    print(f"{which}: {err.max():.2e} at x = {x[err.argmax()]:g}", flush=True)
    assert err.max() <= 4e-15


# The coefficient sums at the smallest and largest order of each kernel
# variant, S and D together, direct and FMM, one and three densities.  The
# bounds are those of the direct and FMM comparisons elsewhere: rounding grows
# with the order (1e-11 up to 40), the FMM adds its eps.
@pytest.mark.parametrize("p", [0, 1, 8, 9, 12, 13, 14, 15, 16, 17, 25, 33, 40])
def test_coefficient_sums_at_variant_edges(ctx, p):
    from paper_1602_05301_amd import qbx
    g = inputs.star(24, 16, lobes=3, amp=0.3)
    omega = 9.0
    ss, sd = _densities(g, 3, 41)
    tc = np.arange(g.n, dtype=np.int32)
    ref = oracle.direct_qbx(omega, p, g, g.sx, g.sy, ss, sd, tgt_ctr=tc)
    for direct, tol in ((True, 1e-11), (False, 1e-9)):
        geo = qbx.Geometry(ctx, g, omega, 1e-9, g.sx, g.sy, tc,
                           qbx.options(p=p, direct=direct, p_add=-1 if p < 20 else 3 * p))
        u = geo.eval(_dev(ss), _dev(sd)).cpu().numpy()
        err = np.linalg.norm(u - ref) / np.linalg.norm(ref)
        print(f"p {p} direct {direct}: {err:.2e}", flush=True)
        assert err <= tol
        one = geo.eval(_dev(ss[1:2]), _dev(sd[1:2])).cpu().numpy()
        assert np.array_equal(one[0], u[1])


# Evaluation of an expansion from the coefficients that the same call returns:
# target counts around a wavefront, targets on their centre, close to it and
# far beyond any disk.  A value of J_n with its share of the normalising sum is
# within 7e-15 of max(|J_n|, its decaying bound) below x = 30, the phase's
# powers add 2 roundings an order: 2e-14 of the sum of moduli; at x in the
# hundreds the recurrence rounds at every order, x 1.1e-16 more.
@pytest.mark.parametrize("p,nt", [(0, 1), (1, 63), (14, 65), (40, 130)])
def test_expansion_evaluation_edges(ctx, p, nt):
    mp = pytest.importorskip("mpmath")
    from paper_1602_05301_amd import qbx
    r = np.random.default_rng(100 + p)
    omega, ns = 3.0, 5
    cx, cy = np.array([0.0, 0.5, -1.0]), np.array([0.0, 0.25, 2.0])
    ang = r.uniform(0, 2 * np.pi, ns)
    pts = inputs.Points(9 * np.cos(ang), 9 * np.sin(ang), np.ones(ns), np.cos(ang), np.sin(ang),
                        np.ones(ns), cx, cy, np.ones(3))
    tc = (np.arange(nt) % 3).astype(np.int32)
    rho = 10.0 ** r.uniform(-6, 0.3, nt)
    rho[::5] = 0.0
    rho[1::16] = 150.0
    th = r.uniform(0, 2 * np.pi, nt)
    tx, ty = cx[tc] + rho * np.cos(th), cy[tc] + rho * np.sin(th)
    geo = qbx.Geometry(ctx, pts, omega, 1e-10, tx, ty, tc, qbx.options(p=p, direct=True))
    sig = _dev(r.standard_normal((2, ns)) + 1j * r.standard_normal((2, ns)))
    u, coef = (a.cpu().numpy() for a in geo.eval(sig, None, coef=True))
    dx, dy = tx - cx[tc], ty - cy[tc]
    x = omega * np.hypot(dx, dy)
    with mp.workdps(30):
        J = np.array([[float(mp.besselj(n, mp.mpf(float(v)))) for v in x] for n in range(p + 1)])
    l = np.arange(-p, p + 1)[:, None]
    Jl = J[abs(l[:, 0])] * np.where((l < 0) & (l % 2 == 1), -1.0, 1.0)
    E = np.exp(-1j * l * np.arctan2(dy, dx)[None])
    a = coef.reshape(2, 2 * p + 1, 3)[:, :, tc]
    ref = (a * Jl * E).sum(1)
    amp = np.where(x > 1.0, np.sqrt(1.0 / np.maximum(x, 1.0)), 0.0)
    size = (abs(a) * np.maximum(abs(Jl), np.where(abs(l) <= x, amp, 0.0))).sum(1)
    err = abs(u - ref) / size
    print(f"p {p} nt {nt}: {err.max():.2e}", flush=True)
    assert (err <= 2e-14 + 1.1e-16 * x).all()


# The locals start from what the X lists' kernel wrote or from nothing: what an
# earlier evaluation left there (here NaN everywhere) has no part in the next
# one.  Alone and batched, one and three densities, FP64 and FP32 far field, a
# tree of a single box, and one on the path that allocates nothing.
@pytest.mark.parametrize("nseg,far32", [(2, False), (60, False), (60, True)])
def test_evaluation_ignores_earlier_locals(ctx, nseg, far32):
    from paper_1602_05301_amd import qbx
    g = inputs.star(nseg, 16, lobes=5, amp=0.45)
    geo = qbx.Geometry(ctx, g, 20.0, 1e-6, g.sx, g.sy, np.arange(g.n, dtype=np.int32),
                       qbx.options(p=6, far_fp32=far32))
    for nd in (1, 3):
        ss, sd = (_dev(a) for a in _densities(g, nd, 77))
        bad = torch.full_like(ss, float("nan"))
        ref = geo.eval(ss, sd)
        out = [torch.empty_like(ref) for _ in range(3)]
        geo.eval(bad, bad)
        geo.eval(ss, sd, u=out[0])
        ctx.eval_batch([geo], [bad], [bad], [out[1]])
        ctx.eval_batch([geo], [ss], [sd], [out[1]])
        geo.eval_noalloc(bad, bad, out[2])
        geo.eval_noalloc(ss, sd, out[2])
        torch.cuda.synchronize()
        assert torch.isfinite(torch.view_as_real(ref)).all()
        for o in out:
            assert torch.equal(torch.view_as_real(o), torch.view_as_real(ref))


# Near-field items on both sides of the rule for larger ones (131072 points in
# leaves of 64 make some 8000, 8192 points 1000): the FMM against the direct mode at every
# target.  eps is 1e-8, ten times that in l2.
@pytest.mark.parametrize("panels,leaf", [(512, 16), (8192, 64)])
def test_near_field_items_on_both_sides_of_the_rule(ctx, panels, leaf):
    from paper_1602_05301_amd import qbx
    g = inputs.star(panels, 16, lobes=7, amp=0.3)
    tc = np.arange(g.n, dtype=np.int32)
    sig = _dev(_densities(g, 1, 51)[0])
    u = [qbx.Geometry(ctx, g, 40.0, 1e-8, g.sx, g.sy, tc, qbx.options(p=10, leaf_max=leaf, direct=d)).eval(sig, sig)
         for d in (False, True)]
    err = float(torch.linalg.norm(u[0] - u[1]) / torch.linalg.norm(u[1]))
    print(f"panels {panels} leaf {leaf}: {err:.2e}", flush=True)
    assert err <= 1e-7


# Gram-Schmidt products with vector counts around the rows of a block and the
# rows of the final sums' blocks, lengths around a chunk and past 64 chunks;
# panel interpolation with panel counts around a block's, and panels too long
# for LDS.  The rounding of sums of n products of unit-variance entries is
# below 1e-12 sqrt(n) at these lengths.
@pytest.mark.parametrize("n,k", [(1, 1), (1023, 3), (1024, 8), (1025, 9), (70001, 5)])
def test_gram_schmidt_edges(ctx, n, k):
    r = np.random.default_rng(n + k)
    V, w = inputs.complex_gaussian(r, (k, n)), inputs.complex_gaussian(r, (n,))
    dV, dw, h = _dev(V), _dev(w), _dev(np.zeros(k, dtype=np.complex128))
    ctx.krylov_dot(dV, k, dw, h)
    ref = V.conj() @ w
    assert np.abs(h.cpu().numpy() - ref).max() <= 1e-13 * max(1.0, np.sqrt(n)) * 10
    ctx.krylov_update(dV, k, h, dw)
    out = w - ref @ V
    assert np.abs(dw.cpu().numpy() - out).max() <= 1e-12 * max(1.0, np.abs(out).max())


@pytest.mark.parametrize("panels,q,qs", [(1, 1, 1), (7, 16, 64), (8, 8, 40), (9, 16, 32), (3, 90, 90)])
def test_upsample_edges(ctx, panels, q, qs):
    r = np.random.default_rng(panels)
    L, x = r.standard_normal((qs, q)), inputs.complex_gaussian(r, (panels * q,))
    ys, yd = _dev(np.zeros(panels * qs, dtype=np.complex128)), _dev(np.zeros(panels * qs, dtype=np.complex128))
    ctx.upsample(_dev(L), q, qs, _dev(x), 2.0 - 1.0j, ys=ys, yd=yd)
    ref = (x.reshape(panels, q) @ L.T).ravel()
    assert np.abs(yd.cpu().numpy() - ref).max() <= 1e-12
    assert np.abs(ys.cpu().numpy() - (2.0 - 1.0j) * ref).max() <= 1e-11


# Offsets of area queries around the sizes of the scan's blocks (2048 counts)
# and past one round of its block sums (256 blocks): one call over n squares
# against calls over parts of them, leaf by leaf.
@pytest.mark.parametrize("n", [0, 1, 2047, 2048, 2049, 530001])
def test_area_query_offsets(ctx, n):
    from paper_1602_05301_amd import qbx
    g = inputs.star(40, 16, lobes=5, amp=0.3)
    geo = qbx.Geometry(ctx, g, 5.0, 1e-8, g.sx, g.sy, np.arange(g.n, dtype=np.int32), qbx.options(p=8))
    r = np.random.default_rng(n)
    x, y = _dev(r.uniform(-1.4, 1.4, n)), _dev(r.uniform(-1.4, 1.4, n))
    rad = _dev(r.uniform(-0.02, 0.06, n))                   # a quarter of them empty
    start, leaves = geo.area_query(x, y, rad)
    starts, parts, base = [], [], 0
    for i in range(0, n, 1000):
        s, l = geo.area_query(x[i:i + 1000].contiguous(), y[i:i + 1000].contiguous(), rad[i:i + 1000].contiguous())
        starts.append(s[:-1] + base)
        parts.append(l)
        base += int(s[-1])
    assert int(start[-1]) == base and leaves.numel() == base
    if n:
        assert torch.equal(start[:-1], torch.cat(starts)) and torch.equal(leaves, torch.cat(parts))
