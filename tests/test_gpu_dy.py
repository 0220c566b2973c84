"""Fused LO Drell-Yan-like integrand (pdfx_eval_dy / pdfx_eval_dy_backward)
against the CPU FP64 oracle: per-point values, partial sums, and the knot
gradient of sum_p I_p against oracle finite differences."""
import math

import numpy as np
import pytest

import oracle
from helpers import cfg0_grid
from paper_2012_08221_amd import workloads as wl

pytestmark = pytest.mark.gpu
XMIN = wl.DY_XMIN
S = wl.SQRT_S_DY ** 2
L = math.log(1.0 / XMIN)


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.fixture(scope="module")
def api(torch):
    from paper_2012_08221_amd import api as a
    return a


@pytest.fixture(scope="module")
def pdf(api):
    return api.mkPDF(cfg0_grid())


def kinematics(grid, u1, u2):
    x1 = np.exp(math.log(XMIN) + u1 * L)
    x2 = np.exp(math.log(XMIN) + u2 * L)
    q2 = np.clip(x1 * x2 * S, grid.q2[0], grid.q2[-1])
    return x1, x2, q2


def scale_of(grid, u1, u2):
    """Error scale: L^2 alpha_s sum_q M_q(x1) M_-q(x2), M = stencil max |v|."""
    x1, x2, q2 = kinematics(grid, u1, u2)
    m1 = oracle.stencil_absmax(grid, [1, 2, 3, 4, 5], x1, q2)
    m2 = oracle.stencil_absmax(grid, [-1, -2, -3, -4, -5], x2, q2)
    a = oracle.alphas(grid.as_q2, grid.as_val, q2)
    return L * L * a * np.sum(m1 * m2, axis=1)


@pytest.mark.parametrize("prec,tol", [("f64", 1e-12), ("f32s", 1e-5)])
def test_integrand_parity_chunk0(pdf, prec, tol):
    g = cfg0_grid()
    u1, u2 = wl.dy_uniforms(0, 1_000_000)
    got, sums = pdf_dy(pdf, u1, u2, prec)
    ora = oracle.dy(g, u1, u2, XMIN, S)
    sc = scale_of(g, u1, u2)
    e = np.abs(got - ora) / np.maximum(np.abs(ora), 0.1 * sc)
    print("integrand %s: max err %.2e; clipped at Q2_min: %.1f%%" %
          (prec, e.max(), 100 * np.mean(kinematics(g, u1, u2)[2] == g.q2[0])))
    assert e.max() <= tol
    rel = abs(sums.sum() - ora.sum()) / np.abs(ora).sum()
    assert rel <= (1e-12 if prec == "f64" else 1e-6)


def pdf_dy(pdf, u1, u2, prec, values=None):
    from paper_2012_08221_amd import api
    res, sums = api.dy_integrand(pdf, u1, u2, XMIN, S, prec=prec, values=values)
    return res.double().cpu().numpy(), sums.cpu().numpy()


def test_integrand_edges(pdf, api, torch):
    res, sums = api.dy_integrand(pdf, np.zeros(0), np.zeros(0))
    assert res.numel() == 0 and sums.numel() == 0
    u1, u2 = wl.dy_uniforms(1, 777)
    u1[:3] = [0.0, 0.999999999, 0.5]
    u2[:3] = [0.0, 0.999999999, 0.0]
    got, sums = pdf_dy(pdf, u1, u2, "f64")
    ora = oracle.dy(cfg0_grid(), u1, u2, XMIN, S)
    np.testing.assert_allclose(got, ora, rtol=1e-12, atol=1e-12 * np.abs(ora).max())
    only_sums, sums2 = api.dy_integrand(pdf, u1, u2, out=False)
    assert only_sums is None
    np.testing.assert_allclose(sums2.cpu().numpy().sum(), ora.sum(), rtol=1e-12)
    v = torch.as_tensor(cfg0_grid().xf, device="cuda")
    got2, _ = pdf_dy(pdf, u1, u2, "f64", values=v)
    np.testing.assert_array_equal(got, got2)


def touched(grid, x, q2, i, k):
    ix, s, iq, inside = oracle.locate(grid, x, q2)
    kg = grid.q_off[s] + iq
    lo = np.maximum(kg - 1, grid.q_off[s])
    hi = np.minimum(kg + 2, grid.q_off[s + 1] - 1)
    return inside & (ix - 1 <= i) & (i <= ix + 2) & (lo <= k) & (k <= hi)


@pytest.mark.parametrize("prec", ["f64", "f32s"])
def test_integrand_gradient_vs_fd(pdf, api, torch, prec):
    g = cfg0_grid()
    n = 100_000
    u1, u2 = wl.dy_uniforms(2, n)
    vals_np = g.xf if prec == "f64" else g.xf.astype(np.float32)
    g64 = wl.GridSpec(pids=g.pids, x=g.x, q2=g.q2, q_off=g.q_off,
                      xf=np.asarray(vals_np, dtype=np.float64), as_q2=g.as_q2, as_val=g.as_val)
    vals = torch.as_tensor(vals_np, device="cuda")
    grad = torch.zeros_like(vals)
    scale = 1.0 / n
    api.dy_backward(pdf, u1, u2, grad, XMIN, S, scale, prec=prec, values=vals)
    grad = grad.double().cpu().numpy()
    x1, x2, q2 = kinematics(g, u1, u2)
    rng = np.random.default_rng(11)
    rows = {int(p): f for f, p in enumerate(g.pids)}
    # flavours outside the luminosity (gluon) get exactly zero
    assert np.all(grad[rows[21]] == 0.0)
    res = []
    h = 1e-4
    while len(res) < 60:
        pid = int(rng.choice([1, 2, 3, 4, 5, -1, -2, -3, -4, -5]))
        f = rows[pid]
        i = int(rng.integers(40, 99))
        k = int(rng.integers(0, g.n_q))
        xs = x1 if pid > 0 else x2
        m = touched(g, xs, q2, i, k)
        if not m.any():
            assert grad[f, i, k] == 0.0
            continue
        gp = wl.GridSpec(pids=g.pids, x=g.x, q2=g.q2, q_off=g.q_off, xf=g64.xf.copy(),
                         as_q2=g.as_q2, as_val=g.as_val)
        gm = wl.GridSpec(pids=g.pids, x=g.x, q2=g.q2, q_off=g.q_off, xf=g64.xf.copy(),
                         as_q2=g.as_q2, as_val=g.as_val)
        gp.xf[f, i, k] += h
        gm.xf[f, i, k] -= h
        fd = scale * np.sum(oracle.dy(gp, u1[m], u2[m], XMIN, S) -
                            oracle.dy(gm, u1[m], u2[m], XMIN, S)) / (2 * h)
        res.append((grad[f, i, k], fd))
    a = np.array(res)
    sc = max(1e-300, 1e-2 * math.sqrt(np.mean(a[:, 1] ** 2)))
    e = np.abs(a[:, 0] - a[:, 1]) / np.maximum(np.abs(a[:, 1]), sc)
    print("integrand gradient %s: max metric %.2e" % (prec, e.max()))
    assert e.max() <= 1e-6


@pytest.mark.parametrize("prec", ["f64", "f32s"])
def test_integrand_kernels_agree(pdf, api, prec):
    """A grid whose partons are not in the standard order -5 .. -1, g, 1 .. 5
    takes the single-slab integrand kernel; the standard grid takes the
    double-buffered one.  Same partons and values: same per-point results."""
    g = cfg0_grid()
    perm = np.arange(g.pids.size)[::-1].copy()
    gp = wl.GridSpec(pids=g.pids[perm], x=g.x, q2=g.q2, q_off=g.q_off, xf=g.xf[perm].copy(),
                     as_q2=g.as_q2, as_val=g.as_val)
    other = api.mkPDF(gp)
    u1, u2 = wl.dy_uniforms(3, 200_000)
    a, sa = pdf_dy(pdf, u1, u2, prec)
    b, sb = pdf_dy(other, u1, u2, prec)
    np.testing.assert_array_equal(a, b)
    assert abs(sa.sum() - sb.sum()) <= 1e-12 * np.abs(a).sum()
    ora = oracle.dy(g, u1, u2, XMIN, S)
    sc = scale_of(g, u1, u2)
    e = np.abs(b - ora) / np.maximum(np.abs(ora), 0.1 * sc)
    assert e.max() <= (1e-12 if prec == "f64" else 1e-5)


@pytest.mark.parametrize("prec", ["f64", "f32s"])
def test_integrand_launch_shapes_agree(pdf, prec):
    u1, u2 = wl.dy_uniforms(4, 150_001)
    keep = pdf.dy_launch(prec)
    ref = None
    try:
        for shape in ((512, 1), (512, 2), (256, 2)) + (((512, 4),) if prec == "f32s" else ()):
            pdf.set_dy_launch(prec, *shape)
            got, sums = pdf_dy(pdf, u1, u2, prec)
            if ref is None:
                ref = got
            else:
                np.testing.assert_array_equal(got, ref)
    finally:
        pdf.set_dy_launch(prec, *keep)
    with pytest.raises(Exception):
        pdf.set_dy_launch(prec, 128, 3)


@pytest.mark.parametrize("prec", ["f64", "f32s"])
def test_integrand_backward_kernels_agree(pdf, api, torch, prec):
    """The standard grid takes the pair-wise knot-gradient pass, a grid with
    reversed parton order the per-flavour one: same gradient (FP64 sums in a
    different order)."""
    g = cfg0_grid()
    perm = np.arange(g.pids.size)[::-1].copy()
    gp = wl.GridSpec(pids=g.pids[perm], x=g.x, q2=g.q2, q_off=g.q_off, xf=g.xf[perm].copy(),
                     as_q2=g.as_q2, as_val=g.as_val)
    other = api.mkPDF(gp)
    u1, u2 = wl.dy_uniforms(5, 300_000)
    dt = api.prec_dtype(prec)
    ga = torch.zeros(g.xf.shape, dtype=dt, device="cuda")
    gb = torch.zeros(g.xf.shape, dtype=dt, device="cuda")
    api.dy_backward(pdf, u1, u2, ga, XMIN, S, 1e-3, prec=prec)
    api.dy_backward(other, u1, u2, gb, XMIN, S, 1e-3, prec=prec)
    a = ga.double().cpu().numpy()
    b = gb.double().cpu().numpy()[perm]
    tol = 1e-12 if prec == "f64" else 1e-6
    np.testing.assert_allclose(a, b, rtol=tol, atol=tol * np.abs(a).max())


@pytest.mark.parametrize("prec", ["f64", "f32s"])
def test_integrand_backward_scale_range_and_nan(pdf, api, torch, prec):
    """The pair pass keeps its knot sums in 64-bit fixed point with a scale
    from a bound on its terms: a scale factor of 1e-200 or 1e200 scales the
    gradient alone; a NaN scale makes the quark and antiquark rows NaN and
    leaves the gluon row at zero."""
    g = cfg0_grid()
    u1, u2 = wl.dy_uniforms(6, 200_000)
    dt = api.prec_dtype(prec)

    def grad(scale):
        gr = torch.zeros(g.xf.shape, dtype=dt, device="cuda")
        api.dy_backward(pdf, u1, u2, gr, XMIN, S, scale, prec=prec)
        return gr.double().cpu().numpy()

    g0 = grad(1.0)
    big = np.abs(g0).max()
    tol = 1e-9 if prec == "f64" else 1e-6
    s_range = (1e-200, 1e200) if prec == "f64" else (1e-30, 1e30)   # FP32 output range
    for s in s_range:
        np.testing.assert_allclose(grad(s) / s, g0, rtol=tol, atol=tol * big)
    gn = grad(float("nan"))
    rows = {int(p): f for f, p in enumerate(g.pids)}
    for p in (1, 2, 3, 4, 5, -1, -2, -3, -4, -5):
        assert np.isnan(gn[rows[p]]).all()
    assert np.all(gn[rows[21]] == 0.0)


@pytest.mark.parametrize("prec", ["f64", "f32s"])
@pytest.mark.parametrize("nx,nq", [(4, 4), (9, 6), (100, 50), (50, 100), (71, 70), (81, 61),
                                   (27, 185), (98, 51)])
def test_gradient_is_the_directional_derivative(api, torch, nx, nq, prec):
    """sum I(v + h) - sum I(v - h) = 2 dI/dv h, exactly, I being quadratic in the knots:
    random values and random h, with the oracle's I, on the smallest grid, on sizes with
    0 to 3 lines in the last block of either axis, and on the largest.  Tolerance:
    FP64 rounding of n terms of 80 products each against the sum of their sizes; in
    FP32 the gradient's own rounding (2^-24 of each entry)."""
    rng = np.random.default_rng(1000 * nx + nq)
    x = np.exp(np.linspace(math.log(XMIN), 0.0, nx))
    q2 = np.exp(np.linspace(math.log(3.0), math.log(S), nq))
    base = cfg0_grid()
    vals = rng.uniform(0.5, 1.5, (len(base.pids), nx, nq)).astype(np.float32).astype(float)

    def spec(xf):
        return wl.GridSpec(pids=base.pids, x=x, q2=q2, q_off=np.array([0, nq], np.int32), xf=xf,
                           as_q2=base.as_q2, as_val=base.as_val)

    pdf = api.mkPDF(spec(vals))
    u1, u2 = wl.dy_uniforms(3, 3000)
    dt = torch.float64 if prec == "f64" else torch.float32
    grad = torch.zeros(pdf.shape, dtype=dt, device="cuda")
    api.dy_backward(pdf, u1, u2, grad, XMIN, S, prec=prec)
    grad = grad.double().cpu().numpy()
    h = rng.uniform(-0.5, 0.5, vals.shape)
    up, dn = (oracle.dy(spec(vals + f * h), u1, u2, XMIN, S) for f in (1, -1))
    size = np.abs(up).sum() + np.abs(dn).sum()
    tol = 1e-12 * size + (0 if prec == "f64" else 2.0 ** -24 * 2 * np.abs(grad * h).sum())
    assert abs((up - dn).sum() - 2 * (grad * h).sum()) <= tol
