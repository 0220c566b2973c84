"""The routed forward kernel (large calls: the grid cut into pieces that stay in
LDS) against the kernels that cycle the grid through LDS, which a set launch
shape selects: same bins, weights and order of sums, so the same bits."""
import numpy as np
import pytest

import oracle
from helpers import capped_rel_err, cfg0_grid
from paper_2012_08221_amd import workloads as wl

pytestmark = pytest.mark.gpu

N = 3_000_003   # past the point where every grid's calls are routed, no multiple of a tile


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


def points(torch, g, n, seed, xlo=1e-9, xhi=1.0):
    """x log-uniform in [xlo, xhi] and Q^2 over the grid, all knots and thresholds
    among them."""
    rng = np.random.default_rng(seed)
    x = np.exp(rng.uniform(np.log(xlo), np.log(xhi), n))
    q2 = np.exp(rng.uniform(np.log(g.q2[0]), np.log(g.q2[-1]), n))
    k = min(n, g.n_x * g.n_q)
    at = rng.choice(n, k, replace=False)
    if xlo <= g.x[0] and xhi >= g.x[-1]:
        x[at] = np.tile(g.x, g.n_q)[:k]
    q2[at] = np.repeat(g.q2, g.n_x)[:k]
    x, q2 = np.clip(x, g.x[0], g.x[-1]), np.clip(q2, g.q2[0], g.q2[-1])
    return torch.as_tensor(x, device="cuda"), torch.as_tensor(q2, device="cuda")


def equal(a, b):
    np.testing.assert_array_equal(a.cpu().numpy(), b.cpu().numpy())


# (n_x, subgrids, n_q): the 100 x 50 grid, grids cut along x and along Q^2 into a
# few and into many pieces, one piece, the smallest axes
GRIDS = [(100, 3, 50), (200, 4, 80), (60, 4, 79), (200, 2, 21), (50, 2, 20), (9, 2, 8)]


@pytest.mark.parametrize("prec", ["f64", "f32s"])
@pytest.mark.parametrize("geo", GRIDS)
def test_same_bits_every_grid(api, torch, geo, prec):
    nx, nsub, nq = geo
    g = wl.make_grid(wl.draw_params(np.random.default_rng(5)), nx, wl.MEMBER_EDGES[nsub], nq)
    pdf = api.PDF(g)
    x, q2 = points(torch, g, N, 1)
    got = pdf.xfxQ2(g.pids, x, q2, prec=prec)
    pdf.set_launch(prec, 512, 1)
    equal(got, pdf.xfxQ2(g.pids, x, q2, prec=prec))


@pytest.mark.parametrize("prec", ["f64", "f32s"])
@pytest.mark.parametrize("n_req", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11])
def test_every_number_of_partons(api, torch, n_req, prec):
    g = cfg0_grid()
    pids = list(np.random.default_rng(n_req).permutation(g.pids)[:n_req])
    routed, cycled = api.PDF(g), api.PDF(g)
    cycled.set_launch(prec, 512, 1)
    x, q2 = points(torch, g, N, 2)
    equal(routed.xfxQ2(pids, x, q2, prec=prec), cycled.xfxQ2(pids, x, q2, prec=prec))


@pytest.mark.parametrize("prec", ["f64", "f32s"])
@pytest.mark.parametrize("domain", ["nan", "clamp", "extrapolate"])
def test_domain_modes_and_counts(api, torch, prec, domain):
    g = cfg0_grid()
    routed, cycled = api.PDF(g), api.PDF(g)
    cycled.set_launch(prec, 512, 1)
    x, q2 = points(torch, g, N, 3)
    x[::97] *= 1e-3
    x[5::101] = 1.5
    q2[::89] *= 1e-2
    q2[7::103] *= 1e8
    x[11::1009] = float("nan")
    q2[13::1013] = float("nan")
    equal(routed.xfxQ2(g.pids, x, q2, prec=prec, domain=domain),
          cycled.xfxQ2(g.pids, x, q2, prec=prec, domain=domain))
    assert routed.domain_errors() == cycled.domain_errors()
    if domain != "extrapolate":
        a, b = (p.xfx_alphasQ2(g.pids, x, q2, prec=prec, domain=domain) for p in (routed, cycled))
        equal(a[0], b[0])
        equal(a[1], b[1])
        assert routed.domain_errors() == cycled.domain_errors()


@pytest.mark.parametrize("prec", ["f64", "f32s"])
@pytest.mark.parametrize("axis", ["x", "q"])
def test_points_where_the_sample_has_none(api, torch, prec, axis):
    """All sampled points (and nearly all others) in a few intervals at the upper
    end, the rest spread over the axis: these belong to no piece."""
    g = wl.make_grid(wl.draw_params(np.random.default_rng(6)), *(
        (200, wl.MEMBER_EDGES[4], 40) if axis == "x" else (60, wl.MEMBER_EDGES[4], 79)))
    routed, cycled = api.PDF(g), api.PDF(g)
    cycled.set_launch(prec, 512, 1)
    x, q2 = points(torch, g, N, 4, xlo=0.1, xhi=0.9)
    if axis == "q":
        q2 = q2.clamp(min=1e6)
    far = torch.ones(N, dtype=torch.bool, device="cuda")
    for s in (1024, 768, 1536):   # leave every point that a sample could take
        far[(torch.arange(s, device="cuda") * N) // s] = False
    far &= torch.rand(N, device="cuda") < 0.01
    fx, fq = points(torch, g, N, 5)
    x, q2 = torch.where(far, fx, x), torch.where(far, fq, q2)
    q2[int(far.nonzero()[0])] = float("nan")
    for domain in ("nan", "clamp"):
        a, b = (p.xfx_alphasQ2(g.pids, x, q2, prec=prec, domain=domain) for p in (routed, cycled))
        equal(a[0], b[0])
        np.testing.assert_allclose(a[1].cpu().numpy(), b[1].cpu().numpy(),
                                   rtol=1e-14 if prec == "f64" else 1e-6)
        assert routed.domain_errors() == cycled.domain_errors()


@pytest.mark.parametrize("prec", ["f64", "f32s"])
def test_caller_values_q_input_odd_requests(api, torch, prec):
    g = cfg0_grid()
    routed, cycled = api.PDF(g), api.PDF(g)
    cycled.set_launch(prec, 512, 1)
    x, q2 = points(torch, g, N, 6)
    vals = torch.as_tensor(g.xf * 1.25 + 0.5, dtype=api.prec_dtype(prec), device="cuda")
    equal(routed.xfxQ(g.pids, x, q2.sqrt(), prec=prec, domain="clamp", values=vals),
          cycled.xfxQ(g.pids, x, q2.sqrt(), prec=prec, domain="clamp", values=vals))
    # repeated and absent partons keep the other kernels
    pids = [21, 3, 21, 22, 0, -3]
    equal(routed.xfxQ2(pids, x, q2, prec=prec), cycled.xfxQ2(pids, x, q2, prec=prec))
    # an output that is aligned to one value only
    size = N * 11
    buf = torch.zeros(size + 1, dtype=api.prec_dtype(prec), device="cuda")
    out = buf[1:].view(N, 11)
    routed.xfxQ2(g.pids, x, q2, prec=prec, out=out)
    equal(out, cycled.xfxQ2(g.pids, x, q2, prec=prec))


@pytest.mark.parametrize("prec,n", [("f64", 48_003), ("f32s", 48_003), ("f64", 65_536), ("f32s", 65_536)])
def test_set_members_equal_single_grids(api, torch, prec, n):
    specs = wl.member_grids(13)
    pset = api.PDFSet(specs)
    x, q2 = points(torch, specs[0], n, 7, xlo=1e-7, xhi=0.99)
    q2 = q2.clamp(4.0, 1e8)
    x[::501] = 2.0
    got = pset.xfxQ2([21, 1, -2, 5, 3], x, q2, prec=prec)
    out = 0
    for m, s in enumerate(specs):
        pdf = api.PDF(s)
        equal(got[m], pdf.xfxQ2([21, 1, -2, 5, 3], x, q2, prec=prec))
        out += pdf.domain_errors()
    assert pset.domain_errors() == out


@pytest.mark.parametrize("prec,tol", [("f64", 1e-12), ("f32s", 1e-5)])
def test_against_the_oracle(api, torch, prec, tol):
    g = cfg0_grid()
    x, q2 = points(torch, g, N, 8)
    got = api.PDF(g).xfxQ2(g.pids, x, q2, prec=prec).double().cpu().numpy()
    at = np.random.default_rng(9).choice(N, 20_000, replace=False)
    xs, qs = x.cpu().numpy()[at], q2.cpu().numpy()[at]
    ref = oracle.xfx(g, g.pids, xs, qs)
    M = oracle.stencil_absmax(g, g.pids, xs, qs)
    assert capped_rel_err(got[at], ref, M).max() <= tol


# ---- the routed integrand ----

def dy_both(api, torch, g, u1, u2, prec, **kw):
    routed, cycled = api.PDF(g), api.PDF(g)
    cycled.set_dy_launch(prec, 512, 1)
    (a, sa), (b, sb) = (api.dy_integrand(p, u1, u2, prec=prec, **kw) for p in (routed, cycled))
    equal(a, b)
    assert routed.domain_errors() == cycled.domain_errors()
    if not torch.isnan(a).any():
        # both sum the same values in FP64, in another order
        bound = a.shape[0] * 2.0 ** -53 * float(a.double().abs().sum())
        assert abs(float(sa.sum()) - float(sb.sum())) <= bound
    return a


@pytest.mark.parametrize("prec", ["f64", "f32s"])
@pytest.mark.parametrize("geo", [(100, 3, 50), (60, 2, 30), (62, 4, 79), (100, 4, 48), (40, 2, 120), (9, 2, 8)])
def test_integrand_same_bits(api, torch, geo, prec):
    nx, nsub, nq = geo
    g = wl.make_grid(wl.draw_params(np.random.default_rng(11)), nx, wl.MEMBER_EDGES[nsub], nq)
    gen = torch.Generator(device="cuda").manual_seed(12)
    u1, u2 = (torch.rand(N, generator=gen, device="cuda", dtype=torch.float64) for _ in range(2))
    # products of x on and beside the thresholds and the ends of the Q^2 axis
    k = 0
    for q2 in list(g.q2[np.array(g.q_off[1:-1])]) + [g.q2[0], g.q2[-1]]:
        lim = np.log(q2 / 13000.0 ** 2) / np.log(1e5) + 2.0      # u1 + u2 at this Q^2
        v = torch.linspace(max(0.0, lim - 1.0), min(1.0, lim), 2000, device="cuda", dtype=torch.float64)
        for d in (-1e-15, 0.0, 1e-15):
            u1[k:k + 2000], u2[k:k + 2000] = v, (lim - v + d).clamp(0.0, 1.0)
            k += 2000
    dy_both(api, torch, g, u1, u2, prec)


@pytest.mark.parametrize("prec", ["f64", "f32s"])
def test_integrand_odd_inputs(api, torch, prec):
    g = wl.make_grid(wl.draw_params(np.random.default_rng(13)), 100, wl.MEMBER_EDGES[3], 50)
    gen = torch.Generator(device="cuda").manual_seed(14)
    u1, u2 = (torch.rand(N, generator=gen, device="cuda", dtype=torch.float64) for _ in range(2))
    u1[::1001] = 1.5        # x > 1: outside
    u2[7::1003] = float("nan")
    dy_both(api, torch, g, u1, u2, prec)
    vals = torch.as_tensor(g.xf * 0.75, dtype=api.prec_dtype(prec), device="cuda")
    dy_both(api, torch, g, u1, u2, prec, values=vals)
    # all sampled points at high Q^2, a few of the others anywhere
    far = torch.rand(N, device="cuda") < 0.01
    for s in (1024, 768, 1536):
        far[(torch.arange(s, device="cuda") * N) // s] = False
    v1, v2 = (torch.where(far, u, 0.9 + 0.1 * u.nan_to_num(0.5).clamp(0.0, 1.0)) for u in (u1, u2))
    dy_both(api, torch, g, v1, v2, prec)


@pytest.mark.parametrize("prec", ["f64", "f32s"])
@pytest.mark.parametrize("quarks", [1, 2, 3, 4])
def test_integrand_fewer_quarks(api, torch, quarks, prec):
    g = wl.make_grid(wl.draw_params(np.random.default_rng(15)), 60, wl.MEMBER_EDGES[3], 40)
    keep = [i for i, p in enumerate(g.pids) if p == 21 or abs(p) <= quarks]
    g.pids, g.xf = g.pids[keep], np.ascontiguousarray(g.xf[keep])
    gen = torch.Generator(device="cuda").manual_seed(16)
    u1, u2 = (torch.rand(N, generator=gen, device="cuda", dtype=torch.float64) for _ in range(2))
    dy_both(api, torch, g, u1, u2, prec)


# ---- the direct kernel of small calls and the group kernel above it ----

@pytest.mark.parametrize("prec", ["f64", "f32s"])
@pytest.mark.parametrize("geo", [(100, 3, 50), (190, 4, 75), (9, 2, 8), (110, 2, 70)])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 3001, 60_001, 300_007])
def test_small_calls_same_bits(api, torch, geo, n, prec):
    nx, nsub, nq = geo
    g = wl.make_grid(wl.draw_params(np.random.default_rng(21)), nx, wl.MEMBER_EDGES[nsub], nq)
    direct, cycled = api.PDF(g), api.PDF(g)
    cycled.set_launch(prec, 512, 1)
    x, q2 = points(torch, g, n, 22)
    if n > 64:
        x[::7] *= 1e-2
        q2[::11] *= 1e6
        x[3::13] = float("nan")
    vals = torch.as_tensor(g.xf * 1.25 + 0.5, dtype=api.prec_dtype(prec), device="cuda")
    buf = torch.zeros(n * 11 + 1, dtype=api.prec_dtype(prec), device="cuda")
    for domain in ("nan", "clamp"):
        for pids in (list(g.pids), [21], [3, -5], [2, 22, 2, 0, 21, -4, 2], [22], list(g.pids[::-1])):
            for v in (None, vals):
                equal(direct.xfxQ2(pids, x, q2, prec=prec, domain=domain, values=v),
                      cycled.xfxQ2(pids, x, q2, prec=prec, domain=domain, values=v))
                assert direct.domain_errors() == cycled.domain_errors()
        a, b = (p.xfx_alphasQ2(g.pids, x, q2, prec=prec, domain=domain) for p in (direct, cycled))
        equal(a[0], b[0])
        # alpha_s from the point's Q^2 weights here, in a pass of its own on the larger grid
        np.testing.assert_allclose(a[1].cpu().numpy(), b[1].cpu().numpy(),
                                   rtol=1e-14 if prec == "f64" else 1e-6)
        assert direct.domain_errors() == cycled.domain_errors()
        out = buf[1:].view(n, 11)
        direct.xfxQ(g.pids, x, q2.sqrt(), prec=prec, domain=domain, out=out)
        equal(out, cycled.xfxQ(g.pids, x, q2.sqrt(), prec=prec, domain=domain))
