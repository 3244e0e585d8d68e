"""The V-cycle and the level diagonals against their definitions, written with the level applies.

A Chebyshev step, a level residual, the smoother's start and the Dirichlet masks run inside the
node gather, the block stencil or a launch after the colours; here the same cycle is composed in
FP64 vectors from pf_apply_jacobian_f32, pf_prolong, pf_restrict and pf_level_diagonal, with the
smoother's bound from the same 15 power iterations on the same start (splitmix64 of the entry).

Tolerance: both sides apply the same FP32 level operators, so they differ by the FP32 rounding of
the vectors between them. At most 30 applies, each followed by some 4 roundings of 6e-8 on terms
that the smoother scales by at most 1.1 lmax / theta = 1.8: 30 * 4 * 6e-8 * 1.8 = 1.3e-5, taken as
2e-5 in the norm of the diagonal. A wrong coefficient, mask or vector is off by 1e-2 or more.
"""
import numpy as np
import pytest

from paper_2607_21150_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
TOL = 2e-5
FACES = {"z0": ("uz",), "z1": ("ux", "uz"), "x0": ("ux", "phi"), "y1": ("uy",)}
AXIS = {"x": 2, "y": 1, "z": 0}
FIELD = {"ux": 0, "uy": 1, "uz": 2, "phi": 3}


@pytest.fixture(scope="module")
def pf():
    from paper_2607_21150_amd import pfmf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    pfmf.load()
    return pfmf


def make_ctx(pf, d, levels, scatter, faces):
    ctx = pf.Context.from_inputs(d)
    ctx.set_scatter(scatter)
    ctx.set_pmg_levels(levels)
    if faces:
        ctx.set_dirichlet(faces)
    ctx.linearize(torch.as_tensor(d["z"]).to("cuda", torch.float64))
    ctx.check()
    return ctx


def free_mask(n_nodes, faces):
    n1 = round(n_nodes ** (1 / 3))
    m = torch.ones((4, n1, n1, n1), dtype=torch.float64, device="cuda")
    for face, fields in (faces or {}).items():
        for f in fields:
            m[FIELD[f]].select(AXIS[face[0]], -1 if face[1] == "1" else 0).zero_()
    return m.reshape(4, -1)


class Cycle:
    def __init__(self, ctx, n_levels, faces):
        self.ctx, self.n = ctx, n_levels
        self.mask = [free_mask(ctx.level_info(l)[1], faces) for l in range(n_levels)]
        self.dinv = [1.0 / ctx.level_diagonal(l).double() for l in range(n_levels)]

    def A(self, l, x):
        return self.mask[l] * self.ctx.apply_jacobian_f32(l, x.float()).double()

    def smooth(self, l, b, x, degree, inv_theta):
        """theta = 0.6 lmax, delta = 0.5 lmax: the interval [0.1, 1.1] lmax."""
        theta = 1.0 / inv_theta
        delta, sigma = theta * 0.5 / 0.6, 0.6 / 0.5
        rho = 1.0 / sigma
        r = b if x is None else b - self.A(l, x)
        d = self.dinv[l] * r / theta
        x = d if x is None else x + d
        for _ in range(degree - 1):
            r = r - self.A(l, d)
            rn = 1.0 / (2.0 * sigma - rho)
            d = rn * rho * d + 2.0 * rn / delta * self.dinv[l] * r
            x = x + d
            rho = rn
        return x

    def lmax(self, l):
        n = self.dinv[l].numel()
        with np.errstate(over="ignore"):
            z = np.uint64(21150 + l) + np.uint64(0x9E3779B97F4A7C15) * np.arange(1, n + 1, dtype=np.uint64)
            z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
            z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
            z = z ^ (z >> np.uint64(31))
        v = torch.as_tensor((z >> np.uint64(11)).astype(np.float64) / 2.0 ** 52 - 1.0).cuda().reshape(4, -1)
        v = v * self.mask[l]
        for _ in range(15):
            v = self.dinv[l] * self.A(l, v / torch.linalg.norm(v))
        return float(torch.linalg.norm(v))

    def run(self, l, b, inv_theta, degree, sweeps):
        if l == self.n - 1:
            x = None
            for _ in range(sweeps):
                x = self.smooth(l, b, x, degree, inv_theta[l])
            return x
        x = self.smooth(l, b, None, degree, inv_theta[l])
        r = b - self.A(l, x)
        rc = self.mask[l + 1] * self.ctx.restrict(l, r.float()).double()
        xc = self.run(l + 1, rc, inv_theta, degree, sweeps)
        x = x + self.mask[l] * self.ctx.prolong(l, xc.float()).double()
        return self.smooth(l, b, x, degree, inv_theta[l])


def dnorm(x, dinv):
    return float(torch.sqrt((x * x / dinv).sum()))


@pytest.mark.parametrize("p,n,levels,scatter,faces", [
    (4, 3, [4, 2, 1], "brick_buffer", FACES), (4, 3, [4, 2], "colour", FACES), (4, 17, [4, 2], "brick_buffer", None),
    (3, 5, [3, 2], "brick_buffer", FACES), (3, 4, [3, 2, 1, 1], "colour", FACES),
    (3, 22, [3, 1], "brick_buffer", FACES), (3, 43, [3, 2], "brick_buffer", FACES),
    (2, 4, [2, 1], "brick_buffer", FACES), (3, 5, [3, 1], "brick_buffer", FACES),  # 125 and 216 coarsest nodes
    (2, 1, [2, 1], "brick_buffer", None), (2, 4, [2, 1, 1], "brick_buffer", FACES), (2, 33, [2, 1], "brick_buffer", None)])
def test_cycle_matches_its_definition(pf, p, n, levels, scatter, faces):
    print(f"case p={p} n={n} {levels} {scatter} faces={bool(faces)}", flush=True)
    d = I.make_inputs("C1", "base", p=p, n=n)
    nn = d["mesh"].n_nodes
    b = torch.as_tensor(np.random.default_rng(5).standard_normal((4, nn))).to("cuda", torch.float32)
    bm = free_mask(nn, faces) * b.double()
    ctx = make_ctx(pf, d, levels, scatter, faces)
    ref = Cycle(ctx, len(levels), faces)
    w = ref.dinv[0]
    inv_theta = [1.0 / (0.6 * ref.lmax(l)) for l in range(len(levels))]
    for degree, sweeps in ((1, 3), (2, 1), (3, 2), (4, 1)):
        x = ctx.pmg_vcycle(b, cheb_degree=degree, coarse_p=levels[-1], coarse_sweeps=sweeps).double()
        y = ref.run(0, bm, inv_theta, degree, sweeps)
        err = dnorm(x - y, w) / dnorm(y, w)
        print(f"  degree {degree} sweeps {sweeps}: {err:.2e}", flush=True)
        assert err <= TOL, (degree, sweeps, err)


@pytest.mark.parametrize("p,n,levels", [(4, 1, [4, 3, 2]), (4, 3, [4, 2]), (3, 3, [3, 2]), (3, 5, [3, 1]), (2, 5, [2, 1])])
@pytest.mark.parametrize("variant", ["plastic", "ex3"])
def test_level_diagonals_match_the_level_applies(pf, p, n, levels, variant):
    """Nodes p + 1 apart share no element, so one apply gives all diagonal entries of a colour.
    Element counts that fill no workgroup, and level lists without an order-1 level. FP32 applies
    and diagonals each within 1e-5 of FP64: 2e-5."""
    d = I.make_inputs("C1", variant, p=p, n=n)
    ctx = make_ctx(pf, d, levels, "brick_buffer", None)
    for l, q in enumerate(levels):
        _, nl = ctx.level_info(l)
        n1 = q * n + 1
        got = ctx.level_diagonal(l).reshape(4, n1, n1, n1)
        ref = torch.zeros_like(got)
        for f in range(4):
            for c in range((q + 1) ** 3):
                s = np.s_[f, c // (q + 1) ** 2::q + 1, c // (q + 1) % (q + 1)::q + 1, c % (q + 1)::q + 1]
                e = torch.zeros_like(got)
                e[s] = 1.0
                ref[s] = ctx.apply_jacobian_f32(l, e.reshape(4, nl)).reshape(4, n1, n1, n1)[s]
        for f in range(4):
            err = float(torch.linalg.norm(got[f] - ref[f]) / torch.linalg.norm(ref[f]))
            assert err <= 2e-5, (l, f, err)


def lagrange(xc, xf):
    B = np.ones((len(xf), len(xc)))
    for j in range(len(xc)):
        for k in range(len(xc)):
            if k != j:
                B[:, j] *= (xf - xc[k]) / (xc[j] - xc[k])
    return B


@pytest.mark.parametrize("p,n,levels", [(4, 20, [4, 3]), (3, 32, [3, 2]), (2, 44, [2, 1, 1]), (4, 2, [4, 3]), (3, 1, [3, 1])])
def test_transfers_match_dense_rows(pf, p, n, levels):
    """Sizes on both sides of the rule for the outputs per thread, masked faces. Three nested sums of
    at most 9 terms in FP32 with weights up to 1.2: 27 * 6e-8 * 1.2^3 = 2.8e-6, taken as 3e-6."""
    d = I.make_inputs("C1", "base", p=p, n=n)
    ctx = make_ctx(pf, d, levels, "brick_buffer", FACES)
    torch.manual_seed(3)
    ne = n
    for l, (q, r) in enumerate(zip(levels[:-1], levels[1:])):
        nc = ne // 2 if q == 1 else ne
        P = np.zeros((q * ne + 1, r * nc + 1))
        if q == 1:
            for i in range(ne + 1):
                P[i, i // 2] += 0.5
                P[i, (i + 1) // 2] += 0.5
        else:
            B = lagrange(np.asarray(I.gll_points(r)), np.asarray(I.gll_points(q)))
            for e in range(ne):
                P[q * e:q * e + q + 1, r * e:r * e + r + 1] = B
        P = torch.as_tensor(P).cuda()
        kf, kc = P.shape
        mf, mc = free_mask(kf ** 3, FACES), free_mask(kc ** 3, FACES)
        ap = lambda M, x: torch.stack([torch.tensordot(M, torch.tensordot(M, torch.tensordot(M, x[f], ([1], [2])), ([1], [2])),
                                                       ([1], [2])) for f in range(4)])
        x = torch.randn(4, kc ** 3, device="cuda")
        ref = ap(P, x.double().reshape(4, kc, kc, kc)).reshape(4, -1) * mf
        err = float(torch.linalg.norm(ctx.prolong(l, x).double() - ref) / torch.linalg.norm(ref))
        assert err <= 3e-6, ("prolong", l, err)
        y = torch.randn(4, kf ** 3, device="cuda")
        ref = ap(P.T.contiguous(), y.double().reshape(4, kf, kf, kf)).reshape(4, -1) * mc
        err = float(torch.linalg.norm(ctx.restrict(l, y).double() - ref) / torch.linalg.norm(ref))
        assert err <= 3e-6, ("restrict", l, err)
        ne = nc


@pytest.mark.parametrize("p", [2, 3, 4])
@pytest.mark.parametrize("stretch", [0.0, 0.25, 0.6, 1.5])
def test_level_apply_at_large_strain_differences(pf, p, stretch):
    """The FP32 record forms the off-diagonal tangent factors from the differences of the principal
    log strains, by a series up to 1/2 and by exponentials above: differences about 0, on both sides
    of the limit and up to 1.3. Bar of the FP32 applies: 1e-5 of FP64."""
    d = I.make_inputs("C1", "base", p=p, n=3)
    m = d["mesh"]
    gll = np.asarray(I.gll_points(p))
    x = I._coords_1d(m.nx, p, m.lx, gll)
    z = np.array(d["z"], copy=True)
    n1 = len(x)
    z[0] += stretch * np.tile(x, n1 * n1)
    z[1] -= 0.25 * stretch * np.tile(np.repeat(x, n1), n1)
    z = torch.as_tensor(z).to("cuda", torch.float64)
    ctx = pf.Context.from_inputs(d)
    ctx.linearize(z)
    ctx.check()
    torch.manual_seed(4)
    v = torch.randn(4, m.n_nodes, device="cuda")
    y, ref = ctx.apply_jacobian_f32(0, v).double(), ctx.apply_jacobian(z, v.double())
    err = float(torch.linalg.norm(y - ref) / torch.linalg.norm(ref))
    assert err <= 1e-5, err
