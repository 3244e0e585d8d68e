"""Boxes whose three sides differ in elements and in length: FP64 applies against the oracle, level
transfers, operators and diagonals against dense products along each axis, and the V-cycle against its
definition. A kernel that takes one direction's nodes, weights or element size for another's is off by
the size of the result.

Tolerances: FP64 1e-12, FP32 level operators 1e-5, transfers 3e-6 (27 FP32 products in nested sums),
diagonals 2e-5 and cycles 2e-5, as for the cubes.
"""
import numpy as np
import pytest

from paper_2607_21150_amd import inputs as I
from test_gpu_mg_smoother import AXIS, FACES, FIELD, TOL, Cycle, dnorm, lagrange

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pf():
    from paper_2607_21150_amd import pfmf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    pfmf.load()
    return pfmf


def box(p, ne, sides=(1.0, 0.7, 1.3), seed=3):
    """Inputs of the form of make_inputs on ne elements: strains of 1 %, a phase-field bump, two phases, an
    isochoric state, random directions."""
    rng = np.random.default_rng(seed)
    mesh = I.Mesh(p, *ne, *sides)
    phases = I.default_phases()
    gll = I.gll_points(p)
    nx1, ny1, nz1 = mesh.node_dims
    X, Y, Z = (I._coords_1d(n, p, s, gll) for n, s in zip(ne, sides))
    x, y, z = X[None, None, :], Y[None, :, None], Z[:, None, None]
    v = np.zeros((4, nz1, ny1, nx1))
    v[0] = 4e-3 * np.sin(2 * x + 3 * y - z)
    v[1] = 3e-3 * np.cos(x - 2 * y + 2 * z)
    v[2] = 1e-2 * z + 3e-3 * np.sin(x + y + 3 * z)
    v[3] = 0.6 * np.exp(-8.0 * ((x - 0.4) ** 2 + (y - 0.2) ** 2 + (z - 0.9) ** 2))
    v = v.reshape(4, -1)
    state = np.zeros((8, mesh.n_q))
    a = rng.uniform(-1e-4, 1e-4, size=(2, mesh.n_q))
    state[0], state[1] = np.expm1(a[0]), np.expm1(a[1])
    state[2] = np.expm1(-a[0] - a[1])
    state[6] = rng.uniform(0.0, 1e-2, size=mesh.n_q)
    state[7] = rng.uniform(0.0, 0.2, size=mesh.n_q)
    unit = lambda: (lambda r: r / np.linalg.norm(r))(rng.standard_normal((4, mesh.n_nodes)))
    return dict(mesh=mesh, phases=phases, fracture=I.default_fracture(mesh, phases), z=v, phi_n=0.99 * v[3], state=state,
                phase=(rng.uniform(size=mesh.n_q) < 0.3).astype(np.uint8), dz=unit(), v_rand=unit())


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).to("cuda", torch.float64)


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("p,ne", [(1, (3, 5, 2)), (2, (3, 5, 4)), (2, (6, 1, 3)), (3, (3, 5, 2)), (3, (1, 4, 6)), (4, (2, 1, 3)),
                                  (4, (3, 4, 1))])
@pytest.mark.parametrize("scatter", ["colour", "brick_buffer"])
def test_fp64_applies(pf, oracle_lib, p, ne, scatter):
    d = box(p, ne)
    ctx, orc = pf.Context.from_inputs(d), oracle_lib.Oracle.from_inputs(d)
    ctx.set_scatter(scatter)
    z, dz, v = dev(d["z"]), dev(d["dz"]), dev(d["v_rand"])
    jac = orc.jacobian(d["z"], d["dz"])
    assert rel(ctx.apply_residual(z).cpu().numpy(), orc.residual(d["z"])) <= 1e-12
    assert rel(ctx.apply_jacobian(z, dz).cpu().numpy(), jac) <= 1e-12
    assert rel(ctx.apply_adjoint(z, v)[0].cpu().numpy(), orc.adjoint(d["z"], d["v_rand"])[0]) <= 1e-12
    if p >= 2:
        ctx.linearize(z)
        assert rel(ctx.apply_jacobian_lin(dz).cpu().numpy(), jac) <= 1e-12
    ctx.check()


def lattices(ne, levels):
    """(order, elements per direction) of every level."""
    out, n = [], tuple(ne)
    for l, q in enumerate(levels):
        if l > 0 and q == 1 and levels[l - 1] == 1:
            n = tuple(k // 2 for k in n)
        out.append((q, n))
    return out


def mask(lat, faces):
    q, n = lat
    m = torch.ones((4, q * n[2] + 1, q * n[1] + 1, q * n[0] + 1), dtype=torch.float64, device="cuda")
    for face, fields in (faces or {}).items():
        for f in fields:
            m[FIELD[f]].select(AXIS[face[0]], -1 if face[1] == "1" else 0).zero_()
    return m.reshape(4, -1)


def rows(fine, coarse, axis):
    """Dense interpolation along one direction (0 = x), coarse to fine level."""
    (q, n), (r, nc) = (fine[0], fine[1][axis]), (coarse[0], coarse[1][axis])
    P = np.zeros((q * n + 1, r * nc + 1))
    if nc != n:
        for i in range(n + 1):
            P[i, i // 2] += 0.5
            P[i, (i + 1) // 2] += 0.5
    else:
        B = lagrange(np.asarray(I.gll_points(r)), np.asarray(I.gll_points(q)))
        for e in range(n):
            P[q * e:q * e + q + 1, r * e:r * e + r + 1] = B
    return torch.as_tensor(P).cuda()


def along(P, x):
    """P = (x, y, z) matrices applied to x[4][nodes]."""
    v = x.double().reshape(4, P[2].shape[1], P[1].shape[1], P[0].shape[1])
    for a in range(3):
        v = torch.movedim(torch.tensordot(v, P[a], ([3 - a], [1])), -1, 3 - a)
    return v.reshape(4, -1)


LISTS = [(3, (3, 5, 4), [3, 2, 1], "brick_buffer"), (2, (6, 2, 4), [2, 1, 1], "brick_buffer"), (4, (3, 2, 5), [4, 2], "colour"),
         (4, (2, 3, 1), [4, 3, 2, 1], "brick_buffer"), (3, (8, 4, 2), [3, 1, 1], "colour"),
         (3, (40, 2, 3), [3, 2], "brick_buffer"), (2, (2, 3, 36), [2, 1], "brick_buffer"), (2, (4, 12, 8), [2, 1, 1, 1], "brick_buffer")]


@pytest.mark.parametrize("p,ne,levels,scatter", LISTS)
@pytest.mark.parametrize("faces", [None, FACES], ids=["free", "faces"])
def test_levels(pf, p, ne, levels, scatter, faces):
    d = box(p, ne)
    lat = lattices(ne, levels)
    ctx = pf.Context.from_inputs(d)
    ctx.set_scatter(scatter)
    ctx.set_pmg_levels(levels)
    if faces:
        ctx.set_dirichlet(faces)
    z = dev(d["z"])
    ctx.linearize(z)
    ctx.check()
    torch.manual_seed(5)
    M = [mask(a, faces) for a in lat]
    total = None  # interpolation from level l to the fine level
    for l in range(len(levels)):
        n = M[l].shape[1]
        assert ctx.level_info(l)[1] == n
        # operator: M P^T J P x with the FP64 Jacobian
        x = torch.randn(4, n, device="cuda")
        f = x.double() if total is None else along(total, x)
        ref = ctx.apply_jacobian(z, f)
        ref = (ref if total is None else along([q.T.contiguous() for q in total], ref)) * M[l]
        y = ctx.apply_jacobian_f32(l, x).double()
        err = float(torch.linalg.norm(y - ref) / torch.linalg.norm(ref))
        assert err <= 1e-5, ("operator", l, err)
        # diagonal against the level's own applies: nodes 2 or order + 1 apart share no element (unmasked entries)
        q, (nx, ny, nz) = lat[l]
        shape = (4, q * nz + 1, q * ny + 1, q * nx + 1)
        got, ref = ctx.level_diagonal(l).reshape(shape).double(), torch.zeros(shape, dtype=torch.float64, device="cuda")
        for f in range(4):
            for c in range((q + 1) ** 3):
                s = np.s_[f, c // (q + 1) ** 2::q + 1, c // (q + 1) % (q + 1)::q + 1, c % (q + 1)::q + 1]
                e = torch.zeros(shape, device="cuda")
                e[s] = 1.0
                ref[s] = ctx.apply_jacobian_f32(l, e.reshape(4, n)).double().reshape(shape)[s]
        free = M[l].reshape(shape)
        err = float(torch.linalg.norm((got - ref) * free) / torch.linalg.norm(ref))
        assert err <= 2e-5, ("diagonal", l, err)
        if l + 1 == len(levels):
            break
        P = [rows(lat[l], lat[l + 1], a) for a in range(3)]
        xc = torch.randn(4, M[l + 1].shape[1], device="cuda")
        ref = along(P, xc) * M[l]
        err = float(torch.linalg.norm(ctx.prolong(l, xc).double() - ref) / torch.linalg.norm(ref))
        assert err <= 3e-6, ("prolong", l, err)
        ref = along([q.T.contiguous() for q in P], x) * M[l + 1]
        err = float(torch.linalg.norm(ctx.restrict(l, x).double() - ref) / torch.linalg.norm(ref))
        assert err <= 3e-6, ("restrict", l, err)
        total = P if total is None else [a @ b for a, b in zip(total, P)]


class BoxCycle(Cycle):
    def __init__(self, ctx, lat, faces):
        self.ctx, self.n = ctx, len(lat)
        self.mask = [mask(a, faces) for a in lat]
        self.dinv = [1.0 / ctx.level_diagonal(l).double() for l in range(len(lat))]


@pytest.mark.parametrize("p,ne,levels,scatter", LISTS)
def test_cycle(pf, p, ne, levels, scatter):
    d = box(p, ne)
    lat = lattices(ne, levels)
    ctx = pf.Context.from_inputs(d)
    ctx.set_scatter(scatter)
    ctx.set_pmg_levels(levels)
    ctx.set_dirichlet(FACES)
    ctx.linearize(dev(d["z"]))
    ctx.check()
    ref = BoxCycle(ctx, lat, FACES)
    b = torch.as_tensor(np.random.default_rng(5).standard_normal((4, d["mesh"].n_nodes))).to("cuda", torch.float32)
    inv_theta = [1.0 / (0.6 * ref.lmax(l)) for l in range(len(levels))]
    for degree, sweeps in ((1, 3), (3, 2)):
        x = ctx.pmg_vcycle(b, cheb_degree=degree, coarse_p=levels[-1], coarse_sweeps=sweeps).double()
        y = ref.run(0, ref.mask[0] * b.double(), inv_theta, degree, sweeps)
        err = dnorm(x - y, ref.dinv[0]) / dnorm(y, ref.dinv[0])
        assert err <= TOL, (degree, sweeps, err)
