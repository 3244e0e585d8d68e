"""FP64 residual, Jacobian and adjoint at homogeneous stretches far outside the small strains of the
other inputs: values against the oracle, and their cost against the cost at small strains.

The log coefficients of the point function are a polynomial sum up to principal log strains 5 % off
their mean and a quadrature rule beyond, chosen by a bound of the ratio of the largest to the
smallest eigenvalue of b_tr (limits 1.45, 4.2, 16, 53, 155, 1250 with the tangent and 1.72, 5.4, 21.9, 74, 245,
2180 without, panels of 12 nodes beyond); the stretches lie on both sides of each limit.
"""
import numpy as np
import pytest

from paper_2607_21150_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pf():
    from paper_2607_21150_amd import pfmf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    pfmf.load()
    return pfmf


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).to("cuda", torch.float64)


def stretched(d, kind, s):
    """The inputs' z plus the homogeneous deformation of stretch s: iso = isochoric uniaxial along z,
    one = along z alone, shear = s along x and 1 / s along y."""
    g = {"iso": (s ** -0.5, s ** -0.5, s), "one": (1.0, 1.0, s), "shear": (s, 1.0 / s, 1.0)}[kind]
    m = d["mesh"]
    gll = I.gll_points(m.p)
    nx1, ny1, nz1 = m.node_dims
    X, Y, Z = (I._coords_1d(n, m.p, 1.0, gll) for n in (m.nx, m.ny, m.nz))
    z = np.array(d["z"], copy=True).reshape(4, nz1, ny1, nx1)
    z[0] += (g[0] - 1.0) * X[None, None, :]
    z[1] += (g[1] - 1.0) * Y[None, :, None]
    z[2] += (g[2] - 1.0) * Z[:, None, None]
    return z.reshape(4, -1)


# ratios of eigenvalues: stretch^3 (iso), stretch^2 (one), stretch^4 (shear)
MODERATE = [("iso", 1.12), ("iso", 1.6), ("iso", 2.4), ("iso", 3.0), ("one", 0.5), ("one", 1.25), ("one", 2.2),
            ("one", 5.0), ("shear", 1.15), ("shear", 1.5), ("shear", 2.0)]
WIDE = [("iso", 5.0), ("iso", 9.0), ("iso", 20.0), ("iso", 0.2), ("one", 10.0), ("one", 0.05), ("shear", 4.0),
        ("shear", 8.0)]


@pytest.mark.parametrize("p,variant", [(1, "base"), (2, "plastic"), (3, "voce"), (4, "plastic"), (3, "ex3")])
@pytest.mark.parametrize("kind,s", MODERATE + WIDE)
def test_values(pf, oracle_lib, p, variant, kind, s):
    """rel-L2 against the oracle within 1e-12, the FP64 bar of the parity tests. The relative error of
    the smallest eigenvalue is that of b_tr's rounding times the ratio r of the eigenvalues: r * 1.1e-16,
    9e-13 at r = 8000, the widest here."""
    print(f"case p={p} {variant} {kind} {s}", flush=True)
    d = I.make_inputs("C1", variant, p=p, n=2)
    d["z"] = stretched(d, kind, s)
    ctx = pf.Context.from_inputs(d)
    orc = oracle_lib.Oracle.from_inputs(d)
    z, dz, v = dev(d["z"]), dev(d["dz"]), dev(d["v_rand"])
    r = ctx.apply_residual(z).cpu().numpy()
    y = ctx.apply_jacobian(z, dz).cpu().numpy()
    gz, gp = (t.cpu().numpy() for t in ctx.apply_adjoint(z, v))
    ctx.check()
    ogz, ogp = orc.adjoint(d["z"], d["v_rand"])
    for name, a, b in (("residual", r, orc.residual(d["z"])), ("jacobian", y, orc.jacobian(d["z"], d["dz"])),
                       ("adjoint", gz, ogz), ("parameters", gp, np.asarray(ogp))):
        err = float(np.linalg.norm(a - b) / np.linalg.norm(b))
        assert err <= 1e-12, (name, err)


@pytest.mark.parametrize("p,n", [(1, 40), (2, 32), (3, 24), (4, 16)])
def test_cost(pf, p, n):
    """A Jacobian of strongly strained elements takes at most 1.5 times one at small strains: a principal
    frame at every point would take 1,152 vector instructions per order-3 element instead of 768, so
    beyond that the tensor form would be the slower one."""
    d = I.make_inputs("C1", "plastic", p=p, n=n)
    ctx = pf.Context.from_inputs(d)
    dz = dev(d["dz"])
    y = torch.empty_like(dz)

    def time(z):
        z = dev(z)
        for _ in range(5):
            ctx.apply_jacobian(z, dz, y)
        got = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                ctx.apply_jacobian(z, dz, y)
            b.record()
            b.synchronize()
            got.append(a.elapsed_time(b))
        return sorted(got)[3]

    small = time(d["z"])
    for kind, s in (("iso", 1.5), ("iso", 3.0), ("one", 4.0), ("shear", 2.5)):
        t = time(stretched(d, kind, s))
        print(f"p={p} {kind} {s}: {t / small:.2f}", flush=True)
        assert t <= 1.5 * small, (kind, s, t / small)
    ctx.check()
