"""pf_prolong and pf_restrict with vectors that share memory: the same result as with vectors apart."""
import pytest

from paper_2607_21150_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("p,n,levels", [(4, 3, [4, 3]), (3, 8, [3, 2]), (2, 8, [2, 1, 1])])
@pytest.mark.parametrize("shift", [0, 37])
def test_overlapping_transfer(p, n, levels, shift):
    """Coarse vector at an offset of `shift` entries into the fine one's memory. Both paths sum at most 27
    products of FP32 weights up to 1.2 in three nested sums: 3e-6, as for the transfers."""
    from paper_2607_21150_amd import pfmf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    d = I.make_inputs("C1", "base", p=p, n=n)
    ctx = pfmf.Context.from_inputs(d)
    ctx.set_pmg_levels(levels)
    ctx.linearize(torch.as_tensor(d["z"]).to("cuda", torch.float64))
    torch.manual_seed(1)
    for l in range(len(levels) - 1):
        nf, nc = ctx.level_info(l)[1], ctx.level_info(l + 1)[1]
        mem = torch.empty(4 * nf + shift, device="cuda")
        fine, coarse = mem[:4 * nf].view(4, nf), mem[shift:shift + 4 * nc].view(4, nc)
        x = torch.randn(4, nc, device="cuda")
        ref = ctx.prolong(l, x).clone()
        coarse.copy_(x)
        got = ctx.prolong(l, coarse, fine)
        assert float(torch.linalg.norm(got - ref) / torch.linalg.norm(ref)) <= 3e-6, ("prolong", l)
        y = torch.randn(4, nf, device="cuda")
        ref = ctx.restrict(l, y).clone()
        fine.copy_(y)
        got = ctx.restrict(l, fine, coarse)
        assert float(torch.linalg.norm(got - ref) / torch.linalg.norm(ref)) <= 3e-6, ("restrict", l)
