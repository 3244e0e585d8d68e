"""A non-physical point's NaN in the multigrid hierarchy stays with the nodes that it reaches."""
import pytest

from paper_2607_21150_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("p,n,levels", [(2, 8, [2, 1, 1, 1]), (3, 4, [3, 2, 1, 1])])
def test_nan_of_the_first_element_stays_local(p, n, levels):
    """NaN displacement at the box's corner node: it lies in the first element only, so on an order-q level
    on the mesh the nodes 0..q per direction, and on a lattice halved h times the nodes 0 and 1, see it."""
    from paper_2607_21150_amd import pfmf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    d = I.make_inputs("C1", "base", p=p, n=n)
    d["z"][0, 0] = float("nan")
    ctx = pfmf.Context.from_inputs(d)
    ctx.set_pmg_levels(levels)
    with pytest.raises(pfmf.PfError) as e:
        ctx.linearize(torch.as_tensor(d["z"]).to("cuda", torch.float64))
    assert e.value.code == pfmf.PF_ENONPHYSICAL
    ne = n
    for l, q in enumerate(levels):
        if l > 0 and q == 1 and levels[l - 1] == 1:
            ne //= 2
        n1 = q * ne + 1
        bad = ~torch.isfinite(ctx.level_diagonal(l).reshape(4, n1, n1, n1)).all(0)
        reach = torch.zeros_like(bad)
        reach[:q + 1, :q + 1, :q + 1] = True
        assert bad[0, 0, 0], l
        assert not (bad & ~reach).any(), (l, bad.nonzero().tolist()[:5])
