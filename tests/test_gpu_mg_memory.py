"""Device memory of a multigrid hierarchy without an order-1 level."""
import pytest

from paper_2607_21150_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_level_list_without_order_1(n=40):
    """Levels 3, 2 on 40^3 elements: what pf_linearize takes is the records (15 and 9 FP32 and 15 FP64 values and
    a flag byte per point), u, two spare and seven vectors per level, the bricks' sums (7^3 nodes of 2^3 elements)
    and 4 * 4^3 FP32 values per element for the diagonals; 64 MB for the allocations' granules. The
    element matrices of an order-1 level (1024 values per element, 262 MB) are not part of it."""
    from paper_2607_21150_amd import pfmf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    pfmf.load()
    d = I.make_inputs("C1", "base", p=3, n=n)
    z = torch.as_tensor(d["z"]).to("cuda", torch.float64)
    first = pfmf.Context.from_inputs(d)  # what the runtime takes for these kernels, once per process
    first.set_pmg_levels([3, 2])
    first.linearize(z)
    first.close()
    ctx = pfmf.Context.from_inputs(d)
    ctx.set_pmg_levels([3, 2])
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    ctx.linearize(z)
    used = free - torch.cuda.mem_get_info()[0]
    m = d["mesh"]
    nodes, coarse = m.n_nodes, (2 * n + 1) ** 3
    need = (m.n_q * (15 * 4 + 9 * 4 + 15 * 8 + 1) + nodes * (24 + 2 * 16) + 7 * 16 * (nodes + coarse)
            + m.n_elem // 8 * 4 * 7 ** 3 * 4 + m.n_elem * 4 * 4 ** 3 * 4)
    print(f"used {used / 2**20:.0f} MB, need {need / 2**20:.0f} MB")
    assert used <= need + (64 << 20), (used, need)
