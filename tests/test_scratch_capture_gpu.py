"""A captured projection and backprojection name the library's device buffer:
they replay correctly after a larger call has outgrown it."""
import pytest

from paper_2512_21180_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    from paper_2512_21180_amd import cbct
    return torch, cbct


def test_replay_after_growth(dev):
    torch, cbct = dev
    print("[scratch] replay after growth", flush=True)
    geo, big = cbct.Geometry(W.cropped(W.C2, n_angles=6, nu=96, nv=40, n=32)), cbct.Geometry(W.C2)
    x, y = torch.rand(geo.vol_shape, device="cuda"), torch.rand(geo.sino_shape, device="cuda")
    fwd, adj = cbct.forward(geo, x), cbct.adjoint(geo, y)
    f, a = torch.empty_like(fwd), torch.empty_like(adj)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cbct.forward(geo, x, out=f)
        cbct.adjoint(geo, y, out=a)

    def replayed():
        f.zero_()
        a.zero_()
        graph.replay()
        torch.cuda.synchronize()
        return torch.equal(f, fwd) and torch.equal(a, adj)

    assert replayed()
    # 3.8 GB of staged projections: the buffer grows (unless an earlier test took as much)
    ys = torch.rand((10,) + big.sino_shape, device="cuda")
    cbct.adjoint(big, ys)
    for _ in range(3):
        assert replayed()
        assert torch.equal(cbct.forward(geo, x), fwd)
        assert torch.equal(cbct.adjoint(geo, y), adj)
