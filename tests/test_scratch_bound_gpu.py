"""The library's device buffer is bounded: stacks and batches whose volume
copies would take more than 4 GiB run in several launches, with the bits of
single calls."""
import pytest

from paper_2512_21180_amd import workloads as W

pytestmark = pytest.mark.gpu

# what the buffer may take: 4 GiB, and the allocator's rounding
BOUND = (4 << 30) + (256 << 20)


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    from paper_2512_21180_amd import cbct
    return torch, cbct


def _taken(torch, call):
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    call()
    torch.cuda.synchronize()
    return free - torch.cuda.mem_get_info()[0]


def test_stack(dev):
    """80 bf16 channels of 256^3, 2.7 GB, whose FP32 copies take 11 GB."""
    torch, cbct = dev
    print("[buffer] stack of 80 x 256^3 bf16", flush=True)
    g = W.geometry(2, 64, 48, 1.6, 1.6, 256, 256, 256, 1.6, angles=[0.0, 1.5])
    geo = cbct.Geometry(g)
    assert geo.plan_info()["fwd_tiled"]
    x = torch.rand((80,) + geo.vol_shape, device="cuda", dtype=torch.bfloat16)
    y = torch.empty((80,) + geo.sino_shape, device="cuda", dtype=torch.bfloat16)
    assert _taken(torch, lambda: cbct.forward(geo, x, out=y)) <= BOUND
    for c in (0, 30, 31, 32, 79):
        assert torch.equal(y[c], cbct.forward(geo, x[c])), c


def test_batch(dev):
    """Ten f16 volumes of 400^3, 1.3 GB, whose FP32 copies take 5.3 GB."""
    torch, cbct = dev
    print("[buffer] batch of 10 x 400^3 f16", flush=True)
    g = W.geometry(2, 64, 48, 1.2, 1.2, 400, 400, 400, 1.0, angles=[0.2, 1.5])
    geos = [cbct.Geometry(g) for _ in range(10)]
    if not geos[0].plan_info()["fwd_tiled"]:
        pytest.fail("the plan is meant to be tiled")
    xs = [torch.rand(g.vol_shape, device="cuda", dtype=torch.float16) for g in geos]
    ys = [torch.empty(g.sino_shape, device="cuda", dtype=torch.float16) for g in geos]
    assert _taken(torch, lambda: cbct.batch_forward(geos, xs, outs=ys)) <= BOUND
    for i in (0, 4, 5, 9):
        assert torch.equal(ys[i], cbct.forward(geos[i], xs[i])), i


def test_adjoint_stack(dev):
    """900 channels of few bricks, whose staged projections and partial volumes
    take 5 GB."""
    torch, cbct = dev
    print("[buffer] adjoint of 900 small channels", flush=True)
    g = W.geometry(64, 128, 96, 3.2, 3.2, 64, 64, 48, 4.0)
    geo = cbct.Geometry(g)
    y = torch.rand((900,) + geo.sino_shape, device="cuda", dtype=torch.float16)
    x = torch.empty((900,) + geo.vol_shape, device="cuda", dtype=torch.float16)
    assert _taken(torch, lambda: cbct.adjoint(geo, y, out=x)) <= BOUND
    for c in (0, 450, 899):
        assert torch.equal(x[c], cbct.adjoint(geo, y[c])), c
